"""The library's own split plan, asked on the CPU."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
PKG = os.path.join(os.path.dirname(HERE), "paper_2502_15075_amd")


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plan") / "plan_check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__=1", "-I", os.path.join(PKG, "csrc"), "-I", os.path.join(os.path.dirname(HERE), "include"),
                    "-isystem", "/opt/rocm/include", "-o", exe, os.path.join(HERE, "plan_check.cpp"), "-L", PKG, "-lkvq", f"-Wl,-rpath,{PKG}",
                    "-L", "/opt/rocm/lib", "-Wl,-rpath,/opt/rocm/lib", "-lamdhip64"], check=True)
    return lambda *a: subprocess.run([exe, *map(str, a)], capture_output=True, text=True)


def _plan(check, *a):
    r = check(*a)
    assert r.returncode == 0, r.stdout + r.stderr
    return tuple(map(int, r.stdout.split()))


@pytest.mark.parametrize("batch,heads,tokens,parts,steps", [(16, 4, 512, 2, 8), (16, 8, 513, 1, 24), (16, 8, 704, 1, 24), (16, 8, 705, 2, 16), (12, 1, 640, 1, 24),
                                                            (16, 4, 641, 2, 16), (11, 4, 577, 1, 24), (11, 4, 768, 2, 16), (10, 4, 577, 3, 8), (17, 4, 577, 1, 24)])
def test_unquantized_sequences_of_two_parts_at_most(check, batch, heads, tokens, parts, steps):
    """Unquantized rows where the chip has room for two parts a sequence: 17 to 20 steps (22 for more than 4 heads) are one part, as two
    would be one of two steps per wavefront and a nearly empty one; with room for three they are three."""
    assert _plan(check, batch, 8, heads, 16, 16, tokens)[:3] == (parts, steps, 8)


def test_plans_stay_inside_the_workspace_and_reach_the_whole_of_it(check):
    """No plan writes more records than the workspace it is given holds or the size query counts, and with the workspace that the
    query reports a call takes the plan of any larger one."""
    r = check()
    assert r.returncode == 0, r.stdout + r.stderr
    assert int(r.stdout.split("plans=")[1].split()[0]) > 1000000


@pytest.mark.parametrize("batch,heads,bits_k,bits_v,tokens,want", [(18, 4, 4, 2, 1400, (1, 48, 8, 0)), (18, 4, 4, 2, 2272, (1, 72, 8, 32)), (18, 4, 4, 2, 2048, (1, 64, 8, 0)),
                                                                   (33, 4, 4, 2, 1281, (1, 44, 4, 64)), (33, 4, 4, 2, 1280, (1, 40, 4, 0)),
                                                                   (18, 4, 8, 8, 1281, (1, 48, 8, 32)), (18, 4, 8, 8, 1024, (1, 32, 8, 0)),
                                                                   (11, 4, 4, 2, 3500, (2, 56, 8, 32)), (9, 4, 4, 2, 12000, (3, 128, 8, 32)),
                                                                   (11, 4, 8, 8, 2048, (2, 32, 8, 32)), (11, 4, 8, 8, 1536, (2, 24, 8, 0)), (11, 4, 8, 4, 1537, (2, 32, 8, 32)),
                                                                   (40, 4, 8, 8, 1153, (1, 40, 4, 64)), (40, 4, 8, 8, 1152, (1, 36, 4, 0))])
def test_which_ragged_batches_may_be_dealt_out(check, batch, heads, bits_k, bits_v, tokens, want):
    """Sequences of one part: from nine steps per wavefront on, half as many of rows twice as wide, of four wavefronts from eleven (ten); of two
    parts from six steps on, of wide rows four."""
    assert _plan(check, batch, 8, heads, bits_k, bits_v, tokens, "ragged")[:4] == want


@pytest.mark.parametrize("batch,heads,bits,tokens,want", [(40, 4, 3, 1400, 16), (40, 4, 3, 2500, 52), (40, 4, 3, 9000, 244), (40, 5, 3, 1400, 8), (40, 8, 3, 3600, 80), (40, 8, 3, 9000, 236),
                                                          (40, 4, 8, 1400, 28), (40, 1, 8, 3600, 88), (40, 4, 8, 9000, 248), (40, 8, 8, 1400, 20), (40, 7, 8, 3600, 84), (40, 8, 8, 9000, 248),
                                                          (18, 8, 3, 2272, 40), (18, 8, 3, 2561, 48), (18, 8, 3, 6500, 168), (18, 8, 3, 9500, 264), (18, 8, 3, 15000, 408), (18, 1, 8, 3000, 72)])
def test_longest_part_that_pays(check, batch, heads, bits, tokens, want):
    """Steps: of four wavefronts at least seven each and 3/10 less than planned, for more than 4 heads nine and a quarter, of wide rows four and
    2/9 (six and a quarter); of eight, five and an eighth (four of up to ten), of wide rows half of
    the five."""
    assert _plan(check, batch, 8, heads, bits, bits, tokens, "ragged")[4] == want
