// The split plan that a decode call takes, and the bounds that the workspace is sized by (256 compute units: without a device the
// plan is the whole part's).
//   plan_check                                                      every length, batch and head count of a range against the bounds;
//                                                                   prints a line per fault and the number of plans
//   plan_check BATCH KV_HEADS HEADS BITS_K BITS_V TOKENS [ragged]   prints parts per sequence, steps per part, wavefronts per
//                                                                   workgroup, the workgroups that are dealt out and the longest
//                                                                   part of those that pays
#include "kvq_internal.h"

#include <cstdio>
#include <cstdlib>
#include <vector>

namespace {
long faults = 0, plans = 0;
void fault(const char* what, const kvq::Geom& g, int heads, int len, long got, long want) {
  if (++faults <= 20)
    printf("%s: %d x %d heads, %d query heads each, bits %d/%d, buffer %d, %d tokens: %ld, %ld\n", what, g.batch, g.kv_heads, heads,
           g.bits_k, g.bits_v, g.resid, len, got, want);
}
// Records per (batch, query head) that a plan's call writes or reads.
long records(const kvq::Geom& g, const kvq::DecodePlan& p) {
  if (p.slots) return (p.slots + g.batch - 1) / g.batch;
  return p.n_splits + (g.resid && g.axis_k != KVQ_AXIS_SEQ ? 1 : 0);
}
bool same(const kvq::DecodePlan& a, const kvq::DecodePlan& b) {
  return a.n_splits == b.n_splits && a.steps_per_split == b.steps_per_split && a.waves_per_wg == b.waves_per_wg && a.slots == b.slots;
}
long room_of(long records) { return records == 1 ? 0 : records; }      // (one record is none: no workspace is asked for)

void check(kvq_layout L, const std::vector<int>& lengths) {
  const kvq::Geom g = kvq::make_geom(L);
  long before = 0;
  for (int len : lengths) {
    const long full = kvq::decode_records_bound(g, len), least = kvq::decode_records_bound(g, len, true);
    if (full < before) fault("the bound shrinks", g, 0, len, full, before);
    if (least > full) fault("the least is more than the bound", g, 0, len, least, full);
    before = full;
    const int n_steps = g.resid ? len / g.resid * (g.resid / 32) : (len + 31) / 32;
    for (int heads : {1, 2, 4, 8})
      for (bool ragged : {false, true}) {
        const kvq::DecodePlan any = kvq::plan_decode(g, len, heads, 1L << 40, ragged);
        if (records(g, any) > 1 && records(g, any) > full) fault(ragged ? "ragged, beyond the bound" : "beyond the bound", g, heads, len, records(g, any), full);
        for (long have : {full, least, (full + least) / 2}) {
          const kvq::DecodePlan p = kvq::plan_decode(g, len, heads, room_of(have), ragged);
          ++plans;
          if (records(g, p) > 1 && records(g, p) > have) fault(ragged ? "ragged, beyond the workspace" : "beyond the workspace", g, heads, len, records(g, p), have);
          if (have == full && !same(p, any)) fault(ragged ? "ragged, not the full plan" : "not the full plan", g, heads, len, records(g, p), records(g, any));
          if (p.n_splits && (long)p.n_splits * p.steps_per_split < n_steps) fault("steps left out", g, heads, len, (long)p.n_splits * p.steps_per_split, n_steps);
          if (p.slots && (p.deal_pays < p.waves_per_wg || p.deal_pays % p.waves_per_wg || 8 * p.deal_pays < p.steps_per_split || p.deal_pays >= p.steps_per_split))
            fault("a part that cannot pay", g, heads, len, p.deal_pays, p.steps_per_split);
          if (p.slots && p.slots < p.n_splits * g.batch) fault("fewer workgroups than parts", g, heads, len, p.slots, p.n_splits * g.batch);
        }
      }
  }
}
}  // namespace

int all() {
  std::vector<int> lengths;
  for (int s = 1; s <= 160; ++s) { lengths.push_back(32 * s - 31); lengths.push_back(32 * s); }
  for (int len = 5121; len <= 131072; len += len / 9 + 13) lengths.push_back(len);
  for (int kv_heads : {1, 2, 4, 5, 8, 16})
    for (int batch = 1; batch <= 80; batch += batch < 66 ? 1 : 7)
      for (int form = 0; form < 6; ++form) {
        kvq_layout L{};
        L.batch = batch; L.kv_heads = kv_heads; L.max_seq = 1 << 18; L.head_dim = 128;
        L.bits_k = form == 1 ? 16 : form == 5 ? 8 : 4; L.bits_v = form == 1 ? 16 : form == 5 ? 8 : 2;
        L.group_k = L.group_v = 64;
        L.axis_k = form == 3 || form == 4 ? KVQ_AXIS_SEQ : KVQ_AXIS_HEAD_DIM; L.axis_v = KVQ_AXIS_HEAD_DIM;
        L.resid_len = form == 2 ? 64 : form == 4 ? 128 : 0;
        check(L, lengths);
      }
  printf("plans=%ld faults=%ld\n", plans, faults);
  return faults != 0;
}

int main(int argc, char** argv) {
  if (argc == 1) return all();
  if (argc < 7) return 2;
  kvq_layout L{};
  L.batch = atoi(argv[1]); L.kv_heads = atoi(argv[2]); L.max_seq = 1 << 18; L.head_dim = 128;
  L.bits_k = atoi(argv[4]); L.bits_v = atoi(argv[5]); L.group_k = L.group_v = 64;
  L.axis_k = L.axis_v = KVQ_AXIS_HEAD_DIM;
  const kvq::DecodePlan p = kvq::plan_decode(kvq::make_geom(L), atoi(argv[6]), atoi(argv[3]), 1L << 40, argc > 7);
  printf("%d %d %d %d %d\n", p.n_splits, p.steps_per_split, p.waves_per_wg, p.slots, p.deal_pays);
  return 0;
}
