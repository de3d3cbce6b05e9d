// The split plan that a decode call takes (256 compute units: without a device the plan is the whole part's).
//   plan_check BATCH KV_HEADS HEADS BITS_K BITS_V TOKENS [ragged]   prints parts per sequence, steps per part, wavefronts per
//                                                                   workgroup and the workgroups that are dealt out
#include "kvq_internal.h"

#include <cstdio>
#include <cstdlib>

int main(int argc, char** argv) {
  if (argc < 7) return 2;
  kvq_layout L{};
  L.batch = atoi(argv[1]); L.kv_heads = atoi(argv[2]); L.max_seq = 1 << 18; L.head_dim = 128;
  L.bits_k = atoi(argv[4]); L.bits_v = atoi(argv[5]); L.group_k = L.group_v = 64;
  L.axis_k = L.axis_v = KVQ_AXIS_HEAD_DIM;
  const kvq::DecodePlan p = kvq::plan_decode(kvq::make_geom(L), atoi(argv[6]), atoi(argv[3]), 1L << 40, argc > 7);
  printf("%d %d %d %d\n", p.n_splits, p.steps_per_split, p.waves_per_wg, p.slots);
  return 0;
}
