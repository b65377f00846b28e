// Prints how decode attention cuts a batch: reads "dtype n_q_heads n_kv_heads head_dim row_pitch batch tokens..." lines
// from stdin and answers each with one line: the workspace size, then per launch
// "| n_split rows:ranges:first ...".  With "waves": per launch the wavefronts of a workgroup over fp32 caches.
#include <cstdio>
#include <vector>

#include "decode_plan.h"

int main(int argc, char **) {
  const bool waves = argc > 1;
  chunkkv_problem p{};
  long long pitch;
  while (std::scanf("%d %d %d %d %lld %d", &p.dtype, &p.n_q_heads, &p.n_kv_heads, &p.head_dim, &pitch, &p.batch) == 6) {
    std::vector<int32_t> n(p.batch);
    for (int32_t &x : n)
      if (std::scanf("%d", &x) != 1) return 1;
    p.seqlen = n.data();
    p.kv_stride_tok = pitch;
    ckv::DecodePlan pl;
    ckv::decode_plan(&p, false, &pl);
    if (!waves) std::printf("%zu", pl.total);
    for (int b0 = 0; b0 < p.batch; b0 += ckv::kMaxBatchPerLaunch) {
      const int nb = p.batch - b0 < ckv::kMaxBatchPerLaunch ? p.batch - b0 : ckv::kMaxBatchPerLaunch;
      ckv::DecodeCut c;
      ckv::decode_cut(&p, false, b0, nb, &c);
      if (waves) {
        std::printf("%d ", ckv::decode_f32_waves(p.head_dim, p.n_q_heads / p.n_kv_heads, p.n_kv_heads, nb, c));
        continue;
      }
      std::printf(" | %d", c.n_split);
      for (int i = 0; i < nb; ++i) std::printf(" %d:%d:%d", c.rows_per_split[i], c.splits[i], c.first_split[i]);
    }
    std::printf("\n");
  }
  return 0;
}
