// Host-only driver for what passes the caches (plan.cpp: WorkItem::peers, rows_past_cache): reads batches from stdin
//   <Hq> <Hkv> <D> <fp8 0|1> <n_cus> <n_seqs> P0 C0 P1 C1 ...
// and prints, for each, "<narrow items> <rows past the caches 0|1>" and then a line "seq kv_head q_tok0 n_tok kv_begin kv_end
// peers" for every one.
#include <cstdio>
#include <iostream>
#include <vector>

#include "cronus_internal.h"

namespace cronus {
int wide_rows_for(int, int) { return kWaves * 32; }
}  // namespace cronus

int main() {
  using namespace cronus;
  int hq, hkv, d, fp8, n_cus, n;
  while (std::cin >> hq >> hkv >> d >> fp8 >> n_cus >> n) {
    std::vector<int32_t> P((size_t)n), C((size_t)n);
    for (int i = 0; i < n; ++i) std::cin >> P[(size_t)i] >> C[(size_t)i];
    cronus_kv_cache c{};
    c.num_blocks = 1 << 30;
    c.num_q_heads = hq;
    c.num_kv_heads = hkv;
    c.head_dim = d;
    c.block_size = 16;
    c.kv_dtype = fp8 ? CRONUS_KV_FP8_E4M3 : CRONUS_KV_BF16;
    Plan plan;
    if (build_plan(&c, P.data(), C.data(), n, 0x7fffffff / 16, n_cus, &plan)) return 1;
    std::vector<unsigned char> image(plan.image_bytes);  // exactly sized
    write_plan(&plan, image.data());
    const WorkItem* w = reinterpret_cast<const WorkItem*>(image.data() + plan.off_items);
    std::printf("%lld %d\n", (long long)(plan.n_items - plan.n_wide), (int)rows_past_cache(&c, P.data(), C.data(), n));
    for (long long i = 0; i < plan.n_items; ++i)
      if (!w[i].wide)
        std::printf("%d %d %d %d %d %d %d\n", w[i].seq, w[i].kv_head, w[i].q_tok0, w[i].n_tok, w[i].kv_begin, w[i].kv_end,
                    w[i].peers);
  }
  return 0;
}
