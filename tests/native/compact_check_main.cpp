// Host-only driver for the compact form of the work list (plan.cpp: compact_plan, and
// expand_item, which the device uses as it is): reads batches from stdin
//   <Hq> <Hkv> <D> <n_cus> <n_seqs> P0 C0 P1 C1 ...
// and prints "<accepted 0|1> <n_items> <bytes> <records that differ>": every record of the
// ordinary list against what its reference expands to.
#include <cstdio>
#include <cstring>
#include <iostream>
#include <vector>

#include "cronus_internal.h"

namespace cronus {
int wide_rows_for(int, int) { return kWaves * 32; }
}  // namespace cronus

int main() {
  using namespace cronus;
  int hq, hkv, d, n_cus, n;
  while (std::cin >> hq >> hkv >> d >> n_cus >> n) {
    std::vector<int32_t> P((size_t)n), C((size_t)n);
    for (int i = 0; i < n; ++i) std::cin >> P[(size_t)i] >> C[(size_t)i];
    cronus_kv_cache c{};
    c.num_blocks = 1 << 30;
    c.num_q_heads = hq;
    c.num_kv_heads = hkv;
    c.head_dim = d;
    c.block_size = 16;
    Plan plan;
    if (build_plan(&c, P.data(), C.data(), n, 0x7fffffff / 16, n_cus, &plan, false)) return 1;
    std::vector<unsigned char> image(plan.image_bytes), buf(plan.image_bytes);  // exactly sized
    write_plan(&plan, image.data());
    CompactPlan m{};
    size_t bytes = 0;
    const bool ok = compact_plan(&c, &plan, &m, buf.data(), buf.size(), &bytes);
    long long bad = 0;
    if (ok) {
      const WorkItem* want = reinterpret_cast<const WorkItem*>(image.data() + plan.off_items);
      const unsigned char* refs = buf.data() + (size_t)m.n_units * sizeof(CompactUnit);
      for (long long i = 0; i < plan.n_items; ++i) {
        uint32_t ref = 0;
        std::memcpy(&ref, refs + (size_t)i * m.ref_bytes, (size_t)m.ref_bytes);
        WorkItem e = expand_item(m, reinterpret_cast<const CompactUnit*>(buf.data()), ref);
        if (e.partial < 0) {  // fields that nothing reads then
          e.first_partial = want[i].first_partial;
          e.merge_key = want[i].merge_key;
        }
        bad += std::memcmp(&e, &want[i], sizeof(e)) != 0;
      }
    }
    std::printf("%d %lld %zu %lld\n", ok ? 1 : 0, (long long)plan.n_items, bytes, bad);
  }
  return 0;
}
