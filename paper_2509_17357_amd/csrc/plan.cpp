// Host-side work decomposition of one mixed iteration (Cronus section 4.4: the batch
// holds continuation chunks and decodes; Eq. 3: chunk cost grows with its prefill
// context, decode cost with the summed decode contexts).  Chunks become wide tiles of
// `wide_rows` (token, head) rows; decodes and short chunks become narrow items whose
// key range is cut into spans so that long contexts spread over the chip.
//
// This runs on the host inside every cronus_attn_mixed call, so it is written to be a
// few tens of microseconds for thousands of items: flat arrays kept per thread, no
// comparison sorts over items (narrow items are bucketed by length, the wide tiles of a
// group are generated in cost order).
#include <algorithm>
#include <cmath>
#include <cstring>
#include <utility>
#include <vector>

#include "cronus_internal.h"

namespace cronus {
namespace {

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

constexpr int kXcds = kQueues;

struct Group {      // the wide tiles of one (sequence, KV head, head group): items [begin, end)
  int32_t begin, end;
  float cost;
};

struct Scratch {
  std::vector<SeqInfo> seqs;
  std::vector<WorkItem> wide, narrow;
  std::vector<float> wide_cost;
  std::vector<Group> groups;
  std::vector<MergeItem> merges;
  std::vector<StageSeq> stages;
  std::vector<int32_t> queue[kXcds];  // item references: >= 0 wide index, < 0 ~narrow index
  struct Tile { int32_t t0, nt, kv_total, n_split, per, first_partial, merge_key; float cost_per_key; };
  std::vector<Tile> tiles;
  std::vector<int32_t> order, bucket_start;
  struct Run { int32_t begin, len; float shortest; };  // a contiguous run of one group's tiles in a queue
  std::vector<Run> runs[kXcds];
  int32_t wide_tok;                    // tokens per wide tile of the last plan
  // compact_plan: the unit of every item (tiles of a sequence back to back, head group by head group), and their number
  std::vector<int32_t> wide_unit, narrow_unit;
  long long n_units;
  std::vector<int32_t> unit_seq, unit_keys, peers;  // build_plan: for WorkItem::peers
  std::vector<uint8_t> whole;          // by sequence: narrow rows that are not cut for want of arrival counters (else empty)
  std::vector<float> row_keys;         // keys of the narrow rows, one entry per sequence
  struct Busy { double until; long long cus; };
  std::vector<Busy> busy;              // list_us: CUs by the time they are free again, a heap
  struct Load { double us; long long items; };
  std::vector<Load> loads;             // items of equal estimated times
  std::vector<std::pair<int32_t, int32_t>> by_length;  // (-keys, sequence) of the narrow rows that are long enough to be cut
};

Scratch& scratch() {
  static thread_local Scratch s;
  return s;
}

}  // namespace

// A narrow item's keys in equal spans of at most `span` (and a quarter: no sliver spans), whole steps.
struct NarrowSplit { int n, per; };
static NarrowSplit split_of(long long kv_total, long long span) {
  long long n = std::max<long long>(1, (kv_total + span - 1) / span);
  if (n > 1 && kv_total - (n - 1) * span <= span / 4) --n;
  const long long per = ((kv_total + n - 1) / n + kNarrowKvStep - 1) / kNarrowKvStep * kNarrowKvStep;
  return NarrowSplit{(int)((kv_total + per - 1) / per), (int)per};
}

// End (us) of the items in `loads`, dealt in their order to `cus` CUs, each to the CU that is free first.
static double list_us(const std::vector<Scratch::Load>& loads, long long cus) {
  auto& busy = scratch().busy;
  auto later = [](const Scratch::Busy& a, const Scratch::Busy& b) { return a.until > b.until; };
  busy.assign(1, Scratch::Busy{0.0, cus});
  double end = 0;
  for (size_t i = 0; i < loads.size();) {
    const Scratch::Load& l = loads[i];
    long long left = 0;
    for (; i < loads.size() && loads[i].us == l.us; ++i) left += loads[i].items;
    while (left > 0) {
      std::pop_heap(busy.begin(), busy.end(), later);
      Scratch::Busy& first = busy.back();
      const long long k = std::min(left, first.cus);
      const double until = first.until + l.us;
      left -= k;
      first.cus -= k;
      if (first.cus == 0) {
        first = Scratch::Busy{until, k};
      } else {
        std::push_heap(busy.begin(), busy.end(), later);
        busy.push_back(Scratch::Busy{until, k});
      }
      std::push_heap(busy.begin(), busy.end(), later);
      end = std::max(end, until);
    }
  }
  return end;
}

// Estimated time (us) of the narrow rows in `row_keys` (`copies` of each) when they are cut into spans of
// `span` keys and run on `cus` CUs, longest first: 8 us and key_us per key an item, 4 us more for each item of a
// launch that cuts any row (partial results, merge).  Lengths are taken in classes of 64 keys, so the cost is
// that of the classes.
static double rounds_us(const std::vector<float>& row_keys, long long copies, long long span, long long cus, double key_us) {
  constexpr int kClass = 64, kClasses = 96;
  long long count[kClasses] = {0};
  bool cut = false;
  for (const float keys : row_keys) {  // as split_of cuts them
    const int n = std::max(1, (int)std::ceil(keys / (float)span - 0.25f));
    count[std::min(kClasses - 1, (int)(keys / (float)n) / kClass)] += n;
    cut = cut || n > 1;
  }
  auto& loads = scratch().loads;
  loads.clear();
  for (int c = kClasses - 1; c >= 0; --c)
    if (count[c] > 0) loads.push_back(Scratch::Load{(cut ? 12.0 : 8.0) + key_us * (kClass * c + kClass / 2), count[c] * copies});
  return list_us(loads, cus);
}

// Time of the chunks' products over `pairs` visible (query, key) pairs a head, at 1.2 PFLOP/s.
static double products_us(const cronus_kv_cache* cache, double pairs) {
  return pairs * 4.0 * cache->num_q_heads * cache->head_dim / 1.2e9;
}

int build_plan(const cronus_kv_cache* cache, const int32_t* prefix_lens, const int32_t* chunk_lens,
               int32_t n_seqs, int32_t max_blocks_per_seq, int n_cus, Plan* plan, bool allow_stage,
               size_t scratch_limit, bool lean) {
  const int D = cache->head_dim, Hq = cache->num_q_heads, Hkv = cache->num_kv_heads;
  const int G = Hq / Hkv;
  const int group = std::min(G, kNarrowRows);          // q heads handled together by one item
  const int n_groups = (G + group - 1) / group;        // > 1 only when G > 32
  const int wide_rows = wide_rows_for(D, cache->kv_dtype);
  // Tokens per wide tile.  A launch whose items would not even fill the CUs once and whose
  // tiles are too short to be cut into key spans (one chunk of a few hundred tokens with
  // little context next to a few decodes: the iteration of section 5.1 early in a request,
  // or a short whole prompt) takes half tiles, 128 rows: four of the eight waves own rows,
  // a tile's time drops by a quarter, and twice as many CUs work.
  // (Measured on MI355X: a 512-token chunk behind 1024 cached tokens 40.6 -> 29.6 us; quarter
  // tiles are slower again, and with the CUs already filled half tiles cost 1.5x the CU time.)
  constexpr int kMinPiece = 16 * kWideKvTile;  // no key span of a wide tile is shorter
  int wide_tok = std::max(1, wide_rows / group);
  // A wide tile addresses its rows by 24-bit products of a token's bytes (Hq x D bf16); where
  // those do not hold them, the chunk is cut into narrow items (64-bit addresses).
  if ((long long)Hq * D * 2 >= 1 << 24) wide_tok = std::max(1, kNarrowRows / group);
  {
    long long full_tiles = 0, narrow_items = 0, longest = 0;
    for (int s = 0; s < n_seqs; ++s) {
      const long long P = prefix_lens[s], C = chunk_lens[s];
      if (C <= 0 || P < 0) continue;
      if (C * group <= kNarrowRows) { narrow_items += (long long)Hkv * n_groups; continue; }
      const long long rem = C % wide_tok, full = C / wide_tok;
      const bool wide_rem = rem && rem * group > kNarrowRows;
      full_tiles += (full + wide_rem) * Hkv * n_groups;
      narrow_items += (rem && !wide_rem) ? (long long)Hkv * n_groups : 0;
      longest = std::max(longest, P + C);
    }
    // (a tile of more than 1.5 minimum spans is cut over its keys below, which serves such a launch better)
    if (full_tiles > 0 && 2 * full_tiles + narrow_items <= std::max(n_cus, 1) && longest <= kMinPiece + kMinPiece / 2 &&
        (wide_tok / 2) * group > kNarrowRows)
      wide_tok /= 2;
  }

  // keys read by narrow items, to size the spans, and the cost of the wide tiles in the
  // planner's unit (one key of a full wide tile = wide_rows / 128, one key of a narrow
  // item = 1/2), to size the spans that long wide tiles are cut into
  long long narrow_keys = 0, decode_keys = 0;
  double wide_cost_total = 0, chunk_pairs = 0;
  long long wide_tiles = 0;
  for (int s = 0; s < n_seqs; ++s) {
    const long long P = prefix_lens[s], C = chunk_lens[s];
    if (P < 0 || C < 0) return CRONUS_ERR_INVALID_ARG;
    if (P + C > (long long)max_blocks_per_seq * kBlock) return CRONUS_ERR_INVALID_ARG;
    if (C == 0) continue;
    if (C * group <= kNarrowRows) {
      narrow_keys += (P + C) * Hkv * n_groups;
      decode_keys += P + C;
    } else {
      chunk_pairs += (double)C * (double)P + 0.5 * (double)C * (double)(C + 1);
      const long long rem = C % wide_tok;
      if (rem && rem * group <= kNarrowRows) narrow_keys += (P + C) * Hkv * n_groups;
      const long long full = C / wide_tok;  // full tiles end at P + wide_tok, P + 2 wide_tok, ...
      double keys = (double)full * P + (double)wide_tok * full * (full + 1) / 2;
      if (rem && rem * group > kNarrowRows) keys += (double)(P + C) * std::max(0.25, (double)(rem * group) / wide_rows);
      wide_cost_total += keys * (wide_rows / 128.0) * Hkv * n_groups;
      wide_tiles += (full + (rem && rem * group > kNarrowRows)) * Hkv * n_groups;
    }
  }
  // no wide item should hold a CU for much longer than three quarters of a CU's fair share
  // (measured on paper-shaped iterations: smaller spans pay more for their prologue and the
  // merge than they gain in balance), and no span is shorter than 16 K/V tiles here
  int wide_piece_keys = 0;
  long long wide_items = -1, wide_slots = 0;  // of the cut chosen below (launches of few tiles)
  // With a limit: that many items and partial slots would exceed it.  (A merge record belongs to at
  // least two slots.  The narrow rows' shares are those of the span that they are counted with: a span that
  // is chosen anew below is counted anew.)
  auto too_large = [&](long long items, long long slots) {
    return scratch_limit > 0 && (size_t)items * sizeof(WorkItem) +
                                        (size_t)slots * (sizeof(float) * partial_floats(D) + sizeof(MergeItem)) + 1024 >
                                    scratch_limit;
  };
  if (wide_cost_total > 0) {
    const double fair = (wide_cost_total + 0.5 * narrow_keys) / std::max(n_cus, 1);
    const double keys = 0.75 * fair / (wide_rows / 128.0);
    wide_piece_keys = (int)std::min<double>(std::max<double>(keys, kMinPiece), 1 << 30);
    wide_piece_keys = (wide_piece_keys + kWideKvTile - 1) / kWideKvTile * kWideKvTile;
  }
  const long long target_items = std::max(n_cus, 1);  // about one span per CU: longer spans mean fewer work-group starts and fewer partial results to merge (measured: 6 % on the Llama-3-8B-shaped batch against four per CU)
  long long span = (narrow_keys + target_items - 1) / target_items;
  span = (span + kNarrowKvStep - 1) / kNarrowKvStep * kNarrowKvStep;
  constexpr int kMaxSpanSteps = 16;  // spans are 2 .. 16 steps of kNarrowKvStep keys
  span = std::min<long long>(std::max<long long>(span, 2 * kNarrowKvStep), kMaxSpanSteps * kNarrowKvStep);

  // A launch with few wide tiles (the paper's own iteration: one chunk of at most 512 tokens
  // = 64 tiles, section 5.1) lives or dies by how its spans pack onto the CUs next to the
  // decodes: 64 tiles in five spans each are 320 items for 256 CUs, two rounds where four
  // spans each need one; next to many decodes long wide items start late and end last.
  // Such a launch therefore picks its span length by estimated duration: for every way of
  // cutting the longest tile into 1 .. 8 equal spans (of at least 8 K/V tiles), the items
  // and their times under a model fitted to measured launches on MI355X (489 iterations of at most
  // two tiles per CU: whole prompts, chunks behind prefixes, with and without decodes, bf16 and fp8,
  // D = 64 and 128, G = 4, 5, 7 and 8, each with every cut: against the measured best cut the model's choice costs
  // 1.6 % on average and 25 % at worst).  Two regimes, by the narrow items' share of the work:
  //  * chunk-dominated (estimated narrow time under 0.34 of the wide tiles'): the wide items
  //    run in rounds over the CUs; the CUs that the last round leaves free take narrow items
  //    meanwhile, the narrow items left after that follow in rounds of their own.  More than one round
  //    of wide items takes 0.3 of (all rounds but one at the mean time, and the longest item) and 0.7 of what
  //    dealing them longest first takes: tiles of one length need whole rounds, those of a whole
  //    prompt (36, 72 .. 1200 keys) do not.  With whole rounds alone, and 14 us an item, one prompt of 1228 tokens, G = 8, was cut
  //    into 384 items instead of 312, 51.6 us instead of 40.0; over the 489 iterations that cost 2.8 % on
  //    average, 34 % at worst against the cut of version 505.  A wide item takes 23 us + 25 ns
  //    per key at 256 rows (three quarters of that per key at half
  //    height), a narrow span 8.4 us + 13 ns per key, a launch with cut
  //    tiles 3 us + 2.4 ns per partial slot.
  //  * decode-rich: the launch cannot end before the items' times summed over the CUs, before
  //    the wide items alone have run in rounds, or before the narrow items' K/V has streamed at
  //    5.2 TB/s; the queues alternate the two kinds with the wide list running ahead (kWideLead), and the
  //    launch ends 0.77 of that time and the longest wide item after its start (0.77 is fitted like
  //    the other constants).
  //    Wide items on at most three quarters of the CUs are queued in front instead (below): the
  //    launch cannot end before the longest of them, 7.8 us + 22.6 ns per key from its start.
  //    Next to streaming CUs a wide item takes 10.5 us + 13 ns per key (the clock is higher than
  //    under a chip-wide MFMA load), a narrow span 8 us + 4.1 ns per key, and a partial slot
  //    costs 14.4 ns (its traffic competes with the decodes'), a launch with cut tiles 7 us.
  // The three quarters are counted over the launch here and per queue below:
  // a queue that was dealt more than its share of the wide items interleaves all the same.
  // A lean plan prices cutting as library versions up to 505 did (a merge launch of its own, no span of
  // less than 12 K/V tiles): where that gives fewer partial slots, it fits a workspace sized by those.
  if (wide_cost_total > 0 && wide_tiles <= 2LL * std::max(n_cus, 1)) {
    const int cus = std::max(n_cus, 1);
    struct Costs { double wide_us0, wide_us_key, narrow_us0, narrow_us_key, slot_us, cut_us0; };
    const Costs chunk_dominated = lean ? Costs{8.0, 0.0237, 6.0, 0.012, 0.003, 13.0} : Costs{23.0, 0.025, 8.4, 0.013, 0.0024, 3.0},
                decode_rich = lean ? Costs{10.0, 0.016, 8.0, 0.0067, 0.0206, 4.0} : Costs{10.5, 0.013, 8.0, 0.0041, 0.0144, 7.0},
                at_once = lean ? Costs{10.0, 0.0255, 0.0, 0.0, 0.0, 0.0} : Costs{7.8, 0.0226, 0.0, 0.0, 0.0, 0.0};
    const double hbm_bytes_per_us = 5.24e6, last_wide_start = 0.77, few_decodes_share = lean ? 0.3 : 0.34, whole_rounds = 0.3;
    const int min_cut_piece = (lean ? 12 : 8) * kWideKvTile;
    long long longest = 0, n_narrow = 0, narrow_slots = 0;
    auto count_narrow = [&](long long keys, long long copies) {
      const long long n = std::max<long long>(1, (keys + span - 1) / span) * copies;
      n_narrow += n;
      if (n > copies) narrow_slots += n;
    };
    for (int s = 0; s < n_seqs; ++s) {
      const long long P = prefix_lens[s], C = chunk_lens[s];
      if (C <= 0) continue;
      const long long copies = (long long)Hkv * n_groups;
      if (C * group > kNarrowRows) {
        longest = std::max(longest, P + C);
        const long long rem = C % wide_tok;
        if (rem && rem * group <= kNarrowRows) count_narrow(P + C, copies);
      } else {
        count_narrow(P + C, copies);
      }
    }
    const double kv_elem_bytes = cache->kv_dtype == CRONUS_KV_FP8_E4M3 ? 1.0 : 2.0;
    const double hbm_us = (double)narrow_keys * 2.0 * D * kv_elem_bytes / hbm_bytes_per_us;  // K and V of every narrow key
    // items, summed and longest time of the wide items, and partial slots for a span length
    auto& loads = scratch().loads;  // the items themselves
    struct WideSide { long long items, slots; double total_us, longest_us, longest_keys; };
    auto wide_side = [&](int piece, const Costs& c) {
      WideSide w{0, 0, 0.0, 0.0, 0.0};
      loads.clear();
      for (int s = 0; s < n_seqs; ++s) {
        const long long P = prefix_lens[s], C = chunk_lens[s];
        if (C * group <= kNarrowRows) continue;
        for (long long t0 = 0; t0 < C; t0 += wide_tok) {
          const long long nt = std::min<long long>(wide_tok, C - t0);
          if (nt * group <= kNarrowRows) continue;
          const long long kv_total = P + t0 + nt;
          long long n_split = kv_total > piece + piece / 2 ? (kv_total + piece - 1) / piece : 1;
          const long long per = ((kv_total + n_split - 1) / n_split + kWideKvTile - 1) / kWideKvTile * kWideKvTile;
          n_split = (kv_total + per - 1) / per;
          const double height = nt * group * 2 <= wide_rows ? 0.75 : 1.0;
          const double us = c.wide_us0 + c.wide_us_key * height * (double)per;
          const long long copies = (long long)Hkv * n_groups;
          loads.push_back(Scratch::Load{us, n_split * copies});
          w.items += n_split * copies;
          w.total_us += us * (double)(n_split * copies);
          w.longest_us = std::max(w.longest_us, us);
          w.longest_keys = std::max(w.longest_keys, height * (double)per);
          if (n_split > 1) w.slots += n_split * copies * kWaves;
        }
      }
      return w;
    };
    auto narrow_item_us = [&](const Costs& c) {
      return n_narrow > 0 ? c.narrow_us0 + c.narrow_us_key * (double)narrow_keys / (double)n_narrow : 0.0;
    };
    const WideSide whole = wide_side(1 << 30, chunk_dominated);  // no tile cut
    const bool few_decodes =
        whole.items == 0 || (double)n_narrow * narrow_item_us(chunk_dominated) < few_decodes_share * whole.total_us;
    const Costs& c = few_decodes ? chunk_dominated : decode_rich;
    const double narrow_us = narrow_item_us(c), narrow_total_us = (double)n_narrow * narrow_us;
    double best_us = 0;
    int best_piece = 0;
    long long best_items = -1;
    for (int cut = 1; cut <= 8; ++cut) {
      int piece = (int)((longest + cut - 1) / cut);
      piece = (piece + kWideKvTile - 1) / kWideKvTile * kWideKvTile;
      if (cut > 1 && piece < min_cut_piece) break;
      const WideSide w = wide_side(piece, c);
      if (w.items == 0) break;
      if (cut > 1 && too_large(w.items + n_narrow, w.slots + narrow_slots)) continue;
      const long long rounds = (w.items + cus - 1) / cus;
      const double mean_us = w.total_us / (double)w.items;
      // narrow items that the CUs left free by the last round of wide items take meanwhile
      auto trailing_us = [&]() {
        if (n_narrow == 0) return 0.0;
        const long long last_round = w.items - (rounds - 1) * cus;
        const long long absorbed = (cus - last_round) * (long long)(mean_us / narrow_us);
        const long long left = std::max<long long>(0, n_narrow - absorbed);
        return (double)((left + cus - 1) / cus) * narrow_us;
      };
      auto launch_us = [&](double wide_alone_us) {
        double us;
        if (few_decodes) {
          us = wide_alone_us + trailing_us();
        } else {
          const double floor_us = std::max(std::max((w.total_us + narrow_total_us) / cus, hbm_us), wide_alone_us);
          const double ratio = narrow_total_us / w.total_us;
          if (ratio < 0.3) us = wide_alone_us + trailing_us();
          else if (4 * w.items <= 3 * cus) us = std::max(floor_us, at_once.wide_us0 + at_once.wide_us_key * w.longest_keys);
          else if (ratio <= 10.0) us = std::max(floor_us, last_wide_start * floor_us + w.longest_us);
          else us = std::max(floor_us, w.longest_us);
        }
        return us + c.slot_us * (double)w.slots + (w.slots ? c.cut_us0 : 0.0);
      };
      const double in_rounds_us = (double)(rounds - 1) * mean_us + w.longest_us;
      double us;
      if (rounds > 1 && !lean) {
        auto wide_alone_us = [&](double dealt_us) { return whole_rounds * in_rounds_us + (1.0 - whole_rounds) * dealt_us; };
        if (best_piece > 0 && launch_us(wide_alone_us(std::max(w.total_us / cus, w.longest_us))) >= best_us) continue;
        std::sort(loads.begin(), loads.end(), [](const Scratch::Load& a, const Scratch::Load& b) { return a.us > b.us; });
        us = launch_us(wide_alone_us(list_us(loads, cus)));
      } else {
        us = launch_us(in_rounds_us);
      }
      if (best_piece == 0 || us < best_us) {
        best_us = us;
        best_piece = piece;
        best_items = w.items;
        wide_slots = w.slots;
      }
    }
    if (best_piece > 0) wide_piece_keys = best_piece;
    wide_items = best_items;
  }

  // The narrow items' span again, now that the wide ones are known: where those leave CUs free
  // from the start, the narrow items run in rounds over the rest, and a few items more than a
  // whole number of rounds cost a round.  (Launches of decodes alone keep the one rule above, keys over
  // CUs, which tests/test_plan_spans_cpu.py states.)  Of the spans that give at most
  // four rounds the one with the least rounds x (8 us + its longest item's keys at the share of
  // 5.3 TB/s that each of those CUs gets, 7 ns a key at least) is a candidate, and it is taken if it also ends
  // before the span above when both are dealt out item by item.  (Measured, us a pass: a chunk
  // behind 16 k in 192 spans next to 16 decodes, 248 -> 192 items on the other 64 CUs, 179.5 -> 163.0; two
  // chunks in 144 items next to 10 decodes of 3400, 232 -> 80 items, 97.4 -> 89.2; fp8, a chunk in 192
  // items next to 7 decodes of 4600, 256 -> 128 items, 70.7 -> 67.0; a chunk in 56 tiles next to 52 decodes,
  // 312 -> 384 items, 128.3 -> 125.4.  With more rounds than that the rounding is a small part.)
  constexpr int kMaxRounds = 4;
  const long long free_cus = std::max(n_cus, 1) - wide_items;
  if (!lean && narrow_keys > 0 && wide_items > 0 && 4 * wide_items <= 3LL * std::max(n_cus, 1)) {
    std::vector<float>& rows = scratch().row_keys;
    rows.clear();
    const long long copies = (long long)Hkv * n_groups;
    const size_t most_rows = (size_t)(kMaxRounds * free_cus / copies);
    for (int s = 0; s < n_seqs && rows.size() <= most_rows; ++s) {
      const long long C = chunk_lens[s];
      if (C == 0) continue;
      const long long rem = C * group <= kNarrowRows ? C : C % wide_tok;
      if (rem > 0 && rem * group <= kNarrowRows) rows.push_back((float)((long long)prefix_lens[s] + C));
    }
    if (rows.size() <= most_rows) {
      const double key_bytes = 2.0 * D * (cache->kv_dtype == CRONUS_KV_FP8_E4M3 ? 1.0 : 2.0);
      auto key_us = [&](long long items) { return std::max(0.007, key_bytes * (double)std::min(items, free_cus) / 5.3e6); };
      double best_us = 0;
      long long best_span = 0, best_items = 0, items_now = 0;
      for (int steps = 2; steps <= kMaxSpanSteps; ++steps) {
        const float inv = 1.0f / (float)(steps * kNarrowKvStep);
        float longest = 0.f;
        long long items = 0, slots = 0;
        for (const float keys : rows) {
          const int n = std::max(1, (int)std::ceil(keys * inv - 0.25f));
          items += n;
          if (n > 1) slots += n;
          longest = std::max(longest, keys / (float)n);
        }
        items *= copies;
        if (steps * kNarrowKvStep == span) items_now = items;
        const long long rounds = (items + free_cus - 1) / free_cus;
        if (rounds > kMaxRounds || too_large(wide_items + items, wide_slots + slots * copies)) continue;
        const double us = (double)rounds * (8.0 + key_us(items) * longest);
        if (best_span == 0 || us < best_us) {
          best_us = us;
          best_span = steps * kNarrowKvStep;
          best_items = items;
        }
      }
      if (best_span > 0 && best_span != span && best_items != items_now &&
          rounds_us(rows, copies, best_span, free_cus, key_us(best_items)) < rounds_us(rows, copies, span, free_cus, key_us(items_now)))
        span = best_span;
    }
  }

  Scratch& sc = scratch();
  sc.wide_tok = wide_tok;
  sc.seqs.resize((size_t)n_seqs);
  sc.wide.clear();
  sc.narrow.clear();
  sc.wide_unit.clear();
  sc.narrow_unit.clear();
  sc.wide_cost.clear();
  sc.groups.clear();
  sc.merges.clear();
  sc.stages.clear();
  int64_t n_partials = 0, n_merge_rows = 0, n_stage_blocks = 0;
  int32_t n_merge_groups = 0;
  // fp8 cache: a chunk of many tiles reads each key of its sequence that many times; its
  // K/V is then converted to bf16 once (into the workspace) and the tiles run on the bf16
  // pipeline (measured on the chunks of the 70B-shaped batch: 7.66 -> 6.6 ms of attention).
  // (measured on 70B-shaped iterations, whole call: 16 tiles gain 5 % behind 2 k cached tokens and 14 %
  // behind 32 k; 8 tiles lose 2 % behind 2 k and gain 10 % behind 32 k)
  constexpr int kStageMinTiles = 16, kStageMinTilesLong = 8, kStageLongKeys = 8192;
  constexpr long long kStageMaxBytes = 1LL << 30;  // of workspace for the copy; later sequences convert on the fly
  const long long stage_block_bytes = 2LL * Hkv * kBlock * D * 2;  // K and V of one block, bf16
  const bool fp8 = cache->kv_dtype == CRONUS_KV_FP8_E4M3 && allow_stage;  // candidates for the bf16 copy
  int32_t q_off = 0;

  // More rows to cut than arrival counters: the longest are cut, the others stay whole.  A row
  // that stays whole is then no longer than any of the nearly kMaxMergeGroups that are cut, so
  // it is a small part of a CU's share of the launch (at most 1/15 at 256 CUs), and the queues
  // take such rows first.  (With the counters dealt in batch order, 512 decodes of 8 k keys and
  // a last one of 128 k left that one whole: 2190 -> 3916 us by the time_of estimates below.)
  sc.whole.clear();
  if ((long long)n_seqs * Hkv * n_groups + wide_tiles > kMaxMergeGroups) {
    const long long copies = (long long)Hkv * n_groups;
    long long cut_tiles = 0;
    sc.by_length.clear();
    for (int s = 0; s < n_seqs; ++s) {
      const long long P = prefix_lens[s], C = chunk_lens[s];
      if (C == 0) continue;
      long long narrow_tok = C * group <= kNarrowRows ? C : 0;
      if (narrow_tok == 0)
        for (long long t0 = 0; t0 < C; t0 += wide_tok) {
          const long long nt = std::min<long long>(wide_tok, C - t0);
          if (nt * group <= kNarrowRows) narrow_tok = nt;
          else cut_tiles += wide_piece_keys > 0 && P + t0 + nt > wide_piece_keys + wide_piece_keys / 2;
        }
      if (narrow_tok > 0 && split_of(P + C, span).n > 1) sc.by_length.push_back({(int32_t)-(P + C), s});
    }
    const size_t cuttable = (size_t)(std::max<long long>(0, kMaxMergeGroups - cut_tiles * copies) / copies);
    if (sc.by_length.size() > cuttable) {
      std::nth_element(sc.by_length.begin(), sc.by_length.begin() + (std::ptrdiff_t)cuttable, sc.by_length.end());
      sc.whole.assign((size_t)n_seqs, 0);
      for (size_t i = cuttable; i < sc.by_length.size(); ++i) sc.whole[(size_t)sc.by_length[i].second] = 1;
    }
  }

  // Sequence and keys of every unit, with 16 empty places on either side, for WorkItem::peers (as expand_item finds them).
  const bool past_cache =
      n_groups == 1 && (decode_keys * 2 * Hkv * D * (cache->kv_dtype == CRONUS_KV_FP8_E4M3 ? 1 : 2) >= kPastCacheBytes ||
                        (decode_keys > 0 && products_us(cache, chunk_pairs) >= kPastCacheProductsUs));
  if (past_cache) {
    sc.unit_seq.assign(kPeersBefore, 0);
    sc.unit_keys.assign(kPeersBefore, 0);
    for (int s = 0; s < n_seqs; ++s) {
      const int32_t C = chunk_lens[s];
      for (int32_t t = C; t > 0; t -= wide_tok) {
        sc.unit_seq.push_back(s);
        sc.unit_keys.push_back(prefix_lens[s] + C);
      }
    }
    sc.unit_seq.insert(sc.unit_seq.end(), kPeersBefore, 0);
    sc.unit_keys.insert(sc.unit_keys.end(), kPeersBefore, 0);
  }
  auto peers_of = [&](int32_t s, int32_t unit, int32_t kv_begin, int32_t kv_end) {
    typedef int32_t Four __attribute__((vector_size(16)));
    static_assert(kPeersBefore == 16 && kPeers == 31, "four vectors a side, without the last place");
    const int32_t first_key = peer_column(kv_begin, kv_end) * kBlock;
    const Four places{0, 1, 2, 3}, bits{1, 2, 4, 8};
    Four mask{0, 0, 0, 0};
    for (int v = 0; v < 8; ++v) {
      Four seq, keys;  // of the units 4 v .. 4 v + 3 places from the first (the unit itself is left out)
      const size_t at = (size_t)unit + 4 * v + (v >= 4);
      std::memcpy(&seq, sc.unit_seq.data() + at, sizeof(seq));
      std::memcpy(&keys, sc.unit_keys.data() + at, sizeof(keys));
      mask |= (keys > first_key) & (seq == places + (s + peer_offset(4 * v))) & (bits << 4 * v);
    }
    return (mask[0] | mask[1] | mask[2] | mask[3]) & 0x7fffffff;
  };

  int32_t peers_unit = -1;  // whose spans sc.peers is of: the same for every KV head
  auto add_narrow = [&](int s, int kvh, int head0, int nh, int q_tok0, int n_tok, int kv_total, int32_t unit) {
    const NarrowSplit split = split_of(kv_total, span);
    int n_split = split.n;
    int per_item = split.per;
    if (n_split > 1 && ((!sc.whole.empty() && sc.whole[(size_t)s]) || n_merge_groups == kMaxMergeGroups)) {
      n_split = 1;
      per_item = kv_total;
    }
    const int32_t first_partial = (int32_t)n_partials, merge_key = n_split * kMaxMergeGroups + n_merge_groups;
    if (n_split > 1) {
      ++n_merge_groups;
      sc.merges.push_back(MergeItem{(int32_t)n_partials, n_split, s, kvh, head0, nh, q_tok0, n_tok, 0, n_tok * nh, 1, 0});
      n_merge_rows += (int64_t)n_tok * nh;
    }
    const bool once = past_cache && n_tok == chunk_lens[s];
    if (once && (unit != peers_unit || n_split != (int)sc.peers.size())) {
      peers_unit = unit;
      sc.peers.resize((size_t)n_split);
      for (int i = 0; i < n_split; ++i) sc.peers[(size_t)i] = peers_of(s, unit, i * per_item, std::min(kv_total, (i + 1) * per_item));
    }
    for (int i = 0; i < n_split; ++i) {
      WorkItem w{};
      w.seq = s; w.kv_head = kvh; w.head0 = head0; w.n_heads = nh; w.q_tok0 = q_tok0; w.n_tok = n_tok;
      w.kv_begin = i * per_item;
      w.kv_end = std::min(kv_total, (i + 1) * per_item);
      w.peers = once ? sc.peers[(size_t)i] : -1;
      w.partial = n_split > 1 ? (int32_t)(n_partials++) : -1;
      w.first_partial = first_partial;
      w.merge_key = merge_key;
      w.wide = 0;
      sc.narrow.push_back(w);
      sc.narrow_unit.push_back(unit);
    }
  };

  long long next_unit = 0;
  for (int s = 0; s < n_seqs; ++s) {
    const int P = prefix_lens[s], C = chunk_lens[s];
    sc.seqs[(size_t)s] = SeqInfo{P, C, q_off, (P + C + kBlock - 1) / kBlock};
    q_off += C;
    if (C == 0) continue;
    const int seq_tiles = (C + wide_tok - 1) / wide_tok;
    const int32_t unit0 = (int32_t)std::min<long long>(next_unit, 1 << 30);  // (that many are never used)
    next_unit += (long long)seq_tiles * n_groups;
    for (int kvh = 0; kvh < Hkv; ++kvh) {
      for (int gidx = 0; gidx < n_groups; ++gidx) {
        const int head0 = kvh * G + gidx * group;
        const int nh = std::min(group, G - gidx * group);
        if (C * group <= kNarrowRows) {
          add_narrow(s, kvh, head0, nh, 0, C, P + C, unit0 + gidx);
          continue;
        }
        int32_t wide_tag = 1;
        if (fp8 && (seq_tiles >= kStageMinTiles || (seq_tiles >= kStageMinTilesLong && P + C >= kStageLongKeys))) {
          const int32_t nb = (P + C + kBlock - 1) / kBlock;
          const bool listed = !sc.stages.empty() && sc.stages.back().seq == s;
          if (!listed && (n_stage_blocks + nb) * stage_block_bytes <= kStageMaxBytes) {
            sc.stages.push_back(StageSeq{s, (int32_t)n_stage_blocks, nb, 0});
            n_stage_blocks += nb;
          }
          if (!sc.stages.empty() && sc.stages.back().seq == s) wide_tag = 2 + sc.stages.back().blk0;
        }
        // the tiles of this (sequence, KV head, head group), shortest first
        sc.tiles.clear();
        int max_split = 0;
        for (int t0 = 0; t0 < C; t0 += wide_tok) {
          const int nt = std::min(wide_tok, C - t0);
          if (nt * group <= kNarrowRows) {
            add_narrow(s, kvh, head0, nh, t0, nt, P + t0 + nt, unit0 + gidx * seq_tiles + t0 / wide_tok);
            continue;
          }
          // A tile whose keys alone would keep one CU busy for much longer than a CU's fair
          // share of the whole launch is cut into spans of whole K/V tiles;
          // each span leaves partial results (one slot per wavefront) for the merge.
          const int kv_total = P + t0 + nt;
          const float rows_frac = std::max(0.25f, (float)(nt * nh) / wide_rows);
          int n_split = 1;
          if (wide_piece_keys > 0 && kv_total > wide_piece_keys + wide_piece_keys / 2)
            n_split = (kv_total + wide_piece_keys - 1) / wide_piece_keys;
          if (n_merge_groups == kMaxMergeGroups) n_split = 1;  // no arrival counters left (more cut tiles than any MI355X launch has)
          const int per = ((kv_total + n_split - 1) / n_split + kWideKvTile - 1) / kWideKvTile * kWideKvTile;
          n_split = (kv_total + per - 1) / per;
          const int rows = nt * nh;
          int32_t first_partial = -1;
          const int32_t merge_key = n_split * kMaxMergeGroups + n_merge_groups;
          if (n_split > 1) {
            ++n_merge_groups;
            first_partial = (int32_t)n_partials;
            for (int wv = 0; wv * kNarrowRows < rows; ++wv)
              sc.merges.push_back(MergeItem{first_partial + wv, n_split, s, kvh, head0, nh, t0, nt,
                                            wv * kNarrowRows, std::min(kNarrowRows, rows - wv * kNarrowRows), kWaves, 0});
            n_merge_rows += rows;
            n_partials += (int64_t)n_split * kWaves;
          }
          sc.tiles.push_back(Scratch::Tile{t0, nt, kv_total, n_split, per, first_partial, merge_key, (wide_rows / 128.0f) * rows_frac});
          max_split = std::max(max_split, n_split);
        }
        // One group per span index: the spans i of all tiles of this (sequence, KV head) cover
        // nearly the same keys, so they are queued together (on one XCD, whose L2 then serves
        // the K/V blocks to all of them); different spans share nothing and may go elsewhere.
        for (int i = 0; i < max_split; ++i) {
          Group g{(int32_t)sc.wide.size(), 0, 0.f};
          for (const Scratch::Tile& t : sc.tiles) {
            if (i >= t.n_split) continue;
            WorkItem w{};
            w.seq = s; w.kv_head = kvh; w.head0 = head0; w.n_heads = nh; w.q_tok0 = t.t0; w.n_tok = t.nt;
            w.kv_begin = i * t.per;
            w.kv_end = std::min(t.kv_total, (i + 1) * t.per);
            w.partial = t.n_split > 1 ? t.first_partial + i * kWaves : -1;
            w.first_partial = t.first_partial;
            w.merge_key = t.merge_key;
            w.wide = wide_tag;
            const float cost = (float)(w.kv_end - w.kv_begin) * t.cost_per_key;
            sc.wide.push_back(w);
            sc.wide_unit.push_back(unit0 + gidx * seq_tiles + t.t0 / wide_tok);
            sc.wide_cost.push_back(cost);
            g.cost += cost;
          }
          g.end = (int32_t)sc.wide.size();
          if (g.end > g.begin) sc.groups.push_back(g);
        }
      }
    }
  }

  // Order of the work.  The main kernel's work-groups stay resident (one per CU) and take
  // items from the queue of the XCD they run on, in queue order, and from the other queues
  // once their own is empty (each XCD has its own L2).  The wide tiles of one (sequence, KV
  // head, span) read the same K/V blocks, so they are queued on one XCD, back to back,
  // longest first (they were generated shortest first), where the 32 CUs of that XCD run
  // them side by side and share the blocks through its L2.  Groups go to the least loaded
  // queue, longest group first; narrow items (no reuse), longest first, even out the queues;
  // the two kinds may then be interleaved (below).
  double load[kXcds] = {0};
  for (auto& q : sc.queue) q.clear();
  for (auto& r : sc.runs) r.clear();
  auto least_loaded = [&]() {
    int x = 0;
    for (int i = 1; i < kXcds; ++i) if (load[i] < load[x]) x = i;
    return x;
  };
  std::sort(sc.groups.begin(), sc.groups.end(), [](const Group& a, const Group& b) { return a.cost > b.cost; });
  double wide_total = 0;
  for (const Group& g : sc.groups) wide_total += g.cost;
  const double piece_max = wide_total / (2 * kXcds);  // balance before locality: no piece above half a fair share
  for (const Group& g : sc.groups) {
    const int n_tiles = g.end - g.begin;
    int pieces = piece_max > 0 ? (int)(g.cost / piece_max) + 1 : 1;
    pieces = std::max(1, std::min(pieces, n_tiles));
    for (int pc = 0; pc < pieces; ++pc) {  // contiguous runs of tiles, longest keys first
      const int hi = g.end - (int)((long long)n_tiles * pc / pieces);
      const int lo = g.end - (int)((long long)n_tiles * (pc + 1) / pieces);
      const int x = least_loaded();
      sc.runs[x].push_back(Scratch::Run{(int32_t)sc.queue[x].size(), hi - lo, sc.wide_cost[(size_t)lo]});
      for (int i = hi - 1; i >= lo; --i) {
        sc.queue[x].push_back(i);
        load[x] += sc.wide_cost[(size_t)i];
      }
    }
  }
  // Within a queue the runs are taken in the order of their shortest tile, longest first: the
  // run that ends with the queue's shortest tiles comes last, so the wide items that start
  // last, and decide when the launch ends, are short ones (runs were dealt by total cost, and
  // a run of many medium tiles would otherwise precede one of few long tiles).  Measured on
  // the prefill-heavy batch: 1 % shorter launch, the other batches unchanged.
  for (int x = 0; x < kXcds; ++x) {
    auto& runs = sc.runs[x];
    if (runs.size() < 2) continue;
    std::stable_sort(runs.begin(), runs.end(), [](const Scratch::Run& a, const Scratch::Run& b) { return a.shortest > b.shortest; });
    sc.order.assign(sc.queue[x].begin(), sc.queue[x].end());
    size_t k = 0;
    for (const Scratch::Run& r : runs)
      for (int32_t j = 0; j < r.len; ++j) sc.queue[x][k++] = sc.order[(size_t)(r.begin + j)];
  }
  {  // narrow items by length, longest first: bucket sort on the number of kNarrowKvStep steps
    // (a span has at most kMaxSpanSteps and a quarter; what is longer is a row left whole above,
    // and those, in the first bucket, are sorted by their length)
    const size_t n = sc.narrow.size();
    sc.bucket_start.assign(kMaxSpanSteps + 3, 0);
    auto bucket_of = [&](const WorkItem& w) {
      const int steps = (w.kv_end - w.kv_begin + kNarrowKvStep - 1) / kNarrowKvStep;
      return (size_t)(steps > kMaxSpanSteps + kMaxSpanSteps / 4 ? 0 : kMaxSpanSteps + 1 - std::min(kMaxSpanSteps, steps));
    };
    for (const WorkItem& w : sc.narrow) ++sc.bucket_start[bucket_of(w) + 1];
    for (int b = 0; b <= kMaxSpanSteps + 1; ++b) sc.bucket_start[(size_t)b + 1] += sc.bucket_start[(size_t)b];
    sc.order.resize(n);
    for (size_t i = 0; i < n; ++i) sc.order[(size_t)sc.bucket_start[bucket_of(sc.narrow[i])]++] = (int32_t)i;
    std::stable_sort(sc.order.begin(), sc.order.begin() + sc.bucket_start[0], [&](int32_t a, int32_t b) {
      const WorkItem &x = sc.narrow[(size_t)a], &y = sc.narrow[(size_t)b];
      return x.kv_end - x.kv_begin > y.kv_end - y.kv_begin;
    });
    for (size_t k = 0; k < n; ++k) {
      const int32_t i = sc.order[k];
      const WorkItem& w = sc.narrow[(size_t)i];
      const int x = least_loaded();
      sc.queue[x].push_back(~i);
      load[x] += 0.5 * (w.kv_end - w.kv_begin);
    }
  }
  // Where decode spans are a large part of a queue's work but not nearly all of it (estimated
  // time at least 0.3 of its wide tiles' and at most ten times theirs), the two kinds alternate in proportion to their estimated times, each
  // kind keeping its order: while some CUs of the XCD compute wide tiles (little HBM
  // traffic), the others stream decode spans, and a CU that streams next to computing CUs
  // gets a larger share of the memory system than one that streams next to 255 others.
  // The wide list runs ahead (its share of time emitted is 1 / kWideLead of the spans'), so that it is used up
  // before the queue's last quarter and only spans, the short items, are left for the tail.  Measured on the
  // Llama-3-8B-shaped batch: 12 % shorter step than with the spans last.  (Lead 0.85: that batch 151.7 -> 150.4 us a step, but
  // 108 mixes take 0.5 % more attention time on average, 22 of them more than 2 % and 9 % at most, 5 less by as much.)  Where
  // wide tiles dominate, the spans stay at the end of the queue anyway.
  constexpr double kWideLead = 0.75;
  // A queue whose wide items are at most three quarters of its XCD's CUs keeps them in front:
  // they all start at once and the rest of the CUs stream beside them, and none is left to
  // start late.  (A chunk of 463 tokens behind 2049 next to 49 decodes, 13 wide items a queue:
  // 88.1 us interleaved, 80.0 with the wide items in front; fp8, a chunk of 201 behind 3000
  // next to 48 decodes, 14 a queue: 110.7 -> 102.2; with as many wide items as CUs, the
  // Llama-3-8B-shaped batch, interleaving is the better one.)
  const size_t wide_at_once = (size_t)(3 * std::max(n_cus, 1) / (4 * kXcds));
  for (auto& q : sc.queue) {
    // microseconds per item, fitted to per-work-group timestamps of the Llama-3-8B-shaped
    // batch on MI355X (D = 128, bf16; only the ratio of the two kinds matters here: wide tiles take
    // 15 % less since, which kWideLead was measured with)
    auto time_of = [&](int32_t ref) {
      if (ref >= 0) {
        const WorkItem& w = sc.wide[(size_t)ref];
        return 5.0 + 0.0286 * (w.kv_end - w.kv_begin);
      }
      const WorkItem& w = sc.narrow[(size_t)~ref];
      return 9.6 + 0.0141 * (w.kv_end - w.kv_begin);
    };
    double total[2] = {0, 0}, done[2] = {0, 0};
    size_t n_wide_q = 0;
    for (int32_t ref : q) {
      total[ref < 0] += time_of(ref);
      n_wide_q += ref >= 0;
    }
    if (n_wide_q <= wide_at_once || n_wide_q == q.size() || total[1] < 0.3 * total[0] || total[0] < 0.1 * total[1]) continue;
    sc.order.assign(q.begin(), q.end());  // wide refs first, then narrow refs
    size_t iw = 0, in = n_wide_q, k = 0;
    while (iw < n_wide_q || in < sc.order.size()) {
      const bool take_narrow =
          iw == n_wide_q || (in < sc.order.size() && done[1] * total[0] < kWideLead * done[0] * total[1]);
      const int32_t ref = take_narrow ? sc.order[in++] : sc.order[iw++];
      done[take_narrow] += time_of(ref);
      q[k++] = ref;
    }
  }
  sc.n_units = next_unit;
  const size_t n_slots = sc.wide.size() + sc.narrow.size();
  {
    int32_t base = 0;
    for (int x = 0; x < kQueues; ++x) {
      plan->q_base[x] = base;
      plan->q_len[x] = (int32_t)sc.queue[x].size();
      base += plan->q_len[x];
    }
  }
  plan->n_workgroups = (int32_t)std::min<size_t>(n_slots, (size_t)std::max(n_cus, 1));

  plan->n_seqs = n_seqs;
  plan->past_cache = past_cache;
  plan->wide_rows = wide_rows;
  plan->n_items = (int64_t)n_slots;
  plan->n_wide = (int64_t)sc.wide.size();
  plan->n_partials = n_partials;
  plan->n_merge = (int64_t)sc.merges.size();
  plan->n_merge_rows = n_merge_rows;
  plan->off_items = 0;
  plan->off_merge = align_up(plan->off_items + sizeof(WorkItem) * n_slots, 256);
  plan->n_stage_seqs = (int32_t)sc.stages.size();
  plan->n_stage_blocks = n_stage_blocks;
  plan->off_stage = align_up(plan->off_merge + sizeof(MergeItem) * sc.merges.size(), 256);
  plan->image_bytes = align_up(plan->off_stage + sizeof(StageSeq) * sc.stages.size(), 256);
  plan->off_partials = 0;
  plan->off_stage_k = align_up(plan->off_partials + sizeof(float) * partial_floats(D) * (size_t)n_partials, 256);
  const size_t stage_bytes = (size_t)n_stage_blocks * Hkv * kBlock * D * 2;  // bf16 copy of K (and of V)
  plan->off_stage_v = align_up(plan->off_stage_k + stage_bytes, 256);
  plan->total_bytes = align_up(plan->off_stage_v + stage_bytes, 256);
  if (plan->total_bytes == 0) plan->total_bytes = 256;

  return CRONUS_OK;
}

void write_plan(const Plan* plan, void* host_buf) {
  // copies the work list that the last build_plan() of this thread left in its scratch
  Scratch& sc = scratch();
  unsigned char* h = static_cast<unsigned char*>(host_buf);
  // (the per-sequence records travel inside the work and merge items; the kernels read nothing else)
  WorkItem* wi = reinterpret_cast<WorkItem*>(h + plan->off_items);
  size_t i = 0;
  for (int x = 0; x < kQueues; ++x) {
    for (const int32_t ref : sc.queue[x]) {
      WorkItem w = ref >= 0 ? sc.wide[(size_t)ref] : sc.narrow[(size_t)~ref];
      const SeqInfo& si = sc.seqs[(size_t)w.seq];
      w.prefix_len = si.prefix_len;
      w.chunk_len = si.chunk_len;
      w.q_off = si.q_off;
      if (w.wide) w.n_blocks = si.n_blocks;
      wi[i++] = w;
    }
  }
  if (!sc.merges.empty()) {
    for (MergeItem& mi : sc.merges) mi.q_off = sc.seqs[(size_t)mi.seq].q_off;
    std::memcpy(h + plan->off_merge, sc.merges.data(), sizeof(MergeItem) * sc.merges.size());
  }
  if (!sc.stages.empty()) std::memcpy(h + plan->off_stage, sc.stages.data(), sizeof(StageSeq) * sc.stages.size());
}

bool compact_plan(const cronus_kv_cache* cache, const Plan* plan, CompactPlan* c, void* buf, size_t capacity, size_t* bytes) {
  Scratch& sc = scratch();
  const int Hkv = cache->num_kv_heads, G = cache->num_q_heads / Hkv;
  const int group = std::min(G, kNarrowRows), n_groups = (G + group - 1) / group;
  if (n_groups > 255) return false;
  const long long n_units = sc.n_units;
  if (plan->n_items <= 0 || n_units > (long long)(capacity / sizeof(CompactUnit)) ||
      (unsigned long long)n_units * sizeof(CompactUnit) + 2ull * (unsigned long long)plan->n_items > capacity)
    return false;
  CompactUnit* units = static_cast<CompactUnit*>(buf);
  std::memset(units, 0, (size_t)n_units * sizeof(CompactUnit));
  uint32_t max_split = 1;
  static_assert(kMaxMergeGroups <= 1 << 12, "a merge group fits in 12 bits");
  // the first span of KV head 0 fills a unit, that of KV head 1 shows the steps between heads
  for (const bool wide : {true, false}) {
    const auto& list = wide ? sc.wide : sc.narrow;
    const auto& unit = wide ? sc.wide_unit : sc.narrow_unit;
    for (size_t k = 0; k < list.size(); ++k) {
      const WorkItem& w = list[k];
      if (w.kv_begin != 0 || w.kv_head > 1) continue;
      CompactUnit& u = units[(size_t)unit[k]];
      const SeqInfo& si = sc.seqs[(size_t)w.seq];
      const bool split = w.partial >= 0;
      const uint32_t merge = (uint32_t)(w.merge_key % kMaxMergeGroups), n_split = split ? (uint32_t)(w.merge_key / kMaxMergeGroups) : 1u;
      if (n_split > 0xffu) return false;
      if (w.kv_head == 0) {
        u = CompactUnit{w.seq, si.prefix_len, si.chunk_len, si.q_off,
                        (uint32_t)(w.q_tok0 / sc.wide_tok) | (uint32_t)((w.head0 / group) << 24),
                        (uint32_t)w.kv_end | (w.wide ? 1u << 31 : 0u), split ? (uint32_t)w.first_partial : 0u,
                        (split ? merge : 0u) | n_split << 24};
        max_split = std::max(max_split, n_split);
        if (u.partial > 0xffffu) return false;
      } else if (split) {
        const int64_t dp = (int64_t)w.first_partial - (u.partial & 0xffffu), dm = (int64_t)merge - (u.merge & 0xfffu);
        if (dp < 0 || dp > 0xffff || dm < 0 || dm > 0xfff) return false;
        u.partial |= (uint32_t)dp << 16;
        u.merge |= (uint32_t)dm << 12;
      }
    }
  }
  auto bits_of = [](uint32_t n) {  // the least b with n <= 2^b
    int32_t b = 0;
    while ((uint64_t)1 << b < n) ++b;
    return b;
  };
  const int32_t head_bits = bits_of((uint32_t)Hkv), span_bits = bits_of(max_split);
  if (head_bits + span_bits > 30) return false;
  const unsigned long long numbers = (unsigned long long)n_units << (head_bits + span_bits);
  if (numbers > 0x7fffffffull) return false;
  *c = CompactPlan{(int32_t)plan->n_items, (int32_t)n_units, head_bits, span_bits, group, G, sc.wide_tok,
                   numbers <= 0x10000ull ? 2 : 4, plan->past_cache};
  const size_t off = (size_t)n_units * sizeof(CompactUnit);
  *bytes = align_up(off + (size_t)plan->n_items * c->ref_bytes, 16);
  if (*bytes > capacity) return false;
  unsigned char* refs = static_cast<unsigned char*>(buf) + off;
  size_t i = 0;
  for (int x = 0; x < kQueues; ++x)
    for (const int32_t q : sc.queue[x]) {
      const WorkItem& w = q >= 0 ? sc.wide[(size_t)q] : sc.narrow[(size_t)~q];
      const uint32_t unit = (uint32_t)(q >= 0 ? sc.wide_unit[(size_t)q] : sc.narrow_unit[(size_t)~q]);
      const uint32_t span = w.partial < 0 ? 0u : (uint32_t)(w.partial - w.first_partial) / (q >= 0 ? kWaves : 1);
      const uint32_t ref = (unit << head_bits | (uint32_t)w.kv_head) << span_bits | span;
      const WorkItem e = expand_unit(*c, units[unit], ref);  // (its peers follow from the other units)
      if (e.seq != w.seq || e.kv_head != w.kv_head || e.head0 != w.head0 || e.n_heads != w.n_heads || e.q_tok0 != w.q_tok0 ||
          e.n_tok != w.n_tok || e.kv_begin != w.kv_begin || e.kv_end != w.kv_end || e.partial != w.partial || e.wide != w.wide ||
          (w.partial >= 0 && (e.first_partial != w.first_partial || e.merge_key != w.merge_key)))
        return false;
      if (c->ref_bytes == 2) reinterpret_cast<uint16_t*>(refs)[i++] = (uint16_t)ref;
      else reinterpret_cast<uint32_t*>(refs)[i++] = ref;
    }
  return true;
}

// Whether an iteration places its rows past the caches: where streaming the decodes' K/V takes at least twice as
// long as the products of the chunks, and 20 us.  Such an iteration is bound by the HBM, which then also takes back what
// the scatter left behind; elsewhere the chunk tiles read the rows from the cache.  us a pass, cached / past the
// caches, behind the times of streaming and products.  This side: 4 chunks next to 64 decodes, 95 and 36, 140.3 / 129.8; a chunk next to 49, 41 and 13,
// 69.4 / 65.8; fp8, 53 and 17, 90.1 / 87.0; a chunk of 256 behind 256 next to 24, 33 and 1, 44.5 / 42.5; 512 behind 1500 next to 32, 44 and 12,
// 80.0 / 69.0; fp8, 100 behind 1000 next to 32, 27 and 3, 52.2 / 50.4; decodes alone, whose rows are few, 22 32.2 / 32.1, 27 45.2 / 45.3,
// 38 43.2 / 42.9, 55 72.6 / 72.0.  The other side: 66 and 36 122.6 / 122.6, 105 and 121 226 / 229, 24 and 113 172.3 / 174.2,
// 0 and 771 799 / 808; 8 and 1 32.2 / 32.8.  (A ratio of 1.6, fp8, 55 and 34, still gained: 108.6 / 106.7.)
bool rows_past_cache(const cronus_kv_cache* cache, const int32_t* prefix_lens, const int32_t* chunk_lens, int32_t n_seqs) {
  const int group = std::min(cache->num_q_heads / cache->num_kv_heads, kNarrowRows);
  double stream_us = 0, product_us = 0;
  for (int s = 0; s < n_seqs; ++s) {
    const double P = prefix_lens[s], C = chunk_lens[s];
    if (C * group > kNarrowRows) product_us += C * P + C * (C + 1) / 2;
    else if (C > 0) stream_us += P + C;
  }
  const double elem_bytes = cache->kv_dtype == CRONUS_KV_FP8_E4M3 ? 1 : 2;
  stream_us *= 2.0 * elem_bytes * cache->num_kv_heads * cache->head_dim / 6e6;  // 6 TB/s
  product_us = products_us(cache, product_us);
  return stream_us >= 20 && stream_us >= 2 * product_us;
}

bool rows_in_launch(const cronus_kv_cache* cache, const cronus_kv_rows* first, const cronus_kv_rows* second, const int32_t* prefix_lens,
                    const int32_t* chunk_lens, int32_t n_seqs, int n_cus) {
  if (!first || second || n_seqs > kMaxNewRows) return false;
  if (cache->num_kv_heads > kMaxScatterHeads) return false;  // (the scatter refuses them)
  long long keys = 0;
  int rows = 0;
  for (int s = 0; s < n_seqs; ++s) {
    if (chunk_lens[s] > 1) return false;
    if (chunk_lens[s] == 0) continue;
    ++rows;
    keys += prefix_lens[s] + 1LL;
  }
  if (first->n_tokens != rows || (rows < n_seqs && n_seqs > kPlacingSkippedSeqs)) return false;
  const int q_heads = cache->num_q_heads / cache->num_kv_heads;
  const long long copies = (long long)cache->num_kv_heads * ((q_heads + kNarrowRows - 1) / kNarrowRows);
  return (keys + kPlacingRowKeys * (long long)rows) * copies <= kPlacingKeysPerCu * (long long)n_cus;
}

}  // namespace cronus
