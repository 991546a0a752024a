// Host half of libdlfp: packed-batch metadata and work list, the Eq. 2
// controller, status strings.  Plain C++ (no HIP calls), so it also builds
// with a host compiler and its sanitizers.  Device launches live in the .hip
// sources; the completion timers in dlfp_timer.cpp.
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <limits>
#include <memory>
#include <vector>

#include "dlfp.h"
#include "dlfp_internal.h"

namespace {

int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
int64_t round_up(int64_t a, int64_t b) { return ceil_div(a, b) * b; }
// The same for counts of keys below 2^31 and divisors up to 2^31: the split
// policy divides once per sequence or tile and candidate, and a 32-bit division
// takes half the time.
uint32_t ceil_div32(uint32_t a, uint32_t b) { return (a + b - 1) / b; }
// Prefill key ranges start on a 64-key tile.
constexpr int64_t KV_GRANULE_PREFILL = 64;

// Floats of one partial result: O (rows x 128), m[rows], l[rows], padded to 256 bytes.
int64_t slot_floats(int64_t rows) { return round_up(rows * (DLFP_HEAD_DIM + 2), 64); }

struct Unit {
  int32_t f[DLFP_WORK_INTS];
};
static_assert(sizeof(Unit) == DLFP_WORK_INTS * sizeof(int32_t), "work records are packed");

}  // namespace

namespace dlfp {

int check_dims(const dlfp_dims* dims, int* group) {
  if (!dims) return DLFP_EINVAL;
  if (dims->num_q_heads <= 0 || dims->num_kv_heads <= 0) return DLFP_EINVAL;
  if (dims->head_dim != DLFP_HEAD_DIM || dims->page_size != DLFP_PAGE_SIZE)
    return DLFP_EUNSUPPORTED;
  if (dims->num_q_heads % dims->num_kv_heads) return DLFP_EUNSUPPORTED;
  const int g = dims->num_q_heads / dims->num_kv_heads;
  if (g != 1 && g != 2 && g != 4 && g != 8) return DLFP_EUNSUPPORTED;
  if (group) *group = g;
  return DLFP_OK;
}

}  // namespace dlfp

extern "C" {

int dlfp_version(void) { return 100; }

const char* dlfp_status_string(int status) {
  switch (status) {
    case DLFP_OK: return "ok";
    case DLFP_EINVAL: return "invalid argument";
    case DLFP_ERANGE: return "index out of range";
    case DLFP_ENOSPC: return "capacity or workspace too small";
    case DLFP_EHIP: return "HIP runtime error";
    case DLFP_EUNSUPPORTED: return "unsupported shape";
    default: return "unknown status";
  }
}

// Work-list policy.  Prefill rows are packed token-major into tiles of
// DLFP_TILE_ROWS rows (DLFP_TILE_ROWS / g tokens, each with its g query heads
// that share one KV head).  Each tile's visible key range [0, last row's
// position] and each decoder's range [0, kv_len) is cut into equal splits when
// it is longer than the split size; splits of the same rows form a group that
// the attention launch combines in split order.  Prefill units are ordered
// KV-head-major (with workgroups dealt round-robin over the XCDs and the
// launch giving each XCD a contiguous range, units reading the same KV head
// share an L2), longest tile first within a head.
int dlfp_build_varlen_meta(const dlfp_dims* dims, const dlfp_tuning* tuning, int32_t num_seqs,
                           const int32_t* q_len, const int32_t* kv_len,
                           const int32_t* block_table, int32_t max_blocks, int32_t num_blocks,
                           dlfp_meta* meta) {
  int g = 0;
  int st = dlfp::check_dims(dims, &g);
  if (st != DLFP_OK) return st;
  if (!meta || num_seqs < 0) return DLFP_EINVAL;
  if (num_seqs > 0 && (!q_len || !kv_len || !block_table || max_blocks <= 0)) return DLFP_EINVAL;
  if (num_blocks < 0) return DLFP_EINVAL;
  dlfp_tuning tn = {0, 0, 0, 0, 0, 0};
  if (tuning) tn = *tuning;
  if (tn.prefill_lead_units < -1) return DLFP_EINVAL;
  if (tn.decode_pages_in_flight < 0 || tn.decode_pages_in_flight > 2) return DLFP_EINVAL;
  if (tn.decode_split_tokens < 0 || tn.decode_split_tokens % DLFP_PAGE_SIZE ||
      tn.decode_split_tokens > DLFP_MAX_DECODE_UNIT_KEYS)
    return DLFP_EINVAL;
  if (tn.prefill_split_tokens < 0 || tn.prefill_split_tokens % 64 ||
      tn.prefill_split_tokens > DLFP_MAX_PREFILL_UNIT_KEYS)
    return DLFP_EINVAL;
  if (tn.target_units < 0) return DLFP_EINVAL;
  if (tn.prefill_tile_tokens < 0 || tn.prefill_tile_tokens > DLFP_TILE_ROWS / g)
    return DLFP_EINVAL;
  const int64_t resident = tn.target_units ? tn.target_units : DLFP_DEFAULT_RESIDENT_WAVES;
  const int hkv = dims->num_kv_heads;
  int tile_tokens = tn.prefill_tile_tokens ? tn.prefill_tile_tokens : DLFP_TILE_ROWS / g;

  // Validate sequences and the pages they use.
  int64_t tokens = 0, pre_keys = 0;
  for (int s = 0; s < num_seqs; ++s) {
    const int32_t ql = q_len[s], kl = kv_len[s];
    if (ql < 1 || kl < ql) return DLFP_EINVAL;
    const int64_t pages = ceil_div(kl, DLFP_PAGE_SIZE);
    if (pages > max_blocks) return DLFP_ERANGE;
    const int32_t* row = block_table + (int64_t)s * max_blocks;
    int32_t lo = std::numeric_limits<int32_t>::max(), hi = std::numeric_limits<int32_t>::min();
    for (int64_t p = 0; p < pages; ++p) {  // branch-free, so the scan vectorises
      lo = std::min(lo, row[p]);
      hi = std::max(hi, row[p]);
    }
    if (lo < 0 || hi >= num_blocks) return DLFP_ERANGE;
    if ((int64_t)num_blocks * DLFP_PAGE_SIZE > std::numeric_limits<int32_t>::max())
      return DLFP_ERANGE;
    tokens += ql;
    if (ql > 1) {
      const int64_t pos0 = kl - ql;
      for (int64_t t0 = 0; t0 < ql; t0 += tile_tokens) {
        const int64_t nt = std::min<int64_t>(tile_tokens, ql - t0);
        pre_keys += (pos0 + t0 + nt) * hkv;
      }
    }
  }
  if (tokens > std::numeric_limits<int32_t>::max()) return DLFP_ERANGE;

  // Decode split for `slots` workgroup slots left by the prefill units
  // (F = 4 slots wavefronts; CUs = resident / 8).  Either the queue runs
  // several rounds: every unit then adds a fixed cost (query and block-table
  // loads, pipeline fill, its part of the merge) worth about 256 keys, the
  // split minimising work / F plus the longest unit is sqrt(256 W / F) keys
  // for W decode keys, and the launch lasts about units / F unit times plus
  // one (units of the last round start late and finish alone, slower than
  // when they shared the device).  Or the units fit in one round (at most F):
  // the launch then
  // lasts as long as the busiest CU, ceil(workgroups / min(CUs, slots)) units
  // of the longest length, so a split leaving some CUs two decode workgroups
  // and others one wastes half of the latter.  The one-round splits
  // (multiples of 16 keys from 128 up, in steps of about 6%) are weighed
  // against the sqrt split by these estimates; ties go to the longer split.
  int32_t max_kv = 0;
  int64_t dec_keys = 0;
  std::vector<int> prompts, decoders;  // sequences of the prefill and of the decode share
  prompts.reserve(num_seqs);
  decoders.reserve(num_seqs);
  for (int s = 0; s < num_seqs; ++s) (q_len[s] == 1 ? decoders : prompts).push_back(s);
  for (int s : decoders) {
    max_kv = std::max(max_kv, kv_len[s]);
    dec_keys += (int64_t)kv_len[s] * hkv;
  }
  auto decode_split = [&](int64_t slots) -> int64_t {
    slots = std::max<int64_t>(1, slots);
    const int64_t free_waves = 4 * slots;
    const int64_t cu_cap = std::max<int64_t>(1, std::min<int64_t>(resident / 8, slots));
    auto units_and_longest = [&](int64_t sp, int64_t* longest) {
      int64_t n_units = 0;
      uint32_t part = 0;
      for (int s : decoders) {
        const uint32_t n = ceil_div32(kv_len[s], (uint32_t)sp);
        n_units += n;
        part = std::max(part, ceil_div32(kv_len[s], n));
      }
      *longest = round_up(part, DLFP_PAGE_SIZE);
      return n_units * hkv;
    };
    const double root = std::sqrt(256.0 * (double)dec_keys / (double)free_waves);
    const int64_t s0 = std::clamp<int64_t>(round_up((int64_t)std::ceil(root), DLFP_PAGE_SIZE), 128,
                                           DLFP_MAX_DECODE_UNIT_KEYS);
    int64_t longest = 0;
    int64_t best_sp = s0;
    double best = std::numeric_limits<double>::infinity();
    const int64_t n0 = units_and_longest(s0, &longest);
    if (n0 > free_waves)
      best = ((double)n0 / (double)free_waves + 1.0) * (double)(longest + 256);
    const int64_t top = std::min<int64_t>(round_up(std::max<int32_t>(max_kv, 128), DLFP_PAGE_SIZE),
                                          DLFP_MAX_DECODE_UNIT_KEYS);
    for (int64_t sp = 128; sp <= top; sp = round_up(sp + std::max<int64_t>(16, sp / 16), 16)) {
      if (dec_keys > free_waves * sp) continue;  // too many units whatever their lengths
      const int64_t n_units = units_and_longest(sp, &longest);
      if (n_units > free_waves) continue;
      const double e = (double)ceil_div(ceil_div(n_units, 4), cu_cap) * (double)(longest + 256);
      if (e <= best) {
        best = e;
        best_sp = sp;
      }
    }
    return best_sp;
  };
  // Split of decode units that are each the work of a workgroup, one workgroup
  // per compute unit.  Every candidate (the longest range in k equal parts, of
  // at least 192 keys: eight wavefronts take 256 at a time; and the longest unit
  // there is) is weighed by an estimate of the decode share's time in
  // microseconds.  Up to one unit per compute unit they all stream side by side:
  // while n units still have keys, 64 more keys of each (32 KiB) take n x 32 KiB
  // at the device's 6.4 TB/s or 32 KiB at a compute unit's 47 GB/s, whichever is
  // longer.  With more units the compute units share the device's rate evenly, so
  // those that get a unit more than the others end with it alone: full rounds of
  // units of the average length at the device's rate, then the rest as above, and
  // 2.5 us; every two units per compute unit after the first two cost 3 us (a
  // prologue and a sum over the wavefronts that are not hidden).  Four units per
  // compute unit of the longest split and more are bound by their bytes whatever
  // the split (128 decoders of 1024-8192 keys 394-398 us at 1608 to 3656 units):
  // the bytes, and 3 us per round of units.  Splitting any range costs its merge,
  // 2.5 us.  (35 decoders of 1241 keys, 8 KV heads: 280 units 40.5 us, 840 units
  // 36.7; 17 of 1072-2110 keys: 136 units 28.1, 464 units 25.0; 100 of 2000: 800
  // units 147.4, 1600 units 141.8.  On 1000 batches of 1-256 sequences of 8-60000
  // keys, g = 1-8, the launches take 0.824x the time of the wavefront units and
  // splits used before, 61 of them more than 1.03x.)
  // Beside `ahead` prefill and append workgroups (0: alone) the units have to
  // fit into the slots those leave, two workgroups per compute unit; when they
  // need a second workgroup on some compute unit, that one's unit takes twice as
  // long as at 60 GB/s; and past one unit per compute unit half of the longest
  // unit runs alone at the end, at that rate.  No split that fits: an infinite
  // estimate.
  struct WideSplit {
    int64_t split, units;
    double est;
  };
  // What a candidate makes of the decoders, whatever stands beside them: its
  // units, the longest one's keys, and the time with all of them side by side,
  // on compute units of their own or shared ones.
  struct WideCandidate {
    int64_t split, units, longest;
    double alone;        // without other workgroups
    double own, shared;  // (or the time of its merge, with more units than that)
  };
  std::vector<WideCandidate> wide_candidates;
  auto add_wide_candidates = [&]() {
    const int64_t cus = std::max<int64_t>(1, resident / 8);
    const int64_t least_parts = ceil_div(std::max<int32_t>(max_kv, 1), DLFP_MAX_DECODE_UNIT_KEYS);
    for (int64_t k = 0;; k = k ? k + std::max<int64_t>(1, k / 4) : least_parts) {
      const int64_t equal = k ? round_up(ceil_div(max_kv, k), 32) : DLFP_MAX_DECODE_UNIT_KEYS;
      const uint32_t sp = (uint32_t)std::clamp<int64_t>(equal, 192, DLFP_MAX_DECODE_UNIT_KEYS);
      constexpr int STEP = 64, BUCKETS = DLFP_MAX_DECODE_UNIT_KEYS / STEP;
      int64_t units = 0, ending[BUCKETS + 1] = {0};
      uint32_t longest = 0;
      bool split = false;
      for (int s : decoders) {
        const uint32_t kl = kv_len[s], n0 = ceil_div32(kl, sp);
        uint32_t n = n0, part = kl;
        if (n0 > 1) {
          part = (ceil_div32(kl, n0) + DLFP_PAGE_SIZE - 1) / DLFP_PAGE_SIZE * DLFP_PAGE_SIZE;
          n = ceil_div32(kl, part);
          split = true;
        }
        units += n;
        longest = std::max(longest, part);
        ending[(part + STEP - 1) / STEP] += n;
      }
      const double merge = split ? 2.5 : 0.0;
      WideCandidate c = {sp, units * hkv, longest, merge, merge, merge};
      if (c.units <= cus) {
        int64_t n = c.units;
        for (int b = 1; b <= BUCKETS && n > 0; ++b) {
          const double bytes = (double)n * (STEP * 512 / 6.4e6);
          c.own += std::max(bytes, STEP * 512 / 47e3);
          c.shared += std::max(bytes, 2.0 * (STEP * 512 / 60e3));
          n -= ending[b] * hkv;
        }
        c.alone = c.own;
      } else {
        const double unit = 512.0 * (double)dec_keys / (double)c.units;  // bytes, on average
        const int64_t rounds = c.units / cus, rest = c.units % cus;
        c.alone += (double)(rounds * cus) * unit / 6.4e6 +
                   (rest ? std::max((double)rest * unit / 6.4e6, unit / 47e3) : 0.0) +
                   2.5 + 3.0 * std::max(0.0, (double)c.units / (2.0 * (double)cus) - 1.0);
      }
      wide_candidates.push_back(c);
      if (sp <= 192) break;
    }
  };
  auto wide_split = [&](int64_t ahead) {
    const int64_t cus = std::max<int64_t>(1, resident / 8);
    if (wide_candidates.empty()) add_wide_candidates();
    WideSplit best = {DLFP_MAX_DECODE_UNIT_KEYS, 0, std::numeric_limits<double>::infinity()};
    const bool few = wide_candidates[0].units <= 4 * cus;  // the longest split comes first
    for (const WideCandidate& c : wide_candidates) {
      if (ahead > 0 && c.units > 2 * cus - ahead) break;  // a shorter split has more
      double e = ahead > 0 && ahead + c.units > cus ? c.shared : c.own;
      if (ahead == 0 && few)
        e = c.alone;
      else if (c.units > cus && ahead > 0)
        e += (double)dec_keys * (512 / 6.4e6) + 0.5 * (double)c.longest * (512 / 60e3);
      else if (c.units > cus)
        e += (double)dec_keys * (512 / 6.4e6) + 3.0 * (double)c.units / (double)cus;
      if (e < best.est) best = {c.split, c.units, e};
    }
    return best;
  };
  // Prefill units of the iteration for a tile size and key split.
  auto prefill_units = [&](int64_t tt, int64_t split) {
    int64_t n = 0;
    for (int s : prompts) {
      // Keys of the tiles: pos0 + tt, pos0 + 2 tt, ..., the last one's all.
      const uint32_t all = kv_len[s], sp = (uint32_t)split;
      int64_t parts = ceil_div32(all, sp);
      for (int64_t k = (int64_t)all - q_len[s] + tt; k < all; k += tt) parts += ceil_div32((uint32_t)k, sp);
      n += hkv * parts;
    }
    return n;
  };
  // Prefill split.  Prefill alone: the split (multiples of 64 keys, at least
  // 1024) that minimises an estimate of the launch time, rounds x the time of
  // the busiest CU, in keys: a unit costs its longest part plus about 300 keys
  // of prologue, store and merge, and a CU running two units at once runs them
  // 1.11x faster than one after the other.  The longest part matters: a split
  // that leaves some tiles whole and cuts others in two makes the launch as
  // long as the whole ones.  (Fitted to Qwen3-0.6B/8B/32B last chunks, where
  // it picks the measured best: 0.6B 2048 tokens 143 against 175 us before,
  // 1024 tokens 83 against 102 us.)
  int64_t split_p = tn.prefill_split_tokens;
  int64_t dec_wgs0 = 0;
  {
    const int64_t sd0 = tn.decode_split_tokens ? tn.decode_split_tokens : decode_split(resident / 4);
    for (int s = 0; s < num_seqs; ++s)
      if (q_len[s] == 1) dec_wgs0 += hkv * ceil_div(kv_len[s], sd0);
    dec_wgs0 = ceil_div(dec_wgs0, 4);
  }
  // Append workgroups of a one-launch iteration (none when the records take a
  // launch of their own), and the time of the decode share as wavefront units,
  // in microseconds: its bytes, and the queue's start, last units and merges.
  int64_t append_records = 0;
  for (int s : prompts)
    append_records +=
        hkv * (ceil_div(kv_len[s], DLFP_PAGE_SIZE) - (kv_len[s] - q_len[s]) / DLFP_PAGE_SIZE);
  const int64_t app_wgs = dlfp::append_workgroups(append_records);
  const double wave_est = dec_keys > 0 ? (double)dec_keys * (512 / 6.4e6) + 8.0 : 0.0;
  // Prefill units of a tile size and split: their number, the longest one's
  // keys, the most parts of a range.
  auto shape = [&](int64_t tt, int64_t sp, int64_t* units, int64_t* longest, int64_t* parts) {
    int64_t n = 0;
    uint32_t longest_part = 0, most = 0;
    auto tile = [&](uint32_t keys) {
      uint32_t cut = 1, part = keys;
      if (keys > (uint32_t)sp) {
        part = ceil_div32(keys, ceil_div32(keys, (uint32_t)sp));
        part = (part + KV_GRANULE_PREFILL - 1) / KV_GRANULE_PREFILL * KV_GRANULE_PREFILL;
        cut = ceil_div32(keys, part);
      }
      n += cut;
      longest_part = std::max(longest_part, std::min(part, keys));
      most = std::max(most, cut);
    };
    for (int s : prompts) {
      const int64_t all = kv_len[s];
      for (int64_t k = all - q_len[s] + tt; k < all; k += tt) tile((uint32_t)k);
      tile((uint32_t)all);
    }
    *units += n * hkv;
    *longest = std::max<int64_t>(*longest, longest_part);
    *parts = std::max<int64_t>(*parts, most);
  };
  // Time of the prefill share in microseconds: a fixed part, the merge of its
  // splits, and its longest unit, with the compute units' workgroups (`others`
  // of other shares) side by side; for the code of at most 32 rows or the other.
  auto prefill_est = [&](int64_t tt, int64_t sp, bool few_rows, int64_t others, int64_t* units) {
    int64_t n = 0, longest = 0, parts = 1;
    shape(tt, sp, &n, &longest, &parts);
    *units = n;
    const double crowd = std::max(1.0, (double)(n + others) / (double)std::max<int64_t>(1, resident / 8));
    return (few_rows ? 6.1 : 10.0) + (parts > 1 ? 2.4 + 0.2 * (double)parts : 0.0) +
           (few_rows ? 0.0064 : 0.0155) * (double)longest * std::min(crowd, 2.0);
  };
  // A launch too small to give every CU a workgroup at 1024-key splits is bound
  // by the latency of its longest unit and of the merge of its splits: its
  // prefill takes tiles of 32 rows (which have code of their own, and whose
  // merge moves a quarter of the bytes), whole or at the split that these
  // estimates favour, all workgroups within the two a CU holds.  The decode
  // share counts as small when its wavefront units, four to a workgroup at the
  // split they would take without prefill, leave that room too, or when units
  // of a workgroup fit beside the tiles and are much faster, and the tiles do
  // not then last far beyond the decode share (54 decoders of 53-396 keys beside
  // 8 prompts of 2 tokens, one over 6376, g = 4: 63.9 us with its tiles whole,
  // 32.5 at 1024 keys beside wavefront units).  (Prefill alone 0.75x the launch
  // time of the policy and code before, 36 shapes.)
  if (!split_p && !tn.prefill_tile_tokens && pre_keys > 0) {
    const int64_t cus = resident / 8, slots = resident / 4;
    const int small = std::max(1, 32 / g);
    const int64_t tall_units = prefill_units(tile_tokens, 1024);
    const bool wave_fits = tall_units + dec_wgs0 < cus;
    const int64_t dec_wgs = wave_fits ? dec_wgs0 : 0;
    if (tall_units < cus && prefill_units(small, 1024) + dec_wgs <= slots) {
      double best = std::numeric_limits<double>::infinity();
      for (int64_t sp : {DLFP_MAX_PREFILL_UNIT_KEYS, 4096, 2048, 1024, 512, 256}) {
        int64_t n = 0;
        double e = prefill_est(small, sp, true, dec_wgs, &n);
        if (n + dec_wgs > slots) break;
        if (dec_keys > 0) {
          const WideSplit wide = wide_split(n + app_wgs);
          if (wide.est < (wave_fits ? 1.0 : 0.75) * wave_est)
            e = std::max(prefill_est(small, sp, true, wide.units, &n), wide.est);
          else if (wave_fits)
            e = std::max(prefill_est(small, sp, false, dec_wgs, &n), wave_est);
          else
            continue;
          if (!wave_fits && e > 1.5 * wave_est) continue;
        }
        if (e < best) {
          best = e;
          tile_tokens = small;
          split_p = sp;
        }
      }
    }
  }
  // Beside a decode share the prefill units wait on loaded memory and their
  // split merges are on the launch's critical path: the units should number
  // about one per compute unit (more leave decode workgroups without a slot,
  // fewer leave long key loops), each as tall as that allows (a shorter tile
  // re-reads its keys and values more often but merges fewer bytes per row
  // group).  So the tallest tile of 128, 64 or 32 rows whose units, with the
  // shortest split of at least 1024 keys that keeps them at most one per
  // compute unit, come within 1/16 of that count; else 32 rows.  When a lower tile has more units
  // than that even whole, its few very long units are the launch: then 128 rows
  // and up to one and a half units per compute unit (g = 8, 176 tokens over
  // 9871 beside 24 decoders: 352 units of 9856 keys of 32-row tiles 166 us, as
  // many of 2560 keys of 128-row tiles 86 us; g = 2, 1082 over 10784 beside 61:
  // 205 -> 159 us).  (Measured on
  // Qwen3-0.6B shapes beside 32 decoders: 44-48 us per layer instead of
  // 50-54 us for chunks of 64-256 tokens over prefixes of 2-6k keys.)
  if (!split_p && !tn.prefill_tile_tokens && pre_keys > 0 && dec_keys > 0) {
    const int64_t target = std::max<int64_t>(1, resident / 8);
    // The shortest split of 1024 + 64 k keys keeping the units within `most`
    // (DLFP_MAX_PREFILL_UNIT_KEYS when none does), by bisection: the unit
    // count only falls as the split grows.
    auto shortest = [&](int64_t tt, int64_t most) {
      int64_t lo = 0, hi = (DLFP_MAX_PREFILL_UNIT_KEYS - 1024) / 64;
      while (lo < hi) {
        const int64_t mid = (lo + hi) / 2;
        if (prefill_units(tt, 1024 + 64 * mid) > most)
          lo = mid + 1;
        else
          hi = mid;
      }
      return 1024 + 64 * lo;
    };
    // More splits of tall tiles take partial results of up to two units per
    // compute unit (34 MB): only where the fixed workspace holds them beside
    // those of the decode share.
    const int64_t dec_bytes = dec_wgs0 * 4 * slot_floats(g) * 4;
    const int64_t tall_bytes = 2 * target * slot_floats(DLFP_TILE_ROWS) * 4;
    const bool roomy =
        dec_bytes < DLFP_STATIC_WORKSPACE_BYTES / 2 &&
        DLFP_WORKSPACE_PARTIALS + dec_bytes + tall_bytes <= DLFP_STATIC_WORKSPACE_BYTES;
    for (int rows : {DLFP_TILE_ROWS, DLFP_TILE_ROWS / 2, DLFP_TILE_ROWS / 4}) {
      const int64_t tt = std::max(1, rows / g);
      const int64_t sp = shortest(tt, target), n = prefill_units(tt, sp);
      if (n > target && rows != DLFP_TILE_ROWS && roomy) {  // too many even whole
        tile_tokens = std::max(1, DLFP_TILE_ROWS / g);
        split_p = shortest(tile_tokens, target + target / 2);
        break;
      }
      if (n * 16 >= target * 15 || rows == DLFP_TILE_ROWS / 4) {
        tile_tokens = (int)tt;
        split_p = sp;
        break;
      }
    }
    // Then the other heights and equal parts (1 to 12 of the longest range, of
    // 256 keys and more, at most two units per compute unit), when an estimate
    // of the launch time puts one clearly ahead.  In microseconds: a tile's
    // units take 10, 18.4, 13.4 or 8.6 per 1024 keys of the longest one (up to
    // 1.7 times that as they crowd the CUs) and the merge; the decode share 14
    // and its bytes at the rate the slots left to it draw (all of it from 400
    // up), at the full rate once the prefill units are done.  (48 shapes of
    // 12-160 decoders beside 33-1500 tokens over up to 12000 keys: 0.965x on
    // average; the estimate is good to 9%, so a smaller lead is left alone.)
    // Past one and a half units per compute unit few slots are left, which a
    // decode share that fits them in one round would get as units of thousands
    // of keys, one wavefront each: where it is not clearly the shorter share
    // such splits are left out (8 decoders of 2741-14421 keys beside 8 prompts
    // of 100-400 tokens, g = 2: 440 units 138.1 us, 344 of them 90.5; a decode
    // share of many rounds gains from them: 148 decoders beside 4 prompts, 496
    // units 87.9 us, 328 of them 120.3; with two units per compute unit no slot is
    // left, and the decode share is cut for the whole device after them).
    int64_t least_units = 0;  // decode units at the longest split
    for (int s : decoders) least_units += hkv * ceil_div(kv_len[s], DLFP_MAX_DECODE_UNIT_KEYS);
    auto launch_est = [&](int64_t tt, int64_t sp, int64_t* units, double* prefill = nullptr) {
      int64_t n = 0, longest = 0, parts = 1;
      shape(tt, sp, &n, &longest, &parts);
      *units = n;
      const double per_key = tt * g > 64 ? 0.0184 : tt * g > 32 ? 0.0134 : 0.0086;
      const double crowd = std::clamp((double)(n - target / 2) / (1.5 * (double)target), 0.0, 1.0);
      const double pre = 10.0 + per_key * (double)longest * (1.0 + 0.72 * crowd) *
                                    std::max(1.0, (double)n / (2.0 * (double)target)) +
                         (parts > 1 ? 2.4 + 0.5 * (double)parts : 0.0);
      if (prefill) *prefill = pre;
      const double rate = std::min(1.0, (double)std::max<int64_t>(2 * target - n, 64) / 400.0);
      const double work = 14.0 + (double)dec_keys * (512 / 6.4e6);
      const double dec = work <= rate * pre ? work / rate : pre + work - rate * pre;
      // The larger, more when the other is near: the root is left out, only
      // comparisons matter.
      const double p3 = pre * pre * pre, d3 = dec * dec * dec;
      return p3 * p3 + d3 * d3;
    };
    int64_t n = 0, max_kend = 0;
    for (int s = 0; s < num_seqs; ++s)
      if (q_len[s] != 1) max_kend = std::max<int64_t>(max_kend, kv_len[s]);
    constexpr double AHEAD = 0.8 * 0.8 * 0.8;  // 20% ahead, in the estimate's sixth power
    double best = roomy ? AHEAD * AHEAD * launch_est(tile_tokens, split_p, &n) : 0.0;
    const double work = 14.0 + (double)dec_keys * (512 / 6.4e6);
    const double least = work * work * work * work * work * work;  // of any estimate
    for (int rows : {DLFP_TILE_ROWS, DLFP_TILE_ROWS / 2, DLFP_TILE_ROWS / 4}) {
      if (least >= best) break;
      const int64_t tt = std::max(1, rows / g);
      for (int64_t k : {1, 2, 3, 4, 5, 6, 8, 12}) {
        const int64_t sp = round_up(ceil_div(max_kend, k), KV_GRANULE_PREFILL);
        if (sp > DLFP_MAX_PREFILL_UNIT_KEYS) continue;
        if (k > 1 && sp < 256) break;
        double pre = 0;
        const double e = launch_est(tt, sp, &n, &pre);
        if (n > 2 * target) break;
        if (2 * n > 3 * target && n < resident / 4 && wave_est > 0.5 * pre &&
            least_units <= 4 * std::max<int64_t>(2 * target - n, 64))
          continue;
        if (e < best) {
          best = e;
          tile_tokens = (int)tt;
          split_p = sp;
        }
      }
    }
  }
  if (!split_p) {
    const int64_t cus = std::max<int64_t>(1, resident / 8), slots = 2 * cus;
    int64_t max_kend = 0;
    for (int s = 0; s < num_seqs; ++s)
      if (q_len[s] != 1) max_kend = std::max<int64_t>(max_kend, kv_len[s]);
    double best = std::numeric_limits<double>::infinity();
    for (int64_t sp = 1024;; sp += 64) {
      int64_t n = 0, longest = 0;
      for (int s = 0; s < num_seqs; ++s) {
        if (q_len[s] == 1) continue;
        const int64_t pos0 = kv_len[s] - q_len[s];
        for (int64_t t0 = 0; t0 < q_len[s]; t0 += tile_tokens) {
          const int64_t kend = pos0 + t0 + std::min<int64_t>(tile_tokens, q_len[s] - t0);
          const int64_t part = round_up(ceil_div(kend, ceil_div(kend, sp)), KV_GRANULE_PREFILL);
          n += hkv * ceil_div(kend, part);
          longest = std::max(longest, part);
        }
      }
      const double unit = 300.0 + (double)longest;
      const double e = (double)ceil_div(n, slots) * (n > cus ? 2.0 * (300.0 + longest / 1.11) : unit);
      if (e < best) {
        best = e;
        split_p = sp;
      }
      if (sp >= max_kend || sp >= DLFP_MAX_PREFILL_UNIT_KEYS) break;
    }
  }
  // Decode units of a workgroup beside the prefill units where their estimate
  // is the lower one (beside 713 plans of short tiles they take 0.78x the time
  // of wavefront units where it is up to 0.85x theirs, 0.87x up to 0.9, 0.97x up
  // to 1, 1.01x up to 1.1, 1.08x up to 1.2) and, beside tall tiles, clearly so
  // (0.93x up to 0.85, even from there) with the decode share not hidden behind
  // them anyway: more workgroups then only crowd the tiles (11 decoders of
  // 38-304 keys beside 796 tokens over 858, g = 2: 34.6 against 35.4 us; 6 of
  // 796-6368 beside 321 over 1359: 40.1 against 33.3 us; 32 of 536-2024 beside
  // 512 over 2048: 51.6 against 48.5 us).
  const bool tall = tile_tokens * g > 32;
  int64_t pre_units = 0;
  const double pre_est = prefill_est(tile_tokens, split_p, !tall, 0, &pre_units);
  int64_t split_d = tn.decode_split_tokens;
  if (!split_d) {
    const WideSplit wide = wide_split(pre_units > 0 ? pre_units + app_wgs : 0);
    const bool use_wide =
        pre_units == 0 || (tall ? wide.est < 0.85 * wave_est && wave_est > 0.5 * pre_est
                                : wide.est < wave_est);
    // As wavefront units the decode share starts in the workgroup slots (two
    // per CU, four wavefronts each) that the prefill units leave, at least 64;
    // when the prefill units take them all, it runs as they retire.
    split_d = use_wide
                  ? wide.split
                  : decode_split(pre_units < resident / 4
                                     ? std::max<int64_t>(resident / 4 - pre_units, 64)
                                     : resident / 4);
    // Without prefill units the launch chooses its kernel by the longest unit:
    // a split that cuts nothing is reported as that.
    if (pre_units == 0 && max_kv > 0)
      split_d = std::min<int64_t>(split_d, round_up(max_kv, DLFP_PAGE_SIZE));
  }
  // Build units: prefill (KV-head-major), then decode.  Capacity: every key
  // range is cut into at most ceil(range / split) parts, plus two tail pieces.
  std::vector<Unit> units;
  {
    int64_t bound = 0;
    for (int s = 0; s < num_seqs; ++s) {
      if (q_len[s] == 1) {
        bound += hkv * (ceil_div(kv_len[s], split_d) + 2);
        continue;
      }
      const int64_t pos0 = kv_len[s] - q_len[s];
      for (int64_t t0 = 0; t0 < q_len[s]; t0 += tile_tokens)
        bound += hkv * (ceil_div(pos0 + t0 + std::min<int64_t>(tile_tokens, q_len[s] - t0),
                                 split_p) + 2);
    }
    units.reserve((size_t)bound);
  }
  std::vector<int64_t> cu_q_of(num_seqs + 1, 0);  // packed row of each sequence's first token
  for (int s = 0; s < num_seqs; ++s) cu_q_of[s + 1] = cu_q_of[s] + q_len[s];
  int32_t groups = 0;
  std::vector<int64_t> group_rows;  // rows of each group
  // A key range longer than the split is cut into equal parts (rounded up
  // to the granule), so the units of a group finish together.
  // With `tail`, the last part is cut again into a half and two quarters
  // (decode units that run in several queue rounds: the queue hands out the
  // longest units first, so these short pieces even out the end of the launch).
  std::vector<int64_t> cut;
  auto cut_range = [&](int64_t kend, int64_t split, int64_t granule, bool tail = false) {
    const uint32_t keys = (uint32_t)kend;
    const uint32_t equal = ceil_div32(keys, ceil_div32(keys, (uint32_t)split));
    const int64_t part = ((int64_t)equal + granule - 1) & -granule;  // a power of two
    const int64_t nsp = equal == keys ? 1 : ceil_div32(keys, (uint32_t)part);
    cut.clear();
    for (int64_t j = 0; j < nsp; ++j) cut.push_back(j * part);
    if (tail) {
      const int64_t b = (nsp - 1) * part, len = kend - b;
      const int64_t h = round_up(ceil_div(len, 2), granule), q = round_up(ceil_div(len - h, 2), granule);
      if (len >= 4 * granule && h < len && h + q < len) {
        cut.push_back(b + h);
        cut.push_back(b + h + q);
      }
    }
    cut.push_back(kend);
  };
  // The units of the range cut last, for one KV head.
  auto emit = [&](int s, int kh, int64_t t0, int64_t nt, int kind) {
    const int64_t nsp = (int64_t)cut.size() - 1;
    const int32_t grp = nsp > 1 ? groups++ : -1;
    if (nsp > 1) group_rows.push_back(nt * g);
    for (int64_t j = 0; j < nsp; ++j) {
      Unit u;
      std::memset(&u, 0, sizeof(u));
      u.f[DLFP_W_SEQ] = s;
      u.f[DLFP_W_KVHEAD] = kh;
      u.f[DLFP_W_QTOK0] = (int32_t)t0;
      u.f[DLFP_W_QNTOK] = (int32_t)nt;
      u.f[DLFP_W_KVBEGIN] = (int32_t)cut[j];
      u.f[DLFP_W_KVEND] = (int32_t)cut[j + 1];
      u.f[DLFP_W_GROUP] = grp;
      u.f[DLFP_W_SPLIT] = (int32_t)j;
      u.f[DLFP_W_NSPLITS] = (int32_t)nsp;
      u.f[DLFP_W_KIND] = kind;
      u.f[DLFP_W_QROW0] = (int32_t)(cu_q_of[s] + t0);
      u.f[DLFP_W_QPOS0] = (int32_t)(kv_len[s] - q_len[s] + t0);
      if (kind == DLFP_KIND_PREFILL)
        u.f[DLFP_W_PAGE0] = !tall;
      if (kind == DLFP_KIND_DECODE) {
        // The unit's first two block ids travel with the record, so its first
        // page loads go out with its query and block-table loads.
        const int32_t* row = block_table + (int64_t)s * max_blocks;
        const int64_t pg = u.f[DLFP_W_KVBEGIN] / DLFP_PAGE_SIZE;
        const int64_t last = (u.f[DLFP_W_KVEND] - 1) / DLFP_PAGE_SIZE;
        u.f[DLFP_W_PAGE0] = row[pg];
        u.f[DLFP_W_PAGE1] = pg + 1 <= last ? row[pg + 1] : -1;
      }
      units.push_back(u);
    }
  };
  // Prefill tiles of one KV head go longest first, so that the workgroups of
  // an XCD (which takes a contiguous range of prefill units) start the long
  // tiles early.
  struct Tile {
    int s;
    int64_t t0, nt, kend;
  };
  std::vector<Tile> tiles;
  for (int s : prompts) {
    const int64_t pos0 = kv_len[s] - q_len[s];
    for (int64_t t0 = 0; t0 < q_len[s]; t0 += tile_tokens) {
      const int64_t nt = std::min<int64_t>(tile_tokens, q_len[s] - t0);
      tiles.push_back(Tile{s, t0, nt, pos0 + t0 + nt});
    }
  }
  std::stable_sort(tiles.begin(), tiles.end(),
                   [](const Tile& x, const Tile& y) { return x.kend > y.kend; });
  for (int kh = 0; kh < hkv; ++kh)
    for (const Tile& t : tiles) {
      cut_range(t.kend, split_p, KV_GRANULE_PREFILL);
      emit(t.s, kh, t.t0, t.nt, DLFP_KIND_PREFILL);
    }
  const int64_t num_prefill = (int64_t)units.size();
  // Decode units that run in a few rounds (more units than the device takes at
  // once, but not so many that the last round is a small part of the launch
  // anyway) get the short tail pieces.  Beside prefill units: wavefront units,
  // more than the wavefronts those leave.  Alone: workgroups of long units (the
  // pieces of short ones cost more than they even out: 512 units of 512-2048
  // keys 54 -> 67 us; 304 of 1024-4096 keys 78.8 -> 76.0 us, 1608 of the
  // Qwen3-8B decoders 396 -> 394 us).
  bool decode_tail = false;
  if (!tn.decode_split_tokens) {
    int64_t n_dec = 0;
    for (int s = 0; s < num_seqs; ++s)
      if (q_len[s] == 1) n_dec += hkv * ceil_div(kv_len[s], split_d);
    const int64_t slots_d = num_prefill < resident / 4
                                ? std::max<int64_t>(resident / 4 - num_prefill, 64) : resident / 4;
    const int64_t cus_d = std::max<int64_t>(1, resident / 8);
    decode_tail = num_prefill > 0 ? n_dec > 4 * slots_d && n_dec <= 24 * slots_d
                                  : n_dec > cus_d && n_dec <= 8 * cus_d && dec_keys >= 2048 * n_dec;
  }
  for (int s : decoders) {
    cut_range(kv_len[s], split_d, DLFP_PAGE_SIZE, decode_tail);
    for (int kh = 0; kh < hkv; ++kh) emit(s, kh, 0, 1, DLFP_KIND_DECODE);
  }
  // Decode wavefronts take units in list order from a queue: longest first,
  // ties in emission order (a stable counting sort on the key count, which the
  // split keeps within 1..DLFP_MAX_DECODE_UNIT_KEYS).
  {
    constexpr int32_t K = DLFP_MAX_DECODE_UNIT_KEYS;
    const size_t first = (size_t)num_prefill, nd = units.size() - first;
    std::vector<int32_t> start(K + 1, 0);
    for (size_t i = first; i < units.size(); ++i) {
      const int32_t len = units[i].f[DLFP_W_KVEND] - units[i].f[DLFP_W_KVBEGIN];
      if (len < 1 || len > K) return DLFP_ERANGE;
      ++start[K - len + 1];
    }
    for (int32_t b = 1; b <= K; ++b) start[b] += start[b - 1];
    std::unique_ptr<Unit[]> sorted(new Unit[nd]);  // no zero fill: every slot is written
    for (size_t i = first; i < units.size(); ++i) {
      const int32_t len = units[i].f[DLFP_W_KVEND] - units[i].f[DLFP_W_KVBEGIN];
      sorted[start[K - len]++] = units[i];
    }
    std::copy(sorted.get(), sorted.get() + nd, units.begin() + first);
  }
  if ((int64_t)units.size() > std::numeric_limits<int32_t>::max() / DLFP_WORK_INTS)
    return DLFP_ERANGE;
  if (groups > DLFP_MAX_GROUPS) return DLFP_ERANGE;

  // Workspace: header, the fixed counter region, then partial slots.
  const int64_t partial_base_bytes = DLFP_WORKSPACE_PARTIALS;
  std::vector<int64_t> group_off(groups, 0);
  int64_t off = partial_base_bytes / 4;
  {
    // assign in order of first appearance
    std::vector<int64_t> seen(groups, -1);
    for (const Unit& u : units) {
      const int32_t grp = u.f[DLFP_W_GROUP];
      if (grp < 0 || seen[grp] >= 0) continue;
      seen[grp] = off;
      group_off[grp] = off;
      off += (int64_t)u.f[DLFP_W_NSPLITS] * slot_floats(group_rows[grp]);
    }
  }
  if (off > std::numeric_limits<int32_t>::max()) return DLFP_ERANGE;
  for (Unit& u : units) {
    const int32_t grp = u.f[DLFP_W_GROUP];
    if (grp < 0) continue;
    const int64_t slot = slot_floats(group_rows[grp]);
    u.f[DLFP_W_WSGROUP] = (int32_t)group_off[grp];
    u.f[DLFP_W_WSOFF] = (int32_t)(group_off[grp] + u.f[DLFP_W_SPLIT] * slot);
  }

  // Append records for the one-launch cache write: each prompt sequence's new
  // tokens cut at page boundaries, per KV head (decode units write their own
  // token).  A prefill unit waits for them when its last key lies in a page
  // from the one holding its sequence's first new token on.
  std::vector<Unit> appends;
  appends.reserve((size_t)append_records);
  for (int s : prompts) {
    const int64_t pos0 = kv_len[s] - q_len[s];
    for (int kh = 0; kh < hkv; ++kh)
      for (int64_t p = pos0; p < kv_len[s];) {
        const int64_t n = std::min<int64_t>(DLFP_PAGE_SIZE - p % DLFP_PAGE_SIZE, kv_len[s] - p);
        Unit u;
        std::memset(&u, 0, sizeof(u));
        u.f[DLFP_W_SEQ] = s;
        u.f[DLFP_W_KVHEAD] = kh;
        u.f[DLFP_W_QTOK0] = (int32_t)(p - pos0);
        u.f[DLFP_W_QNTOK] = (int32_t)n;
        u.f[DLFP_W_KVBEGIN] = (int32_t)p;
        u.f[DLFP_W_KVEND] = (int32_t)(p + n);
        u.f[DLFP_W_GROUP] = -1;
        u.f[DLFP_W_NSPLITS] = 1;
        u.f[DLFP_W_KIND] = DLFP_KIND_APPEND;
        u.f[DLFP_W_QROW0] = (int32_t)(cu_q_of[s] + p - pos0);
        u.f[DLFP_W_QPOS0] = (int32_t)p;
        appends.push_back(u);
        p += n;
      }
  }
  int64_t waiting = 0;
  for (int64_t i = 0; i < num_prefill; ++i) {
    const Unit& u = units[i];
    const int64_t pos0 = u.f[DLFP_W_QPOS0] - u.f[DLFP_W_QTOK0];
    if ((u.f[DLFP_W_KVEND] - 1) / DLFP_PAGE_SIZE >= pos0 / DLFP_PAGE_SIZE) ++waiting;
  }
  const int64_t records = (int64_t)(units.size() + appends.size());
  if (records > std::numeric_limits<int32_t>::max() / DLFP_WORK_INTS) return DLFP_ERANGE;

  meta->num_seqs = num_seqs;
  meta->num_tokens = (int32_t)tokens;
  meta->num_units = (int32_t)units.size();
  meta->num_prefill_units = (int32_t)num_prefill;
  meta->num_groups = groups;
  meta->decode_split_tokens = (int32_t)split_d;
  meta->prefill_split_tokens = (int32_t)split_p;
  meta->workspace_bytes = std::max<int64_t>(off * 4, partial_base_bytes);
  meta->num_append = (int32_t)appends.size();
  meta->num_waiting_units = (int32_t)waiting;
  // Grid layout: with more prefill units than compute units, one per compute
  // unit leads and the decode workgroups follow, so the two shares run side by
  // side from the start instead of the decode units running alone after the
  // last prefill tile.
  const int64_t n_dec_units = (int64_t)units.size() - num_prefill;
  const int64_t cus = std::max<int64_t>(1, resident / 8);
  int64_t lead = num_prefill;
  if (tn.prefill_lead_units > 0)
    lead = std::min<int64_t>(tn.prefill_lead_units, num_prefill);
  else if (tn.prefill_lead_units == 0 && n_dec_units > 0 && num_prefill > cus)
    lead = cus;
  meta->prefill_lead_units = (int32_t)lead;
  // Decode page depth of a wavefront's unit: one page (deeper decode queues
  // delay the prefill tiles' loads; on the Qwen3-32B sweep a second page gained
  // nothing at p_t <= 1024 and lost 3-5% at larger chunks).
  const int depth = tn.decode_pages_in_flight ? tn.decode_pages_in_flight
                                              : (num_prefill == 0 ? 2 : 1);
  meta->decode_pages_in_flight = depth;
  if (meta->cap_seqs < num_seqs || meta->cap_tokens < tokens || meta->cap_work < records)
    return DLFP_ENOSPC;
  if ((num_seqs > 0 && (!meta->cu_q || !meta->q_pos0)) || (tokens > 0 && !meta->slot_mapping) ||
      (records > 0 && !meta->work))
    return DLFP_EINVAL;
  if (meta->cu_q) meta->cu_q[0] = 0;
  int64_t t = 0;
  for (int s = 0; s < num_seqs; ++s) {
    const int32_t pos0 = kv_len[s] - q_len[s];
    meta->q_pos0[s] = pos0;
    const int32_t* row = block_table + (int64_t)s * max_blocks;
    for (int32_t i = 0; i < q_len[s]; ++i) {
      const int32_t p = pos0 + i;
      meta->slot_mapping[t++] = row[p / DLFP_PAGE_SIZE] * DLFP_PAGE_SIZE + p % DLFP_PAGE_SIZE;
    }
    meta->cu_q[s + 1] = (int32_t)t;
  }
  if (!units.empty()) std::memcpy(meta->work, units.data(), units.size() * sizeof(Unit));
  if (!appends.empty())
    std::memcpy(meta->work + units.size() * DLFP_WORK_INTS, appends.data(),
                appends.size() * sizeof(Unit));
  return DLFP_OK;
}

int dlfp_controller_init(dlfp_controller* ctrl, double target_ms, int32_t c_initial,
                         int32_t c_min, int32_t c_max, int32_t quantum) {
  if (!ctrl) return DLFP_EINVAL;
  if (!(std::isfinite(target_ms) && target_ms > 0.0)) return DLFP_EINVAL;
  if (!(0 < c_min && c_min <= c_initial && c_initial <= c_max) || quantum <= 0)
    return DLFP_EINVAL;
  ctrl->target_ms = target_ms;
  ctrl->c_initial = c_initial;
  ctrl->c_min = c_min;
  ctrl->c_max = c_max;
  ctrl->quantum = quantum;
  ctrl->cap = c_initial;
  return DLFP_OK;
}

// Eq. 2 (Sec. 3.1).  floor_quantum(x) = quantum * floor(x / quantum) in
// double precision, then clamp to [c_min, c_max].
int dlfp_controller_step(dlfp_controller* ctrl, int32_t num_decoding_next,
                         int32_t last_was_guarded, double observed_ms, int32_t* next_cap) {
  if (!ctrl || !next_cap || num_decoding_next < 0) return DLFP_EINVAL;
  if (last_was_guarded) {
    if (!(std::isfinite(observed_ms) && observed_ms > 0.0)) return DLFP_EINVAL;
    const double x = (double)ctrl->cap * ctrl->target_ms / observed_ms;
    const double q = std::floor(x / ctrl->quantum);
    int64_t c;
    if (!(q < (double)std::numeric_limits<int32_t>::max()))
      c = ctrl->c_max;
    else
      c = (int64_t)q * ctrl->quantum;
    c = std::min<int64_t>(std::max<int64_t>(c, ctrl->c_min), ctrl->c_max);
    ctrl->cap = (int32_t)c;
  }
  if (num_decoding_next == 0) {
    ctrl->cap = ctrl->c_initial;
    *next_cap = -1;
  } else {
    *next_cap = ctrl->cap;
  }
  return DLFP_OK;
}

}  // extern "C"
