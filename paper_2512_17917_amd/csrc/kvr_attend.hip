// kvr_attend_decode: cache rebuild (Algorithm 4) fused with decode attention and
// the accumulation of per-token attention probabilities (Overview, Calculation
// Phase).  Retained tokens are streamed from their slots, Vague tokens are
// rebuilt on the fly from the sketch (Algorithm 2) and never written out.
//
// A unit's tokens are numbered t = 0 .. ret_cap-1 (retained slots) followed by
// ret_cap .. ret_cap+n_vague-1 (Vague index list) and cut into slices; every
// slice leaves a partial (max, sum, weighted V) per query head, and the merge
// kernel combines the partials, writes `out`, and turns the spilled logits into
// probabilities that are added to the cumulative scores.
//
// This file: the plan, the generic slice kernel (any storage type, any r, any
// sign setting; Vague rows gathered straight from global memory), the merge
// kernel and the dispatch.  The LDS-staged kernel for the Vague list is in
// kvr_attend_staged.hip.
#include "kvr_launch.h"

#include <algorithm>
#include <cmath>

namespace kvr {

static inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Tokens per slice: about 1280 slices per launch (measured on the 32k workloads: fewer, larger slices leave
// the merge kernel fewer partials to fold and cost the retained kernel nothing), in multiples of
// 64 tokens, at least 128 when a unit has a long list (a workgroup of four waves with a single 16-token tile
// per wave is mostly start-up), at most 1024.
static int slice_tokens_for(long long tokens, long long units) {
  long long st = (tokens * units + 1279) / 1280;
  st = (st + 63) / 64 * 64;
  const long long mn = tokens >= 1024 ? 128 : 64;
  if (st < mn) st = mn;
  if (st > 1024) st = 1024;
  return (int)st;
}

int attend_slice_tokens(long long tokens, long long units) { return slice_tokens_for(tokens, units); }

// The chip in these plans: 256 CUs, 32 on an XCD.  (Written in: plans are made without a GPU too, for the size of a workspace.)
constexpr double RET_RATE = 38e3, RET_CHIP = 5.0e6, RET_SLICE = 6.0;   // bytes per us of a CU, of all; us a slice ends with
// us for n_wgs workgroups, each on a CU of its own, to stream `bytes` of retained rows
static double ret_time(double bytes, int n_wgs) {
  return RET_SLICE + std::max(bytes / (RET_RATE * n_wgs), bytes / RET_CHIP);
}
// Slices of a unit's retained slots for n_wgs workgroups of `waves` waves: a number that spreads evenly over them, of slices as
// large as LDS allows and at most `most`.  45 KB per us is what one CU gets with few others beside it (43 measured on 8, 41 on 32),
// 38 what it gets in a launch (37 on 64).  40 units of 4104 slots, eight heads, 56 workgroups: one slice a unit (16 workgroups
// with none) 51 us, four 57.
static int ret_slices(long long units, int ret_cap, int n_wgs, int n_col, int waves, int most) {
  const int tiles = (ret_cap + 15) / 16, biggest = ret_stream_most(n_col, waves), least = std::max(1, (tiles + biggest - 1) / biggest);
  int slices = least;
  double best = 1e30;
  for (int s = least, end = std::min({tiles, least + 31, most}); s <= end; ++s) {
    const double t = (double)((units * s + n_wgs - 1) / n_wgs) * ((double)((tiles + s - 1) / s) * 8192.0 / 45e3 + RET_SLICE);
    if (t < best - 1e-9) { best = t; slices = s; }
  }
  return slices;
}

// The plans below price the slots by their bytes.  A workgroup walks whole slices, one after another, and where it has several,
// or the slots many CUs, that is too little: this is the estimate by turns of slices.  us, fitted to 644 calls of 20 .. 512 units x
// 7 .. 9000 slots x 65 .. 8000 listed tokens, each measured in all the ways below, and checked on 52 of 8 .. 128 units, up to 131072 tokens, in 1800 splits: a
// slice streams at 40 KB per us, less where many CUs share memory (128 of them 30, 256 17), and then ends (8 waves, of the 64- and
// 16-channel kernels: 3.5 .. 5; 16 waves, of the streaming kernel: 10 .. 14).
constexpr double RET_TURN_RATE = 40e3, RET_TURN_CHIP = 5.4e6;      // bytes per us of one CU, of all
static double ret_turns(long long units, int ret_cap, int slices, int n_wgs, int n_col, int waves) {
  const double shared = RET_TURN_RATE * (double)std::min<long long>(n_wgs, units * slices) / RET_TURN_CHIP;
  const double end = waves == 8 ? 3.0 + 0.45 * n_col : 10.0 + 0.25 * n_col;
  const int tiles = ((ret_cap + 15) / 16 + slices - 1) / slices;
  return (double)((units * slices + n_wgs - 1) / n_wgs) * (tiles * 8192.0 / RET_TURN_RATE * std::sqrt(1.0 + shared * shared) + end);
}

// List workgroups per unit (each takes `wg` us), workgroups for the slots (256: all CUs, before the list) and slices of a unit's slots.
struct RetChoice {
  int n;
  double wg;
  int n_wgs, slices;
  bool own;                 // the slots in a launch of their own
};
struct ListChoice {
  int n;
  double wg;
};
// The plan's choice c, or the slots ahead of the list or elsewhere, where that is better by turns of slices:
//  * the slots first, on all CUs of the launch: eight heads, 246 units of 585 + 1755 tokens 446 us a call on the 8 CUs left, 71 first
//    (as launches of their own 85), four heads, 246 units of 1441 + 4325 111 on 64, 100 first (125);
//  * in a launch of their own, whose small workgroups share CUs, for hardly any slots of many units: 400 units of 4 + 220, eight
//    heads 59.1 on 56 CUs, 50.8 own (72 + 300: 62.4, 56.1), four heads 47.8, 42.1; up to 64 slots, beside the streaming kernel 256
//    (four heads, 512 units of 130 + 600 60.7 first, 64.1 own).
//  * where the plan has workgroups walk six slices or more, on other CUs that the list can leave: 400 units of 1441 + 4325, four
//    heads 201 on 56, 184 on 80, 512 units, one head 202 on 80, 174 on 128 (fewer slices each: 20 units of 7000 + 1400, one head
//    25.5 us, by this estimate 34).  Beside the streaming kernel from three on: eight heads, 320 units of 3000 + 900 219 -> 154, 144 of
//    11000 + 2800 307 -> 250; not with 16 columns, whose slices LDS keeps short (100 units of 11000 + 2800 219, by this 260).
// Only for a gain of 5 % by this estimate (streaming kernel 10 %): within it the plans' own figures are the better ones.
static RetChoice ret_ahead(RetChoice c, const ListChoice* lists, int n_lists, long long units, int ret_cap, int n_col, int waves,
                              int most, int own_slices) {
  if (c.n_wgs == 0) return c;
  const long long units8 = (units + 7) / 8;
  const int tiles = (ret_cap + 15) / 16, biggest = ret_stream_most(n_col, waves), least = std::max(1, (tiles + biggest - 1) / biggest);
  const long long left = 32 - c.n_wgs / 8;
  double best = ret_turns(units, ret_cap, c.slices, c.n_wgs, n_col, waves);
  best = left > 0 ? std::max((double)((units8 * c.n + left - 1) / left) * c.wg, best) : (double)((units8 * c.n + 31) / 32) * c.wg + best;
  best *= waves == 8 ? 0.95 : 0.9;
  // the slots' time on n_wgs workgroups: as many slices as a number of turns holds
  int slices = 1;
  const bool many = units * c.slices >= (waves == 16 && n_col <= 8 ? 3ll : 6ll) * c.n_wgs;
  const auto slots = [&](int n, int n_wgs) {
    const int top = std::min(tiles, most - n);
    const long long first = (units * least + n_wgs - 1) / n_wgs;
    double us = 1e30;
    for (long long turns = first; turns < first + 3; ++turns) {
      const int s = std::max(least, (int)std::min<long long>(turns * n_wgs / units, top));
      const double t = ret_turns(units, ret_cap, s, n_wgs, n_col, waves);
      if (t < us) { us = t; slices = s; }
      if (s >= top) break;
    }
    return us;
  };
  for (int i = 0; i < n_lists; ++i) {
    const int n = lists[i].n;
    const double wg = lists[i].wg;
    const long long turns = (units8 * n + 31) / 32;
    if ((double)turns * wg >= best || n + least > most) continue;
    for (long long k = turns; many && k <= turns + 2 && (double)k * wg < best; ++k) {
      const int n_wgs = 8 * (32 - (int)((units8 * n + k - 1) / k));
      if (n_wgs <= 0) continue;
      const double t = std::max((double)k * wg, slots(n, n_wgs));
      if (t < best) { best = t; c = {n, wg, n_wgs, slices, false}; }
    }
    const double list = (double)turns * wg, t = list + slots(n, 256);
    if (t < best) { best = t; c = {n, wg, 256, slices, false}; }
    const double own = list + (waves == 8 ? 5.0 : 10.0) + 512.0 * (double)units * ret_cap / 4.2e6;
    if (own < best && ret_cap <= (waves == 8 ? 64 : 256) && n + own_slices <= most) { best = own; c = {n, wg, 0, own_slices, true}; }
  }
  return c;
}

// One launch for the retained slots and the Vague list (64- and 16-channel kernels): n_vslices workgroups per unit over the
// list and n_ret_wgs workgroups over the slots, at most `most` slices of both kinds per unit (what callers' workspaces hold).
// A workgroup of either kind has a CU to itself (its registers fill the SIMDs) and a unit's workgroups share an XCD of 32
// CUs, so the launch takes turns * (time of a list workgroup) on the CUs that the slots leave; where it leaves none, the slots
// go first, on all of them.  In us, measured: a list workgroup of the 64-channel kernel takes 11.5 at 273 slots per row, 7 at six,
// and 5 per round of 64 tokens a wave (one head 3.5), at 25 rounds as at two; of the 16-channel kernel 27 at 1050 sketch rows,
// 68 at 3276, and 5.5 a round (four rows 10.5).  A CU streams 35 .. 40 KB of retained rows per us whatever its waves have in
// flight, and a slice ends with 6 us of merging and starting anew.
// Before, slots and list were launches of their own, one behind the other or on two streams, with at most 6 rounds (16
// channels: 13) a wave.  Both, us from the first start to the last end of a call: 64 channels: 8 units of 25395 + 7374 tokens
// 42.1 -> 32.6 (25 list workgroups per unit, 56 for the slots; 16 and 128: 38), 32 units 104.5 -> 70 (6 and 64; 5 and 96: 73, 8
// and none: 80 with every list workgroup taking a slice along), 128 units 311 (on two streams 258 .. 284) -> 230 .. 255 (3 and
// 64), 64 units of 1862 + 187 33.4 -> 27.4, 96 units of 3753 + 1128, one head 45.2 -> 36.0.  16 channels: 16 units of 101580 +
// 29492 206 -> 174 (13 and 48; 12 and 64: 191, 14 and 32: 198), 24 units of 70000 tokens in all 164 -> 132, 8 of 42000 65 -> 50; four
// rows: 32 units of 101580 + 29492 520 -> 476 .. 506 (14 and 32; 21 and 32: 499), 16 of 60000 in all 151 -> 125, 128 of 9000, one head
// 130 -> 122 (slots first; 3 and 64: 142).
static void plan_pair(AttendPlan& p, const DevDesc& d, long long units, int ret_cap, int vague_cap, int most) {
  const bool s64 = p.ch == 64;
  const int kmax = s64 ? STAGED64_KMAX : staged16_kmax(d.r);
  const double fixed = s64 ? 6.5 + 0.018 * d.w : 8.5 + 0.018 * d.r * d.w, round = s64 ? 3.0 + 0.5 * d.G : d.r == 3 ? 5.5 : 10.5;
  const int wr = (vague_cap + 63) / 64;
  const long long units8 = (units + 7) / 8;
  const double bytes = 512.0 * units * ret_cap;
  const int biggest = 16 * ret_stream_most(d.G, 8), least = (ret_cap + biggest - 1) / biggest;
  double best = 1e30, best_wg = 0.0;
  int best_n = 1, best_r = 0, last = 0, n_lists = 0;
  ListChoice lists[std::max(STAGED64_KMAX, staged16_kmax(4))];
  for (int rho = 1; rho <= kmax; ++rho) {
    const int n = (wr + 8 * rho - 1) / (8 * rho);
    if (n == last || (n + least > most && rho < kmax)) continue;
    last = n;
    const double wg = fixed + round * ((wr + 8 * n - 1) / (8 * n));
    const long long per_xcd = units8 * n, turns = (per_xcd + 31) / 32;
    lists[n_lists++] = {n, wg};
    for (long long k = turns; k <= turns + 2; ++k) {
      int r = ret_cap > 0 ? 8 * (32 - (int)((per_xcd + k - 1) / k)) : 0;
      double t = (double)k * wg;
      if (r > 0) {
        t = std::max(t, ret_time(bytes, r));
      } else if (ret_cap > 0) {              // no CU is left: the slots first, on all of them
        r = 256;
        t += 2.0 + ret_time(bytes, r);
      }
      if (t < best - 1e-9) { best = t; best_n = n; best_r = r; best_wg = wg; }
    }
  }
  const int slices = best_r > 0 ? ret_slices(units, ret_cap, best_r, d.G, 8, most - best_n) : 1;
  const RetChoice c = ret_ahead({best_n, best_wg, best_r, slices, false}, lists, n_lists, units, ret_cap, d.G, 8, most, p.n_rslices);
  p.n_vslices = c.n;
  p.ret_own = c.own;
  p.pair_lds = p.lds_bytes;
  if (c.own) return;                         // slices as that launch has them anyway
  p.rslice_tokens = std::max(1, ((ret_cap + 15) / 16 + c.slices - 1) / c.slices) * 16;
  p.n_rslices = (ret_cap + p.rslice_tokens - 1) / p.rslice_tokens;
  p.n_ret_wgs = (int)std::min<long long>(c.n_wgs, (units * p.n_rslices + 7) / 8 * 8);
  if (ret_cap > 0) p.pair_lds = std::max(p.pair_lds, ret_stream_lds(d.G, 8, p.rslice_tokens));
}

// The streaming kernel's launch, likewise: one of its workgroups per CU (16 waves, 17 us and 17 ns per token of its part).  It
// takes as many parts as one turn holds; with enough slots to matter, fewer where the CUs that leaves them gain more.  us
// from the first start to the last end of a call, slots and list before as two launches: eight heads, 40 units of 12307 + 4104
// tokens 88 -> 65 (5 parts and 56 workgroups; 4 and 96: 69, 6 and 16: 150), 16 units of 32768 79 -> 55 (13 and 48; 12 and 64: 56,
// 16 parts, the slots first: 65), 64 units 194 -> 167 (3 and 64; slots first 203), 8 of 900 34 -> 22.
StreamPlan plan_stream(const DevDesc& d, int n_col, long long units, int ret_cap, int vague_cap, int most) {
  constexpr double FIXED = 17.0, TOKEN = 0.017;
  StreamPlan p = {};
  const long long units8 = (units + 7) / 8;
  const double bytes = 512.0 * units * ret_cap;
  const int full = multi_staged_part_tokens(vague_cap, units), n_full = (vague_cap + full - 1) / full;
  double best = 1e30, best_wg = 0.0;
  int best_r = 0, n_lists = 0;
  constexpr int LISTS = 32;
  ListChoice lists[LISTS];
  int list_tokens[LISTS];
  p.vslice_tokens = full;
  const auto parts = [&](int tokens) { return (vague_cap + tokens - 1) / tokens; };
  for (int n = n_full; n >= 1 && n >= n_full / 2; --n) {
    const int tokens = n == n_full ? full : (vague_cap + 16 * n - 1) / (16 * n) * 16;
    const long long per_xcd = units8 * parts(tokens), turns = (per_xcd + 31) / 32;
    int r = ret_cap > 0 ? 8 * (32 - (int)((per_xcd + turns - 1) / turns)) : 0;
    const double wg = FIXED + TOKEN * tokens;
    double t = (double)turns * wg;
    if (n_lists < LISTS) { lists[n_lists] = {parts(tokens), wg}; list_tokens[n_lists++] = tokens; }
    if (r > 0) {
      t = std::max(t, ret_time(bytes, r));
    } else if (ret_cap > 0) {
      r = 256;
      t += 2.0 + ret_time(bytes, r);
    }
    if (t < best - 1e-9) { best = t; best_r = r; best_wg = wg; p.vslice_tokens = tokens; }
    // a few slots go first, on all CUs; from 256 on it is measured that fewer parts can be better: eight heads, 42 units of 400 + 12000
    // 85 -> 58 us, 60 units of 300 + 1200 37 -> 30 (181 calls of 256 .. 510 slots: 3 % on average, one slower by more than 3 %)
    if (ret_cap < 256) break;
  }
  const int best_parts = parts(p.vslice_tokens);
  const int slices = best_r > 0 ? ret_slices(units, ret_cap, best_r, n_col, 16, most - best_parts) : 1;
  const RetChoice c = ret_ahead({best_parts, best_wg, best_r, slices, false}, lists, n_lists, units, ret_cap, n_col, 16, most, 1);
  for (int i = 0; c.n != best_parts && i < n_lists; ++i)
    if (lists[i].n == c.n) p.vslice_tokens = list_tokens[i];
  p.n_vslices = parts(p.vslice_tokens);
  p.own = c.own;
  p.lds = multi_staged_lds(d, n_col);
  p.rslice_tokens = std::max(1, ((ret_cap + 15) / 16 + c.slices - 1) / c.slices) * 16;
  p.n_rslices = (ret_cap + p.rslice_tokens - 1) / p.rslice_tokens;
  p.n_ret_wgs = (int)std::min<long long>(c.n_wgs, (units * p.n_rslices + 7) / 8 * 8);
  if (p.n_ret_wgs > 0) p.lds = std::max(p.lds, ret_stream_lds(n_col, 16, p.rslice_tokens));
  return p;
}

AttendPlan attend_plan(const DevDesc& d, int dtype, long long ret_cap, long long vague_cap) {
  AttendPlan p;
  const long long units = (long long)d.B * d.Hkv;
  const long long tot_cap = ret_cap + vague_cap;
  p.staged = p.pair = p.ret_own = false;
  p.n_vslices = 0;
  p.ch = 0;
  p.lds_bytes = 0;
  p.n_ret_wgs = p.pair_lds = 0;
  // staged kernel: bf16, the paper's sign setting, G <= 4, r = 3 or 4, bucket fits 15 bits
  if (dtype == KVR_BF16 && d.sign_mask == 2 && d.G <= 4 && (d.r == 3 || d.r == 4) && d.w <= 32768 &&
      vague_cap >= 64) {
    const bool s64 = staged64_applies(d), s16 = staged16_applies(d);
    p.lds_bytes = s64 ? staged64_lds(d.w, d.G) : s16 ? staged16_lds(d) : 0;
    p.ch = s64 ? 64 : s16 ? 16 : 0;
    // The general kernel: 16 channels where they fit (four heads: 5056 rows), else 8, up to 8000 rows with four heads, 8288
    // with two, 8432 with one (the gather takes more workspace, so the line stays where callers' workspaces know it): a chunk then
    // passes through LDS 32 times for fewer and fewer tokens per row, and the gather of the generic kernel is no slower.
    // 16 units, 31 tokens per row, us with 8 channels / by the gather: four rows, four heads 7000 rows 924 / 995, 8000
    // 1030 / 1076, 9000 1165 / 1150; one head 6000 560 / 665, 7000 865 / 714; three rows, four heads 5100 483 / 502,
    // 6000 558 / 534, 7000 867 / 723 (three rows, and one head, lose from a narrower sketch on than the line says).
    // 16 against 8 channels: 32 units of 139000 tokens, 4500 rows, 1360 -> 946 us a call.
    for (int c = 16; c >= 8 && p.ch == 0; c >>= 1)
      if (staged_lds(d.r * d.w, d.G, c) <= STAGED_LDS_LIMIT && (c == 16 || d.r * d.w <= 8576 - 144 * d.G)) {
        p.ch = c;
        p.lds_bytes = staged_lds(d.r * d.w, d.G, c);
      }
    if (p.ch) {
      const long long wr = (vague_cap + 63) / 64;          // wave-rounds to cover the list
      // Cost model: a workgroup that gives every wave rho
      // rounds of 64 tokens takes about (fixed + rho) round times (fixed part: staging the sketch chunks,
      // hashes, softmax, reductions), and the launch runs ceil(workgroups / 256)
      // such workgroups one after another on each CU.  It decides for the general kernel; for the other two it only bounds
      // the number of slices (plan_pair), so that no call needs a larger workspace than it did when it decided for them.
      const int kmax = s16 ? 13 : STAGED_KMAX;
      const double fixed_rounds = s16 ? 7.5 : 2.8;
      double best = 1e30;
      int best_n = 1;
      for (int rho = 1; rho <= kmax; ++rho) {
        const long long n = (wr + 8 * rho - 1) / (8 * rho);
        const long long rho_eff = (wr + 8 * n - 1) / (8 * n);      // rounds the busiest wave really gets
        const long long waves_of_wgs = (units * n + 255) / 256;
        const double cost = (double)waves_of_wgs * (fixed_rounds + (double)rho_eff);
        if (cost < best - 1e-9) { best = cost; best_n = (int)n; }
      }
      p.staged = true;
      p.pair = s64 || s16;
      p.n_vslices = best_n;
    }
  }
  p.mfma_retained = (dtype == KVR_BF16);
  // 8 query heads per kv head: too many logits per token for the register-resident staged kernels; the
  // streaming kernel of kvr_attend_multi takes the list with the 8 heads as its columns (one query)
  p.streamed = !p.staged && dtype == KVR_BF16 && d.G == 8 && multi_staged_applies(d, vague_cap);
  p.vslice_tokens = 0;
  if (p.mfma_retained || p.staged) {
    // retained slots and the Vague list are cut separately
    p.rslice_tokens = slice_tokens_for(ret_cap, units);
    p.n_rslices = (int)((ret_cap + p.rslice_tokens - 1) / p.rslice_tokens);
    if (p.streamed) {
      const int full = multi_staged_part_tokens(vague_cap, units);
      p.stream = plan_stream(d, d.G, units, (int)ret_cap, (int)vague_cap, p.n_rslices + (int)((vague_cap + full - 1) / full));
      p.rslice_tokens = p.stream.rslice_tokens;
      p.n_rslices = p.stream.n_rslices;
      p.vslice_tokens = p.stream.vslice_tokens;
      p.n_vslices = p.stream.n_vslices;
    } else if (p.pair) {
      plan_pair(p, d, units, (int)ret_cap, (int)vague_cap, p.n_rslices + p.n_vslices);
    } else if (!p.staged && vague_cap > 0) {
      p.vslice_tokens = slice_tokens_for(vague_cap, units);
      p.n_vslices = (int)((vague_cap + p.vslice_tokens - 1) / p.vslice_tokens);
    }
    p.n_slices = p.n_rslices + p.n_vslices;
  } else {
    // one generic launch over all tokens
    p.rslice_tokens = slice_tokens_for(tot_cap, units);
    p.n_rslices = (int)((tot_cap + p.rslice_tokens - 1) / p.rslice_tokens);
    if (p.n_rslices < 1) p.n_rslices = 1;
    p.n_slices = p.n_rslices;
  }
  size_t off = 0;
  p.off_part_o = off;
  off = align_up(off + (size_t)units * p.n_slices * d.G * D * sizeof(float), 256);
  p.off_part_ml = off;
  off = align_up(off + (size_t)units * p.n_slices * d.G * 2 * sizeof(float), 256);
  p.off_logits = off;
  off = align_up(off + (size_t)units * (size_t)(p.streamed ? ret_cap : tot_cap) * d.G * sizeof(float), 256);
  p.off_rec = p.off_tiles = off;
  if (p.streamed) {
    const size_t tokens = multi_staged_scratch_tokens(units, vague_cap);
    off = align_up(off + tokens * sizeof(uint32_t), 256);
    p.off_tiles = off;
    off = align_up(off + tokens * d.G * sizeof(float), 256);
  }
  p.total_bytes = off;
  return p;
}

int attend_side_lds(const DevDesc& d, const AttendPlan& p) {
  if (!p.staged || !p.mfma_retained) return 0;
  // Registers: two waves of a staged kernel of up to 192 and one of the retained kernel's capped form (128) share a SIMD's
  // 512.  Four rows and four heads take more in the general kernel, four rows always in the 16-channel kernel, and the retained
  // kernel only finds room where a workgroup has just ended: 4400 rows in four, four heads 1105 us side by side, 1087 back to
  // back.  (The 16-channel kernel's launch holds the slots: there the answer decides nothing.)  Where they fit: three rows of 1500 slots (general kernel), 32 units 907 / 947.
  if (d.r != 3 && (staged16_applies(d) || d.G == 4)) return 0;
  // LDS: room for a slice's logits, or for 512 tokens' and the sums.
  constexpr int UNIT = 1280;                   // LDS is handed out in these
  const int room = (STAGED_LDS_LIMIT / UNIT - (p.lds_bytes + UNIT - 1) / UNIT) * UNIT -
                   2 * 4 * d.G * (int)sizeof(float);                               // statistics of the four waves
  const int whole = retained_lds(d.G, p.rslice_tokens), least = retained_lds(d.G, 0);
  return whole <= room ? whole : least <= room ? least : 0;
}

// ---------------------------------------------------------------------------
// generic slice kernel
// ---------------------------------------------------------------------------
// NW waves per workgroup walk a slice, WAVE / LPT tokens a wave at a time, each a chain of its own (position -> sketch rows ->
// lane sums -> exponential).  Launches that leave CUs without a workgroup take 16 waves instead of four, so that a slice is
// walked in a quarter of the steps; elsewhere four waves and several workgroups per CU do the same with smaller merges.
template <typename T, int G, int R, int NW>
__global__ __launch_bounds__(64 * NW) void attend_main_kernel(DevDesc d, AttendArgs a) {
  constexpr int VEC = Store<T>::VEC;
  constexpr int LPT = D / VEC;       // lanes that share one token
  constexpr int TPW = WAVE / LPT;    // tokens per wave per iteration
  const int unit = blockIdx.y, slice = blockIdx.x;
  const int b = unit / d.Hkv, hk = unit % d.Hkv;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int sub = lane % LPT, tl = lane / LPT;
  const int c0 = sub * VEC;

  float qf[G][VEC];
  {
    const T* q = (const T*)a.q + ((size_t)b * d.Hq + (size_t)hk * G) * D + c0;
#pragma unroll
    for (int g = 0; g < G; ++g) Store<T>::load16(q + (size_t)g * D, qf[g]);
  }
  const int nv = a.n_vague ? clampi(a.n_vague[unit], 0, a.vague_cap) : 0;
  const int tot_cap = a.ret_cap + a.vague_cap;
  const int total = min(a.ret_cap + nv, a.tok_limit);
  const int t_begin = a.tok_start + slice * a.slice_tokens;
  const int t_end = min(t_begin + a.slice_tokens, total);

  const T* kret = (const T*)a.k_ret + (size_t)unit * a.ret_cap * D;
  const T* vret = (const T*)a.v_ret + (size_t)unit * a.ret_cap * D;
  const size_t sk_unit = (size_t)unit * d.r * d.w * D;
  const T* sk = (const T*)a.sk + sk_unit;
  const T* sv = (const T*)a.sv + sk_unit;
  const bool flip_k = (d.sign_mask & 1) != 0, flip_v = (d.sign_mask & 2) != 0;

  float m[G], l[G], acc[G][VEC];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    m[g] = -__builtin_inff();
    l[g] = 0.f;
#pragma unroll
    for (int c = 0; c < VEC; ++c) acc[g][c] = 0.f;
  }

  for (int t0 = t_begin + wave * TPW; t0 < t_end; t0 += NW * TPW) {
    const int t = t0 + tl;
    bool valid = t < t_end;
    float kf[VEC], vf[VEC];
#pragma unroll
    for (int c = 0; c < VEC; ++c) { kf[c] = 0.f; vf[c] = 0.f; }
    if (valid) {
      if (t < a.ret_cap) {
        const int pos = a.ret_pos ? a.ret_pos[(size_t)unit * a.ret_cap + t] : t;
        if (pos < 0) {
          valid = false;
        } else {
          Store<T>::load16(kret + (size_t)t * D + c0, kf);
          Store<T>::load16(vret + (size_t)t * D + c0, vf);
        }
      } else {
        const int J = a.vague_pos[(size_t)unit * a.vague_cap + (t - a.ret_cap)];
        query_chunk<T, R>(d, sk, J, c0, flip_k, kf);
        query_chunk<T, R>(d, sv, J, c0, flip_v, vf);
      }
    }
    float s[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      float x = 0.f;
#pragma unroll
      for (int c = 0; c < VEC; ++c) x = fmaf(qf[g][c], kf[c], x);
#pragma unroll
      for (int off = LPT / 2; off >= 1; off >>= 1) x += __shfl_xor(x, off);
      s[g] = valid ? x * d.scale : -__builtin_inff();
    }
    if (a.logits != nullptr && sub == 0 && t < t_end) {
      float* lg = a.logits + ((size_t)unit * tot_cap + t) * G;
#pragma unroll
      for (int g = 0; g < G; ++g) lg[g] = s[g];
    }
    if (valid) {
#pragma unroll
      for (int g = 0; g < G; ++g) {
        if (s[g] > m[g]) {
          const float corr = expf(m[g] - s[g]);     // exp(-inf) = 0 on the first token
          m[g] = s[g];
          l[g] = l[g] * corr + 1.f;
#pragma unroll
          for (int c = 0; c < VEC; ++c) acc[g][c] = fmaf(acc[g][c], corr, vf[c]);
        } else {
          const float pr = expf(s[g] - m[g]);
          l[g] += pr;
#pragma unroll
          for (int c = 0; c < VEC; ++c) acc[g][c] = fmaf(pr, vf[c], acc[g][c]);
        }
      }
    }
  }

  // merge the token lane groups of a wave (they hold the same channels)
#pragma unroll
  for (int off = LPT; off < WAVE; off <<= 1) {
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const float m2 = __shfl_xor(m[g], off);
      const float l2 = __shfl_xor(l[g], off);
      const float mn = fmaxf(m[g], m2);
      const float e1 = (m[g] == -__builtin_inff()) ? 0.f : expf(m[g] - mn);
      const float e2 = (m2 == -__builtin_inff()) ? 0.f : expf(m2 - mn);
      l[g] = l[g] * e1 + l2 * e2;
#pragma unroll
      for (int c = 0; c < VEC; ++c) {
        const float a2 = __shfl_xor(acc[g][c], off);
        acc[g][c] = acc[g][c] * e1 + a2 * e2;
      }
      m[g] = mn;
    }
  }

  __shared__ float s_acc[NW][G][D];
  __shared__ float s_m[NW][G], s_l[NW][G];
  if (tl == 0) {
#pragma unroll
    for (int g = 0; g < G; ++g) {
#pragma unroll
      for (int c = 0; c < VEC; ++c) s_acc[wave][g][c0 + c] = acc[g][c];
      if (sub == 0) { s_m[wave][g] = m[g]; s_l[wave][g] = l[g]; }
    }
  }
  __syncthreads();
  float* po = a.part_o + ((size_t)unit * a.n_slices + a.slice0 + slice) * G * D;
  float* pml = a.part_ml + ((size_t)unit * a.n_slices + a.slice0 + slice) * G * 2;
  for (int idx = threadIdx.x; idx < G * D; idx += 64 * NW) {
    const int g = idx / D, c = idx % D;
    float M = s_m[0][g];
#pragma unroll
    for (int w_ = 1; w_ < NW; ++w_) M = fmaxf(M, s_m[w_][g]);
    float L = 0.f, O = 0.f;
#pragma unroll
    for (int w_ = 0; w_ < NW; ++w_) {
      const float e = (s_m[w_][g] == -__builtin_inff()) ? 0.f : expf(s_m[w_][g] - M);
      L += s_l[w_][g] * e;
      O += s_acc[w_][g][c] * e;
    }
    po[idx] = O;
    if (c == 0) { pml[g * 2] = M; pml[g * 2 + 1] = L; }
  }
}

// ---------------------------------------------------------------------------
// merge kernel
// ---------------------------------------------------------------------------

// Waves per SIMD: the most whose registers hold the kernel without a spill (64 registers: 1 spilled with four heads, 62
// with eight; 80: 9 with eight; 96: 6 with sixteen columns).
template <int G, bool TILES>
__global__ __launch_bounds__(256, (G <= 2 ? 8 : G <= 4 ? 7 : G == 8 ? 5 : 4)) void attend_combine_kernel(DevDesc d, AttendArgs a) {
  const int unit = blockIdx.y;
  const int b = unit / d.Hkv, hk = unit % d.Hkv;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  __shared__ float sM[G], sL[G];
  const float* pml = a.part_ml + (size_t)unit * a.n_slices * G * 2;

  // ---- the unit's output: spread over the first nb workgroups of the unit (a power
  //      of two): workgroup bx takes G*D/nb output elements in rounds of 256/tpe, `tpe`
  //      threads per element, each summing every tpe-th slice with eight loads in
  //      flight.  tpe is the one of 4, 8, 16 that takes the fewest batches of loads, rounds
  //      x batches per round, on the grid there is.  The first batch is requested here,
  //      ahead of the statistics.  Against 4 or 16 threads by the slice count alone, at most 8 or 32 workgroups and
  //      no look-ahead, us: 8 units, 83 slices 10.1 -> 8.8; 64 units, 12 slices, 3 workgroups per unit 9.6 -> 7.4;
  //      40 units, 35 slices, 8 heads 18.7 -> 15.0; 16 units, 93 slices 22 -> 20. ----------
  int tpe = 4, best = 1 << 30;
#pragma unroll
  for (int c = 4; c <= 16; c *= 2) {
    int n = 1;
    while (n * 2 <= (int)gridDim.x && G * D / (n * 2) >= 256 / c) n *= 2;
    const int cost = (G * D / n) / (256 / c) * ((a.n_slices + 8 * c - 1) / (8 * c));
    if (cost < best) { best = cost; tpe = c; }
  }
  const int epw = 256 / tpe;                  // output elements per workgroup and round
  int nb = 1;
  while (nb * 2 <= (int)gridDim.x && G * D / (nb * 2) >= epw) nb *= 2;
  const bool do_out = (int)blockIdx.x < nb;
  const int per_wg = G * D / nb;              // a multiple of epw
  const int el = tid % epw, sq = tid / epw;
  const float* po = a.part_o + (size_t)unit * a.n_slices * G * D;
  float bv[8];
  float2 bm[8];                               // (maximum, sum) of the slice
  auto load_batch = [&](int idx, int s0) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int s_ = s0 + tpe * j;
      bv[j] = 0.f;
      bm[j] = make_float2(0.f, 0.f);
      if (s_ < a.n_slices) {
        bv[j] = po[(size_t)s_ * G * D + idx];
        bm[j] = *reinterpret_cast<const float2*>(pml + (s_ * G + idx / D) * 2);
      }
    }
  };
  constexpr bool EARLY = G < 16;              // 16 columns: the logits take the registers (four waves per SIMD)
  if (EARLY && do_out) load_batch(blockIdx.x * per_wg + el, sq);

  // ---- score pass, first half: everything that does not depend on the global
  //      statistics is requested before they are formed (token positions, the
  //      spilled logits and the old scores), so that the two chains of memory
  //      round trips (slice statistics -> reduction, position -> old score) run
  //      side by side instead of one after the other.  Four tokens per thread. ----
  constexpr int U = 4;
  const bool do_scores = a.scores != nullptr;
  const int logit_rows = TILES ? a.ret_cap : a.ret_cap + a.vague_cap;      // of a unit
  int total = 0;
  int pos[U];
  float x[U][G], old[U];
  float* sc = do_scores ? a.scores + (size_t)unit * a.n_cap : nullptr;
  // TILES: the streaming kernel leaves its tokens' logits by tile, [column][16 tokens]; there a thread takes four neighbouring
  // tokens (a 16-byte load per column), in workgroups of their own behind those of the retained slots.
  const int ret_wgs = (a.ret_cap + 256 * U - 1) / (256 * U);
  const bool tiled = TILES && (int)blockIdx.x >= ret_wgs;
  const int v0 = ((int)blockIdx.x - ret_wgs) * 256 * U + tid * U;             // tiled: first of the thread's tokens in the list
  const int t0 = tiled ? a.ret_cap + v0 : blockIdx.x * 256 * U + tid, dt = tiled ? 1 : 256;
  if (do_scores) {
    const int nv = a.n_vague ? clampi(a.n_vague[unit], 0, a.vague_cap) : 0;
    total = (TILES && !tiled) ? a.ret_cap : a.ret_cap + nv;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int t = t0 + u * dt;
      pos[u] = -1;
      if (t < total) {
        if (t < a.ret_cap) pos[u] = a.ret_pos ? a.ret_pos[(size_t)unit * a.ret_cap + t] : t;
        else pos[u] = a.vague_pos[(size_t)unit * a.vague_cap + (t - a.ret_cap)];
        if (pos[u] >= a.n_cap) pos[u] = -1;
      }
    }
    if (tiled) {
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int g = 0; g < G; ++g) x[u][g] = -__builtin_inff();
      if (v0 < nv) {
        const int tile0 = v0 & ~15, pitch = min(16, ((nv + 3) & ~3) - tile0);
        const float* lg = a.tiles + ((size_t)unit * ((a.vague_cap + 3) & ~3) + tile0) * G + (v0 - tile0);
#pragma unroll
        for (int g = 0; g < G; ++g) {
          const float4 v = *reinterpret_cast<const float4*>(lg + g * pitch);
          x[0][g] = v.x; x[1][g] = v.y; x[2][g] = v.z; x[3][g] = v.w;
        }
      }
    } else {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int t = t0 + u * 256;
#pragma unroll
        for (int g = 0; g < G; ++g) x[u][g] = -__builtin_inff();
        if (t < total) {
          const float* lg = a.logits + ((size_t)unit * logit_rows + t) * G;
          if constexpr (G % 4 == 0) {
#pragma unroll
            for (int g4 = 0; g4 < G; g4 += 4) {
              const float4 v = *reinterpret_cast<const float4*>(lg + g4);
              x[u][g4] = v.x; x[u][g4 + 1] = v.y; x[u][g4 + 2] = v.z; x[u][g4 + 3] = v.w;
            }
          } else {
#pragma unroll
            for (int g = 0; g < G; ++g) x[u][g] = lg[g];
          }
        }
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) old[u] = (pos[u] >= 0) ? sc[pos[u]] : 0.f;
  }

  // ---- global max and sum per head: wave w takes heads w, w + 4, ...; their chains of loads, exponentials and
  //      lane exchanges run side by side ---------------------------------------------------------------------
  {
    constexpr int NG = (G + 3) / 4;             // heads per wave
    float M[NG], L[NG];
#pragma unroll
    for (int j = 0; j < NG; ++j) { M[j] = -__builtin_inff(); L[j] = 0.f; }
    for (int s = lane; s < a.n_slices; s += WAVE) {
      float2 ml[NG];
#pragma unroll
      for (int j = 0; j < NG; ++j)
        ml[j] = *reinterpret_cast<const float2*>(pml + (s * G + min(wave + 4 * j, G - 1)) * 2);
#pragma unroll
      for (int j = 0; j < NG; ++j) {
        if (ml[j].y > 0.f) {
          const float mn = fmaxf(M[j], ml[j].x);
          L[j] = L[j] * expf(M[j] - mn) + ml[j].y * expf(ml[j].x - mn);
          M[j] = mn;
        }
      }
    }
    // the wave's maximum first (no exponentials), then one rescaling per lane and a plain sum
    float Mw[NG], Lw[NG];
#pragma unroll
    for (int j = 0; j < NG; ++j) Mw[j] = M[j];
#pragma unroll
    for (int off = 1; off < WAVE; off <<= 1)
#pragma unroll
      for (int j = 0; j < NG; ++j) Mw[j] = fmaxf(Mw[j], __shfl_xor(Mw[j], off));
#pragma unroll
    for (int j = 0; j < NG; ++j) Lw[j] = (L[j] > 0.f) ? L[j] * expf(M[j] - Mw[j]) : 0.f;
#pragma unroll
    for (int off = 1; off < WAVE; off <<= 1)
#pragma unroll
      for (int j = 0; j < NG; ++j) Lw[j] += __shfl_xor(Lw[j], off);
#pragma unroll
    for (int j = 0; j < NG; ++j)
      if (lane == 0 && wave + 4 * j < G) { sM[wave + 4 * j] = Mw[j]; sL[wave + 4 * j] = Lw[j]; }
  }
  __syncthreads();

  // ---- score pass, second half ----------------------------------------------------
  if (do_scores) {
    float acc[U];
#pragma unroll
    for (int u = 0; u < U; ++u) acc[u] = 0.f;
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const float M = sM[g], L = sL[g];
      const float invL = L > 0.f ? 1.f / L : 0.f;
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (x[u][g] != -__builtin_inff()) acc[u] += __expf(x[u][g] - M) * invL;
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (pos[u] >= 0) sc[pos[u]] = old[u] + acc[u];
  }

  // ---- the output elements ------------------------------------------------------------
  if (do_out) {
    __shared__ float sO[256];                  // [slice share][output element of this round]
    for (int o0 = 0; o0 < per_wg; o0 += epw) {
      const int idx = blockIdx.x * per_wg + o0 + el;
      const int g = idx / D;
      const float M = sM[g];
      float o = 0.f;
      for (int s0 = sq; s0 < a.n_slices; s0 += tpe * 8) {
        if (!EARLY || o0 != 0 || s0 != sq) load_batch(idx, s0);
#pragma unroll
        for (int j = 0; j < 8; ++j) o = fmaf(bv[j], (bm[j].y > 0.f) ? expf(bm[j].x - M) : 0.f, o);
      }
      __syncthreads();                         // previous round's readers are done with sO
      sO[sq * epw + el] = o;
      __syncthreads();
      if (sq == 0) {
        float tot = 0.f;
        for (int k = 0; k < tpe; k += 4)
          tot += (sO[k * epw + el] + sO[(k + 1) * epw + el]) + (sO[(k + 2) * epw + el] + sO[(k + 3) * epw + el]);
        const float L = sL[g];
        // column g of the partials = (query tq, head gh of the group); out is [B, n_q, Hq, D]
        const int tq = g / d.G, gh = g % d.G;
        a.out[((((size_t)b * a.n_q + tq) * d.Hq) + (size_t)hk * d.G + gh) * D + (idx % D)] = (L > 0.f) ? tot / L : 0.f;
      }
    }
  }
}

// ---------------------------------------------------------------------------
// compute units of the current device (the runtime answers from its own tables; nothing is cached here)
static int cu_count() {
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
    cus = 256;
  return cus;
}

template <typename T, int G, int NW>
static void launch_main_nw(const DevDesc& d, const AttendArgs& a, dim3 grid, hipStream_t st) {
  switch (d.r) {
    case 3: hipLaunchKernelGGL((attend_main_kernel<T, G, 3, NW>), grid, dim3(64 * NW), 0, st, d, a); break;
    case 4: hipLaunchKernelGGL((attend_main_kernel<T, G, 4, NW>), grid, dim3(64 * NW), 0, st, d, a); break;
    default: hipLaunchKernelGGL((attend_main_kernel<T, G, 0, NW>), grid, dim3(64 * NW), 0, st, d, a); break;
  }
}
template <typename T, int G>
static void launch_main_r(const DevDesc& d, const AttendArgs& a, dim3 grid, hipStream_t st) {
  // 16 waves hold 128 registers each (bf16 with four heads needs 156).  us a call, four and 16 waves: float32, 1 unit of 2049 tokens, one
  // head 21.3 and 14.8, four heads 29.1 and 18.6; 2 units of 6700 tokens, four heads 32.2 and 20.1; bf16, 1 unit of 6700 tokens, two heads,
  // five rows 51.8 and 40.5
  if constexpr (G <= (sizeof(T) == 4 ? 4 : 2)) {
    if ((long long)grid.x * grid.y <= cu_count()) return launch_main_nw<T, G, 16>(d, a, grid, st);
  }
  launch_main_nw<T, G, 4>(d, a, grid, st);
}

hipError_t launch_attend_combine(const DevDesc& d, const AttendArgs& a, int n_cols, hipStream_t st) {
  const int units = d.B * d.Hkv;
  const long long tot_cap = (long long)a.ret_cap + a.vague_cap;
  int cx = (int)(a.tiles ? (a.ret_cap + 1023ll) / 1024 + (a.vague_cap + 1023ll) / 1024 : (tot_cap + 1023) / 1024);
  // few tokens and few units: workgroups for the output alone, 64 elements each, as long as the chip has room
  const int want = std::min(n_cols * D / 64, 512 / units);
  if (cx < want) cx = want;
  if (cx < 1) cx = 1;
  const dim3 grid(cx, units), block(256);
#define KVR_COMBINE(N)                                                                        \
  case N:                                                                                     \
    if (a.tiles) hipLaunchKernelGGL((attend_combine_kernel<N, true>), grid, block, 0, st, d, a); \
    else hipLaunchKernelGGL((attend_combine_kernel<N, false>), grid, block, 0, st, d, a);     \
    break;
  switch (n_cols) {
    KVR_COMBINE(1)
    KVR_COMBINE(2)
    KVR_COMBINE(4)
    KVR_COMBINE(8)
    KVR_COMBINE(16)
    default: return hipErrorInvalidValue;
  }
#undef KVR_COMBINE
  return hipGetLastError();
}

template <int G>
static hipError_t launch_g(const DevDesc& d, int dtype, const AttendArgs& a0, const AttendPlan& plan,
                           hipStream_t st, const AttendSide& sd) {
  const int units = d.B * d.Hkv;
  AttendArgs a = a0;
  a.n_slices = plan.n_slices;
  a.n_rslices = plan.n_rslices;
  a.n_vslices = plan.n_vslices;
  if (sd.prof_start) (void)hipEventRecord(sd.prof_start, st);
  hipError_t e = hipSuccess;
  // 1. retained slots (or, for f32 storage without staging, everything at once)
  a.slice_tokens = plan.rslice_tokens;
  a.tok_start = 0;
  a.slice0 = 0;
  // Where the general staged kernel takes the list (the others hold the slots in their own launch): the retained kernel is
  // bound by HBM, the staged kernel by the vector ALUs and LDS, so when the caller lends a second stream they run side by
  // side, the retained kernel on that stream, forked from and joined back into `st` with the caller's two events.
  // Only when the staged kernel fills the chip several times over: a launch of a few workgroups is
  // short, the fork and join then cost more than the overlap saves, and the retained kernel is better
  // off with a launch as wide as its item count than with one workgroup per CU.
  const int cus = cu_count();
  const bool big = (long long)units * plan.n_vslices >= 2ll * cus;
  // And only where a CU holds a workgroup of each.
  const int side_lds = !plan.pair && sd.stream != nullptr && big ? attend_side_lds(d, plan) : 0;
  const bool side = side_lds > 0;
  if (plan.pair) {
    if (plan.ret_own) e = launch_attend_retained(d, a, plan.n_rslices, 0, 0, st);
    if (e == hipSuccess) e = plan.ch == 64 ? launch_attend_pair64(d, a, plan, st) : launch_attend_pair16(d, a, plan, st);
  } else if (side) {
    e = hipEventRecord(sd.fork, st);
    if (e == hipSuccess) e = hipStreamWaitEvent(sd.stream, sd.fork, 0);
    if (e == hipSuccess) {
      // From here on the side stream may hold work that writes the caller's workspace: whatever
      // fails below, `st` is made to wait for it before this call returns.
      e = launch_attend_retained(d, a, plan.n_rslices, cus, side_lds, sd.stream);
      const hipError_t ej = hipEventRecord(sd.join, sd.stream);
      if (e == hipSuccess && ej == hipSuccess) e = launch_attend_vague_staged(d, a, plan, st);
      hipError_t ew = (ej == hipSuccess) ? hipStreamWaitEvent(st, sd.join, 0) : ej;
      if (ew != hipSuccess) {
        (void)hipStreamSynchronize(sd.stream);      // no event to order by: wait on the host (error path only)
        if (e == hipSuccess) e = ew;
      }
    }
  } else if (plan.streamed) {
    // no causal mask in a decode call: every listed token is visible (n_ctx = null)
    e = launch_attend_multi_staged(d, a, nullptr, 1, plan.stream, st);
  } else if (plan.mfma_retained) {
    e = launch_attend_retained(d, a, plan.n_rslices, 0, 0, st);
  } else {
    a.tok_limit = plan.staged ? a.ret_cap : a.ret_cap + a.vague_cap;
    dim3 grid(plan.n_rslices, units);
    if (dtype == KVR_F32) launch_main_r<float, G>(d, a, grid, st);
    else launch_main_r<bf16_t, G>(d, a, grid, st);
    e = hipGetLastError();
  }
  // 2. the Vague list
  if (side || plan.pair || plan.streamed) {
    // already launched above
  } else if (e == hipSuccess && plan.staged) {
    e = launch_attend_vague_staged(d, a, plan, st);
  } else if (e == hipSuccess && plan.mfma_retained && plan.n_vslices > 0) {
    a.slice_tokens = plan.vslice_tokens;
    a.tok_start = a.ret_cap;
    a.tok_limit = a.ret_cap + a.vague_cap;
    a.slice0 = plan.n_rslices;
    dim3 grid(plan.n_vslices, units);
    launch_main_r<bf16_t, G>(d, a, grid, st);
    e = hipGetLastError();
  }
  // 3. merge
  if (e == hipSuccess) e = launch_attend_combine(d, a, G, st);
  if (sd.prof_stop) (void)hipEventRecord(sd.prof_stop, st);
  return e;
}

hipError_t launch_attend(const DevDesc& d, int dtype, const AttendArgs& a, const AttendPlan& plan,
                         hipStream_t st, const AttendSide& sd) {
  switch (d.G) {
    case 1: return launch_g<1>(d, dtype, a, plan, st, sd);
    case 2: return launch_g<2>(d, dtype, a, plan, st, sd);
    case 4: return launch_g<4>(d, dtype, a, plan, st, sd);
    case 8: return launch_g<8>(d, dtype, a, plan, st, sd);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace kvr
