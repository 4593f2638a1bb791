// kvr_swap_back: the swap loop of Algorithm 3 (Recent and Candidate; its second
// while-loop): as long as the weakest Candidate's score times ReplaceRate is below
// the strongest Vague token's score, that Vague token is queried from the sketch
// and deleted from it, the Candidate is popped and inserted into the sketch, and
// the queried estimate is pushed into the Candidate part in its place.
//
// One workgroup per unit, at most max_swaps rounds.
//
// Ranking.  Every token gets the 64-bit key
//     (order-preserving image of its float32 score) << 32 | ~position,
// the key kvr_select ranks by: "highest score, then earlier position" is the
// largest key, "lowest score, then later position" the smallest, and all keys are
// distinct.  V.Max is the largest key of the Vague index list, C.Min the smallest
// key of the retained slots outside the Recent window.
//
// One scan serves many rounds.  It leaves the m = min(max_swaps, 16) largest Vague
// keys and m smallest Candidate keys in two sorted lists in LDS.  REG: up to 26
// Vague tokens and 8 slots per thread, keys loaded once into registers, and both
// lists by one floor each in three barriers; longer parts: m workgroup-wide
// reductions, keys read again from memory.  A swap pops both heads and inserts each token's key into the
// other list; since a round removes only the head, the head of a list stays the
// true extreme of its part for m rounds (the j-th extreme of the scanned part is
// in the list for j <= m, and every key that entered the part since is in it
// too).  After m swaps the parts are scanned again.
//
// A swap.  Thread c < D owns channel c of the key tensors, thread D + c channel c
// of the value tensors: it reads its channel of the r sketch rows of the Vague
// token, takes the median (Algorithm 2), reads the Candidate's channel, writes
// sketch = round(float32(old) - estimate) and round(float32(old) + candidate)
// (one sum, one rounding, if both fall into the same slot of a row: delete first,
// then insert), and stores the estimate into the Candidate's slot.  A channel is
// only ever touched by its own thread, so no barrier is needed between the query
// and the update.  Thread 2 D exchanges the two positions in ret_pos / vague_pos.
//
// Bound by memory round trips.  All swaps of a scan are decided before the first is carried out, so the values of four
// swaps are requested together; a value that an earlier one of the four has just written (the same slot of a sketch row, the
// same retained slot: equal for all channels) is taken from registers instead.  One swap at a time, each waiting for its loads behind
// the stores of the one before, and wave extremes by 64-bit shuffles: 32 units, 4 swaps 41 -> 32.5 us.
#include "kvr_launch.h"
#include "kvr_update.h"

namespace kvr {

constexpr int SWP_THREADS = 1024;
constexpr int SWP_WAVES = SWP_THREADS / WAVE;
constexpr int SWP_KV = 26;                             // REG: Vague keys per thread
constexpr int SWP_KC = 8;                              // REG: slot keys per thread
constexpr int SWP_LIST = 16;                           // list length per scan
constexpr int SWP_ROOM = SWP_KV * SWP_LIST;            // keys of SWP_LIST threads
constexpr unsigned long long SWP_NONE_MAX = 0ull;      // below every key (the low word ~position of a key is never 0)
constexpr unsigned long long SWP_NONE_MIN = ~0ull;     // above every key of a finite score

struct SwapShared {
  unsigned long long wmax[2][SWP_WAVES], wmin[2][SWP_WAVES];
  unsigned long long vkey[SWP_LIST + 1], ckey[SWP_LIST + 1];   // sorted: vkey descending, ckey ascending
  int vidx[SWP_LIST + 1], cslot[SWP_LIST + 1];                 // Vague list index / retained slot of each entry
  int nvl, ncl;                                                // entries in use
  int go;                                                      // swaps decided for this scan
  // REG, [0] Vague keys, [1] Candidate keys inverted, so that both parts look for their largest (0 = none)
  unsigned long long top[2][SWP_WAVES * SWP_LIST];             // each wave's largest thread maxima
  unsigned long long floor[2];                                 // the m-th largest thread maximum of the workgroup
  unsigned long long lkey[2][SWP_ROOM];                        // keys from the floor up, in any order
  int lidx[2][SWP_ROOM], ln[2];
  int dec[SWP_LIST][4];                                        // per swap: Vague position, Candidate position, list index, slot
};

// key of (score, position): larger = higher score, then earlier position.  -0 ranks as +0.
// Never 0 and never ~0 for a valid position (0 <= pos < 2^30) and a finite score.
__device__ __forceinline__ unsigned long long swap_key(float score, int pos) {
  uint32_t b = __float_as_uint(score);
  if (b == 0x80000000u) b = 0u;
  const uint32_t mono = b ^ ((b >> 31) ? 0xffffffffu : 0x80000000u);
  return ((unsigned long long)mono << 32) | (uint32_t)(~(uint32_t)pos);
}
// the score a key was made from (-0 comes back as +0, which compares and multiplies alike)
__device__ __forceinline__ float key_score(unsigned long long key) {
  const uint32_t mono = (uint32_t)(key >> 32);
  return __uint_as_float(mono ^ ((mono >> 31) ? 0x80000000u : 0xffffffffu));
}

__device__ __forceinline__ unsigned long long vague_key_at(const int32_t* vp, const float* sc, int i, int nv,
                                                           long long n_cap) {
  if (i >= nv) return SWP_NONE_MAX;
  const int pos = vp[i];
  return (pos >= 0 && pos < n_cap) ? swap_key(sc[pos], pos) : SWP_NONE_MAX;
}
__device__ __forceinline__ unsigned long long cand_key_at(const int32_t* rp, const float* sc, int s, int ret_cap,
                                                          int recent_from, long long n_cap) {
  if (s >= ret_cap) return SWP_NONE_MIN;
  const int pos = rp[s];
  return (pos >= 0 && pos < recent_from && pos < n_cap) ? swap_key(sc[pos], pos) : SWP_NONE_MIN;
}

// Scan both parts of a unit and leave the m largest Vague keys and the m
// smallest Candidate keys, in order, in sh (with the Vague list index / the
// retained slot of each).  Not inlined: the keys it holds in registers are
// dead when it returns and must not count against the caller's registers.
//
// Every one of the m largest keys is at least as large as the m-th largest of the threads' maxima (m threads have a key from
// there up).  So: a maximum per thread, the m largest per wave, the m-th largest of all (one wave per part), the keys from
// there up into a list (at most those of m threads), and the list's m largest in order (one wave per part): three barriers whatever m
// is, and every key is looked at twice, where m rounds of a workgroup-wide extreme took two barriers and another look each.
__device__ __noinline__ void swap_build_lists(SwapShared& sh, const int32_t* vp, const int32_t* rp,
                                              const float* sc, int nv, int ret_cap, int recent_from,
                                              long long n_cap, int m) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // all positions first, then all scores (clamped addresses, no branches): two
  // rounds of independent loads instead of one dependent pair per token
  int pv[SWP_KV], pc[SWP_KC];
#pragma unroll
  for (int j = 0; j < SWP_KV; ++j) {
    const int i = j * SWP_THREADS + tid;
    pv[j] = vp[min(i, max(nv - 1, 0))];
    if (i >= nv || pv[j] >= n_cap) pv[j] = -1;
  }
#pragma unroll
  for (int j = 0; j < SWP_KC; ++j) {
    const int s_ = j * SWP_THREADS + tid;
    pc[j] = rp[min(s_, ret_cap - 1)];
    if (s_ >= ret_cap || pc[j] >= recent_from || pc[j] >= n_cap) pc[j] = -1;
  }
  float fv[SWP_KV], fc[SWP_KC];
#pragma unroll
  for (int j = 0; j < SWP_KV; ++j) fv[j] = sc[max(pv[j], 0)];
#pragma unroll
  for (int j = 0; j < SWP_KC; ++j) fc[j] = sc[max(pc[j], 0)];
  if (tid < 2) sh.ln[tid] = 0;
  // the halves of a key: the score's image, and ~position (Vague) or, of the inverted key, the position (Candidate)
  uint32_t hv[SWP_KV], hc[SWP_KC];
  uint32_t bv = 0u, bc = 0u;
#pragma unroll
  for (int j = 0; j < SWP_KV; ++j) {
    hv[j] = pv[j] >= 0 ? (uint32_t)(swap_key(fv[j], 0) >> 32) : 0u;
    bv = max(bv, hv[j]);
  }
#pragma unroll
  for (int j = 0; j < SWP_KC; ++j) {
    hc[j] = pc[j] >= 0 ? ~(uint32_t)(swap_key(fc[j], 0) >> 32) : 0u;
    bc = max(bc, hc[j]);
  }
  uint32_t lv = 0u, lc = 0u;
#pragma unroll
  for (int j = 0; j < SWP_KV; ++j) lv = max(lv, hv[j] == bv ? ~(uint32_t)pv[j] : 0u);
#pragma unroll
  for (int j = 0; j < SWP_KC; ++j) lc = max(lc, hc[j] == bc ? (uint32_t)pc[j] : 0u);
  const unsigned long long tv = bv ? ((unsigned long long)bv << 32) | lv : 0ull;
  const unsigned long long tc = bc ? ((unsigned long long)bc << 32) | lc : 0ull;
  {
    unsigned long long xv = tv, xc = tc;
    for (int k = 0; k < m; ++k) {
      const unsigned long long gv = wave_max_u64(xv), gc = wave_max_u64(xc);
      if (lane == 0) { sh.top[0][wave * m + k] = gv; sh.top[1][wave * m + k] = gc; }
      if (xv == gv) xv = 0ull;
      if (xc == gc) xc = 0ull;
    }
  }
  wg_lds_barrier();
  if (wave < 2) {
    unsigned long long x[SWP_LIST / 4];              // SWP_WAVES * m entries over 64 lanes
#pragma unroll
    for (int e = 0; e < SWP_LIST / 4; ++e) x[e] = (e * 64 + lane < SWP_WAVES * m) ? sh.top[wave][e * 64 + lane] : 0ull;
    unsigned long long g = 0ull;
    for (int k = 0; k < m; ++k) {
      unsigned long long y = x[0];
#pragma unroll
      for (int e = 1; e < SWP_LIST / 4; ++e) y = x[e] > y ? x[e] : y;
      g = wave_max_u64(y);
#pragma unroll
      for (int e = 0; e < SWP_LIST / 4; ++e)
        if (x[e] == g) x[e] = 0ull;
    }
    if (lane == 0) sh.floor[wave] = g;               // 0: fewer than m threads have a key
  }
  wg_lds_barrier();
  const unsigned long long floor_v = sh.floor[0], floor_c = sh.floor[1];
  if (tv >= floor_v && tv != 0ull) {
#pragma unroll
    for (int j = 0; j < SWP_KV; ++j) {
      const unsigned long long key = ((unsigned long long)hv[j] << 32) | ~(uint32_t)pv[j];
      if (hv[j] != 0u && key >= floor_v) {
        const int at = atomicAdd(&sh.ln[0], 1);
        if (at < SWP_ROOM) { sh.lkey[0][at] = key; sh.lidx[0][at] = j * SWP_THREADS + tid; }
      }
    }
  }
  if (tc >= floor_c && tc != 0ull) {
#pragma unroll
    for (int j = 0; j < SWP_KC; ++j) {
      const unsigned long long key = ((unsigned long long)hc[j] << 32) | (uint32_t)pc[j];
      if (hc[j] != 0u && key >= floor_c) {
        const int at = atomicAdd(&sh.ln[1], 1);
        if (at < SWP_ROOM) { sh.lkey[1][at] = key; sh.lidx[1][at] = j * SWP_THREADS + tid; }
      }
    }
  }
  wg_lds_barrier();
  if (wave < 2) {
    const int n = min(sh.ln[wave], SWP_ROOM);      // more only if a position is listed twice
    unsigned long long prev = ~0ull;
    int found = 0;
    for (int k = 0; k < m; ++k) {
      unsigned long long best = 0ull;
      int at = 0;
      for (int e = lane; e < n; e += 64) {
        const unsigned long long key = sh.lkey[wave][e];
        if (key < prev && key > best) { best = key; at = e; }
      }
      const unsigned long long g = wave_max_u64(best);
      if (g == 0ull) break;
      if (best == g) {                               // keys are distinct: one owner
        if (wave == 0) { sh.vkey[k] = g; sh.vidx[k] = sh.lidx[0][at]; }
        else { sh.ckey[k] = ~g; sh.cslot[k] = sh.lidx[1][at]; }
      }
      prev = g;
      ++found;
    }
    if (lane == 0) { if (wave == 0) sh.nvl = found; else sh.ncl = found; }
  }
  wg_lds_barrier();
}

// The same for parts that do not fit registers: m rounds of a workgroup-wide extreme, keys read again from memory by the
// threads that need their next one.
__device__ __noinline__ void swap_build_lists_long(SwapShared& sh, const int32_t* vp, const int32_t* rp,
                                              const float* sc, int nv, int ret_cap, int recent_from,
                                              long long n_cap, int m) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // A thread offers the best key it still has; only the thread whose key was taken
  // looks for its next one (the taken keys are exactly those beyond the last extreme).
  unsigned long long vprev = SWP_NONE_MIN, cprev = SWP_NONE_MAX;       // previous extremes (exclusive bounds)
  int n_vl = 0, n_cl = 0;
  unsigned long long kmax = SWP_NONE_MAX, kmin = SWP_NONE_MIN;
  int imax = -1, smin = -1;
  bool redo_v = true, redo_c = true;
  for (int k = 0; k < m; ++k) {
    if (redo_v) {
      kmax = SWP_NONE_MAX;
      imax = -1;
      for (int i = tid; i < nv; i += SWP_THREADS) {
        const unsigned long long key = vague_key_at(vp, sc, i, nv, n_cap);
        if (key < vprev && key > kmax) { kmax = key; imax = i; }
      }
      redo_v = false;
    }
    if (redo_c) {
      kmin = SWP_NONE_MIN;
      smin = -1;
      for (int s_ = tid; s_ < ret_cap; s_ += SWP_THREADS) {
        const unsigned long long key = cand_key_at(rp, sc, s_, ret_cap, recent_from, n_cap);
        if (key > cprev && key < kmin) { kmin = key; smin = s_; }
      }
      redo_c = false;
    }
    const unsigned long long wmx = wave_max_u64(kmax), wmn = wave_min_u64(kmin);
    if (lane == 0) { sh.wmax[k & 1][wave] = wmx; sh.wmin[k & 1][wave] = wmn; }
    __syncthreads();
    unsigned long long gmax = sh.wmax[k & 1][0], gmin = sh.wmin[k & 1][0];
#pragma unroll
    for (int w_ = 1; w_ < SWP_WAVES; ++w_) {
      gmax = sh.wmax[k & 1][w_] > gmax ? sh.wmax[k & 1][w_] : gmax;
      gmin = sh.wmin[k & 1][w_] < gmin ? sh.wmin[k & 1][w_] : gmin;
    }
    // keys are distinct: each extreme has exactly one owner
    if (gmax != SWP_NONE_MAX) {
      if (kmax == gmax) { sh.vkey[n_vl] = gmax; sh.vidx[n_vl] = imax; redo_v = true; }
      ++n_vl;
      vprev = gmax;
    }
    if (gmin != SWP_NONE_MIN) {
      if (kmin == gmin) { sh.ckey[n_cl] = gmin; sh.cslot[n_cl] = smin; redo_c = true; }
      ++n_cl;
      cprev = gmin;
    }
    if (gmax == SWP_NONE_MAX && gmin == SWP_NONE_MIN) break;             // both parts exhausted (uniform)
  }
  if (tid == 0) { sh.nvl = n_vl; sh.ncl = n_cl; }
  __syncthreads();
}

// Carry out the swaps [k0, k0 + n) of sh.dec, n <= NB, on this thread's channel.  sx: the channel in the unit's sketch, xr: in the
// unit's retained rows.  RR: rows there is room for, r <= RR.
template <typename T, int NB, int RR>
__device__ __forceinline__ void swap_apply(const DevDesc& d, const SwapShared& sh, int k0, int n, T* sx, T* xr, bool flip) {
  int off_d[NB][RR], off_c[NB][RR], slot[NB];        // uniform
  uint32_t neg_d[NB], neg_c[NB];
  float val_d[NB][RR], val_c[NB][RR], cand[NB];
#pragma unroll
  for (int k = 0; k < NB; ++k) {
    // past n: the last swap's addresses again, nothing is stored
    const int kk = k0 + min(k, n - 1);
    const int J = __builtin_amdgcn_readfirstlane(sh.dec[kk][0]), pc = __builtin_amdgcn_readfirstlane(sh.dec[kk][1]);
    slot[k] = __builtin_amdgcn_readfirstlane(sh.dec[kk][3]);
    neg_d[k] = neg_c[k] = 0u;
#pragma unroll
    for (int i = 0; i < RR; ++i) {
      off_d[k][i] = off_c[k][i] = 0;
      val_d[k][i] = val_c[k][i] = 0.f;
      if (i < d.r) {
        off_d[k][i] = (i * d.w + bucket_of(d, i, J)) * D;
        off_c[k][i] = (i * d.w + bucket_of(d, i, pc)) * D;
        if (flip && sign_neg(d, i, J)) neg_d[k] |= 1u << i;
        if (flip && sign_neg(d, i, pc)) neg_c[k] |= 1u << i;
        val_d[k][i] = Store<T>::load1(sx + off_d[k][i]);
        val_c[k][i] = Store<T>::load1(sx + off_c[k][i]);
      }
    }
    cand[k] = Store<T>::load1(xr + (size_t)slot[k] * D);
  }
#pragma unroll
  for (int k = 0; k < NB; ++k) {
    if (k >= n) break;
    // what the earlier swaps of this call have written since
#pragma unroll
    for (int j = 0; j < k; ++j) {
#pragma unroll
      for (int i = 0; i < RR; ++i) {
        if (i < d.r) {
          if (off_d[k][i] == off_d[j][i]) val_d[k][i] = val_d[j][i];
          if (off_d[k][i] == off_c[j][i]) val_d[k][i] = val_c[j][i];
          if (off_c[k][i] == off_d[j][i]) val_c[k][i] = val_d[j][i];
          if (off_c[k][i] == off_c[j][i]) val_c[k][i] = val_c[j][i];
        }
      }
      if (slot[k] == slot[j]) cand[k] = cand[j];
    }
    float rows[KVR_MAX_ROWS];
#pragma unroll
    for (int i = 0; i < KVR_MAX_ROWS; ++i) rows[i] = (i < RR) ? (((neg_d[k] >> i) & 1u) ? -val_d[k][i < RR ? i : 0] : val_d[k][i < RR ? i : 0]) : 0.f;
    const float est = median_rows<0, T>(rows, d.r, d.median_mode);
#pragma unroll
    for (int i = 0; i < RR; ++i) {
      if (i < d.r) {
        // delete first, then insert; float32 sums, one rounding per touched slot
        const float gd = ((neg_d[k] >> i) & 1u) ? -1.f : 1.f;
        const float gc = ((neg_c[k] >> i) & 1u) ? -1.f : 1.f;
        float acc = val_d[k][i] + (-gd) * est;
        if (off_c[k][i] == off_d[k][i]) {
          acc = acc + gc * cand[k];
          Store<T>::store1(sx + off_d[k][i], acc);
          val_d[k][i] = val_c[k][i] = Store<T>::round(acc);
        } else {
          const float ins = val_c[k][i] + gc * cand[k];
          Store<T>::store1(sx + off_d[k][i], acc);
          Store<T>::store1(sx + off_c[k][i], ins);
          val_d[k][i] = Store<T>::round(acc);
          val_c[k][i] = Store<T>::round(ins);
        }
      }
    }
    Store<T>::store1(xr + (size_t)slot[k] * D, est);
    cand[k] = Store<T>::round(est);                  // from here on: what the slot holds
  }
}

template <typename T, bool REG>
__global__ __launch_bounds__(SWP_THREADS) void swap_back_kernel(
    DevDesc d, const float* __restrict__ scores, long long n_cap, T* k_ret, T* v_ret, int32_t* ret_pos,
    int ret_cap, const int32_t* __restrict__ n_ctx, int n_recent, float replace_rate, int max_swaps, T* sk,
    T* sv, int32_t* vague_pos, const int32_t* __restrict__ n_vague, int vague_cap,
    int32_t* __restrict__ n_swapped, int32_t* __restrict__ swap_log) {
  const int unit = blockIdx.x;
  const int b = unit / d.Hkv;
  const int tid = threadIdx.x;
  __shared__ SwapShared sh;
  int32_t* rp = ret_pos + (size_t)unit * ret_cap;
  int32_t* vp = vague_pos + (size_t)unit * vague_cap;
  const float* sc = scores + (size_t)unit * n_cap;
  const int recent_from = n_ctx[b] - n_recent;
  const int nv = clampi(n_vague[unit], 0, vague_cap);
  int done = 0;

  while (done < max_swaps) {
    const int m = min(max_swaps - done, SWP_LIST);
    if constexpr (REG) swap_build_lists(sh, vp, rp, sc, nv, ret_cap, recent_from, n_cap, m);
    else swap_build_lists_long(sh, vp, rp, sc, nv, ret_cap, recent_from, n_cap, m);

    // ---- up to m swaps on the lists.  Which tokens change places depends on scores and
    //      positions only, not on sketch contents: the first wave decides all swaps of this
    //      scan first and leaves the pairs in LDS, then the channel threads carry them out one
    //      after the other without a barrier in between (a later swap that touches a slot
    //      or a retained row of an earlier one is ordered by the thread's own program
    //      order: a channel is only ever touched by its own thread). -------------------------
    if (tid < WAVE) {
      // lane i holds entry i of both lists
      int nvl = sh.nvl, ncl = sh.ncl, n_dec = 0;
      unsigned long long vk = tid < nvl ? sh.vkey[tid] : SWP_NONE_MAX, ck = tid < ncl ? sh.ckey[tid] : SWP_NONE_MIN;
      int vi = tid < nvl ? sh.vidx[tid] : 0, cs = tid < ncl ? sh.cslot[tid] : 0;
      auto next = [](unsigned long long v) {                              // of the lane above
        const uint32_t lo = __shfl_down((int)(uint32_t)v, 1), hi = __shfl_down((int)(uint32_t)(v >> 32), 1);
        return ((unsigned long long)hi << 32) | lo;
      };
      auto first = [](unsigned long long v) {
        const uint32_t lo = __builtin_amdgcn_readfirstlane((int)(uint32_t)v), hi = __builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
        return ((unsigned long long)hi << 32) | lo;
      };
      while (n_dec < m && nvl > 0 && ncl > 0) {
        const unsigned long long kv = first(vk), kc = first(ck);
        const float lhs = key_score(kc) * replace_rate;                   // float32 product, float32 compare
        if (!(lhs < key_score(kv))) break;
        const int v_idx = __builtin_amdgcn_readfirstlane(vi), c_slot = __builtin_amdgcn_readfirstlane(cs);
        if (tid == 0) {
          sh.dec[n_dec][0] = (int)(~(uint32_t)kv);
          sh.dec[n_dec][1] = (int)(~(uint32_t)kc);
          sh.dec[n_dec][2] = v_idx;
          sh.dec[n_dec][3] = c_slot;
        }
        ++n_dec;
        // pop both heads; the Candidate's key enters the Vague list (at the Vague token's list
        // index), the Vague token's key enters the Candidate list (in the Candidate's slot).  What stays in front of the
        // new entry moves up by one, what comes behind it stays where it was.
        const unsigned long long vn = next(vk), cn = next(ck);
        const int vin = __shfl_down(vi, 1), csn = __shfl_down(cs, 1);
        const int va = __popcll(__ballot(tid < nvl - 1 && vn > kc)), ca = __popcll(__ballot(tid < ncl - 1 && cn < kv));
        if (tid < va) { vk = vn; vi = vin; }
        else if (tid == va) { vk = kc; vi = v_idx; }
        if (tid < ca) { ck = cn; cs = csn; }
        else if (tid == ca) { ck = kv; cs = c_slot; }
      }
      if (tid == 0) sh.go = n_dec;
    }
    __syncthreads();
    const int swaps_here = sh.go;
    const bool stop = swaps_here < m;                                       // the loop condition failed (uniform)
    if (tid < 2 * D) {
      const bool is_v = tid >= D;
      const int c = is_v ? tid - D : tid;
      T* sx = (is_v ? sv : sk) + (size_t)unit * d.r * d.w * D + c;
      T* xr = (is_v ? v_ret : k_ret) + (size_t)unit * ret_cap * D + c;
      const bool flip = is_v ? (d.sign_mask & 2) != 0 : (d.sign_mask & 1) != 0;
      if (d.r <= 4) {
        for (int k = 0; k < swaps_here; k += 4) swap_apply<T, 4, 4>(d, sh, k, min(4, swaps_here - k), sx, xr, flip);
      } else {
        for (int k = 0; k < swaps_here; k += 2) swap_apply<T, 2, KVR_MAX_ROWS>(d, sh, k, min(2, swaps_here - k), sx, xr, flip);
      }
    } else if (tid == 2 * D) {
      for (int k = 0; k < swaps_here; ++k) {
        const int J = sh.dec[k][0], pc = sh.dec[k][1];
        rp[sh.dec[k][3]] = J;
        vp[sh.dec[k][2]] = pc;
        if (swap_log) {
          swap_log[((size_t)unit * max_swaps + done + k) * 2] = J;
          swap_log[((size_t)unit * max_swaps + done + k) * 2 + 1] = pc;
        }
      }
    }
    __syncthreads();             // sh.go / the pairs may be overwritten; positions visible to a later scan
    done += swaps_here;
    if (stop) break;
  }
  if (tid == 0 && n_swapped) n_swapped[unit] = done;
}

template <typename T>
static void launch_swap_t(const DevDesc& d, const float* scores, long long n_cap, void* k_ret, void* v_ret,
                          int32_t* ret_pos, int ret_cap, const int32_t* n_ctx, int n_recent, float replace_rate,
                          int max_swaps, void* sk, void* sv, int32_t* vague_pos, const int32_t* n_vague,
                          int vague_cap, int32_t* n_swapped, int32_t* swap_log, hipStream_t st) {
  const dim3 grid(d.B * d.Hkv), block(SWP_THREADS);
  // keys in registers when both parts fit (vague_cap bounds n_vague)
  if (vague_cap <= SWP_KV * SWP_THREADS && ret_cap <= SWP_KC * SWP_THREADS)
    hipLaunchKernelGGL((swap_back_kernel<T, true>), grid, block, 0, st, d, scores, n_cap, (T*)k_ret, (T*)v_ret,
                       ret_pos, ret_cap, n_ctx, n_recent, replace_rate, max_swaps, (T*)sk, (T*)sv, vague_pos,
                       n_vague, vague_cap, n_swapped, swap_log);
  else
    hipLaunchKernelGGL((swap_back_kernel<T, false>), grid, block, 0, st, d, scores, n_cap, (T*)k_ret, (T*)v_ret,
                       ret_pos, ret_cap, n_ctx, n_recent, replace_rate, max_swaps, (T*)sk, (T*)sv, vague_pos,
                       n_vague, vague_cap, n_swapped, swap_log);
}

hipError_t launch_swap_back(const DevDesc& d, int dtype, const float* scores, long long n_cap, void* k_ret,
                            void* v_ret, int32_t* ret_pos, int ret_cap, const int32_t* n_ctx, int n_recent,
                            float replace_rate, int max_swaps, void* sk, void* sv, int32_t* vague_pos,
                            const int32_t* n_vague, int vague_cap, int32_t* n_swapped, int32_t* swap_log,
                            hipStream_t st) {
  if (dtype == KVR_F32)
    launch_swap_t<float>(d, scores, n_cap, k_ret, v_ret, ret_pos, ret_cap, n_ctx, n_recent, replace_rate,
                         max_swaps, sk, sv, vague_pos, n_vague, vague_cap, n_swapped, swap_log, st);
  else
    launch_swap_t<bf16_t>(d, scores, n_cap, k_ret, v_ret, ret_pos, ret_cap, n_ctx, n_recent, replace_rate,
                          max_swaps, sk, sv, vague_pos, n_vague, vague_cap, n_swapped, swap_log, st);
  return hipGetLastError();
}

}  // namespace kvr
