// Device bodies of the three small per-step updates of a unit's storage
// (Recent and Candidate, Algorithm 3; Vague Sketch, Algorithm 1):
//   append_body        R.Push of the new token into the lowest empty slot
//   select_body        which retained tokens leave for the Vague part
//   encode_small_body  V.Insert of up to 64 listed tokens
// Each is called by all threads of a workgroup for one unit.  The stand-alone
// kernels of kvr_append / kvr_select / kvr_encode and the fused kvr_step_update
// kernel are thin wrappers around them.
#pragma once
#include "kvr_dev.h"

namespace kvr {

constexpr int SEL_THREADS = 1024;
constexpr int SEL_WAVES = SEL_THREADS / WAVE;
constexpr int SEL_SMALL = 8;                     // up to this many evictions: repeated minimum
constexpr unsigned long long KEY_NONE = ~0ull;   // not a valid key (it would be a NaN score at position 0)
constexpr int ENC_SMALL_CAP = 64;
constexpr int SEL_DIGIT = 11;                    // bits per radix pass
constexpr int SEL_BINS = 1 << SEL_DIGIT;         // two per thread
constexpr int SEL_PLACE_CHUNKS = 128;            // chunks of SEL_THREADS slots that are emitted together

struct SelShared {
  union {
    unsigned hist[SEL_BINS];                       // radix select
    int place[SEL_PLACE_CHUNKS * SEL_WAVES];       // emission: evictions per (chunk, wave), then where each starts
  };
  unsigned long long wmin[SEL_WAVES];
  unsigned long long prefix;
  int wsum[SEL_WAVES];
  int krem, cnt, whole;
  int nlist, list[SEL_SMALL];        // small eviction counts: the evicted slots, in any order
};

// Eviction list of one unit in LDS: how the fused update kernel hands the selection's result to the
// insert without a round trip through global memory (the lists in global memory are written as well).
struct EvictHandOver {
  int cnt;                           // 0 if nothing is evicted or the lists would overflow
  int slot[ENC_SMALL_CAP];
  int pos[ENC_SMALL_CAP];
};

// Barrier for what a workgroup exchanges through LDS: unlike __syncthreads it does not wait for the wave's global stores
// (lists, freed slots, the new row), a memory round trip each time.
__device__ __forceinline__ void wg_lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// ---------------------------------------------------------------------------
// append
// ---------------------------------------------------------------------------
// NT = threads of the workgroup.  Returns (in every thread) the slot used, or -1.
template <typename T, int NT>
__device__ __forceinline__ int append_body(const DevDesc& d, int unit, const T* __restrict__ k_new,
                                           const T* __restrict__ v_new, const int32_t* __restrict__ n_ctx,
                                           T* __restrict__ k_ret, T* __restrict__ v_ret,
                                           int32_t* __restrict__ ret_pos, int ret_cap) {
  constexpr int VEC = Store<T>::VEC;
  constexpr int LPT = D / VEC;     // 16 (bf16) or 32 (f32) lanes copy one row
  const int tid = threadIdx.x;
  int32_t* rp = ret_pos + (size_t)unit * ret_cap;
  __shared__ int s_free;
  if (tid == 0) s_free = 0x7fffffff;
  __syncthreads();
  int mine = 0x7fffffff;
  for (int s0 = 0; s0 < ret_cap; s0 += NT * 8) {       // lowest empty slot, 8 independent loads a round
    int p[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int s = s0 + u * NT + tid;
      p[u] = (s < ret_cap) ? rp[s] : 0;
    }
#pragma unroll
    for (int u = 7; u >= 0; --u) {
      const int s = s0 + u * NT + tid;
      if (s < ret_cap && p[u] < 0 && s < mine) mine = s;
    }
  }
  if (mine != 0x7fffffff) atomicMin(&s_free, mine);
  __syncthreads();
  const int s = s_free;
  if (s >= ret_cap) return -1;
  const size_t dst = ((size_t)unit * ret_cap + s) * D;
  if (tid < LPT) {
    const uint4 v = *reinterpret_cast<const uint4*>(k_new + (size_t)unit * D + tid * VEC);
    *reinterpret_cast<uint4*>(k_ret + dst + tid * VEC) = v;
  } else if (tid < 2 * LPT) {
    const int l2 = tid - LPT;
    const uint4 v = *reinterpret_cast<const uint4*>(v_new + (size_t)unit * D + l2 * VEC);
    *reinterpret_cast<uint4*>(v_ret + dst + l2 * VEC) = v;
  }
  if (tid == 0) rp[s] = n_ctx[unit / d.Hkv] - 1;
  return s;
}

// The stores of the append into slot s (>= ret_cap: there is no empty slot).  row_in: this thread's 16 bytes of the new K row
// (tid < LPT) or V row (tid < 2 LPT), loaded by the caller ahead of time.
template <typename T>
__device__ __forceinline__ void append_store(const DevDesc& d, int unit, const int32_t* __restrict__ n_ctx,
                                             T* __restrict__ k_ret, T* __restrict__ v_ret,
                                             int32_t* __restrict__ ret_pos, int ret_cap, int s, uint4 row_in) {
  constexpr int VEC = Store<T>::VEC;
  constexpr int LPT = D / VEC;
  const int tid = threadIdx.x;
  if (s >= ret_cap) return;
  const size_t dst = ((size_t)unit * ret_cap + s) * D;
  if (tid < LPT) *reinterpret_cast<uint4*>(k_ret + dst + tid * VEC) = row_in;
  else if (tid < 2 * LPT) *reinterpret_cast<uint4*>(v_ret + dst + (tid - LPT) * VEC) = row_in;
  if (tid == 0) ret_pos[(size_t)unit * ret_cap + s] = n_ctx[unit / d.Hkv] - 1;
}

// ---------------------------------------------------------------------------
// select
// ---------------------------------------------------------------------------
// key of a slot from its position and the token's score there (scv is read only if the position is eligible)
__device__ __forceinline__ bool pos_key(int pos, float scv, int slot, int ret_cap, int recent_from, long long n_cap,
                                        unsigned long long& key) {
  if (slot >= ret_cap) return false;
  if (pos < 0 || pos >= recent_from || pos >= n_cap) return false;
  uint32_t b = __float_as_uint(scv);
  if (b == 0x80000000u) b = 0u;                                   // -0 ranks as +0
  const uint32_t mono = b ^ ((b >> 31) ? 0xffffffffu : 0x80000000u);
  key = ((unsigned long long)mono << 32) | (uint32_t)(~(uint32_t)pos);
  return true;
}

__device__ __forceinline__ int key_pos(unsigned long long key) { return (int)(~(uint32_t)key); }

// Minimum over a wave, in every lane: row rotations (DPP) and row exchanges on the vector ALUs.
template <int CTRL>
__device__ __forceinline__ unsigned long long dpp_min_u64(unsigned long long v) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, CTRL, 0xf, 0xf, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), CTRL, 0xf, 0xf, true);
  const unsigned long long o = ((unsigned long long)hi << 32) | lo;
  return o < v ? o : v;
}
__device__ __forceinline__ unsigned long long wave_min_u64(unsigned long long v) {
  v = dpp_min_u64<0x121>(v);
  v = dpp_min_u64<0x122>(v);
  v = dpp_min_u64<0x124>(v);
  v = dpp_min_u64<0x128>(v);
  {
    const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)v, (uint32_t)v, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(v >> 32), (uint32_t)(v >> 32), false, false);
    const unsigned long long a = ((unsigned long long)hi[0] << 32) | lo[0], b = ((unsigned long long)hi[1] << 32) | lo[1];
    v = a < b ? a : b;
  }
  const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)v, (uint32_t)v, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(v >> 32), (uint32_t)(v >> 32), false, false);
  const unsigned long long a = ((unsigned long long)hi[0] << 32) | lo[0], b = ((unsigned long long)hi[1] << 32) | lo[1];
  return a < b ? a : b;
}

__device__ __forceinline__ unsigned long long wave_max_u64(unsigned long long v) { return ~wave_min_u64(~v); }

// Sum over a wave, in every lane.
template <int CTRL>
__device__ __forceinline__ int dpp_add_i(int v) {
  return v + __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true);
}
__device__ __forceinline__ int wave_sum(int v) {
  v = dpp_add_i<0x128>(dpp_add_i<0x124>(dpp_add_i<0x122>(dpp_add_i<0x121>(v))));
  const auto a = __builtin_amdgcn_permlane16_swap((uint32_t)v, (uint32_t)v, false, false);
  v = (int)(a[0] + a[1]);
  const auto b = __builtin_amdgcn_permlane32_swap((uint32_t)v, (uint32_t)v, false, false);
  return (int)(b[0] + b[1]);
}

// Block-wide minimum of one value per thread (KEY_NONE = nothing).
__device__ __forceinline__ unsigned long long block_min(unsigned long long v, SelShared& sh) {
  v = wave_min_u64(v);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  wg_lds_barrier();                      // wmin may still be read from the previous round
  if (lane == 0) sh.wmin[wave] = v;
  wg_lds_barrier();
  unsigned long long r = sh.wmin[0];
#pragma unroll
  for (int w_ = 1; w_ < SEL_WAVES; ++w_) r = sh.wmin[w_] < r ? sh.wmin[w_] : r;
  return r;
}

// Inclusive scan of one value per thread over the workgroup; total (may be null): the sum.  The caller's barrier
// must separate two calls.
__device__ __forceinline__ int block_scan(int v, SelShared& sh, int* total = nullptr) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int incl = v;
#pragma unroll
  for (int off = 1; off < WAVE; off <<= 1) {
    const int y = __shfl_up(incl, off);
    if (lane >= off) incl += y;
  }
  if (lane == WAVE - 1) sh.wsum[wave] = incl;
  wg_lds_barrier();
  int before = 0, tot = 0;
#pragma unroll
  for (int w_ = 0; w_ < SEL_WAVES; ++w_) {
    const int c = sh.wsum[w_];
    before += (w_ < wave) ? c : 0;
    tot += c;
  }
  if (total) *total = tot;
  return incl + before;
}

// The bins, scanned from the top: pick the one where the running count reaches
// krem; updates sh.krem, ors the digit into sh.prefix and says in sh.whole whether
// all keys of that bin are among the krem.  All threads call it, two bins each.
__device__ __forceinline__ void pick_digit(SelShared& sh, int shift) {
  static_assert(SEL_BINS == 2 * SEL_THREADS, "two bins per thread");
  const int hi_bin = SEL_BINS - 1 - 2 * (int)threadIdx.x;
  const int a = (int)sh.hist[hi_bin], b = (int)sh.hist[hi_bin - 1];
  const int krem = sh.krem;
  const int incl = block_scan(a + b, sh);            // its barrier: everyone has read krem
  const int excl = incl - a - b;
  if (excl < krem && krem <= incl) {                 // exactly one thread
    const bool first = krem <= excl + a;
    const int left = first ? krem - excl : krem - excl - a;
    sh.krem = left;
    sh.whole = left == (first ? a : b);
    sh.prefix |= (unsigned long long)(first ? hi_bin : hi_bin - 1) << shift;
  }
  wg_lds_barrier();
}

// Workgroup of SEL_THREADS threads.  REG: ret_cap <= SEL_THREADS * KPT, keys live
// in registers (KPT per thread: 8 for the retained slots of a decode step, 32 for
// a 32k prompt).  Writes the eviction lists, frees the slots, appends to the Vague
// list, sets n_evict (negative = needed count on overflow, nothing evicted).
// pre, pre_sc (REG only): positions of this thread's slots and the scores at those
// positions (valid where the position is eligible), read by the caller ahead of time.
// The fused update kernel reads them before it appends the new token: while that token
// is Recent it ranks like an empty slot, so the stale value serves; with an empty Recent
// window the kernel patches the one entry.
template <bool REG, int KPT>
__device__ __forceinline__ void select_body(
    const DevDesc& d, int unit, const float* __restrict__ scores, long long n_cap,
    int32_t* __restrict__ ret_pos, int ret_cap, const int32_t* __restrict__ n_ctx, int n_recent, int k_cand,
    int32_t* __restrict__ evict_slot, int32_t* __restrict__ evict_pos, int32_t* __restrict__ n_evict,
    int evict_cap, int32_t* __restrict__ vague_pos, int32_t* __restrict__ n_vague, int vague_cap,
    const int* pre = nullptr, const float* pre_sc = nullptr, EvictHandOver* ho = nullptr,
    int eligible = -1, int nv_ahead = 0) {
  // eligible >= 0: the caller has counted the unit's eligible slots, and nv_ahead is what it read from n_vague
  const int b = unit / d.Hkv;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  int32_t* rp = ret_pos + (size_t)unit * ret_cap;
  const float* sc = scores + (size_t)unit * n_cap;
  const int recent_from = n_ctx[b] - n_recent;
  if (k_cand < 0) k_cand = 0;
  __shared__ SelShared sh;

  // keys of this thread's slots: slot = j * SEL_THREADS + tid
  unsigned long long rkey[REG ? KPT : 1];
  const int n_chunks = (ret_cap + SEL_THREADS - 1) / SEL_THREADS;
  // f(chunk, eligible, key) for the chunks [jb, je) in order, the same ones in all threads; without registers the
  // positions, then the scores of eight chunks are requested together
  auto for_keys = [&](int jb, int je, auto&& f) {
    if constexpr (REG) {
#pragma unroll
      for (int j = 0; j < KPT; ++j) f(j, rkey[j] != KEY_NONE, rkey[j]);
    } else {
      for (int j0 = jb; j0 < je; j0 += 8) {
        int p8[8];
        float s8[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int slot = (j0 + u) * SEL_THREADS + tid;
          p8[u] = (j0 + u < je && slot < ret_cap) ? rp[slot] : -1;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
          s8[u] = (p8[u] >= 0 && p8[u] < recent_from && p8[u] < n_cap) ? sc[p8[u]] : 0.f;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          unsigned long long key = KEY_NONE;
          const bool ok = pos_key(p8[u], s8[u], (j0 + u) * SEL_THREADS + tid, ret_cap, recent_from, n_cap, key);
          if (j0 + u < je) f(j0 + u, ok, key);
        }
      }
    }
  };

  // read ahead of its use, which is many barriers away
  const int nv_read = eligible >= 0 ? nv_ahead : (vague_pos && n_vague) ? n_vague[unit] : 0;
  if (tid == 0) { sh.cnt = 0; sh.prefix = 0ull; sh.krem = k_cand; sh.nlist = 0; }
  wg_lds_barrier();
  int c = 0;
  {
    if constexpr (REG) {
#pragma unroll
      for (int j = 0; j < KPT; ++j) {
        unsigned long long key = KEY_NONE;
        const bool ok = pos_key(pre[j], pre_sc[j], j * SEL_THREADS + tid, ret_cap, recent_from, n_cap, key);
        rkey[j] = ok ? key : KEY_NONE;
        c += ok ? 1 : 0;
      }
    } else {
      for_keys(0, n_chunks, [&](int, bool ok, unsigned long long) { c += ok ? 1 : 0; });
    }
  }
  if (eligible < 0) {
    if (c) atomicAdd(&sh.cnt, c);
    wg_lds_barrier();
    eligible = sh.cnt;
  }
  const int n_e = eligible - k_cand;
  if (n_e <= 0) {
    if (tid == 0) {
      n_evict[unit] = 0;
      if (ho) ho->cnt = 0;
    }
    return;
  }
  const int nv_old = (vague_pos && n_vague) ? clampi(nv_read, 0, vague_cap) : 0;
  if (n_e > evict_cap || (vague_pos && n_vague && nv_old + n_e > vague_cap)) {
    if (tid == 0) {
      n_evict[unit] = -n_e;
      if (ho) ho->cnt = 0;
    }
    return;
  }

  // cut: evict every eligible key <= cut
  unsigned long long cut;
  if (k_cand == 0) {
    cut = KEY_NONE - 1;
  } else if (REG && n_e <= SEL_SMALL) {
    unsigned long long last = 0;
    bool have = false;
    for (int it = 0; it < n_e; ++it) {
      unsigned long long mine = KEY_NONE;
#pragma unroll
      for (int j = 0; j < (REG ? KPT : 1); ++j) {
        const unsigned long long key = rkey[j];
        if (key != KEY_NONE && (!have || key > last) && key < mine) mine = key;
      }
      last = block_min(mine, sh);
      have = true;
    }
    cut = last;
  } else {
    // the pass stops where a bin is taken whole: with distinct scores after two or three digits, and no later than
    // the last bit, since all keys are distinct
    for (int shift = 64 - SEL_DIGIT, known = 64; ;
         known = shift, shift = shift > SEL_DIGIT ? shift - SEL_DIGIT : 0) {     // bits from `known` up are decided
      for (int i = tid; i < SEL_BINS; i += SEL_THREADS) sh.hist[i] = 0u;
      wg_lds_barrier();
      const unsigned long long prefix = sh.prefix;
      for_keys(0, n_chunks, [&](int, bool ok, unsigned long long key) {
        const bool match = known >= 64 || (key >> known) == (prefix >> known);
        if (ok && match) atomicAdd(&sh.hist[(unsigned)(key >> shift) & (SEL_BINS - 1)], 1u);
      });
      wg_lds_barrier();
      pick_digit(sh, shift);
      if (sh.whole || shift == 0) break;             // uniform: read behind pick_digit's barrier
    }
    cut = sh.prefix - 1;       // the k largest keys are those from the prefix up; they stay
  }

  if (REG && n_e <= SEL_SMALL) {
    // a handful of evictions: the owners put their slots into a short list (any
    // order), and each then takes the rank of its slot as its place in the output
    if constexpr (REG) {
#pragma unroll
      for (int j = 0; j < KPT; ++j)
        if (rkey[j] != KEY_NONE && rkey[j] <= cut) sh.list[atomicAdd(&sh.nlist, 1)] = j * SEL_THREADS + tid;
      wg_lds_barrier();
#pragma unroll
      for (int j = 0; j < KPT; ++j) {
        if (rkey[j] != KEY_NONE && rkey[j] <= cut) {
          const int slot = j * SEL_THREADS + tid;
          int idx = 0;
          for (int x = 0; x < n_e; ++x) idx += (sh.list[x] < slot) ? 1 : 0;
          const int pos = key_pos(rkey[j]);
          evict_slot[(size_t)unit * evict_cap + idx] = slot;
          evict_pos[(size_t)unit * evict_cap + idx] = pos;
          if (ho && idx < ENC_SMALL_CAP) { ho->slot[idx] = slot; ho->pos[idx] = pos; }
          rp[slot] = -1;
          if (vague_pos && n_vague) vague_pos[(size_t)unit * vague_cap + nv_old + idx] = pos;
        }
      }
    }
    if (tid == 0) {
      n_evict[unit] = n_e;
      if (ho) ho->cnt = n_e;
      if (vague_pos && n_vague) n_vague[unit] = nv_old + n_e;
    }
    return;
  }

  // Ascending slot order = (chunk, wave, lane) order: count the evictions of every wave and chunk, scan, place.
  static_assert(SEL_PLACE_CHUNKS * SEL_WAVES == 2 * SEL_THREADS, "two counters per thread");
  int base = 0;
  for (int c0 = 0; c0 < n_chunks; c0 += SEL_PLACE_CHUNKS) {
    const int c1 = min(c0 + SEL_PLACE_CHUNKS, n_chunks);
    const int n_cnt = (REG ? KPT : c1 - c0) * SEL_WAVES;
    wg_lds_barrier();                                 // nobody reads hist / the previous places any more
    for_keys(c0, c1, [&](int j, bool ok, unsigned long long key) {
      const unsigned long long bal = __ballot(ok && key <= cut);
      if (lane == 0) sh.place[(j - c0) * SEL_WAVES + wave] = __popcll(bal);
    });
    wg_lds_barrier();
    const int a = (2 * tid < n_cnt) ? sh.place[2 * tid] : 0, b_ = (2 * tid + 1 < n_cnt) ? sh.place[2 * tid + 1] : 0;
    int total;
    const int excl = base + block_scan(a + b_, sh, &total) - a - b_;
    if (2 * tid < n_cnt) sh.place[2 * tid] = excl;
    if (2 * tid + 1 < n_cnt) sh.place[2 * tid + 1] = excl + a;
    wg_lds_barrier();
    for_keys(c0, c1, [&](int j, bool ok, unsigned long long key) {
      const bool flag = ok && key <= cut;
      const unsigned long long bal = __ballot(flag);
      if (flag) {
        const int slot = j * SEL_THREADS + tid;
        const int idx = sh.place[(j - c0) * SEL_WAVES + wave] + __popcll(bal & ((1ull << lane) - 1ull));   // < n_e
        const int pos = key_pos(key);
        evict_slot[(size_t)unit * evict_cap + idx] = slot;
        evict_pos[(size_t)unit * evict_cap + idx] = pos;
        if (ho && idx < ENC_SMALL_CAP) { ho->slot[idx] = slot; ho->pos[idx] = pos; }
        rp[slot] = -1;
        if (vague_pos && n_vague) vague_pos[(size_t)unit * vague_cap + nv_old + idx] = pos;
      }
    });
    base += total;
  }
  if (tid == 0) {
    n_evict[unit] = n_e;
    if (ho) ho->cnt = n_e;
    if (vague_pos && n_vague) n_vague[unit] = nv_old + n_e;
  }
}

// ---------------------------------------------------------------------------
// encode, up to ENC_SMALL_CAP listed tokens
// ---------------------------------------------------------------------------
// Called by a workgroup of at least D threads; the hashes of the listed tokens go
// to LDS, then thread (row group, channel) walks the list and owns the slots it
// meets first (list order = summation order, one rounding per slot).
template <typename T>
__device__ __forceinline__ void encode_small_body(
    const DevDesc& d, int unit, const T* __restrict__ k_src, const T* __restrict__ v_src, int src_rows,
    const int32_t* __restrict__ src_slot, const int32_t* __restrict__ tok_pos,
    const int32_t* __restrict__ count, int cap, T* __restrict__ sk, T* __restrict__ sv,
    int32_t* __restrict__ out_bucket, uint8_t* __restrict__ out_sign, const EvictHandOver* ho = nullptr) {
  __shared__ int s_bucket[ENC_SMALL_CAP][KVR_MAX_ROWS];
  __shared__ int s_slot[ENC_SMALL_CAP];
  __shared__ unsigned s_sign[ENC_SMALL_CAP];
  const int tid = threadIdx.x;
  // the list comes from LDS when the selection ran in this workgroup just before (fused update)
  const int cnt = clampi(ho ? ho->cnt : count[unit], 0, min(cap, ENC_SMALL_CAP));
  if (tid < cnt) {
    const int J = ho ? ho->pos[tid] : tok_pos[(size_t)unit * cap + tid];
    const int slot = ho ? ho->slot[tid] : src_slot[(size_t)unit * cap + tid];
    s_slot[tid] = (slot >= 0 && slot < src_rows) ? slot : -1;
    unsigned sg = 0;
    for (int i = 0; i < d.r; ++i) {
      const int bk = bucket_of(d, i, J);
      s_bucket[tid][i] = bk;
      if (sign_neg(d, i, J)) sg |= 1u << i;
      if (out_bucket) out_bucket[((size_t)unit * cap + tid) * d.r + i] = bk;
    }
    s_sign[tid] = sg;
    if (out_sign) out_sign[(size_t)unit * cap + tid] = (uint8_t)sg;
  }
  wg_lds_barrier();
  // thread = (row group, channel): rows i0, i0 + groups, ... (groups = blockDim / D)
  const int c = tid % D;
  const int groups = blockDim.x / D;
  const int i0 = tid / D;
  if (i0 >= groups) return;
  const bool fk = (d.sign_mask & 1) != 0, fv = (d.sign_mask & 2) != 0;
  for (int i = i0; i < d.r; i += groups) {
    for (int e = 0; e < cnt; ++e) {
      if (s_slot[e] < 0) continue;
      const int bk = s_bucket[e][i];
      bool first = true;
      for (int e2 = 0; e2 < e; ++e2) first = first && !(s_slot[e2] >= 0 && s_bucket[e2][i] == bk);
      if (!first) continue;
      const size_t idx = (((size_t)unit * d.r + i) * d.w + bk) * D + c;
      float ak = Store<T>::load1(sk + idx), av = Store<T>::load1(sv + idx);
      for (int e2 = e; e2 < cnt; ++e2) {
        if (s_slot[e2] >= 0 && s_bucket[e2][i] == bk) {
          const bool neg = (s_sign[e2] >> i) & 1u;
          const size_t src = ((size_t)unit * src_rows + s_slot[e2]) * D + c;
          const float kv = Store<T>::load1(k_src + src), vv = Store<T>::load1(v_src + src);
          ak += (fk && neg) ? -kv : kv;
          av += (fv && neg) ? -vv : vv;
        }
      }
      Store<T>::store1(sk + idx, ak);
      Store<T>::store1(sv + idx, av);
    }
  }
}

}  // namespace kvr
