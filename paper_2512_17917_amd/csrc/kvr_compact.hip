// kvr_compact: the rows that stay after a prompt's selection move, in slot order,
// from the full cache into the small slot array of the decode steps.
//
// Bound by memory: every kept K and V row is read once and written once.  The
// place of a row is its slot number minus the number of evicted slots below it,
// which a workgroup finds for the start of its range of source slots by a 64-ary
// search of the (ascending) eviction list: three dependent reads at 32k slots, no
// second launch and no workspace.  Ranges are short because the kept rows are not
// spread evenly: half of them are the newest tokens, one solid block at the end.
// 64 units of 32768 slots, 7373 kept each (483 MB of rows read and written): 113 us
// = 4.3 TB/s, against 151 us with ranges of 512 slots and 211 us with ranges of
// 2048 (a large copy reaches 5.1 TB/s).
#include "kvr_launch.h"

namespace kvr {

constexpr int CP_THREADS = 256;
constexpr int CP_RANGE = 256;             // source slots per workgroup

// entries of the ascending list[0 .. n) that are below x; called by a whole wave
__device__ __forceinline__ int count_below(const int32_t* __restrict__ list, int n, int x, int lane) {
  int lo = 0;
  while (n > 0) {                                            // the answer lies in lo .. lo + n
    const int step = (n + WAVE - 1) / WAVE;
    const int i = (lane + 1) * step - 1;                     // last entry of this lane's piece
    const bool below = i < n && list[lo + i] < x;
    const int k = __popcll(__ballot(below));                 // whole pieces below x
    lo += k * step;
    n = min(step - 1, n - k * step);                         // the piece after them, without its last entry
  }
  return lo;
}

template <typename T>
__global__ __launch_bounds__(CP_THREADS) void compact_kernel(
    const T* __restrict__ k_src, const T* __restrict__ v_src, const int32_t* __restrict__ src_pos, int src_cap,
    const int32_t* __restrict__ evict_slot, const int32_t* __restrict__ n_evict, int evict_cap,
    T* __restrict__ k_ret, T* __restrict__ v_ret, int32_t* __restrict__ ret_pos, int ret_cap, int max_keep) {
  constexpr int VEC = Store<T>::VEC;
  constexpr int LPR = D / VEC;                               // lanes per row
  constexpr int NWV = CP_THREADS / WAVE;
  const int unit = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int32_t* sp = src_pos + (size_t)unit * src_cap;
  const int s0 = blockIdx.x * CP_RANGE, s1 = min(s0 + CP_RANGE, src_cap);
  __shared__ int s_slot[CP_RANGE], s_pos[CP_RANGE];
  __shared__ int s_w[NWV], s_before;

  // slots of the range, in thread order
  int pos[CP_RANGE / CP_THREADS];
  int mine = 0;
#pragma unroll
  for (int u = 0; u < CP_RANGE / CP_THREADS; ++u) {
    const int s = s0 + tid * (CP_RANGE / CP_THREADS) + u;
    pos[u] = s < s1 ? sp[s] : -1;
    mine += pos[u] >= 0 ? 1 : 0;
  }
  if (wave == 0) {
    const int gone = count_below(evict_slot + (size_t)unit * evict_cap, clampi(n_evict[unit], 0, evict_cap), s0, lane);
    if (lane == 0) s_before = s0 - gone;
  }
  int incl = mine;
#pragma unroll
  for (int off = 1; off < WAVE; off <<= 1) {
    const int y = __shfl_up(incl, off);
    if (lane >= off) incl += y;
  }
  if (lane == WAVE - 1) s_w[wave] = incl;
  __syncthreads();
  const int before = s_before;
  int at = incl - mine, n = 0;
#pragma unroll
  for (int w_ = 0; w_ < NWV; ++w_) {
    at += (w_ < wave) ? s_w[w_] : 0;
    n += s_w[w_];
  }
#pragma unroll
  for (int u = 0; u < CP_RANGE / CP_THREADS; ++u)
    if (pos[u] >= 0) {
      s_slot[at] = s0 + tid * (CP_RANGE / CP_THREADS) + u;
      s_pos[at] = pos[u];
      ++at;
    }
  __syncthreads();

  const int limit = min(max_keep, ret_cap);
  n = max(0, min(n, limit - before));                        // rows of this range that have a place
  const size_t src0 = (size_t)unit * src_cap * D, dst0 = (size_t)unit * ret_cap * D;
  int32_t* rp = ret_pos + (size_t)unit * ret_cap;
  for (int i = tid; i < n; i += CP_THREADS) rp[before + i] = s_pos[i];
  // four rows of K and of V in flight per lane; read once, written once
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  constexpr int RPI = CP_THREADS / LPR;                      // rows per step of the workgroup
  const int sub = tid % LPR;
  for (int i0 = tid / LPR; i0 < n; i0 += 4 * RPI) {
    u32x4 k[4], v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = min(i0 + u * RPI, n - 1);
      const size_t src = src0 + (size_t)s_slot[i] * D + sub * VEC;
      k[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(k_src + src));
      v[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(v_src + src));
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = i0 + u * RPI;
      if (i < n) {
        const size_t dst = dst0 + (size_t)(before + i) * D + sub * VEC;
        __builtin_nontemporal_store(k[u], reinterpret_cast<u32x4*>(k_ret + dst));
        __builtin_nontemporal_store(v[u], reinterpret_cast<u32x4*>(v_ret + dst));
      }
    }
  }
  // the slots that stay empty: the workgroup of the last range knows how many there are
  if (blockIdx.x == gridDim.x - 1) {
    const u32x4 zero = {0u, 0u, 0u, 0u};
    for (int i = min(before + n, limit) + tid / LPR; i < ret_cap; i += RPI) {
      const size_t dst = dst0 + (size_t)i * D + sub * VEC;
      *reinterpret_cast<u32x4*>(k_ret + dst) = zero;
      *reinterpret_cast<u32x4*>(v_ret + dst) = zero;
      if (sub == 0) rp[i] = -1;
    }
  }
}

hipError_t launch_compact(const DevDesc& d, int dtype, const void* k_src, const void* v_src, const int32_t* src_pos,
                          int src_cap, const int32_t* evict_slot, const int32_t* n_evict, int evict_cap, void* k_ret,
                          void* v_ret, int32_t* ret_pos, int ret_cap, int max_keep, hipStream_t st) {
  const dim3 grid((src_cap + CP_RANGE - 1) / CP_RANGE, d.B * d.Hkv), block(CP_THREADS);
  if (dtype == KVR_F32)
    hipLaunchKernelGGL(compact_kernel<float>, grid, block, 0, st, (const float*)k_src, (const float*)v_src, src_pos,
                       src_cap, evict_slot, n_evict, evict_cap, (float*)k_ret, (float*)v_ret, ret_pos, ret_cap,
                       max_keep);
  else
    hipLaunchKernelGGL(compact_kernel<bf16_t>, grid, block, 0, st, (const bf16_t*)k_src, (const bf16_t*)v_src,
                       src_pos, src_cap, evict_slot, n_evict, evict_cap, (bf16_t*)k_ret, (bf16_t*)v_ret, ret_pos,
                       ret_cap, max_keep);
  return hipGetLastError();
}

}  // namespace kvr
