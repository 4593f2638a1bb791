// Attention over the retained slots (raw Recent + Candidate tokens), bf16.
//
// This part of the step is a plain stream over HBM: every retained K and V row
// is read exactly once.  q.k for the G query heads of the kv head is a small
// dense contraction and goes to the matrix cores: per 16-token tile, four
// v_mfma_f32_16x16x32_bf16 with the K rows as the A operand (lane l supplies
// token l mod 16, channels 8 (l div 16) .. +7 of each 32-channel block) and q as
// the B operand (column n = head n, zero for n >= G).  The result leaves lane l
// with the logits of tokens 4 (l div 16) + {0,1,2,3} for head l mod 16.  The V
// rows are loaded so that lane l holds channels 8 (l mod 16) .. +7 of exactly
// those four tokens; the weight of (token, head g) then sits in lane g of the
// same 16-lane row and is fetched with a DPP row broadcast.  p * v is
// accumulated in float32 on the vector ALUs (an MFMA would need V transposed).
// Online softmax per wave; the four waves of a workgroup are merged through LDS
// into one partial per slice.
//
// Bound by HBM.  Alone, a wave requests the next tile's rows while it computes (168 registers keep three waves
// per SIMD); the logits wait in LDS and leave together, 16 bytes a lane.  32 units x 29492 slots, 4 heads: 107 ->
// 102 us = 4.7 TB/s (a large copy reaches 5.1); 40 units x 4104 slots, 8 heads: 32.4 -> 30.0 us.  Next to a staged kernel
// there are no registers for it; the logits wait in what LDS the staged kernel leaves, of a whole slice or of 512 tokens
// at a time.
//
// A workgroup walks over (unit, slice) items with a grid stride, so the launch
// can be as wide as the item count (stand-alone: many workgroups per CU hide the
// HBM latency) or as narrow as one workgroup per CU (next to the general staged
// kernel, whose registers and LDS leave room for exactly that).
#include "kvr_launch.h"

namespace kvr {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

// value held by lane N of the caller's 16-lane row
template <int N>
__device__ __forceinline__ float row_bcast(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x150 + N, 0xf, 0xf, true));
}

template <int G, int I>
struct AccStep {
  __device__ static __forceinline__ void fma(float (&acc)[G][8], float p, const float (&v)[8]) {
    const float pg = row_bcast<I>(p);
#pragma unroll
    for (int c = 0; c < 8; ++c) acc[I][c] = fmaf(pg, v[c], acc[I][c]);
    AccStep<G, I + 1>::fma(acc, p, v);
  }
  __device__ static __forceinline__ void scale(float (&acc)[G][8], float corr) {
    const float cg = row_bcast<I>(corr);
#pragma unroll
    for (int c = 0; c < 8; ++c) acc[I][c] *= cg;
    AccStep<G, I + 1>::scale(acc, corr);
  }
};
template <int G>
struct AccStep<G, G> {
  __device__ static __forceinline__ void fma(float (&)[G][8], float, const float (&)[8]) {}
  __device__ static __forceinline__ void scale(float (&)[G][8], float) {}
};

struct RetTile {
  uint4 ka[4];   // K: token t0 + (lane mod 16), channels 32 kk + 8 (lane div 16) .. +7
  uint4 vv[4];   // V: token t0 + 4 (lane div 16) + j, channels 8 (lane mod 16) .. +7
  int pos[4];    // position of token t0 + 4 (lane div 16) + j, -1 = empty slot / past the slice
};

// 16 bytes that are read exactly once: non-temporal, so that the stream does not
// push the sketch (which the staged kernel reads many times) out of L2
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 stream_load16(const bf16_t* p) {
  const u32x4_t v = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(p));
  return make_uint4(v[0], v[1], v[2], v[3]);
}

__device__ __forceinline__ void load_k(RetTile& t, const bf16_t* __restrict__ kret, int t0, int ret_cap, int r16,
                                       int col) {
  const int tk = min(t0 + col, ret_cap - 1);
#pragma unroll
  for (int kk = 0; kk < 4; ++kk)
    t.ka[kk] = stream_load16(kret + (size_t)tk * D + 32 * kk + 8 * r16);
}
__device__ __forceinline__ void load_pos_v(RetTile& t, const bf16_t* __restrict__ vret,
                                           const int32_t* __restrict__ rp, int t0, int t_end, int ret_cap, int r16,
                                           int col) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int tt = t0 + 4 * r16 + j;
    const int x = rp ? rp[min(tt, ret_cap - 1)] : tt;
    t.pos[j] = (tt < t_end) ? x : -1;
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int tc = min(t0 + 4 * r16 + j, ret_cap - 1);
    t.vv[j] = stream_load16(vret + (size_t)tc * D + 8 * col);
  }
}

// One 16-token tile.  NEXT: the tile at t_next follows, and its K rows are requested as soon as this tile's are
// consumed, its positions and V rows behind this tile's p.v, all into the same registers.  No global store may sit
// between these loads (reads and writes complete in no common order, so a wait for a read with a write outstanding
// is a wait for everything): the logits go to s_log.
template <int G, bool NEXT>
__device__ __forceinline__ void compute_tile(RetTile& t, const uint4 (&qb)[4], const bf16_t* __restrict__ kret,
                                             const bf16_t* __restrict__ vret, const int32_t* __restrict__ rp,
                                             float scale, int t0, int t_next, int t_end, int ret_cap, int r16, int col,
                                             float* __restrict__ s_log, float& m_run, float& l_run,
                                             float (&acc)[G][8]) {
  const float NEG_INF = -__builtin_inff();
  f32x4_t S = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int kk = 0; kk < 4; ++kk)
    S = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, t.ka[kk]),
                                                __builtin_bit_cast(bf16x8_t, qb[kk]), S, 0, 0, 0);
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (NEXT) {
    load_k(t, kret, t_next, ret_cap, r16, col);
    __builtin_amdgcn_sched_barrier(0);
  }
  float s[4];
  bool invalid = false;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const bool ok = t.pos[i] >= 0 && col < G;
    s[i] = ok ? S[i] * scale : NEG_INF;
    invalid = invalid || t.pos[i] < 0;
  }
  if (col < G) {
#pragma unroll
    for (int i = 0; i < 4; ++i) s_log[(4 * r16 + i) * G + col] = s[i];
  }
  float mx = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
  mx = fmaxf(mx, __shfl_xor(mx, 16));
  mx = fmaxf(mx, __shfl_xor(mx, 32));
  const float m_new = fmaxf(m_run, mx);
  if (__any(m_new > m_run)) {
    const float corr = (m_run == NEG_INF) ? 0.f : __expf(m_run - m_new);
    l_run *= corr;
    AccStep<G, 0>::scale(acc, corr);
  }
  m_run = m_new;
  float p[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    p[i] = (s[i] == NEG_INF) ? 0.f : __expf(s[i] - m_new);
    l_run += p[i];
  }
  const bool any_invalid = __any(invalid);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    float v[8] = {__uint_as_float(t.vv[j].x << 16), __uint_as_float(t.vv[j].x & 0xffff0000u),
                  __uint_as_float(t.vv[j].y << 16), __uint_as_float(t.vv[j].y & 0xffff0000u),
                  __uint_as_float(t.vv[j].z << 16), __uint_as_float(t.vv[j].z & 0xffff0000u),
                  __uint_as_float(t.vv[j].w << 16), __uint_as_float(t.vv[j].w & 0xffff0000u)};
    if (any_invalid) {            // an empty slot may hold anything, even NaN: weight 0 is not enough
      const bool dead = t.pos[j] < 0;
#pragma unroll
      for (int c = 0; c < 8; ++c) v[c] = dead ? 0.f : v[c];
    }
    AccStep<G, 0>::fma(acc, p[j], v);
    if constexpr (NEXT) __builtin_amdgcn_sched_barrier(0);       // one row's floats at a time: registers
  }
  if constexpr (NEXT) {
    load_pos_v(t, vret, rp, t_next, t_end, ret_cap, r16, col);
  }
}

template <int G, bool AHEAD>
__device__ __forceinline__ void attend_retained_body(const DevDesc& d, const AttendArgs& a, int n_rslices,
                                                     int seg_tiles) {
  constexpr int NW = 4;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r16 = lane >> 4, col = lane & 15;
  const int tot_cap = a.ret_cap + a.vague_cap;
  const int n_items = d.B * d.Hkv * n_rslices;
  const float NEG_INF = -__builtin_inff();
  // logits while the slice is walked (AHEAD: of the whole slice, else of seg_tiles tiles at a time), then the waves' sums
  // [NW][G][D]
  extern __shared__ __align__(16) float s_dyn[];
  __shared__ float s_m[NW][G], s_l[NW][G];

  // Same issue priority as the lower of the two levels that the staged kernel's
  // waves alternate between: measured best when the two kernels share the CUs.
  __builtin_amdgcn_s_setprio(1);
  for (int item = blockIdx.x; item < n_items; item += gridDim.x) {
    const int unit = item / n_rslices, slice = item % n_rslices;
    const int b = unit / d.Hkv, hk = unit % d.Hkv;
    const int t_begin = slice * a.slice_tokens;
    const int t_end = min(t_begin + a.slice_tokens, a.ret_cap);
    const bf16_t* kret = (const bf16_t*)a.k_ret + (size_t)unit * a.ret_cap * D;
    const bf16_t* vret = (const bf16_t*)a.v_ret + (size_t)unit * a.ret_cap * D;
    const int32_t* rp = a.ret_pos ? a.ret_pos + (size_t)unit * a.ret_cap : nullptr;
    float* logits_unit = a.logits ? a.logits + (size_t)unit * tot_cap * G : nullptr;

    const int n_tiles = (t_end > t_begin) ? (t_end - t_begin + 15) >> 4 : 0;
    int ti = wave;
    RetTile tile;
    if (AHEAD && ti < n_tiles) {
      load_k(tile, kret, t_begin + ti * 16, a.ret_cap, r16, col);
      load_pos_v(tile, vret, rp, t_begin + ti * 16, t_end, a.ret_cap, r16, col);
    }
    uint4 qb[4];
    {
      const bf16_t* q = (const bf16_t*)a.q + ((size_t)b * d.Hq + (size_t)hk * G + (col < G ? col : 0)) * D + 8 * r16;
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        qb[kk] = *reinterpret_cast<const uint4*>(q + 32 * kk);
        if (col >= G) qb[kk] = make_uint4(0u, 0u, 0u, 0u);
      }
    }
    float m_run = NEG_INF, l_run = 0.f;
    float acc[G][8];
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int c = 0; c < 8; ++c) acc[g][c] = 0.f;

    // logits of n_tok tokens from the slice's token `first` on leave LDS together, 16 bytes a lane
    auto store_logits = [&](int first, int n_tok) {
      if (logits_unit == nullptr) return;
      const int n = n_tok * G;                     // floats
      float* dst = logits_unit + (size_t)(t_begin + first) * G;
      if constexpr (G % 4 == 0) {
        for (int i = threadIdx.x * 4; i < n; i += 1024)
          *reinterpret_cast<float4*>(dst + i) = *reinterpret_cast<const float4*>(s_dyn + i);
      } else {
        for (int i = threadIdx.x; i < n; i += 256) dst[i] = s_dyn[i];
      }
    };
    if constexpr (AHEAD) {
      for (; ti + NW < n_tiles; ti += NW)
        compute_tile<G, true>(tile, qb, kret, vret, rp, d.scale, t_begin + ti * 16, t_begin + (ti + NW) * 16, t_end,
                              a.ret_cap, r16, col, s_dyn + ti * 16 * G, m_run, l_run, acc);
      if (ti < n_tiles)
        compute_tile<G, false>(tile, qb, kret, vret, rp, d.scale, t_begin + ti * 16, 0, t_end, a.ret_cap, r16, col,
                               s_dyn + ti * 16 * G, m_run, l_run, acc);
      __syncthreads();             // the slice's logits are complete
      store_logits(0, t_end - t_begin);
      __syncthreads();             // everyone has read them: the sums may take their place
    } else {
      for (int s0 = 0; s0 < n_tiles; s0 += seg_tiles) {
        for (; ti < min(s0 + seg_tiles, n_tiles); ti += NW) {
          load_k(tile, kret, t_begin + ti * 16, a.ret_cap, r16, col);
          load_pos_v(tile, vret, rp, t_begin + ti * 16, t_end, a.ret_cap, r16, col);
          compute_tile<G, false>(tile, qb, kret, vret, rp, d.scale, t_begin + ti * 16, 0, t_end, a.ret_cap, r16, col,
                                 s_dyn + (ti - s0) * 16 * G, m_run, l_run, acc);
        }
        __syncthreads();
        store_logits(s0 * 16, min(t_end - t_begin - s0 * 16, seg_tiles * 16));
        __syncthreads();
      }
    }

    // the four 16-lane rows of the wave hold different tokens: add them
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        acc[g][c] += __shfl_xor(acc[g][c], 16);
        acc[g][c] += __shfl_xor(acc[g][c], 32);
      }
    l_run += __shfl_xor(l_run, 16);
    l_run += __shfl_xor(l_run, 32);

    float (*s_acc)[G][D] = reinterpret_cast<float (*)[G][D]>(s_dyn);
    if (r16 == 0) {
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int c = 0; c < 8; ++c) s_acc[wave][g][col * 8 + c] = acc[g][c];
      if (col < G) { s_m[wave][col] = m_run; s_l[wave][col] = l_run; }
    }
    __syncthreads();
    float* po = a.part_o + ((size_t)unit * a.n_slices + slice) * G * D;
    float* pml = a.part_ml + ((size_t)unit * a.n_slices + slice) * G * 2;
    for (int idx = threadIdx.x; idx < G * D; idx += 256) {
      const int g = idx / D, c = idx % D;
      float M = s_m[0][g];
#pragma unroll
      for (int w_ = 1; w_ < NW; ++w_) M = fmaxf(M, s_m[w_][g]);
      float L = 0.f, O = 0.f;
#pragma unroll
      for (int w_ = 0; w_ < NW; ++w_) {
        const float e = (s_m[w_][g] == NEG_INF) ? 0.f : __expf(s_m[w_][g] - M);
        L += s_l[w_][g] * e;
        O += s_acc[w_][g][c] * e;
      }
      po[idx] = O;
      if (c == 0) { pml[g * 2] = M; pml[g * 2 + 1] = L; }
    }
    __syncthreads();             // the next item writes its logits over the sums
  }
}

// Two kernels around the same body.  Alone, the kernel may use what three waves per SIMD leave (one head: four).  Next to
// a staged kernel it is capped at 124 + 4 accumulation registers (the attribute counts in units of two on
// this target): 2 x 192 (two waves of the staged kernel, which then needs no spills) + 128 fill a SIMD's 512
// registers exactly; the few spills of this kernel, which waits for HBM most of the time, cost nothing.
template <int G>
__global__ __launch_bounds__(256, (G <= 1 ? 4 : G <= 4 ? 3 : 2)) void attend_retained_kernel(DevDesc d, AttendArgs a, int n_rslices) {
  attend_retained_body<G, true>(d, a, n_rslices, 0);
}
template <int G>
__global__ __launch_bounds__(256) __attribute__((amdgpu_num_vgpr(62))) void attend_retained_shared_kernel(
    DevDesc d, AttendArgs a, int n_rslices, int seg_tiles) {
  attend_retained_body<G, false>(d, a, n_rslices, seg_tiles);
}

hipError_t launch_attend_retained(const DevDesc& d, const AttendArgs& a, int n_rslices, int max_wgs,
                                  int side_lds, hipStream_t st) {
  int n_wgs = d.B * d.Hkv * n_rslices;
  if (max_wgs > 0 && n_wgs > max_wgs) n_wgs = max_wgs;
  if (n_wgs < 1) return hipSuccess;
  const dim3 grid(n_wgs), block(256);
  const int lds = side_lds ? side_lds : retained_lds(d.G, a.slice_tokens);
  if (side_lds) {
    if (side_lds < retained_lds(d.G, 0)) return hipErrorInvalidValue;
    const int seg = side_lds / (d.G * 4 * 16) / 4 * 4;         // tiles, the same number for each of the four waves
    switch (d.G) {
      case 1: hipLaunchKernelGGL(attend_retained_shared_kernel<1>, grid, block, lds, st, d, a, n_rslices, seg); break;
      case 2: hipLaunchKernelGGL(attend_retained_shared_kernel<2>, grid, block, lds, st, d, a, n_rslices, seg); break;
      case 4: hipLaunchKernelGGL(attend_retained_shared_kernel<4>, grid, block, lds, st, d, a, n_rslices, seg); break;
      default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
  }
  switch (d.G) {
    case 1: hipLaunchKernelGGL(attend_retained_kernel<1>, grid, block, lds, st, d, a, n_rslices); break;
    case 2: hipLaunchKernelGGL(attend_retained_kernel<2>, grid, block, lds, st, d, a, n_rslices); break;
    case 4: hipLaunchKernelGGL(attend_retained_kernel<4>, grid, block, lds, st, d, a, n_rslices); break;
    case 8: hipLaunchKernelGGL(attend_retained_kernel<8>, grid, block, lds, st, d, a, n_rslices); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace kvr
