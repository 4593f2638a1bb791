// The retained slots of a unit as one role of a launch whose other workgroups rebuild the Vague list (bf16, G <= 4).
//
// Eight waves walk the 16-token tiles of an item (a slice of one unit's slots).  q.k as in kvr_attend_retained.hip:
// four v_mfma_f32_16x16x32_bf16 per tile, K rows straight from memory as the A operand, q as the B operand.  Here q
// stands in the 16 columns four times over (column = 4 part + head): lane (row group, column) ends up with the logits
// of tokens 4 (l div 16) + i for head l mod 4, forms their weights and keeps the `part`-th bf16 part of each: three
// parts are all 24 bits of a float32 weight.  They are the A operand of p.v as they lie (v_mfma_f32_16x16x16, row =
// 4 part + head), the V rows its B operand after sixteen v_perm_b32, and row group `part` of the result holds the sums
// of that part, for all four heads.  The matrix instruction cuts its smaller addends off towards minus infinity: odd
// waves sum with the opposite sign.
//
// Bound by the latency of memory: a CU gets 35 .. 40 KB per us whether a wave has one, two or three tiles in flight (8 CUs, 30
// MB: 105.7, 105.7, 106.5 us), so one is enough.
#pragma once
#include "kvr_staged.h"

namespace kvr {

typedef __bf16 rs_bf16x8_t __attribute__((ext_vector_type(8)));

struct RsTile {
  uint4 ka[4];   // K: token t0 + (lane mod 16), channels 32 kk + 8 (lane div 16) .. +7
  uint4 vv[4];   // V: token t0 + 4 (lane div 16) + j, channels 8 (lane mod 16) .. +7
  int pos;       // position of token t0 + (lane mod 16), -1 = empty slot / past the slice
};

// (plain loads: non-temporal ones, as in kvr_attend_retained.hip, are slower where few CUs stream: 128 units of 7374 slots,
// 64 workgroups 249 against 208 us, 32 units 66 against 58)
__device__ __forceinline__ uint4 rs_load16(const bf16_t* p) { return *reinterpret_cast<const uint4*>(p); }

// rows of the 16 tokens from t0 on, of a slice that ends at t_end <= ret_cap
__device__ __forceinline__ void rs_load(RsTile& t, const bf16_t* __restrict__ k, const bf16_t* __restrict__ v,
                                        const int32_t* __restrict__ rp, int t0, int t_end, int r16, int col) {
  const int tk = min(t0 + col, t_end - 1);
  t.pos = rp ? rp[tk] : tk;
  if (t0 + col >= t_end) t.pos = -1;
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) t.ka[kk] = rs_load16(k + (size_t)tk * D + 32 * kk + 8 * r16);
#pragma unroll
  for (int j = 0; j < 4; ++j) t.vv[j] = rs_load16(v + (size_t)min(t0 + 4 * r16 + j, t_end - 1) * D + 8 * col);
}

template <int N>
__device__ __forceinline__ float rs_row_bcast(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x150 + N, 0xf, 0xf, true));
}

template <int G>
__device__ __forceinline__ void rs_compute(const RsTile& t, const uint4 (&qb)[4], float scale, int r16, int col,
                                           uint32_t neg, float* __restrict__ s_log, float& m_run, float& l_run,
                                           f32x4_t (&acc)[8]) {
  const float NEG_INF = -__builtin_inff();
  f32x4_t S = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int kk = 0; kk < 4; ++kk)
    S = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(rs_bf16x8_t, t.ka[kk]),
                                                __builtin_bit_cast(rs_bf16x8_t, qb[kk]), S, 0, 0, 0);
  const uint32_t valid16 = (uint32_t)__ballot(t.pos >= 0) & 0xffffu;      // of the tile's tokens (lanes 0-15 hold them all)
  const uint32_t mine = valid16 >> (4 * r16);
  const bool head_ok = (col & 3) < G;
  float s[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) s[i] = (((mine >> i) & 1u) && head_ok) ? S[i] * scale : NEG_INF;
  if (col < G) {
#pragma unroll
    for (int i = 0; i < 4; ++i) s_log[(4 * r16 + i) * G + col] = s[i];
  }
  const float m_new = fmaxf(m_run, rows_max(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]))));
  if (__any(m_new > m_run)) {
    const float corr = (m_run == NEG_INF) ? 0.f : __expf(m_run - m_new);
    l_run *= corr;
    const float c4[4] = {rs_row_bcast<0>(corr), rs_row_bcast<1>(corr), rs_row_bcast<2>(corr), rs_row_bcast<3>(corr)};
#pragma unroll
    for (int e = 0; e < 8; ++e)
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[e][i] *= c4[i];
  }
  m_run = m_new;
  uint32_t x[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float p = (s[i] == NEG_INF) ? 0.f : __expf(s[i] - m_new);
    l_run += p;
    const uint32_t h0 = __float_as_uint(p) & 0xffff0000u;
    const float r1 = p - __uint_as_float(h0);
    const uint32_t h1 = __float_as_uint(r1) & 0xffff0000u;
    const uint32_t h2 = __float_as_uint(r1 - __uint_as_float(h1));
    x[i] = (col < 4 ? h0 : col < 8 ? h1 : col < 12 ? h2 : 0u) ^ neg;
  }
  const short4_t w = pack_k4(pair_hi(x[0], x[1]), pair_hi(x[2], x[3]));
  uint4 v[4] = {t.vv[0], t.vv[1], t.vv[2], t.vv[3]};
  if (valid16 != 0xffffu) {       // an empty slot may hold anything, even NaN: weight 0 is not enough
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (!((mine >> j) & 1u)) v[j] = make_uint4(0u, 0u, 0u, 0u);
  }
#define KVR_RS_PV(c, dw)                                                                                            \
  acc[2 * dw] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(w, pack_k4(pair_lo(v[0].c, v[1].c), pair_lo(v[2].c, v[3].c)), \
                                                          acc[2 * dw], 0, 0, 0);                                    \
  acc[2 * dw + 1] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(                                                      \
      w, pack_k4(pair_hi(v[0].c, v[1].c), pair_hi(v[2].c, v[3].c)), acc[2 * dw + 1], 0, 0, 0);
  KVR_RS_PV(x, 0)
  KVR_RS_PV(y, 1)
  KVR_RS_PV(z, 2)
  KVR_RS_PV(w, 3)
#undef KVR_RS_PV
}

// One slice (a.slice_tokens slots) of a unit's retained slots, by a whole workgroup; ends with a barrier.
template <int G>
__device__ __forceinline__ void ret_stream_slice(const DevDesc& d, const AttendArgs& a, int unit, int slice,
                                                 unsigned char* smem) {
  constexpr int NW = ST_WAVES;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r16 = lane >> 4, col = lane & 15;
  const uint32_t neg = (wave & 1) ? 0x80000000u : 0u;
  float (*s_acc)[G][D] = reinterpret_cast<float (*)[G][D]>(smem);
  float* s_m = reinterpret_cast<float*>(smem + NW * G * D * 4);        // [NW][4]
  float* s_l = s_m + NW * 4;
  float* s_log = s_l + NW * 4;

  const int t_begin = slice * a.slice_tokens, t_end = min(t_begin + a.slice_tokens, a.ret_cap);
  const int n_tiles = t_end > t_begin ? (t_end - t_begin + 15) >> 4 : 0;
  const bf16_t* k = (const bf16_t*)a.k_ret + (size_t)unit * a.ret_cap * D;
  const bf16_t* v = (const bf16_t*)a.v_ret + (size_t)unit * a.ret_cap * D;
  const int32_t* rp = a.ret_pos ? a.ret_pos + (size_t)unit * a.ret_cap : nullptr;
  RsTile t;
  if (n_tiles > 0) rs_load(t, k, v, rp, t_begin + wave * 16, t_end, r16, col);
  uint4 qb[4];
  {
    const int b = unit / d.Hkv, hk = unit % d.Hkv, head = col & 3;
    const bf16_t* q = (const bf16_t*)a.q + ((size_t)b * d.Hq + (size_t)hk * G + (head < G ? head : 0)) * D + 8 * r16;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) qb[kk] = *reinterpret_cast<const uint4*>(q + 32 * kk);
  }
  float m_run = -__builtin_inff(), l_run = 0.f;
  f32x4_t acc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  // every wave walks as many tiles; past the slice's last one they ask for its last row over and over
  for (int ti = wave; ti - wave < n_tiles; ti += NW) {
    rs_compute<G>(t, qb, d.scale, r16, col, neg, s_log + ti * 16 * G, m_run, l_run, acc);
    __builtin_amdgcn_sched_barrier(0);
    rs_load(t, k, v, rp, t_begin + (ti + NW) * 16, t_end, r16, col);
  }
  // Parts (row groups) of the sums, then the waves'.  An infinite value gives the first part its infinity and the others a
  // NaN where their share of the weight is zero: there the first part, which the storing lanes hold, is the sum.
  float o[G][8];
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float all = rows_sum(acc[e][g]);
      o[g][e] = __uint_as_float(__float_as_uint(fabsf(acc[e][g]) < __builtin_inff() ? all : acc[e][g]) ^ neg);
    }
  l_run = rows_sum(l_run);
  if (r16 == 0) {
#pragma unroll
    for (int g = 0; g < G; ++g) {
      *reinterpret_cast<float4*>(&s_acc[wave][g][col * 8]) = make_float4(o[g][0], o[g][1], o[g][2], o[g][3]);
      *reinterpret_cast<float4*>(&s_acc[wave][g][col * 8 + 4]) = make_float4(o[g][4], o[g][5], o[g][6], o[g][7]);
    }
    if (col < G) { s_m[wave * 4 + col] = m_run; s_l[wave * 4 + col] = l_run; }
  }
  lds_barrier();
  if (a.logits != nullptr) {
    const int n = (t_end - t_begin) * G;
    float* dst = a.logits + ((size_t)unit * (a.ret_cap + a.vague_cap) + t_begin) * G;
    if constexpr (G % 4 == 0) {
      for (int i = threadIdx.x * 4; i < n; i += ST_THREADS * 4)
        *reinterpret_cast<float4*>(dst + i) = *reinterpret_cast<const float4*>(s_log + i);
    } else {
      for (int i = threadIdx.x; i < n; i += ST_THREADS) dst[i] = s_log[i];
    }
  }
  const size_t part = (size_t)unit * a.n_slices + slice;
  for (int idx = threadIdx.x; idx < G * D; idx += ST_THREADS) {
    const int g = idx / D, c = idx % D;
    float M = s_m[g];
#pragma unroll
    for (int x = 1; x < NW; ++x) M = fmaxf(M, s_m[x * 4 + g]);
    float L = 0.f, O = 0.f;
#pragma unroll
    for (int x = 0; x < NW; ++x) {
      const float m = s_m[x * 4 + g];
      const float e = (m == -__builtin_inff()) ? 0.f : __expf(m - M);
      L += s_l[x * 4 + g] * e;
      O += s_acc[x][g][c] * e;
    }
    a.part_o[part * G * D + idx] = O;
    if (c == 0) { a.part_ml[(part * G + g) * 2] = M; a.part_ml[(part * G + g) * 2 + 1] = L; }
  }
  lds_barrier();                             // LDS is free again
}

}  // namespace kvr
