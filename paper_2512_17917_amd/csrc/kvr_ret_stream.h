// The retained slots as one role of a launch whose other workgroups rebuild the Vague list (bf16): columns c = (query t, head
// g) = t * G + g, NCOL = n_q * G of them (kvr_attend_decode: one query).
//
// NW waves walk the 16-token tiles of a slice of one unit's slots.  q.k: four v_mfma_f32_16x16x32_bf16 per tile, K rows
// straight from memory as the A operand (lane l supplies token l mod 16, channels 8 (l div 16) .. +7 of each 32-channel block),
// the query vectors as the B operand, repeated over the 16 columns as often as they fit: lane (row group, column) ends up with
// the logits of tokens 4 (l div 16) + i for its query vector, forms their weights and keeps one bf16 part of each (the place of
// the repetition says which): three parts are all 24 bits of a float32 weight.  They are the A operand of p.v as they lie
// (v_mfma_f32_16x16x16), the V rows its B operand after sixteen v_perm_b32; eight columns need a second product for the third
// part, sixteen one per part.  The matrix instruction cuts its smaller addends off towards minus infinity: odd waves sum with
// the opposite sign.
//
// Bound by the latency of memory: a CU gets 35 .. 40 KB per us whether a wave has one, two or three tiles in flight (8 CUs, 30
// MB: 105.7, 105.7, 106.5 us), so one is enough.
#pragma once
#include "kvr_staged.h"

namespace kvr {

typedef __bf16 rs_bf16x8_t __attribute__((ext_vector_type(8)));

struct RetStream {
  const bf16_t* q;          // [B, n_q, Hq, D]
  const bf16_t* k;          // [units, cap, D]
  const bf16_t* v;
  const int32_t* pos;       // [units, cap], -1: empty slot; null: slot = position
  const int32_t* n_ctx;     // [B]: query t sees positions up to n_ctx - n_q + t; null: everything
  int n_q, cap;
  int slice_tokens, n_rslices, n_slices;    // slices of a unit (the partials' first ones), partials of a unit
  int logit_rows;           // of a unit
  float* part_o;            // [units, n_slices, NCOL, D]
  float* part_ml;           // [units, n_slices, NCOL, 2]
  float* logits;            // [units, logit_rows, NCOL] or null
};
__device__ __forceinline__ RetStream ret_stream_of(const AttendArgs& a) {
  return RetStream{(const bf16_t*)a.q, (const bf16_t*)a.k_ret, (const bf16_t*)a.v_ret, a.ret_pos, nullptr, 1, a.ret_cap,
                   a.slice_tokens, a.n_rslices, a.n_slices, a.ret_cap + a.vague_cap, a.part_o, a.part_ml, a.logits};
}

struct RsTile {
  uint4 ka[4];   // K: token t0 + (lane mod 16), channels 32 kk + 8 (lane div 16) .. +7
  uint4 vv[4];   // V: token t0 + 4 (lane div 16) + j, channels 8 (lane mod 16) .. +7
  int pos;       // position of token t0 + (lane mod 16), -1 = empty slot / past the slice
};

// (plain loads: non-temporal ones, as in kvr_attend_retained.hip, are slower where few CUs stream: 128 units of 7374 slots,
// 64 workgroups 249 against 208 us, 32 units 66 against 58)
__device__ __forceinline__ uint4 rs_load16(const bf16_t* p) { return *reinterpret_cast<const uint4*>(p); }

// rows of the 16 tokens from t0 on, of a slice that ends at t_end <= cap
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

// both halves zero, or the one that is no finite number
__device__ __forceinline__ uint32_t rs_finite(uint32_t x) {
  if ((x & 0x7f80u) == 0x7f80u) x &= 0xffff0000u;
  if ((x & 0x7f800000u) == 0x7f800000u) x &= 0xffffu;
  return x;
}

// Query vectors in the 16 columns: NC apart, REP times over; product number o takes parts o * REP + (column / NC).
template <int NCOL, int PARTS>
struct RsShape {
  static constexpr int NC = NCOL < 4 ? 4 : NCOL, REP = 16 / NC, OPS = (PARTS + REP - 1) / REP;
  // Parts in two products share accumulators: an infinite value would give the sums of the first part a NaN where the part of
  // the second product is zero.  Three parts: the second product leaves what is not finite out.  Two, with 16 columns, where that
  // cost 64 units of 7374 + 25395 tokens 203.3 -> 209.1 us a call: the second part is no less than 2^-30 of the weight
  // (of which two parts keep 16 bits).
  static constexpr bool GUARD = OPS > 1 && PARTS == 3, FLOOR = OPS > 1 && PARTS == 2;
};

template <int NCOL, int PARTS>
__device__ __forceinline__ void rs_compute(const RsTile& t, const uint4 (&qb)[4], float scale, int r16, int col, int q_first,
                                           int q_pos, uint32_t neg, float* __restrict__ s_log, float& m_run, float& l_run,
                                           f32x4_t (&acc)[8]) {
  using SH = RsShape<NCOL, PARTS>;
  const float NEG_INF = -__builtin_inff();
  f32x4_t S = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int kk = 0; kk < 4; ++kk)
    S = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(rs_bf16x8_t, t.ka[kk]),
                                                __builtin_bit_cast(rs_bf16x8_t, qb[kk]), S, 0, 0, 0);
  const uint32_t valid16 = (uint32_t)__ballot(t.pos >= 0) & 0xffffu;      // of the tile's tokens (lanes 0-15 hold them all)
  const uint32_t mine = valid16 >> (4 * r16);
  const bool live = col % SH::NC < NCOL;
  float s[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) s[i] = (((mine >> i) & 1u) && live) ? S[i] * scale : NEG_INF;
  if (__any(t.pos > q_first)) {             // a position that some query must not see
    const int lane16 = (threadIdx.x & 48) + 4 * r16;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (__shfl(t.pos, lane16 + i) > q_pos) s[i] = NEG_INF;
  }
  if (col < NCOL) {
#pragma unroll
    for (int i = 0; i < 4; ++i) s_log[(4 * r16 + i) * NCOL + col] = s[i];
  }
  const float m_new = fmaxf(m_run, rows_max(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]))));
  if (__any(m_new > m_run)) {
    const float corr = (m_run == NEG_INF) ? 0.f : __expf(m_run - m_new);
    l_run *= corr;
#pragma unroll
    for (int i = 0; i < 4; ++i) {           // accumulator i belongs to row 4 r16 + i
      const float c = __shfl(corr, (threadIdx.x & 48) + (4 * r16 + i) % SH::NC);
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e][i] *= c;
    }
  }
  m_run = m_new;
  uint32_t x[SH::OPS][4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float p = (s[i] == NEG_INF) ? 0.f : __expf(s[i] - m_new);
    l_run += p;
    uint32_t h[4] = {__float_as_uint(p) & 0xffff0000u, 0u, 0u, 0u};
    float r1 = p - __uint_as_float(h[0]);
    if constexpr (SH::FLOOR) r1 = fmaxf(r1, p * 0x1p-30f);
    h[1] = __float_as_uint(r1) & 0xffff0000u;
    if constexpr (PARTS > 2) h[2] = __float_as_uint(r1 - __uint_as_float(h[1]));
#pragma unroll
    for (int o = 0; o < SH::OPS; ++o) {
      uint32_t y = h[o * SH::REP];
#pragma unroll
      for (int c = 1; c < SH::REP; ++c)
        if (col >= c * SH::NC) y = o * SH::REP + c < 4 ? h[o * SH::REP + c] : 0u;
      x[o][i] = y ^ neg;
    }
  }
  uint4 v[4] = {t.vv[0], t.vv[1], t.vv[2], t.vv[3]};
  if (valid16 != 0xffffu) {       // an empty slot may hold anything, even NaN: weight 0 is not enough
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (!((mine >> j) & 1u)) v[j] = make_uint4(0u, 0u, 0u, 0u);
  }
#pragma unroll
  for (int o = 0; o < SH::OPS; ++o) {
    if (SH::GUARD && o == 1) {
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = make_uint4(rs_finite(v[j].x), rs_finite(v[j].y), rs_finite(v[j].z), rs_finite(v[j].w));
    }
    const short4_t w = pack_k4(pair_hi(x[o][0], x[o][1]), pair_hi(x[o][2], x[o][3]));
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
}

// One slice of a unit's retained slots, by a whole workgroup of NW waves; ends with a barrier.
template <int NCOL, int PARTS, int NW>
__device__ __forceinline__ void ret_stream_slice(const DevDesc& d, const RetStream& a, int unit, int slice,
                                                 unsigned char* smem) {
  using SH = RsShape<NCOL, PARTS>;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r16 = lane >> 4, col = lane & 15;
  const uint32_t neg = (wave & 1) ? 0x80000000u : 0u;
  float* s_m = reinterpret_cast<float*>(smem);                         // [NW][16]
  float* s_l = s_m + NW * 16;
  float* s_log = s_l + NW * 16;                                        // logits of the slice, then the waves' sums
  float (*s_acc)[NCOL][D] = reinterpret_cast<float (*)[NCOL][D]>(s_log);

  const int t_begin = slice * a.slice_tokens, t_end = min(t_begin + a.slice_tokens, a.cap);
  const int n_tiles = t_end > t_begin ? (t_end - t_begin + 15) >> 4 : 0;
  const bf16_t* k = a.k + (size_t)unit * a.cap * D;
  const bf16_t* v = a.v + (size_t)unit * a.cap * D;
  const int32_t* rp = a.pos ? a.pos + (size_t)unit * a.cap : nullptr;
  RsTile t;
  if (n_tiles > 0) rs_load(t, k, v, rp, t_begin + wave * 16, t_end, r16, col);
  const int b = unit / d.Hkv, hk = unit % d.Hkv;
  const int c_ = col % SH::NC < NCOL ? col % SH::NC : 0, tq = c_ / d.G;
  uint4 qb[4];
  {
    const bf16_t* q = a.q + (((size_t)b * a.n_q + tq) * d.Hq + (size_t)hk * d.G + c_ % d.G) * D + 8 * r16;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) qb[kk] = *reinterpret_cast<const uint4*>(q + 32 * kk);
  }
  const int q_first = a.n_ctx ? a.n_ctx[b] - a.n_q : 0x7fffffff, q_pos = a.n_ctx ? q_first + tq : 0x7fffffff;
  float m_run = -__builtin_inff(), l_run = 0.f;
  f32x4_t acc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  // every wave walks as many tiles; past the slice's last one they ask for its last row over and over
  for (int ti = wave; ti - wave < n_tiles; ti += NW) {
    rs_compute<NCOL, PARTS>(t, qb, d.scale, r16, col, q_first, q_pos, neg, s_log + ti * 16 * NCOL, m_run, l_run, acc);
    __builtin_amdgcn_sched_barrier(0);
    rs_load(t, k, v, rp, t_begin + (ti + NW) * 16, t_end, r16, col);
  }
  l_run = rows_sum(l_run);
  if (r16 == 0 && col < NCOL) { s_m[wave * 16 + col] = m_run; s_l[wave * 16 + col] = l_run; }
  lds_barrier();                             // the slice's logits are complete
  if (a.logits != nullptr) {
    const int n = (t_end - t_begin) * NCOL;
    float* dst = a.logits + ((size_t)unit * a.logit_rows + t_begin) * NCOL;
    if constexpr (NCOL % 4 == 0) {
      for (int i = threadIdx.x * 4; i < n; i += NW * 256)
        *reinterpret_cast<float4*>(dst + i) = *reinterpret_cast<const float4*>(s_log + i);
    } else {
      for (int i = threadIdx.x; i < n; i += NW * 64) dst[i] = s_log[i];
    }
  }
  lds_barrier();                             // everyone has read them
  // Row 4 r16 + i of the sums is part (row / NC) of column (row mod NC): the parts, then the waves.  An infinite value gives
  // the first part its infinity and the others a NaN where their share of the weight is zero: there the first part, which
  // the storing lanes hold, is the sum.
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float o[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float own = acc[e][i];
      float all = own;
      if constexpr (SH::NC == 4) {
        all = rows_sum(own);
      } else if constexpr (SH::NC == 8) {
        const auto y = __builtin_amdgcn_permlane32_swap(__float_as_uint(own), __float_as_uint(own), false, false);
        all = __uint_as_float(y[0]) + __uint_as_float(y[1]);
      }
      o[e] = __uint_as_float(__float_as_uint(fabsf(own) < __builtin_inff() ? all : own) ^ neg);
    }
    const int c = 4 * r16 + i;
    if (c < NCOL) {
      *reinterpret_cast<float4*>(&s_acc[wave][c][col * 8]) = make_float4(o[0], o[1], o[2], o[3]);
      *reinterpret_cast<float4*>(&s_acc[wave][c][col * 8 + 4]) = make_float4(o[4], o[5], o[6], o[7]);
    }
  }
  lds_barrier();
  const size_t part = (size_t)unit * a.n_slices + slice;
  for (int idx = threadIdx.x; idx < NCOL * D; idx += NW * 64) {
    const int g = idx / D, c = idx % D;
    float M = s_m[g];
#pragma unroll
    for (int x = 1; x < NW; ++x) M = fmaxf(M, s_m[x * 16 + g]);
    float L = 0.f, O = 0.f;
#pragma unroll
    for (int x = 0; x < NW; ++x) {
      const float m = s_m[x * 16 + g];
      const float e = (m == -__builtin_inff()) ? 0.f : __expf(m - M);
      L += s_l[x * 16 + g] * e;
      O += s_acc[x][g][c] * e;
    }
    a.part_o[part * NCOL * D + idx] = O;
    if (c == 0) { a.part_ml[(part * NCOL + g) * 2] = M; a.part_ml[(part * NCOL + g) * 2 + 1] = L; }
  }
  lds_barrier();                             // the next slice's logits and statistics go over these
}

// Workgroup `wg` of `n_wgs`: slices wg, wg + n_wgs, ... of all units.
template <int NCOL, int PARTS, int NW>
__device__ __forceinline__ void ret_stream_role(const DevDesc& d, const RetStream& a, int wg, int n_wgs, unsigned char* smem) {
  for (int item = wg; item < d.B * d.Hkv * a.n_rslices; item += n_wgs)
    ret_stream_slice<NCOL, PARTS, NW>(d, a, item / a.n_rslices, item % a.n_rslices, smem);
}

}  // namespace kvr
