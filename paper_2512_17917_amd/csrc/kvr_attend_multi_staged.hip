// kvr_attend_multi, Vague index list, LDS-staged (bf16, three sketch rows, values
// signed only, 3 w <= 1024 so that a 64-channel chunk of a sketch fits LDS).
//
// Rebuilding a Vague token (Algorithm 2) needs three rows of the K sketch and three
// of the V sketch; gathered out of L2 that is 5 GB per layer of the 32k workload.
// Here a workgroup copies one 64-channel chunk of a unit's sketch into LDS and
// walks ALL of its tokens against it, four times (K chunk 0, K chunk 1, V chunk 0,
// V chunk 1).  Nothing about a token stays in registers between the phases: the
// token's record (slots and signs), its partial logits after the first K chunk and
// its final logits go through scratch memory, 16-token tile by tile, so a
// workgroup's share of the list is not limited by registers and a unit's sketch is
// staged by as few workgroups as fill the chip.
//
// Per 16-token tile, with lane = (r16, col) = (lane / 16, lane mod 16):
//   K phases: token t0 + col, 16-byte piece 4 kx + r16 of the chunk (kx = 0, 1) is
//     rebuilt from LDS and is directly the A operand of v_mfma_f32_16x16x32_bf16;
//     the NCOL query vectors are the B operand (column c = query t * G + head g).
//     The lane receives the logits of tokens t0 + 4 r16 + {0..3} for column col.
//   V phases: the weights of those same four tokens for column col are the A operand
//     of v_mfma_f32_16x16x16_bf16 (bf16 hi + lo); the lane rebuilds channels
//     4 col .. 4 col + 3 of the chunk for the four tokens (8 bytes per row) and a
//     register transpose gives the four B operands; instruction c leaves the lane
//     with the sums of columns 4 r16 + {0..3} for channel 4 col + c.
// Softmax: the K-chunk-1 phase knows the final logits, so each wave takes the
// maximum of its tiles per column there; the V phases form the weights against
// the workgroup's maximum (the waves' maxima meet in LDS in between).
// Tiles are handed to the waves through a counter in LDS, phase by phase.
//
// Bound by the vector ALUs, so the layouts are chosen for few instructions per tile:
//   * scratch memory holds the logits of a tile column by column (a lane's four tokens are one 16-byte load or store)
//     and a token's record in four bytes (a lane's four records are one 16-byte load);
//   * what lies past the end of the list is written so that nothing has to be masked when it is read: records 0, logits
//     -inf; positions are looked at once per token, by the thread that hashes it, and again only in a workgroup that has a
//     position some query must not see;
//   * LDS rows are 144 bytes apart: the 16 lanes that read the same piece of 16 random slots spread over all bank groups, and
//     a row's address is one multiply-add (V chunks: 128, a row is read by 16 lanes at once).
// us a phase, 64 units x 25395 tokens, 16 columns, 273 slots per row, one workgroup per CU: K 17 (what LDS delivers with three lanes in
// 16 on the same bank group) and 25 (with the logits of the first pass read and the final ones written), V 26 and 26 (130 vector
// instructions per tile and phase), everything else 26.  Against records of eight bytes, logits token by token, in two arrays, and 538
// vector instructions per tile instead of 400: call of four queries 254 -> 227, decode step of 5 x 8 units, 12706 tokens, eight heads,
// two layers 204 -> 193.
#include "kvr_ret_stream.h"

#include <algorithm>

namespace kvr {

typedef __bf16 bf16x8ms_t __attribute__((ext_vector_type(8)));

constexpr int MS_THREADS = 1024;          // 16 waves: four per SIMD cover each other's memory round trips
constexpr int MS_WAVES = MS_THREADS / 64;
constexpr int MS_PITCH = 144;             // K chunks: bytes from one sketch slot to the next in LDS (128 of them used)
__host__ __device__ constexpr int ms_chunk_lds(int rows, int n_col) {     // a chunk in whole kilobytes; later [waves][n_col][64] floats
  const int chunk = (rows * MS_PITCH + 1023) & ~1023, sums = MS_WAVES * n_col * 64 * 4;
  return chunk > sums ? chunk : sums;
}

struct MultiStagedArgs {
  const bf16_t* q;          // [B, n_q, Hq, D]
  const int32_t* n_ctx;     // [B], or null: every listed token is visible to every query
  int n_q;
  const bf16_t* sk;         // [units, 3, w, D]
  const bf16_t* sv;
  const int32_t* pos;       // Vague index list [units, cap]
  const int32_t* n_valid;   // [units]
  int cap;
  int part_tokens, n_parts; // tokens per workgroup (a multiple of 16), workgroups per unit
  int slice0, n_slices;     // partial index of part 0 / partials per unit
  float* part_o;            // [units, n_slices, NCOL, D]
  float* part_ml;           // [units, n_slices, NCOL, 2]
  float* tiles;             // scratch [units, cap4, NCOL], cap4 = cap in whole fours: per 16-token tile [NCOL][16] (the last
                            // tile: [NCOL][its tokens in whole fours]), partial logits, then final ones (which the merge
                            // kernel reads here)
  uint32_t* rec;            // scratch [units, cap4]: token records
  RetStream ret;            // the retained slots: the first n_ret_wgs workgroups
  int n_ret_wgs;            // a multiple of 8 (XCDs)
};

// Token record: LDS row indices i * w + h_i < 1024 of the three rows at bits 0, 10 and 20, bit 31 = the sign two of the three
// rows agree on (1 = minus, folded into the token's weight), bit 30 = the third listed row has the other sign.  The row whose
// sign differs from the other two, if any, is listed third.
__device__ __forceinline__ uint32_t make_record3(const DevDesc& d, int w, int J) {
  const uint32_t r0 = (uint32_t)bucket_of(d, 0, J), r1 = (uint32_t)(w + bucket_of(d, 1, J)),
                 r2 = (uint32_t)(2 * w + bucket_of(d, 2, J));
  const uint32_t s0 = sign_neg(d, 0, J) ? 1u : 0u, s1 = sign_neg(d, 1, J) ? 1u : 0u, s2 = sign_neg(d, 2, J) ? 1u : 0u;
  const uint32_t maj = (s0 & s1) | (s0 & s2) | (s1 & s2);
  const bool odd0 = s0 != maj, odd1 = s1 != maj;
  const uint32_t ra = odd0 ? r2 : r0, rbk = odd1 ? r2 : r1, rc = odd0 ? r0 : (odd1 ? r1 : r2);
  const uint32_t flip = (s0 ^ s1) | (s0 ^ s2);
  return ra | (rbk << 10) | (rc << 20) | (flip << 30) | (maj << 31);
}
// byte address of listed row I in LDS, plus base: two instructions (left to itself the compiler takes a shift, a mask and an
// addition where the pitch is a power of two)
template <int I, int PITCH>
__device__ __forceinline__ int record_row(uint32_t rec, int base) {
  const uint32_t row = __builtin_amdgcn_ubfe(rec, 10 * I, 10);
  if constexpr (PITCH == 128) {
    int a;
    asm("v_lshl_add_u32 %0, %1, 7, %2" : "=v"(a) : "v"(row), "v"(base));
    return a;
  } else {
    return (int)__umul24(row, PITCH) + base;
  }
}

// Copy chunk cc (64 channels) of a sketch tensor [rows][128] into LDS: PITCH / 16 16-byte places per row, a ninth is unused
// (its lanes read the row's last piece).
template <int PITCH>
__device__ __forceinline__ void stage_issue_pitch(const unsigned char* __restrict__ g, unsigned char* s_sk, int rows,
                                                  int cc, int tid) {
  const int lane = tid & 63, wave = tid >> 6;
  const int n_places = rows * (PITCH / 16);
  for (int p0 = wave * 64; p0 < n_places; p0 += MS_THREADS) {
    const uint32_t idx = (uint32_t)min(p0 + lane, n_places - 1);
    const uint32_t row = idx / (PITCH / 16), c = min(idx - row * (PITCH / 16), 7u);
    __builtin_amdgcn_global_load_lds(
        (const __attribute__((address_space(1))) void*)(g + (size_t)row * (D * 2) + cc * 128 + c * 16),
        (__attribute__((address_space(3))) void*)(s_sk + p0 * 16), 16, 0, 0);
  }
}

// Parts of a retained slot's weight: three (as many bits as float32) but for 16 columns, where two take two products as well.
constexpr int ret_parts(int n_col) { return n_col <= 8 ? 3 : 2; }

// The retained slots alone, before the list's launch, in workgroups of four waves of which many share a CU (StreamPlan::own).
constexpr int RA_WAVES = 4;
template <int NCOL>
__global__ __launch_bounds__(64 * RA_WAVES) void attend_slots_kernel(DevDesc d, RetStream a) {
  extern __shared__ __align__(16) unsigned char smem[];
  ret_stream_role<NCOL, ret_parts(NCOL), RA_WAVES>(d, a, blockIdx.x, gridDim.x, smem);
}

template <int NCOL>
__global__ __launch_bounds__(MS_THREADS) void attend_multi_staged_kernel(DevDesc d, MultiStagedArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int CH = 64;
  const float NEG_INF = -__builtin_inff();
  const int units = d.B * d.Hkv;
  // workgroup ids go round-robin to the 8 XCDs: all parts of a unit get ids that are equal modulo 8
  if ((int)blockIdx.x < a.n_ret_wgs) {
    ret_stream_role<NCOL, ret_parts(NCOL), MS_WAVES>(d, a.ret, blockIdx.x, a.n_ret_wgs, smem);
    return;
  }
  const int lin = blockIdx.x - a.n_ret_wgs;
  const int unit = ((lin >> 3) / a.n_parts) * 8 + (lin & 7);
  const int part_i = (lin >> 3) % a.n_parts;
  if (unit >= units) return;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r16 = lane >> 4, col = lane & 15;
  const int w = d.w;
  unsigned char* s_sk = smem;                                        // chunk; later [waves][NCOL][64] floats
  float* s_max = reinterpret_cast<float*>(smem + ms_chunk_lds(3 * w, NCOL));   // [waves][16]
  float* s_sum = s_max + MS_WAVES * 16;                              // [waves][16]
  int* s_ctr = reinterpret_cast<int*>(s_sum + MS_WAVES * 16);        // next tile of the running phase
  int* s_hidden = s_ctr + 1;                                         // some query must not see some token of this workgroup

  const int b = unit / d.Hkv, hk = unit % d.Hkv;
  const int rows = clampi(a.n_valid[unit], 0, a.cap);
  const int t_begin = min(part_i * a.part_tokens, rows);
  const int t_end = min(t_begin + a.part_tokens, rows);
  const int n_tiles = (t_end - t_begin + 15) >> 4;
  const int cap4 = (a.cap + 3) & ~3;
  const int32_t* pp = a.pos + (size_t)unit * a.cap;
  uint32_t* recs = a.rec + (size_t)unit * cap4;
  float* tiles = a.tiles + (size_t)unit * cap4 * NCOL;
  const size_t sk_unit = (size_t)unit * 3 * w * D;
  const unsigned char* skg = reinterpret_cast<const unsigned char*>(a.sk + sk_unit);
  const unsigned char* svg = reinterpret_cast<const unsigned char*>(a.sv + sk_unit);

  // this lane's column: query tq, head g
  const int tq = col / d.G, g = col % d.G;
  const bool col_live = col < NCOL;
  const int col_c = col_live ? col : 0;
  const int qpos = a.n_ctx ? a.n_ctx[b] - a.n_q + tq : 0x7fffffff;   // no n_ctx: no causal mask (decode call)

  // Tiles are handed out through a counter in LDS, phase by phase: of the four waves that share a SIMD the
  // ones started first win the issue arbitration, and with a fixed share each the workgroup would wait for
  // its slowest wave at the end of every phase.  One at a time: groups of four leave the last ones to a few waves (5 x 8 units
  // of 12706 tokens, 8 columns: 14 of 48 us), and asking for their inputs together gains nothing.
  const uint32_t ctr_at = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) int*)s_ctr;
  auto next_tile = [&]() {
    int t = 0;
    if (lane == 0)         // one lane: written out, because the compiler would first count the active lanes of an atomicAdd
      asm volatile("ds_add_rtn_u32 %0, %1, %2\n\ts_waitcnt lgkmcnt(0)" : "=v"(t) : "v"(ctr_at), "v"(1) : "memory");
    return __builtin_amdgcn_readfirstlane(t);
  };
  // tokens of a tile in whole fours (16 but for the list's last tile) = distance of its columns in `tiles`
  auto tile_pitch = [&](int ti) { return min(16, ((t_end - t_begin + 3) & ~3) - ti * 16); };

  // ---- K phases -----------------------------------------------------------------------------------
  // What a tile needs from memory is requested one tile ahead with unconditional loads, and what a tile leaves in memory
  // is stored one tile late.  Vector memory returns reads in order and writes in order, but not the two against each
  // other, so a wait for any read with a write outstanding drains everything: arranged like this, every such wait
  // only covers requests that are a whole tile old.  A look-ahead past the last tile reads the last tile again.
  struct KIn {
    uint32_t rec;       // record of token t0 + col
    float4 prev;        // second chunk: partial logits of tokens t0 + 4 r16 + i, this lane's column
  };
  float m_run = NEG_INF;
  if (tid == 0) { *s_ctr = 0; *s_hidden = 0; }
  for (int cc = 0; cc < 2; ++cc) {
    lds_barrier();                                            // every wave is done with the previous chunk
    stage_issue_pitch<MS_PITCH>(skg, s_sk, 3 * w, cc, tid);
    if (cc == 0) {
      // under the first chunk copy: the record of every token of this workgroup, one token per thread
      // (hashed once, not once per lane group that needs it); published by the barrier below
      const int q_first = a.n_ctx ? a.n_ctx[b] - a.n_q : 0x7fffffff;
      bool hidden = false;
      for (int t = t_begin + tid; t < ((t_end + 3) & ~3); t += MS_THREADS) {
        const int J = t < t_end ? pp[t] : 0;
        hidden = hidden || J < 0 || J > q_first;
        recs[t] = t < t_end ? make_record3(d, w, J) : 0u;
      }
      if (hidden) *s_hidden = 1;
    }
    // q of this lane's column, channels 64 cc + 32 kx + 8 r16 .. + 7
    uint4 qb[2];
    {
      const bf16_t* q = a.q + (((size_t)b * a.n_q + (col_live ? tq : 0)) * d.Hq + (size_t)hk * d.G + (col_live ? g : 0)) * D +
                        64 * cc + 8 * r16;
#pragma unroll
      for (int kx = 0; kx < 2; ++kx) {
        qb[kx] = *reinterpret_cast<const uint4*>(q + 32 * kx);
        if (!col_live) qb[kx] = make_uint4(0u, 0u, 0u, 0u);
      }
    }
    if (cc > 0 && tid == 0) *s_ctr = 0;
    stage_wait();
    lds_barrier();
    const bool hidden = *s_hidden != 0;
    auto k_loads = [&](int ti, KIn& in) {
      ti = min(ti, n_tiles - 1);
      const int t0 = t_begin + ti * 16, cp = tile_pitch(ti);
      in.rec = recs[t0 + min(col, cp - 1)];
      if (cc == 1)
        in.prev = *reinterpret_cast<const float4*>(tiles + (size_t)t0 * NCOL + col_c * cp + min(4 * r16, cp - 4));
    };
    // results of the previous tile, not yet stored
    int st_ti = n_tiles;
    float4 st_v = make_float4(0.f, 0.f, 0.f, 0.f);
    auto k_stores = [&]() {
      if (st_ti >= n_tiles) return;
      const int t0 = t_begin + st_ti * 16, cp = tile_pitch(st_ti);
      if (col_live && 4 * r16 < cp) *reinterpret_cast<float4*>(tiles + (size_t)t0 * NCOL + col * cp + 4 * r16) = st_v;
    };
    // Two input buffers take the tiles in turn (copying a buffer would wait for its loads).
    auto k_tile = [&](const KIn& cur, KIn& nxt, int ti, int ti_next) {
      const int t0 = t_begin + ti * 16;
      // the tile's inputs must have arrived here (empty statement that reads them), before the
      // previous tile's stores and the next tile's loads are issued
      if (cc == 0) asm volatile("" ::"v"(cur.rec));
      else asm volatile("" ::"v"(cur.rec), "v"(cur.prev.x), "v"(cur.prev.y), "v"(cur.prev.z), "v"(cur.prev.w));
      __builtin_amdgcn_sched_barrier(0);
      k_stores();
      __builtin_amdgcn_sched_barrier(0);
      k_loads(ti_next, nxt);
      __builtin_amdgcn_sched_barrier(0);
      st_ti = ti;
      if (ti >= n_tiles) return;                  // uniform: the wave's tiles are done
      const int a0 = record_row<0, MS_PITCH>(cur.rec, 16 * r16), a1 = record_row<1, MS_PITCH>(cur.rec, 16 * r16),
                a2 = record_row<2, MS_PITCH>(cur.rec, 16 * r16);
      uint4 ka[2];
#pragma unroll
      for (int kx = 0; kx < 2; ++kx) {
        const uint4 x0 = *reinterpret_cast<const uint4*>(s_sk + a0 + 64 * kx);
        const uint4 x1 = *reinterpret_cast<const uint4*>(s_sk + a1 + 64 * kx);
        const uint4 x2 = *reinterpret_cast<const uint4*>(s_sk + a2 + 64 * kx);
        ka[kx] = med3_fast_piece(x0, x1, x2);
      }
      f32x4_t S = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kx = 0; kx < 2; ++kx)
        S = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8ms_t, ka[kx]),
                                                    __builtin_bit_cast(bf16x8ms_t, qb[kx]), S, 0, 0, 0);
      st_v = make_float4(S[0], S[1], S[2], S[3]);
      if (cc == 1) {
        float4 x = make_float4((S[0] + cur.prev.x) * d.scale, (S[1] + cur.prev.y) * d.scale,
                               (S[2] + cur.prev.z) * d.scale, (S[3] + cur.prev.w) * d.scale);
        const int n = t_end - t0 - 4 * r16;       // tokens of the lane's four that the list still has
        if (t_end - t0 < 16) {                    // uniform: the list's last tile
          if (n < 1) x.x = NEG_INF;
          if (n < 2) x.y = NEG_INF;
          if (n < 3) x.z = NEG_INF;
          if (n < 4) x.w = NEG_INF;
        }
        if (hidden) {                             // uniform
          const int32_t* p4 = pp + t0 + 4 * r16;
          if (n > 0 && (p4[0] < 0 || p4[0] > qpos)) x.x = NEG_INF;
          if (n > 1 && (p4[1] < 0 || p4[1] > qpos)) x.y = NEG_INF;
          if (n > 2 && (p4[2] < 0 || p4[2] > qpos)) x.z = NEG_INF;
          if (n > 3 && (p4[3] < 0 || p4[3] > qpos)) x.w = NEG_INF;
        }
        if (col_live) m_run = fmaxf(fmaxf(fmaxf(x.x, x.y), fmaxf(x.z, x.w)), m_run);
        st_v = x;
      }
    };
    if (n_tiles > 0) {
      KIn in_a, in_b;
      int ti = next_tile();
      k_loads(ti, in_a);
      while (ti < n_tiles) {
        const int t1 = next_tile();
        k_tile(in_a, in_b, ti, t1);
        const int t2 = next_tile();
        k_tile(in_b, in_a, t1, t2);
        ti = t2;
      }
      k_stores();
    }
  }
  // the wave's maximum per column (the four 16-lane rows hold different tokens of the same column)
  m_run = rows_max(m_run);
  if (r16 == 0) s_max[wave * 16 + col] = m_run;

  // ---- V phases -----------------------------------------------------------------------------------
  const size_t part = (size_t)unit * a.n_slices + a.slice0 + part_i;
  float l_run = 0.f;
  for (int cc = 0; cc < 2; ++cc) {
    lds_barrier();                                            // every wave is done with the previous chunk
    stage_issue_pitch<128>(svg, s_sk, 3 * w, cc, tid);
    if (tid == 0) *s_ctr = 0;
    if (cc == 0) {
      // a wave meets other tiles here than in the K phases: weights against the workgroup's maximum
      float M = s_max[col];
#pragma unroll
      for (int w_ = 1; w_ < MS_WAVES; ++w_) M = fmaxf(M, s_max[w_ * 16 + col]);
      m_run = M;
    }
    stage_wait();                                             // also: this wave's logits stores have landed
    lds_barrier();
    f32x4_t acc[4];                                           // acc[c][i]: column 4 r16 + i, channel 64 cc + 4 col + c
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    // this lane's four tokens of a tile: records, and their logits for this lane's column; requested two
    // tiles ahead with unconditional loads (no stores in these phases: the waits are exact).  One tile ahead: 8.4 instead of
    // 5.5 us a phase of 8 tiles per wave
    struct VIn {
      uint4 rec;
      float4 s;
    };
    // a column without any visible token: all weights 0; a column that is none: the same
    const float m_safe = !col_live ? -NEG_INF : (m_run == NEG_INF) ? 0.f : m_run;
    auto v_loads = [&](int ti, VIn& in) {
      ti = min(ti, n_tiles - 1);
      const int t0 = t_begin + ti * 16, cp = tile_pitch(ti), f = min(4 * r16, cp - 4);
      in.rec = *reinterpret_cast<const uint4*>(recs + t0 + f);
      in.s = *reinterpret_cast<const float4*>(tiles + (size_t)t0 * NCOL + col_c * cp + f);
    };
    auto v_tile = [&](const VIn& cur, VIn& nxt, int ti, int ti_next) {
      const int t0 = t_begin + ti * 16;
      v_loads(ti_next, nxt);
      __builtin_amdgcn_sched_barrier(0);
      if (ti >= n_tiles) return;                              // uniform
      const uint32_t rj[4] = {cur.rec.x, cur.rec.y, cur.rec.z, cur.rec.w};
      const float sl[4] = {cur.s.x, cur.s.y, cur.s.z, cur.s.w};
      // past the list's last four these lanes read what is not theirs
      float m = m_safe;
      if (t_end - t0 < 16 && 4 * r16 >= t_end - t0) m = -NEG_INF;
      float p[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        p[j] = __expf(sl[j] - m);                         // -inf (masked, or past the end) gives 0
        l_run += p[j];
        // the sign two of the token's three rows agree on goes onto the weight
        p[j] = __uint_as_float(__float_as_uint(p[j]) ^ (rj[j] & 0x80000000u));
      }
      uint32_t hb[4], lb[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        hb[i] = __float_as_uint(p[i]) & 0xffff0000u;
        lb[i] = __float_as_uint(p[i] - __uint_as_float(hb[i]));
      }
      const short4_t a_hi = pack_k4(pair_hi(hb[0], hb[1]), pair_hi(hb[2], hb[3]));
      const short4_t a_lo = pack_k4(pair_hi(lb[0], lb[1]), pair_hi(lb[2], lb[3]));
      // channels 4 col .. + 3 of the chunk for the four tokens: 8 bytes at offset 8 col of each row (the results go
      // through v_perm_b32 before they reach a matrix instruction)
      uint2 vt[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint2 x0 = *reinterpret_cast<const uint2*>(s_sk + record_row<0, 128>(rj[j], 8 * col));
        const uint2 x1 = *reinterpret_cast<const uint2*>(s_sk + record_row<1, 128>(rj[j], 8 * col));
        uint2 x2 = *reinterpret_cast<const uint2*>(s_sk + record_row<2, 128>(rj[j], 8 * col));
        const uint32_t fm = (uint32_t)((int)(rj[j] << 1) >> 31) & 0x80008000u;
        x2.x ^= fm;
        x2.y ^= fm;
        vt[j] = make_uint2(med3_fast_alu(x0.x, x1.x, x2.x), med3_fast_alu(x0.y, x1.y, x2.y));
      }
      short4_t bop[4];
      bop[0] = pack_k4(pair_lo(vt[0].x, vt[1].x), pair_lo(vt[2].x, vt[3].x));
      bop[1] = pack_k4(pair_hi(vt[0].x, vt[1].x), pair_hi(vt[2].x, vt[3].x));
      bop[2] = pack_k4(pair_lo(vt[0].y, vt[1].y), pair_lo(vt[2].y, vt[3].y));
      bop[3] = pack_k4(pair_hi(vt[0].y, vt[1].y), pair_hi(vt[2].y, vt[3].y));
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[c] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a_hi, bop[c], acc[c], 0, 0, 0);
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[c] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a_lo, bop[c], acc[c], 0, 0, 0);
    };
    if (n_tiles > 0) {
      VIn in_a, in_b, in_c;
      int ta = next_tile();
      v_loads(ta, in_a);
      int tb = next_tile();
      v_loads(tb, in_b);
      while (ta < n_tiles) {
        const int t2 = next_tile();
        v_tile(in_a, in_c, ta, t2);
        ta = next_tile();
        v_tile(in_b, in_a, tb, ta);
        tb = next_tile();
        v_tile(in_c, in_b, t2, tb);
      }
    }
    if (cc == 0) {
      // a lane's sum of weights covers its own four tokens of every tile: add the four 16-lane rows
      const float l = rows_sum(l_run);
      if (r16 == 0) s_sum[wave * 16 + col] = l;
    }
    lds_barrier();                                            // the chunk is free: the waves' sums meet in it
    float* s_acc = reinterpret_cast<float*>(s_sk);            // [waves][NCOL][64]
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int c_ = 4 * r16 + i;
      if (c_ < NCOL) {
        *reinterpret_cast<float4*>(s_acc + ((size_t)wave * NCOL + c_) * CH + 4 * col) =
            make_float4(acc[0][i], acc[1][i], acc[2][i], acc[3][i]);
      }
    }
    lds_barrier();
    for (int idx = tid; idx < NCOL * CH; idx += MS_THREADS) {
      const int c_ = idx / CH, ch = idx % CH;
      float M = s_max[c_];
#pragma unroll
      for (int w_ = 1; w_ < MS_WAVES; ++w_) M = fmaxf(M, s_max[w_ * 16 + c_]);
      float L = 0.f, O = 0.f;
#pragma unroll
      for (int w_ = 0; w_ < MS_WAVES; ++w_) {
        L += s_sum[w_ * 16 + c_];
        O += s_acc[((size_t)w_ * NCOL + c_) * CH + ch];
      }
      a.part_o[(part * NCOL + c_) * D + cc * CH + ch] = O;
      if (cc == 0 && ch == 0) {
        a.part_ml[(part * NCOL + c_) * 2] = M;
        a.part_ml[(part * NCOL + c_) * 2 + 1] = L;
      }
    }
  }
}

// ---- host side ----------------------------------------------------------------------------------------
bool multi_staged_applies(const DevDesc& d, long long vague_cap) {
  return d.r == 3 && d.sign_mask == 2 && 3 * d.w <= 1024 && vague_cap >= 64;
}

// Tokens per workgroup, at least 256 (below, its fixed part is nearly all there is).  One workgroup (16 waves, the chunk in
// LDS) runs per CU, so a launch takes ceil(workgroups / 256) turns of (fixed part + tokens of a workgroup), and a unit gets
// as many parts as one turn holds: with n parts on one turn, n + 1 on two cost 2 (fixed + tokens / (n + 1)), never less
// than fixed + tokens / n.  40 units x 12706 tokens, 8 columns: 7 parts (280 workgroups, the last 24 on a turn of their own)
// 82 us, 6 parts 49 us.  A turn of 256 workgroups, 8 columns, 273 slots per row: 34.7 us at 1024 tokens each, 87.5 at 4096.
int multi_staged_part_tokens(long long vague_cap, long long units) {
  const long long turn = units < 256 ? 256 / units : 1;
  const long long n = std::max(1ll, std::min(turn, (vague_cap - 1) / 255));       // ceil(vague_cap / n) >= 256
  const long long t = std::max(256ll, (vague_cap + n - 1) / n);
  return (int)((t + 15) / 16 * 16);
}

template <int NCOL>
static hipError_t launch_n(const DevDesc& d, const MultiStagedArgs& a, int lds, bool own, hipStream_t st) {
  auto kern = attend_multi_staged_kernel<NCOL>;
  static std::once_flag once;
  static hipError_t attr_rc = hipSuccess;
  std::call_once(once, [&]() {
    attr_rc = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                  160 * 1024);
  });
  if (attr_rc != hipSuccess) return attr_rc;
  if (lds < multi_staged_lds(d, NCOL) || lds > STAGED_LDS_LIMIT) return hipErrorInvalidValue;
  const int units = d.B * d.Hkv;
  const int units_pad = (units + 7) / 8 * 8;
  if (own) {
    const int slots_lds = ret_stream_lds(NCOL, RA_WAVES, a.ret.slice_tokens);
    if (slots_lds > 64 * 1024) return hipErrorInvalidValue;
    hipLaunchKernelGGL(attend_slots_kernel<NCOL>, dim3(units * a.ret.n_rslices), dim3(64 * RA_WAVES), slots_lds, st, d, a.ret);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kern, dim3(a.n_ret_wgs + units_pad * a.n_parts), dim3(MS_THREADS), lds, st, d, a);
  return hipGetLastError();
}

int multi_staged_lds(const DevDesc& d, int n_col) {
  return ms_chunk_lds(3 * d.w, n_col) + 2 * MS_WAVES * 16 * (int)sizeof(float) + 16;
}

hipError_t launch_attend_multi_staged(const DevDesc& d, const AttendArgs& a0, const int32_t* n_ctx, int n_q,
                                      const StreamPlan& plan, hipStream_t st) {
  if (!multi_staged_applies(d, a0.vague_cap) || plan.n_vslices < 1 || (plan.vslice_tokens & 15) != 0) return hipErrorInvalidValue;
  MultiStagedArgs a;
  a.q = (const bf16_t*)a0.q;
  a.n_ctx = n_ctx;
  a.n_q = n_q;
  a.sk = (const bf16_t*)a0.sk;
  a.sv = (const bf16_t*)a0.sv;
  a.pos = a0.vague_pos;
  a.n_valid = a0.n_vague;
  a.cap = a0.vague_cap;
  a.part_tokens = plan.vslice_tokens;
  a.n_parts = plan.n_vslices;
  a.slice0 = plan.n_rslices;
  a.n_slices = plan.n_rslices + plan.n_vslices;
  a.part_o = a0.part_o;
  a.part_ml = a0.part_ml;
  a.tiles = a0.tiles;
  a.rec = (uint32_t*)a0.scratch_rec;
  a.ret = RetStream{(const bf16_t*)a0.q, (const bf16_t*)a0.k_ret, (const bf16_t*)a0.v_ret, a0.ret_pos, n_ctx, n_q, a0.ret_cap,
                    plan.rslice_tokens, plan.n_rslices, a.n_slices, a0.ret_cap, a0.part_o, a0.part_ml, a0.logits};
  a.n_ret_wgs = plan.n_ret_wgs;
  switch (n_q * d.G) {
    case 1: return launch_n<1>(d, a, plan.lds, plan.own, st);
    case 2: return launch_n<2>(d, a, plan.lds, plan.own, st);
    case 4: return launch_n<4>(d, a, plan.lds, plan.own, st);
    case 8: return launch_n<8>(d, a, plan.lds, plan.own, st);
    case 16: return launch_n<16>(d, a, plan.lds, plan.own, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace kvr
