// Staged attention kernel over the Vague list in chunks of 16 channels: four sketch
// rows, or three whose sketch is too wide for the 64-channel kernel (bf16 storage,
// values signed only, G <= 4 query heads per kv head).  Same contract and the same
// token -> wave mapping as the general staged kernel (kvr_attend_staged.hip), which
// takes what is wider still (more than 4096 rows in all).
//
// Such a sketch is large (131k tokens: 4 x 819 or 3 x 1092 slots of 256 bytes per
// tensor), so it goes through LDS in chunks of 16 channels
// (32 bytes per slot; eight chunks of the K sketch, then eight of the V sketch).
// Inside a chunk the unit of work is a *half piece*: 4 channels = 8 bytes, which
// is exactly the contraction length of v_mfma_f32_4x4x4.
//
// Vector ALUs 71 % busy with four rows; with three 58 % at 1092 slots per row and 68 % at 350, where the sixteen chunk
// phases (copy, barriers, reduction) are worth 66 of a turn's 140 us and 30 of its 111.  Three rows against the general
// kernel: 131072 tokens, 16 units 353 -> 136 us; one layer's whole decode step, with what else changed in it: 454 -> 231 us,
// 8 units 263 -> 172; 70000 tokens, 24 units 235 -> 184; 42000 tokens, 48 units 260 -> 199, 8 units 92 -> 86.  (A sketch with
// about as many slots as tokens loses: 256 units, 1500 tokens, 3 x 400 slots 182 -> 200 us a call.)
// The launch also holds workgroups that stream the retained slots (kvr_ret_stream.h) on CUs of their own, and a wave takes up
// to 17 rounds of 64 tokens (four rows: 24) in 256 registers, where it took 13: 16 units of 101580 + 29492 tokens, us a call
// 206 -> 174, four rows, 32 units 520 -> 476 .. 506.
// Error of a call's output against float64, relative in the 2-norm, three rows: 1.6e-7 (200 tokens) .. 3.0e-7 (101580), as
// with the general kernel's float32 multiply-adds (1.7e-7 .. 3.2e-7); weights as two bf16 parts: 8e-6 .. 1.1e-5, three
// parts cost 1 % of the time.  Four rows: two parts, 7e-6 .. 1.1e-5.
//
//  * K phases: one lane = one token.  The 4 lanes of a block read the same half
//    piece of their tokens' rows (neighbouring blocks take different half pieces,
//    so the 16 lanes served together spread over the banks), the median is taken on
//    packed bf16 bits, and one matrix instruction per
//    half piece multiplies the block's 4 rebuilt tokens (A, one row per lane) with
//    q (B, column j = head j): lane j receives the logits of the block's 4 tokens
//    for head j -- already the layout the V phases want for their A operand, so the
//    softmax needs no transposition afterwards.
//  * V phases: a quad rebuilds the 4 tokens its own lanes own, lane `sub` taking
//    half piece `sub` of every row; a token's row offsets and flip masks reach the
//    quad by DPP quad broadcasts.  With the mean-of-the-middle-two rule (an odd
//    function of the four values) g_0 is folded into the token's weight and the
//    other rows are flipped relative to row 0; with the lower-middle rule every row
//    is flipped by its own sign.  p.v on the same matrix instruction with the 4
//    tokens as the contraction index; weights as two or three bf16 parts.
//  * Every loop over LDS reads is a pinned software pipeline (rows of the step
//    after next requested, medians of the next step formed, matrix instruction of
//    this step issued): two waves per SIMD cannot hide LDS latency for each other.
//  * The copy of the next chunk is started as soon as every wave is done with the
//    current one and overlaps the reduction of the V partial sums, which have LDS
//    of their own (two sets that take turns, so that a chunk needs two barriers).
#include "kvr_ret_stream.h"

namespace kvr {
namespace {

constexpr int S16_CH = 16;                 // channels per chunk
constexpr int S16_ROWB = 32;               // bytes per LDS row
constexpr int S16_NHP = 4;                 // 8-byte half pieces per LDS row
constexpr int S16_NCHUNK = D / S16_CH;      // chunks per tensor
constexpr int S16_NROW = ST_WAVES * 4;     // 16-lane rows per workgroup

template <int R>
struct Rows {
  uint2 r[R];
};

template <int R>
__device__ __forceinline__ void load_rows(Rows<R>& o, const unsigned char* s_sk, const int (&rb)[R], int co) {
#pragma unroll
  for (int i = 0; i < R; ++i) o.r[i] = *reinterpret_cast<const uint2*>(s_sk + rb[i] + co);
}

template <int R, int MODE>
__device__ __forceinline__ uint2 median_rows_of(const Rows<R>& v) {
  if constexpr (R == 3) {
    return med3_fast_half_piece(v.r[0], v.r[1], v.r[2]);
  } else {
    const uint32_t x[4] = {v.r[0].x, v.r[1].x, v.r[2].x, v.r[3].x};
    const uint32_t y[4] = {v.r[0].y, v.r[1].y, v.r[2].y, v.r[3].y};
    return make_uint2(median_dword<4>(x, MODE), median_dword<4>(y, MODE));
  }
}

// value of lane J of this lane's quad
template <int J>
__device__ __forceinline__ uint32_t quad_bcast(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, J | (J << 2) | (J << 4) | (J << 6), 0xf, 0xf, true);
}

// Token record (2 dwords).  LDS row indices (i * w + h_i(J) < 4096) are stored
// pre-multiplied by the 32-byte row pitch: row 0 in x[5..16], row 1 in x[17..28],
// row 2 in y[5..16], row 3 in y[17..28].  Bit 0 of x is a sign that is folded into
// the token's weight; bit 30 of x, bit 31 of x, bit 31 of y and bit 30 of y say
// whether rows 0, 1, 2, 3 are flipped before the median.
//
// Four rows: the mean of the two middle values is an odd function of the four
// values, so there g_0 goes onto the weight and the rows are flipped relative to
// row 0 (row 0 never is); the lower of the two middle values is not odd, so there
// nothing is folded and every row is flipped by its own sign.
// Three rows: two of the three signs always agree; theirs goes onto the weight and
// the row with the other sign, if there is one, is listed last (a median does not
// care about the order), so that only "row 2" is ever flipped.
template <int R, int MODE>
__device__ __forceinline__ uint2 make_record(const DevDesc& d, int w, int J) {
  uint32_t r[R], s[R];
#pragma unroll
  for (int i = 0; i < R; ++i) {
    r[i] = (uint32_t)(i * w + bucket_of(d, i, J));
    s[i] = sign_neg(d, i, J) ? 1u : 0u;
  }
  if constexpr (R == 3) {
    const uint32_t maj = (s[0] & s[1]) | (s[2] & (s[0] | s[1]));
    const uint32_t flip = (s[0] ^ s[1]) | (s[0] ^ s[2]);
    const bool last0 = (s[0] != maj), last1 = (s[1] != maj);
    const uint32_t q0 = last0 ? r[2] : r[0];
    const uint32_t q1 = last1 ? r[2] : r[1];
    const uint32_t q2 = last0 ? r[0] : (last1 ? r[1] : r[2]);
    return make_uint2((q0 << 5) | (q1 << 17) | maj, (q2 << 5) | (flip << 31));
  } else {
    const uint32_t fold = (MODE == KVR_MEDIAN_MIDMEAN) ? s[0] : 0u;
    return make_uint2((r[0] << 5) | (r[1] << 17) | fold | ((s[0] ^ fold) << 30) | ((s[1] ^ fold) << 31),
                      (r[2] << 5) | (r[3] << 17) | ((s[2] ^ fold) << 31) | ((s[3] ^ fold) << 30));
  }
}
template <int R>
__device__ __forceinline__ void rec_offsets(uint2 rec, int (&rb)[R]) {
  rb[0] = (int)(rec.x & 0x1ffe0u);
  rb[1] = (int)((rec.x >> 12) & 0x1ffe0u);
  rb[2] = (int)(rec.y & 0x1ffe0u);
  if constexpr (R > 3) rb[3] = (int)((rec.y >> 12) & 0x1ffe0u);
}

// first row that a V phase may have to flip
template <int R, int MODE>
__host__ __device__ constexpr int first_flip() {
  return R == 3 ? 2 : (MODE == KVR_MEDIAN_MIDMEAN ? 1 : 0);
}

// V phases: what a lane derives from its own token's record (row offsets and flip
// masks); the other lanes of the quad fetch it with quad broadcasts, so a record is
// taken apart once per quad.
template <int R>
struct VOwn {
  int o[R];
  uint32_t f[R];
};
template <int R>
__device__ __forceinline__ VOwn<R> v_own(uint2 rec) {
  VOwn<R> v;
  rec_offsets<R>(rec, v.o);
  v.f[0] = (uint32_t)((int)(rec.x << 1) >> 31) & 0x80008000u;
  v.f[1] = (uint32_t)((int)rec.x >> 31) & 0x80008000u;
  v.f[2] = (uint32_t)((int)rec.y >> 31) & 0x80008000u;
  if constexpr (R > 3) v.f[3] = (uint32_t)((int)(rec.y << 1) >> 31) & 0x80008000u;
  return v;
}
template <int R>
struct VItem {
  Rows<R> rows;
  uint32_t f[R];
};
template <int J, int R, int MODE>
__device__ __forceinline__ void v_fetch(VItem<R>& o, const VOwn<R>& own, const unsigned char* s_sk, int co) {
  int rb[R];
#pragma unroll
  for (int i = 0; i < R; ++i) {
    rb[i] = (int)quad_bcast<J>((uint32_t)own.o[i]) + co;
    o.f[i] = (i < first_flip<R, MODE>()) ? 0u : quad_bcast<J>(own.f[i]);
  }
  load_rows<R>(o.rows, s_sk, rb, 0);
}
template <int R, int MODE>
__device__ __forceinline__ uint2 v_median(const VItem<R>& it) {
  Rows<R> x = it.rows;
#pragma unroll
  for (int i = first_flip<R, MODE>(); i < R; ++i) x.r[i] = make_uint2(it.rows.r[i].x ^ it.f[i], it.rows.r[i].y ^ it.f[i]);
  return median_rows_of<R, MODE>(x);
}

// A weight goes into the matrix instruction as a sum of bf16 parts, each the upper half of what the parts before it
// leave.  Three rows: three parts, which hold all 24 bits of the float32 weight, as the float32 multiply-adds of the
// general kernel do.  Four rows: two parts (16 bits).
template <int R>
__host__ __device__ constexpr int weight_parts() {
  return R == 3 ? 3 : 2;
}

// acc[c] (4 head sums of channel c of the half piece) += weights (4 heads x 4 tokens, packed parts W: two dwords
// each, largest first) x values (4 tokens x 4 channels)
template <int NP>
__device__ __forceinline__ void pv_half_piece(const uint2 (&med)[4], const uint32_t (&W)[2 * NP], f32x4_t (&acc)[4]) {
  short4_t b[4];
  b[0] = pack_k4(pair_lo(med[0].x, med[1].x), pair_lo(med[2].x, med[3].x));
  b[1] = pack_k4(pair_hi(med[0].x, med[1].x), pair_hi(med[2].x, med[3].x));
  b[2] = pack_k4(pair_lo(med[0].y, med[1].y), pair_lo(med[2].y, med[3].y));
  b[3] = pack_k4(pair_hi(med[0].y, med[1].y), pair_hi(med[2].y, med[3].y));
#pragma unroll
  for (int p = 0; p < NP; ++p)
#pragma unroll
    for (int c = 0; c < 4; ++c)
      acc[c] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(pack_k4(W[2 * p], W[2 * p + 1]), b[c], acc[c], 0, 0, 0);
}

// The same value, but the compiler can no longer tell: whatever is derived from
// it is computed where it is used instead of once per kernel and kept in
// registers through all phases.
__device__ __forceinline__ uint2 opaque(uint2 v) {
  asm volatile("" : "+v"(v.x), "+v"(v.y));
  return v;
}
__device__ __forceinline__ int opaque_s(int v) {
  asm volatile("" : "+s"(v));
  return v;
}

#define KVR_PIN() __builtin_amdgcn_sched_barrier(0)

// The two waves that share a SIMD take turns in having the higher issue priority,
// round by round; both levels are above the default 0.
__device__ __forceinline__ void take_turn(int t) {
  if (t & 1) __builtin_amdgcn_s_setprio(2);
  else __builtin_amdgcn_s_setprio(1);
}

// K pass over the rounds of one chunk.  qx[j]: the 4 channels of q for head (lane
// mod 4) that belong to the half piece this lane's block reads at step j (byte
// offset co[j] of the row).  s[k][i]: logit of token i of this lane's quad in round
// k, for head (lane mod 4).  Pipeline over the steps t = 4 k + j: rows of step t + 2
// requested, median of step t + 1 formed, matrix instruction of step t issued.  (Behind the last round it reads rows that a
// zero record names, and drops them.)
template <int KMAX, int R, int MODE>
__device__ __forceinline__ void k_pass(const unsigned char* s_sk, const uint2 (&info)[KMAX], int n_k,
                                       const uint2 (&qx)[S16_NHP], const int (&co)[S16_NHP], int turn,
                                       float (&s)[KMAX][4]) {
  Rows<R> buf[3];                        // rows of step t live in buf[t % 3]
  int rb[R];
  rec_offsets<R>(opaque(info[0]), rb);
  load_rows<R>(buf[0], s_sk, rb, co[0]);
  load_rows<R>(buf[1], s_sk, rb, co[1]);
  uint2 m[2];                            // median of step t in m[t % 2]
  m[0] = median_rows_of<R, MODE>(buf[0]);
  for_rounds<KMAX>(n_k, [&](auto kc) __attribute__((always_inline)) {
    constexpr int k = decltype(kc)::value;
    int rn[R];
    rec_offsets<R>(opaque(info[k + 1 < KMAX ? k + 1 : k]), rn);
    f32x4_t ax = {0.f, 0.f, 0.f, 0.f};
    take_turn(k + turn);
#pragma unroll
    for (int j = 0; j < S16_NHP; ++j) {
      const int t = S16_NHP * k + j;
      if (j + 2 < S16_NHP) load_rows<R>(buf[(t + 2) % 3], s_sk, rb, co[j + 2]);
      else load_rows<R>(buf[(t + 2) % 3], s_sk, rn, co[j + 2 - S16_NHP]);
      KVR_PIN();
      m[(t + 1) & 1] = median_rows_of<R, MODE>(buf[(t + 1) % 3]);
      KVR_PIN();
      const uint2 mc = m[t & 1];
      ax = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(pack_k4(mc.x, mc.y), pack_k4(qx[j].x, qx[j].y), ax, 0, 0, 0);
      KVR_PIN();
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      s[k][i] += ax[i];
      asm volatile("" : "+v"(s[k][i]));        // formed here, not where it is used next
    }
#pragma unroll
    for (int i = 0; i < R; ++i) rb[i] = rn[i];
  });
  __builtin_amdgcn_s_setprio(1);
}

// V pass over the rounds of one chunk for the half piece at byte offset co of each
// row: the quad's 4 tokens per round, same kind of pipeline.
template <int KMAX, int R, int MODE>
__device__ __forceinline__ void v_pass(const unsigned char* s_sk, const uint2 (&info)[KMAX], int n_k,
                                       const uint32_t (&W)[KMAX][2 * weight_parts<R>()], int co, int turn,
                                       f32x4_t (&acc)[4]) {
  VItem<R> buf[4];
  VOwn<R> own = v_own<R>(opaque(info[0]));
  v_fetch<0, R, MODE>(buf[0], own, s_sk, co);
  v_fetch<1, R, MODE>(buf[1], own, s_sk, co);
  for_rounds<KMAX>(n_k, [&](auto kc) __attribute__((always_inline)) {
    constexpr int k = decltype(kc)::value;
    uint2 med[4];
    take_turn(k + turn);
    v_fetch<2, R, MODE>(buf[2], own, s_sk, co);
    KVR_PIN();
    med[0] = v_median<R, MODE>(buf[0]);
    KVR_PIN();
    v_fetch<3, R, MODE>(buf[3], own, s_sk, co);
    own = v_own<R>(opaque(info[k + 1 < KMAX ? k + 1 : k]));
    KVR_PIN();
    med[1] = v_median<R, MODE>(buf[1]);
    KVR_PIN();
    v_fetch<0, R, MODE>(buf[0], own, s_sk, co);
    KVR_PIN();
    med[2] = v_median<R, MODE>(buf[2]);
    KVR_PIN();
    v_fetch<1, R, MODE>(buf[1], own, s_sk, co);
    KVR_PIN();
    med[3] = v_median<R, MODE>(buf[3]);
    pv_half_piece<weight_parts<R>()>(med, W[k], acc);
    KVR_PIN();
  });
  __builtin_amdgcn_s_setprio(1);
}

// LDS of a workgroup: one chunk, two sets of V partial sums [NROW][G][CH], wave statistics, q
__host__ __device__ constexpr int chunk_bytes(int r, int w) { return (r * w * S16_ROWB + 1023) & ~1023; }
__host__ __device__ constexpr int stat_floats(int G) { return 3 * ST_WAVES * G; }

}  // namespace

// One workgroup's share (part vs of a.n_vslices) of a unit's Vague list.
template <int G, int R, int MODE>
__device__ __forceinline__ void vague16_part(const DevDesc& d, const AttendArgs& a, int unit, int vs, unsigned char* smem) {
  constexpr int KMAX = staged16_kmax(R), CH = S16_CH;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int b = unit / d.Hkv, hk = unit % d.Hkv;
  const int w = d.w;
  const int cb = chunk_bytes(R, w);
  unsigned char* s_sk = smem;                                             // one 16-channel chunk
  float* s_part = reinterpret_cast<float*>(smem + cb);                    // [2][NROW][G][CH]
  float* s_stat = s_part + 2 * S16_NROW * G * CH;                          // [8 waves][G] maxima, sums, factors
  uint2* s_q = reinterpret_cast<uint2*>(s_stat + stat_floats(G));         // [G][32] half pieces of q

  const int nv = clampi(a.n_vague[unit], 0, a.vague_cap);
  const int rounds_total = (nv + 63) >> 6;
  const int NWT = a.n_vslices * ST_WAVES;
  const int gw = vs * ST_WAVES + wave;
  int n_k = gw < rounds_total ? (rounds_total - gw + NWT - 1) / NWT : 0;
  if (n_k > KMAX) n_k = KMAX;             // cannot happen when the plan was made for vague_cap
  n_k = __builtin_amdgcn_readfirstlane(n_k);      // equal in all lanes of a wave; now the compiler knows
  const int turn = __builtin_amdgcn_readfirstlane(wave >> 2);   // waves i and i + 4 share a SIMD

  const size_t sk_unit = (size_t)unit * R * w * D;      // elements
  const unsigned char* skg = reinterpret_cast<const unsigned char*>((const bf16_t*)a.sk + sk_unit);
  const unsigned char* svg = reinterpret_cast<const unsigned char*>((const bf16_t*)a.sv + sk_unit);
  const int n_pieces = R * w * (S16_ROWB / 16);          // 16-byte pieces of a chunk

  __builtin_amdgcn_s_setprio(1);
  // ---- loads first: Vague positions of this wave's tokens and q ---------------
  int Jv[KMAX];
  const int32_t* vpos = a.vague_pos + (size_t)unit * a.vague_cap;
  for_rounds<KMAX>(n_k, [&](auto kc) __attribute__((always_inline)) {
    constexpr int k = decltype(kc)::value;
    const int tok = (gw + k * NWT) * 64 + lane;
    Jv[k] = vpos[min(tok, nv - 1)];        // (a choice made here would wait for the load, round by round)
  });
  uint4 qv = make_uint4(0u, 0u, 0u, 0u);
  if (tid < G * 16)
    qv = reinterpret_cast<const uint4*>((const bf16_t*)a.q + ((size_t)b * d.Hq + (size_t)hk * G) * D)[tid];
  // Wait for them here, so that the hashes below do not have to wait for the chunk
  // copy that is started next: memory operations complete in order.
  __builtin_amdgcn_s_waitcnt(0x0F70);

  // ---- the first K chunk is on its way while the hashes are computed ----------
  stage_issue<S16_ROWB / 16, S16_ROWB>(skg, s_sk, n_pieces, 0, tid);

  uint2 info[KMAX];
#pragma unroll
  for (int k = 0; k < KMAX; ++k) info[k] = make_uint2(0u, 0u);
  for_rounds<KMAX>(n_k, [&](auto kc) __attribute__((always_inline)) {
    constexpr int k = decltype(kc)::value;
    const int J = Jv[k];
    if (J >= 0 && (gw + k * NWT) * 64 + lane < nv) info[k] = make_record<R, MODE>(d, w, J);
  });
  if (tid < G * 16) reinterpret_cast<uint4*>(s_q)[tid] = qv;

  // ---- K phases: logits -----------------------------------------------------
  // s[k][i]: token i of this lane's quad in round k, head (lane mod 4)
  float s[KMAX][4];
#pragma unroll
  for (int k = 0; k < KMAX; ++k)
#pragma unroll
    for (int i = 0; i < 4; ++i) s[k][i] = 0.f;

  const int sub = lane & 3, tl = lane >> 2;
  for (int cc = 0; cc < S16_NCHUNK; ++cc) {
    stage_wait();
    lds_barrier();                         // chunk cc is complete
    {
      uint2 qx[S16_NHP];
      int co[S16_NHP];
#pragma unroll
      for (int j = 0; j < S16_NHP; ++j) {
        const int hp = (tl + j) & (S16_NHP - 1);       // the block's half piece at step j
        co[j] = hp * 8;
        qx[j] = (sub < G) ? s_q[sub * 32 + cc * S16_NHP + hp] : make_uint2(0u, 0u);
      }
      k_pass<KMAX, R, MODE>(s_sk, info, n_k, qx, co, turn, s);
    }
    lds_barrier();                         // every wave is done with chunk cc
    if (cc + 1 < S16_NCHUNK) stage_issue<S16_ROWB / 16, S16_ROWB>(skg, s_sk, n_pieces, cc + 1, tid);
    else stage_issue<S16_ROWB / 16, S16_ROWB>(svg, s_sk, n_pieces, 0, tid);       // the first V chunk, under the softmax
  }

  // ---- softmax weights against the wave's own maximum ---------------------------
  // Lane (quad t, sub) holds the logits of the quad's 4 tokens for head `sub` (nothing
  // of use if there is no such head).
  const int tot_cap = a.ret_cap + a.vague_cap;
  const int unit_l = opaque_s(__builtin_amdgcn_readfirstlane(unit));
  const int gw_l = opaque_s(__builtin_amdgcn_readfirstlane(gw));
  const bool head_ok = sub < G;
  float mx = -__builtin_inff();
  for_rounds<KMAX>(n_k, [&](auto kc) __attribute__((always_inline)) {
    constexpr int k = decltype(kc)::value;
    const int tok0 = (gw_l + k * NWT) * 64 + (lane & ~3);        // first token of the quad in this round
    const int n_ok = nv - tok0;                                   // tokens i < n_ok of the quad exist
    float* lg = a.logits + ((size_t)unit_l * tot_cap + a.ret_cap + tok0) * G + sub;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool valid = i < n_ok;
      s[k][i] = valid ? s[k][i] * d.scale : -__builtin_inff();
      mx = fmaxf(mx, s[k][i]);
      if (a.logits != nullptr && valid && head_ok) lg[i * G] = s[k][i];
    }
  });
  // Weights are formed against the wave's own maximum, which needs no barrier; the
  // workgroup's maximum is put together after the barrier that publishes the first
  // V chunk, and each wave's sums are rescaled by exp(own maximum - workgroup
  // maximum) when they are merged.  s_stat: [8 waves][G] maxima, [8 waves][G] sums.
  {
    // maximum over the lanes of this head: the quads of a 16-lane row, then the four rows
    float x = dpp_max<0x124>(mx);
    x = dpp_max<0x128>(x);
    x = fmaxf(x, __shfl_xor(x, 16));
    x = fmaxf(x, __shfl_xor(x, 32));
    if (lane < G) s_stat[wave * G + lane] = x;
    float lsum = 0.f;
    for_rounds<KMAX>(n_k, [&](auto kc) __attribute__((always_inline)) {
      constexpr int k = decltype(kc)::value;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float p = (s[k][i] == -__builtin_inff()) ? 0.f : __expf(s[k][i] - x);
        s[k][i] = p;                 // from here on s holds the weights
        lsum += p;
      }
    });
    lsum = row_sum<4>(lsum);
    lsum += __shfl_xor(lsum, 16);
    lsum += __shfl_xor(lsum, 32);
    if (lane < G) s_stat[ST_WAVES * G + wave * G + lane] = lsum;
  }
  const size_t part = (size_t)unit_l * a.n_slices + a.n_rslices + opaque_s(__builtin_amdgcn_readfirstlane(vs));

  // ---- weights into matrix-core operand form ----------------------------------
  // The A operand of the V phases is, per lane, the weights of head `sub` for the
  // quad's 4 tokens: what the lane holds already.  The sign g_0 of each token (bit 0
  // of its record, which lives in the lane that owns the token) is folded in, and the
  // weight's bf16 parts are packed as the A operands of a round.
  // Three rows: odd quads take the negative weights, and their sums are negated back when quads are added.  The matrix
  // instruction cuts the smaller addends off towards minus infinity where it aligns them; the same small loss at every
  // token would grow with the list (101580 tokens, error against float64 4.0e-7 of the result), in opposite senses it
  // cancels.
  constexpr int NP = weight_parts<R>();
  const uint32_t neg_quad = (R == 3) ? (uint32_t)(lane & 4) << 29 : 0u;
  uint32_t W[KMAX][2 * NP];                // (of the rounds there are)
  for_rounds<KMAX>(n_k, [&](auto kc) __attribute__((always_inline)) {
    constexpr int k = decltype(kc)::value;
    const uint32_t rx = info[k].x;
    const uint32_t sg[4] = {quad_bcast<0>(rx) << 31, quad_bcast<1>(rx) << 31, quad_bcast<2>(rx) << 31,
                            quad_bcast<3>(rx) << 31};
    float rest[4];
#pragma unroll
    for (int t = 0; t < 4; ++t)
      rest[t] = head_ok ? __uint_as_float(__float_as_uint(s[k][t]) ^ (sg[t] ^ neg_quad)) : 0.f;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      uint32_t part[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        part[t] = __float_as_uint(rest[t]) & 0xffff0000u;
        rest[t] -= __uint_as_float(part[t]);                // exact
      }
      W[k][2 * p] = pair_hi(part[0], part[1]);
      W[k][2 * p + 1] = pair_hi(part[2], part[3]);
    }
  });

  // ---- V phases: weighted values ------------------------------------------------
  float* s_fw = s_stat + 2 * ST_WAVES * G;          // [8 waves][G]: exp(wave maximum - workgroup maximum)
  const int prow = wave * 4 + (lane >> 4);
  static_assert(G * S16_CH <= ST_THREADS, "one output element per thread and chunk");
  for (int cc = 0; cc < S16_NCHUNK; ++cc) {
    stage_wait();
    lds_barrier();             // V chunk cc complete; partial sums of chunk cc - 1 visible
    if (cc == 0) {
      // every wave's maximum and sum are visible now (this wave's own maximum is read
      // back too: it would not survive in registers without being spilled)
      float mo[G], mw[G], so[G];
#pragma unroll
      for (int g = 0; g < G; ++g) {
        mo[g] = s_stat[(lane & 7) * G + g];                          // maximum of wave (lane mod 8)
        so[g] = s_stat[ST_WAVES * G + (lane & 7) * G + g];           // its sum
        mw[g] = s_stat[wave * G + g];
      }
#pragma unroll
      for (int g = 0; g < G; ++g) {
        float M = dpp_max<0x121>(mo[g]);
        M = dpp_max<0x122>(M);
        M = dpp_max<0x124>(M);                               // over 8 neighbouring lanes = all 8 waves
        if (lane == 0) s_fw[wave * G + g] = (mw[g] == -__builtin_inff()) ? 0.f : __expf(mw[g] - M);
        if (wave == 0) {
          float x = so[g] * ((mo[g] == -__builtin_inff()) ? 0.f : __expf(mo[g] - M));
          x = dpp_add<0x121>(x);
          x = dpp_add<0x122>(x);
          x = dpp_add<0x124>(x);                             // sum over the 8 waves
          if (lane == 0) {
            a.part_ml[(part * G + g) * 2] = M;
            a.part_ml[(part * G + g) * 2 + 1] = x;
          }
        }
      }
    } else if (tid < G * CH) {
      // chunk cc - 1's output element: the NROW rows of partial sums that the barrier just published
      const float* sp = s_part + ((cc - 1) & 1) * (S16_NROW * G * CH);
      float v = 0.f;
#pragma unroll
      for (int pr = 0; pr < S16_NROW; ++pr) v += sp[pr * G * CH + tid];
      a.part_o[part * G * D + (tid / CH) * D + (cc - 1) * CH + (tid % CH)] = v;
    }
    f32x4_t acc[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    v_pass<KMAX, R, MODE>(s_sk, info, n_k, W, sub * 8, turn, acc);
    lds_barrier();                         // every wave is done with this V chunk
    if (cc + 1 < S16_NCHUNK) stage_issue<S16_ROWB / 16, S16_ROWB>(svg, s_sk, n_pieces, cc + 1, tid);

    // Reduction over the workgroup's tokens.  Lane (quad, sub) holds, per head, the 4
    // channels of half piece `sub` summed over the tokens of its quad; the four quads of
    // a 16-lane row are added with two DPP rotations, and the NROW rows meet in LDS.
    {
      float* sp = s_part + (cc & 1) * (S16_NROW * G * CH);
      float o[G][4];
      // odd quads hold the negative sums (formed here anew: in a register through the V passes it would not fit)
      const uint32_t neg_back = (R == 3) ? (opaque(make_uint2((uint32_t)lane, 0u)).x & 4u) << 29 : 0u;
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const float f = s_fw[wave * G + g];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          float x = acc[c][g];
          if constexpr (R == 3) x = __uint_as_float(__float_as_uint(x) ^ neg_back);
          o[g][c] = row_sum<4>(x) * f;
        }
      }
      if ((lane & 15) < 4) {
#pragma unroll
        for (int g = 0; g < G; ++g)
          *reinterpret_cast<float4*>(sp + (prow * G + g) * CH + sub * 4) = make_float4(o[g][0], o[g][1], o[g][2], o[g][3]);
      }
    }
  }
  lds_barrier();
  if (tid < G * CH) {
    const float* sp = s_part + ((S16_NCHUNK - 1) & 1) * (S16_NROW * G * CH);
    float v = 0.f;
#pragma unroll
    for (int pr = 0; pr < S16_NROW; ++pr) v += sp[pr * G * CH + tid];
    a.part_o[part * G * D + (tid / CH) * D + (S16_NCHUNK - 1) * CH + (tid % CH)] = v;
  }
}

// The first n_ret_wgs workgroups walk slices of the retained slots, the others take parts of the Vague lists.
template <int G, int R, int MODE>
__global__ __launch_bounds__(ST_THREADS, 2) void attend_pair16_kernel(DevDesc d, AttendArgs a, int n_ret_wgs) {
  extern __shared__ __align__(16) unsigned char smem[];
  if ((int)blockIdx.x < n_ret_wgs) {
    ret_stream_role<G, 3, ST_WAVES>(d, ret_stream_of(a), blockIdx.x, n_ret_wgs, smem);
    return;
  }
  // XCD-aware mapping: workgroup ids are dealt round-robin to the 8 XCDs, so all
  // workgroups of a unit get ids that are equal modulo 8 (they share one L2).
  const int lin = blockIdx.x - n_ret_wgs;
  const int xcd = lin & 7, jj = lin >> 3;
  const int unit = (jj / a.n_vslices) * 8 + xcd;
  if (unit >= d.B * d.Hkv) return;
  vague16_part<G, R, MODE>(d, a, unit, jj % a.n_vslices, smem);
}

template <int G, int R, int MODE>
static hipError_t launch16(const DevDesc& d, const AttendArgs& a, const AttendPlan& plan, hipStream_t st) {
  auto kern = attend_pair16_kernel<G, R, MODE>;
  static std::once_flag once;
  static hipError_t attr_rc = hipSuccess;
  std::call_once(once, [&]() {
    attr_rc = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                  160 * 1024);
  });
  if (attr_rc != hipSuccess) return attr_rc;
  const int units = d.B * d.Hkv;
  const int units_pad = (units + 7) / 8 * 8;
  hipLaunchKernelGGL(kern, dim3(plan.n_ret_wgs + units_pad * plan.n_vslices), dim3(ST_THREADS), plan.pair_lds, st, d, a,
                     plan.n_ret_wgs);
  return hipGetLastError();
}

template <int G>
static hipError_t launch16_r(const DevDesc& d, const AttendArgs& a, const AttendPlan& plan, hipStream_t st) {
  if (d.r == 3) return launch16<G, 3, KVR_MEDIAN_MIDMEAN>(d, a, plan, st);      // one median, whatever the rule
  return d.median_mode == KVR_MEDIAN_LOWER ? launch16<G, 4, KVR_MEDIAN_LOWER>(d, a, plan, st)
                                           : launch16<G, 4, KVR_MEDIAN_MIDMEAN>(d, a, plan, st);
}

int staged16_lds(const DevDesc& d) {
  return chunk_bytes(d.r, d.w) + 2 * S16_NROW * d.G * S16_CH * 4 + stat_floats(d.G) * 4 + d.G * 256;
}

bool staged16_applies(const DevDesc& d) {
  if (staged64_applies(d)) return false;
  return (d.r == 3 || d.r == 4) && d.r * d.w <= 4096 && d.G <= 4 && d.sign_mask == 2 &&
         staged16_lds(d) <= STAGED_LDS_LIMIT;
}

hipError_t launch_attend_pair16(const DevDesc& d, const AttendArgs& a, const AttendPlan& plan,
                                        hipStream_t st) {
  if (!staged16_applies(d) || plan.n_vslices < 1 || plan.pair_lds < staged16_lds(d)) return hipErrorInvalidValue;    // 12-bit LDS row indices, LDS size
  switch (d.G) {
    case 1: return launch16_r<1>(d, a, plan, st);
    case 2: return launch16_r<2>(d, a, plan, st);
    case 4: return launch16_r<4>(d, a, plan, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace kvr
