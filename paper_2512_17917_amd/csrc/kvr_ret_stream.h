// The retained slots of a short list, taken along by the waves of the 64-channel staged kernel: a wave requests a 16-token tile
// (8 KB of K and V) before a K phase and takes it in at the end of that phase, under the copy of the next sketch chunk.  Two tiles a
// wave cost next to nothing there, and the retained kernel's launch (7 us for a few slots) is gone.
//
// q.k: as in kvr_attend_retained.hip, with the query of head h in the four columns 4 h .. 4 h + 3 of the B operand, so that
// lane (r16 = l / 16, col = l mod 16) receives the logits of tokens 4 r16 .. 4 r16 + 3 for head col / 4.  p.v goes to the
// matrix cores too, and V needs no transposition: a dword of a V row (channels 2 i, 2 i + 1 of one token) stands for two
// consecutive entries of the contraction index, and row m = 4 h + 2 e + s of A has the weight of head h in the entries
// of channel 2 i + e and zero in the others.  s = 0, 1 are the first two of the weight's three bf16 parts (24 bits, all
// of it); the third goes through a second instruction.  Lane (r16, col) ends up with head r16, channels 8 col .. + 7.
#pragma once
#include "kvr_staged.h"

namespace kvr {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

template <int G>
struct RetStream {
  // what the wave walks over; uniform
  const bf16_t* kret;
  const bf16_t* vret;
  const int32_t* rp;        // null: every slot holds its own number
  int ret_cap;
  int t0, step;             // first token of the tile that is in flight (>= ret_cap: none), distance to the next
  // the tile
  u32x4_t ka[4];            // K: token t0 + col, channels 32 kk + 8 r16 .. + 7
  u32x4_t vv[4];            // V: token t0 + 4 r16 + j, channels 8 col .. + 7
  int pos;                  // position of token t0 + col, -1: empty slot or past the end
  // state
  f32x4_t acc[4];           // [dword of the piece][2 e + s], head r16
  float m_run, l_run;       // maximum (equal in all lanes of a head), sum over this lane's tokens: head col / 4

  __device__ __forceinline__ void init(const AttendArgs& a, int unit, int first_tile, int tile_step) {
    kret = (const bf16_t*)a.k_ret + (size_t)unit * a.ret_cap * D;
    vret = (const bf16_t*)a.v_ret + (size_t)unit * a.ret_cap * D;
    rp = a.ret_pos ? a.ret_pos + (size_t)unit * a.ret_cap : nullptr;
    ret_cap = a.ret_cap;
    t0 = first_tile * 16;
    step = tile_step * 16;
    m_run = -__builtin_inff();
    l_run = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  }

  // request the tile at t0 (read once: non-temporal, so that it does not push the sketch out of L2)
  __device__ __forceinline__ void issue(int lane) {
    if (t0 >= ret_cap) return;
    asm volatile("" : "+v"(lane));        // what depends on the lane is formed here, not kept through all phases
    const int r16 = lane >> 4, col = lane & 15;
    const int last = ret_cap - 1 - t0;                  // >= 0
    const int tk = min(col, last);
    pos = rp ? rp[t0 + tk] : t0 + tk;
    if (col > last) pos = -1;
    const bf16_t* kb = kret + (size_t)t0 * D;
    const bf16_t* vb = vret + (size_t)t0 * D;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
      ka[kk] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(kb + tk * D + 32 * kk + 8 * r16));
#pragma unroll
    for (int j = 0; j < 4; ++j)
      vv[j] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(vb + min(4 * r16 + j, last) * D + 8 * col));
  }

  // take in the tile that is in flight and move on to the next one (not yet requested).  s_q: q in LDS,
  // [G][16 pieces]; logits_unit: where the unit's retained logits go, may be null
  __device__ __forceinline__ void consume(int lane, const uint4* s_q, float scale, float* logits_unit) {
    if (t0 >= ret_cap) return;
    asm volatile("" : "+v"(lane));
    const float NEG_INF = -__builtin_inff();
    const int r16 = lane >> 4, col = lane & 15, head = col >> 2, x = col & 3;
    const uint4* qp = s_q + min(head, G - 1) * 16 + r16;
    f32x4_t S = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
      S = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, ka[kk]),
                                                  __builtin_bit_cast(bf16x8_t, qp[4 * kk]), S, 0, 0, 0);
    const uint32_t live16 = (uint32_t)__ballot(pos >= 0) & 0xffffu;       // bit t: token t0 + t
    const uint32_t live = (head < G) ? (live16 >> (4 * r16)) : 0u;        // bit i: token t0 + 4 r16 + i
    float s[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) s[i] = ((live >> i) & 1u) ? S[i] * scale : NEG_INF;
    if (logits_unit != nullptr) {
      // the four columns of a head hold the same four logits: column x stores token 4 r16 + x, 256 bytes a wave with four heads
      const float y = (x & 2) ? ((x & 1) ? s[3] : s[2]) : ((x & 1) ? s[1] : s[0]);
      const int t = t0 + 4 * r16 + x;
      if (head < G && t < ret_cap) logits_unit[(size_t)t * G + head] = y;
    }
    float mx = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
    mx = rows_max(mx);
    const float m_new = fmaxf(m_run, mx);
    if (__any(m_new > m_run)) {
      const float corr = (m_run == NEG_INF) ? 0.f : __expf(m_run - m_new);
      l_run *= corr;
      const float ch = __shfl(corr, (lane & 48) + 4 * r16);               // of head r16
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[j][i] *= ch;
    }
    m_run = m_new;
    if (live16 != 0xffffu) {          // an empty slot may hold anything, even NaN: weight 0 is not enough
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (!((live16 >> (4 * r16 + j)) & 1u)) vv[j] = u32x4_t{0u, 0u, 0u, 0u};
    }
    const uint32_t down = (col & 2) ? 0u : 16u;          // e: which half of the dword this row's weight belongs to
    u32x4_t a1, a2;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float p = (s[i] == NEG_INF) ? 0.f : __expf(s[i] - m_new);
      l_run += p;
      const uint32_t hi = __float_as_uint(p) & 0xffff0000u;
      const float r1 = p - __uint_as_float(hi);
      const uint32_t mid = __float_as_uint(r1) & 0xffff0000u;
      const uint32_t lo = __float_as_uint(r1 - __uint_as_float(mid));     // eight bits left: the low half is zero
      a1[i] = ((col & 1) ? mid : hi) >> down;
      a2[i] = ((col & 1) ? 0u : lo) >> down;
    }
    const bf16x8_t w1 = __builtin_bit_cast(bf16x8_t, a1), w2 = __builtin_bit_cast(bf16x8_t, a2);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const u32x4_t bj = {vv[0][j], vv[1][j], vv[2][j], vv[3][j]};
      const bf16x8_t b = __builtin_bit_cast(bf16x8_t, bj);
      acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1, b, acc[j], 0, 0, 0);
      acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w2, b, acc[j], 0, 0, 0);
    }
    t0 += step;
  }

  // sum of the weights of head col / 4 over the wave's tokens, in every lane of the head
  __device__ __forceinline__ float sum() const { return rows_sum(l_run); }

  // the wave's sums, head r16 (zero for r16 >= G), channels 8 col .. + 7
  __device__ __forceinline__ void result(int lane, int first_t0, const uint4* s_q, float scale, float (&o)[8]) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      o[2 * j] = acc[j][0] + acc[j][1];
      o[2 * j + 1] = acc[j][2] + acc[j][3];
    }
    bool nan = false;
#pragma unroll
    for (int c = 0; c < 8; ++c) nan = nan || o[c] != o[c];
    if (!__any(nan)) return;
    // Something is not finite.  The zeros in A times an infinite value would put NaN where there is none, so the
    // wave's tokens are summed once more, one multiply-add each.
    const int r16 = lane >> 4, col = lane & 15, h = min(r16, G - 1);
    const float m = __shfl(m_run, 4 * h);
#pragma unroll
    for (int c = 0; c < 8; ++c) o[c] = 0.f;
    for (int tb = first_t0; tb < ret_cap; tb += step) {
      for (int t = tb; t < min(tb + 16, ret_cap); ++t) {
        if (rp && rp[t] < 0) continue;
        float kf[8], qf[8], vf[8];
        Store<bf16_t>::load16(kret + (size_t)t * D + 8 * col, kf);
        Store<bf16_t>::load16(reinterpret_cast<const bf16_t*>(s_q) + h * D + 8 * col, qf);
        Store<bf16_t>::load16(vret + (size_t)t * D + 8 * col, vf);
        float y = 0.f;
#pragma unroll
        for (int c = 0; c < 8; ++c) y = fmaf(qf[c], kf[c], y);
#pragma unroll
        for (int off = 1; off < 16; off <<= 1) y += __shfl_xor(y, off);
        y *= scale;
        const float p = (y == -__builtin_inff()) ? 0.f : __expf(y - m);
#pragma unroll
        for (int c = 0; c < 8; ++c) o[c] = fmaf(p, vf[c], o[c]);
      }
    }
  }
};

}  // namespace kvr
