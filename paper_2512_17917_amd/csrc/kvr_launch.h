// Host-side launcher declarations: one per kernel family.  Each launcher
// receives already validated arguments and returns the hipError_t of its last
// launch.
#pragma once
#include <hip/hip_runtime.h>

#include <mutex>

#include "kvr_dev.h"

namespace kvr {

// Launch of the streaming kernel of kvr_attend_multi: parts of the Vague lists, slices of the retained slots and workgroups for them; at most `most` parts and
// slices of a unit.
struct StreamPlan {
  int vslice_tokens, n_vslices, rslice_tokens, n_rslices, n_ret_wgs, lds;
  bool own;             // the slots have a launch of their own before it
};

// How one kvr_attend_decode call is cut into workgroups.  Slices 0 .. n_rslices-1
// cover the retained slots, slices n_rslices .. n_slices-1 the Vague index list.
struct AttendPlan {
  bool staged;          // Vague tokens by the LDS-staged kernel (else by the generic kernel)
  bool mfma_retained;   // retained slots by the MFMA kernel (bf16) (else by the generic kernel)
  int n_slices;         // partial results per unit
  int n_rslices;        // of which: retained slices
  int rslice_tokens;    // tokens per retained slice
  int n_vslices;        // slices (generic) or workgroups (staged) per unit over the Vague list
  int vslice_tokens;    // generic kernel over the Vague list: tokens per slice
  int ch;               // staged: channels per LDS phase
  int lds_bytes;        // staged: dynamic LDS per workgroup
  bool streamed;        // Vague tokens by the streaming LDS-staged kernel of kvr_attend_multi with one query
                        // (8 query heads per kv head; vslice_tokens / n_vslices are its parts)
  bool pair;            // staged, and its launch takes the retained slots along (64- and 16-channel kernels)
  bool ret_own;         // pair: the slots have a launch of their own before it after all
  int n_ret_wgs;        // pair: workgroups for the retained slots (0: none, or ret_own)
  int pair_lds;         // and its dynamic LDS (a workgroup of either kind)
  StreamPlan stream;    // streamed
  size_t off_part_o, off_part_ml, off_logits, off_rec, off_tiles, total_bytes;
};
AttendPlan attend_plan(const DevDesc& d, int dtype, long long ret_cap, long long vague_cap);
// Dynamic LDS of the retained kernel's capped form next to the plan's staged kernel; 0 = a CU has no room for both.  (Used
// where the general kernel takes the list; the others have the slots in their own launch.)
int attend_side_lds(const DevDesc& d, const AttendPlan& p);

struct AttendArgs {
  const void* q;
  const void* k_ret;
  const void* v_ret;
  const int32_t* ret_pos;
  int ret_cap;
  const void* sk;
  const void* sv;
  const int32_t* vague_pos;
  const int32_t* n_vague;
  int vague_cap;
  float* out;
  float* scores;
  long long n_cap;
  // workspace carve-up
  float* part_o;     // [units, n_slices, G, D]
  float* part_ml;    // [units, n_slices, G, 2]
  float* logits;     // [units, ret_cap + vague_cap, G] (tiles: [units, ret_cap, G]) or nullptr when scores == nullptr
  void* scratch_rec; // streaming kernel: token records
  float* tiles;      // and the logits of its tokens, by tile, which the merge kernel reads there (null: no streaming kernel)
  int n_slices;      // partial results per unit (all kinds)
  int slice_tokens;  // generic / retained kernel: tokens per slice
  int tok_start;     // generic kernel: first token it handles
  int tok_limit;     // generic kernel: it handles tokens t < min(tok_limit, ret_cap + n_vague)
  int slice0;        // generic kernel: index of its first partial
  int n_rslices;     // staged kernel: index of its first partial
  int n_vslices;     // staged kernel: workgroups per unit
  int n_q;           // merge kernel: query tokens per sequence (1 for kvr_attend_decode); the partials'
                     // columns are then (query t, head g) = t * G + g and out is [B, n_q, Hq, D]
};

// Retained slots by the MFMA kernel (bf16): slices 0 .. n_rslices-1 of a.slice_tokens slots.
// max_wgs > 0 caps the launch width (the workgroups then walk the items with a grid stride).
// side_lds > 0: the form capped at 128 registers, for the launch that shares the CUs with a staged kernel (G <= 4), with
// that much dynamic LDS (attend_side_lds).
// Dynamic LDS of a workgroup: the sums of its four waves and, in the same place, the logits of as many tokens.
constexpr int retained_lds(int G, int tokens) {
  const int sums = 4 * D, logits = (tokens + 15) / 16 * 16;
  return G * 4 * (sums > logits ? sums : logits);          // <= 32 KB (1024 tokens, G = 8)
}
hipError_t launch_attend_retained(const DevDesc& d, const AttendArgs& a, int n_rslices, int max_wgs,
                                  int side_lds, hipStream_t st);

// kept rows of a prompt's cache into the small slot array
hipError_t launch_compact(const DevDesc& d, int dtype, const void* k_src, const void* v_src, const int32_t* src_pos,
                          int src_cap, const int32_t* evict_slot, const int32_t* n_evict, int evict_cap, void* k_ret,
                          void* v_ret, int32_t* ret_pos, int ret_cap, int max_keep, hipStream_t st);

struct EncodePlan {
  bool bulk;
  size_t off_bucket, off_order, off_start, total_bytes;
};
EncodePlan encode_plan(const DevDesc& d, long long cap);

hipError_t launch_reconstruct(const DevDesc& d, int dtype, const void* sk, const void* sv,
                              const int32_t* tok_pos, const int32_t* count, int cap,
                              void* k_out, void* v_out, hipStream_t st);

// What the caller of kvr_attend_decode lends to a call (all may be null): a second stream with a fork and a
// join event for running the retained-slot kernel next to the staged kernel, and two events that are
// recorded on `st` right before the call's first and right after its last kernel.
struct AttendSide {
  hipStream_t stream;
  hipEvent_t fork, join;
  hipEvent_t prof_start, prof_stop;
};
hipError_t launch_attend(const DevDesc& d, int dtype, const AttendArgs& a, const AttendPlan& plan,
                         hipStream_t st, const AttendSide& sd);

// tokens per slice when `tokens` tokens of each of `units` units are cut for about 1280 workgroups
int attend_slice_tokens(long long tokens, long long units);

// merge kernel alone: n_cols = partial columns per unit (G for one query, n_q * G for several)
hipError_t launch_attend_combine(const DevDesc& d, const AttendArgs& a, int n_cols, hipStream_t st);

// LDS-staged kernel of kvr_attend_multi over the Vague list (bf16, r = 3, values signed only, 3 w <= 1024)
bool multi_staged_applies(const DevDesc& d, long long vague_cap);
int multi_staged_part_tokens(long long vague_cap, long long units);
int multi_staged_lds(const DevDesc& d, int n_col);
StreamPlan plan_stream(const DevDesc& d, int n_col, long long units, int ret_cap, int vague_cap, int most);
// its scratch: a record (4 bytes) and n_col floats for every listed token, each unit's in whole fours of tokens
constexpr size_t multi_staged_scratch_tokens(long long units, long long vague_cap) {
  return (size_t)units * (size_t)((vague_cap + 3) / 4 * 4);
}
// a: the call's arguments, with the workspace's areas, slice counts and a.tiles (logits by tile) / a.scratch_rec (records)
hipError_t launch_attend_multi_staged(const DevDesc& d, const AttendArgs& a, const int32_t* n_ctx, int n_q,
                                      const StreamPlan& plan, hipStream_t st);
// kvr_attend_multi: workspace carve-up and launch (bf16, n_q * G in {1, 2, 4, 8, 16})
struct MultiPlan {
  int rslice_tokens, n_rslices, vslice_tokens, n_vslices, n_slices;
  bool staged;           // Vague list through the LDS-staged kernel (its launch: stream)
  StreamPlan stream;
  size_t off_khat, off_vhat, off_part_o, off_part_ml, off_logits, total_bytes;
};
MultiPlan attend_multi_plan(const DevDesc& d, int n_q, long long ret_cap, long long vague_cap);
hipError_t launch_attend_multi(const DevDesc& d, const AttendArgs& a, const int32_t* n_ctx, int n_q,
                               const MultiPlan& plan, void* ws, hipStream_t st);

// Staged kernel over the Vague list (bf16, values signed only, G <= 4, r in {3,4}).
hipError_t launch_attend_vague_staged(const DevDesc& d, const AttendArgs& a, const AttendPlan& plan,
                                      hipStream_t st);
// LDS per workgroup (bytes): the sketch chunk in whole kilobytes (a wave copies 1 KB at a time; it doubles as the reduction
// scratch [32 rows][G][channels] floats), wave statistics [2][32 rows][G] and q [G][16 pieces]
constexpr int STAGED_KMAX = 6;                    // wave-rounds (64 tokens) per wave
constexpr int STAGED_LDS_LIMIT = 160 * 1024;      // LDS per workgroup on gfx950
__host__ __device__ constexpr int staged_chunk_lds(int rows, int G, int channels) {
  const int chunk = (rows * channels * 2 + 1023) & ~1023, scratch = 32 * G * channels * 4;
  return chunk > scratch ? chunk : scratch;
}
__host__ __device__ constexpr int staged_stat_lds(int G) { return 2 * 32 * G * 4; }
constexpr int staged_lds(int rows, int G, int channels) {
  return staged_chunk_lds(rows, G, channels) + staged_stat_lds(G) + G * 256;
}
// Its specialisation for chunks of 16 channels (kvr_attend_staged16.hip): four rows, and three rows whose sketch is too
// wide for the 64-channel kernel.  Its launch takes the retained slots along, and a wave up to staged16_kmax rounds of 64 tokens,
// what 256 registers hold (every workgroup stages the unit's whole sketch, sixteen chunks of it, so few large workgroups are
// better than many small ones).
__host__ __device__ constexpr int staged16_kmax(int r) { return r == 3 ? 17 : 24; }
bool staged16_applies(const DevDesc& d);
int staged16_lds(const DevDesc& d);               // bytes of a workgroup
hipError_t launch_attend_pair16(const DevDesc& d, const AttendArgs& a, const AttendPlan& plan,
                                         hipStream_t st);
// Its specialisation for r = 3 and 64-channel chunks, whose launch also takes the retained slots; 10-bit row indices.
// Its chunk stays whole through the V phases, so the reduction scratch is a place of its own.
constexpr int staged64_lds(int w, int G) {
  return ((3 * w * 128 + 1023) & ~1023) + 32 * G * 64 * 4 + staged_stat_lds(G) + G * 256;
}
// Range: with four heads what LDS holds (less the last kilobyte: w <= 333), with fewer what ten bits hold (w <= 341).
inline bool staged64_applies(const DevDesc& d) {
  return d.r == 3 && d.G <= 4 && d.sign_mask == 2 && 3 * d.w <= (d.G == 4 ? 1000 : 1024);
}
static_assert(staged64_lds(1000 / 3, 4) <= STAGED_LDS_LIMIT && staged64_lds(1024 / 3, 2) <= STAGED_LDS_LIMIT, "LDS");
constexpr int STAGED64_KMAX = 25;                 // wave-rounds (64 tokens) per wave: what 256 registers hold
// LDS of a workgroup (8 or 16 waves) of such a launch that takes retained slots: the waves' statistics, then the logits of a
// slice (a tile of 16 tokens for every wave at a time) and in the same place their sums
constexpr int ret_stream_lds(int n_col, int waves, int tokens) {
  const int logits = (tokens + 16 * waves - 1) / (16 * waves) * (16 * waves), sums = waves * D;
  return 2 * waves * 16 * 4 + n_col * 4 * (logits > sums ? logits : sums);
}
// and the largest slice that fits, in tiles of 16 tokens
constexpr int ret_stream_most(int n_col, int waves) {
  return (STAGED_LDS_LIMIT - 2 * waves * 16 * 4) / (n_col * 4 * 16 * waves) * waves;
}
hipError_t launch_attend_pair64(const DevDesc& d, const AttendArgs& a, const AttendPlan& plan, hipStream_t st);

hipError_t launch_select(const DevDesc& d, const float* scores, long long n_cap, int32_t* ret_pos,
                         int ret_cap, const int32_t* n_ctx, int n_recent, int k_candidate,
                         int32_t* evict_slot, int32_t* evict_pos, int32_t* n_evict, int evict_cap,
                         int32_t* vague_pos, int32_t* n_vague, int vague_cap, hipStream_t st);

hipError_t launch_append(const DevDesc& d, int dtype, const void* k_new, const void* v_new,
                         const int32_t* n_ctx, void* k_ret, void* v_ret, int32_t* ret_pos, int ret_cap,
                         int32_t* out_slot, hipStream_t st);

// append -> select -> encode of every unit in one launch (ret_cap <= 32768, evict_cap <= 64)
hipError_t launch_step_update(const DevDesc& d, int dtype, const void* k_new, const void* v_new,
                              const int32_t* n_ctx, void* k_ret, void* v_ret, int32_t* ret_pos, int ret_cap,
                              const float* scores, long long n_cap, int n_recent, int k_candidate,
                              int32_t* evict_slot, int32_t* evict_pos, int32_t* n_evict, int evict_cap,
                              int32_t* vague_pos, int32_t* n_vague, int vague_cap, void* sk, void* sv,
                              hipStream_t st);

// swap loop of Algorithm 3: at most max_swaps exchanges between the Candidate and the Vague part per unit
hipError_t launch_swap_back(const DevDesc& d, int dtype, const float* scores, long long n_cap, void* k_ret,
                            void* v_ret, int32_t* ret_pos, int ret_cap, const int32_t* n_ctx, int n_recent,
                            float replace_rate, int max_swaps, void* sk, void* sv, int32_t* vague_pos,
                            const int32_t* n_vague, int vague_cap, int32_t* n_swapped, int32_t* swap_log,
                            hipStream_t st);

hipError_t launch_encode(const DevDesc& d, int dtype, const void* k_src, const void* v_src, int src_rows,
                         const int32_t* src_slot, const int32_t* tok_pos, const int32_t* count, int cap,
                         void* sk, void* sv, int32_t* out_bucket, uint8_t* out_sign,
                         void* ws, const EncodePlan& plan, hipStream_t st);

}  // namespace kvr
