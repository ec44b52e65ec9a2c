// Host launchers of the device kernels (argument checks happen in the C ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "device.hpp"

namespace tbias {

hipError_t launch_init_states(const ArenaView& A, int32_t B, int32_t K, const int32_t* model_ids,
                              int32_t* states, float* scores, hipStream_t st);
hipError_t launch_empty(int32_t grid, int32_t block, int32_t lds_bytes, hipStream_t st);
hipError_t launch_reset_stream(int32_t b, int32_t m, int32_t K, int32_t* model_ids,
                               int32_t* states, float* scores, hipStream_t st);

// Greedy: T steps for B streams. Requires V1 <= kMaxV1.
hipError_t launch_greedy(const ArenaView& A, const void* logits, int32_t dtype, int32_t T,
                         int32_t B, int64_t row_stride, const int32_t* model_ids, int32_t* states,
                         int32_t* out_tok, int32_t* out_state, float* out_score, hipStream_t st);

hipError_t launch_beam(const ArenaView& A, const void* logits, int32_t dtype, int32_t T, int32_t B,
                       int32_t K, int64_t row_stride, const int32_t* model_ids, int32_t* states,
                       float* scores, int32_t* out_tok, int32_t* out_parent, int32_t* out_state,
                       float* out_step, float* out_cum, hipStream_t st);

// Streaming beam (recombination and tree): launch_init_beam_stream starts the
// carry.
hipError_t launch_init_beam_stream(const ArenaView& A, int32_t B, int32_t K,
                                   const int32_t* model_ids, int32_t* states, float* scores,
                                   tb_hyp* hyps, int32_t* tree_len, hipStream_t st);
hipError_t launch_beam_stream(const ArenaView& A, const void* logits, int32_t dtype, int32_t T,
                              int32_t B, int32_t K, int64_t row_stride, const int32_t* model_ids,
                              int32_t* states, float* scores, tb_hyp* hyps, int32_t* tree,
                              int32_t tree_cap, int32_t* tree_len, int32_t recombine,
                              int32_t* out_tok, int32_t* out_parent, int32_t* out_state,
                              float* out_step, float* out_cum, hipStream_t st);

// Segmented greedy kernel (plus its boundary fix-up); hipErrorNotSupported
// when V+1 is too large for it.
hipError_t launch_greedy_seg(const ArenaView& A, const void* logits, int32_t dtype, int32_t T,
                             int32_t B, int64_t row_stride, const int32_t* model_ids,
                             int32_t* states, int32_t* out_tok, int32_t* out_state,
                             float* out_score, hipStream_t st);

// Calls of few steps over rows of more than 2048 values; hipErrorNotSupported
// for calls that row summaries and walk (greedy_list.hpp) serve better.
hipError_t launch_greedy_wide(const ArenaView& A, const void* logits, int32_t dtype, int32_t T,
                              int32_t B, int64_t row_stride, const int32_t* model_ids,
                              int32_t* states, int32_t* out_tok, int32_t* out_state,
                              float* out_score, hipStream_t st);

// Workgroups a launch may have: a dispatch holds at most 2^32 - 1 work-items.
constexpr int64_t most_groups(int32_t threads) { return 0xffffffffll / threads; }

// Byte ranges of a call's buffers.
struct Span {
  const void* p;
  int64_t bytes;
};
inline bool overlap(const Span& a, const Span& b) {
  const uintptr_t x = (uintptr_t)a.p, y = (uintptr_t)b.p;
  return x < y + (uint64_t)b.bytes && y < x + (uint64_t)a.bytes;
}
// Whether one of the first n_out spans (a call's outputs) shares memory with
// another span. The list kernels keep row summaries in the outputs, so such a
// call (a frame-synchronous one that lets out_state be states, or one buffer for
// two outputs that nobody reads) takes the reference kernel, which writes a
// step's outputs after it has read what the step needs.
template <int N>
inline bool outputs_shared(const Span (&s)[N], int n_out) {
  for (int i = 0; i < n_out; ++i)
    for (int j = i + 1; j < N; ++j)
      if (overlap(s[i], s[j])) return true;
  return false;
}

// Largest V+1 the step kernels accept: the compiler's limit (the reference
// kernels' per-class LDS table, 4 B and one bit per class, fits up to it).
constexpr int32_t kMaxV1 = 32768;

// Test hooks (tb_debug_select_kernels, tb_debug_set_spin_limit): kernel
// choices forced by tests, and the poll limit of the greedy hand-off wait
// (0 = the kernel's default). Plain process-wide values, read per call.
enum { kGreedyAuto = 0, kGreedyRef = 1 };
enum { kBeamAuto = 0, kBeamRef = 1, kBeamNoPipe = 2 };
int32_t debug_greedy_kernel();
int32_t debug_beam_kernel();
uint32_t debug_spin_limit();

}  // namespace tbias
