// Boosted greedy step for calls of few steps over wide rows (V+1 > 2048): one
// workgroup of 256 threads per stream reads each row once and scores every
// token from the current state, step after step.
//
// Row summaries and walk (greedy_list.hpp) are two launches, and the walk starts
// with a chain of dependent loads, so they take some 14 us before the first
// step's answer; scoring every token takes 3 to 8 us a step, so it is the faster
// way for the first few. most_steps() holds the line, which follows from both
// sides' times.
//
// Thread i holds tokens v = i + 256 j (j < TPV) and keeps, in registers, their
// logits (the next row's already in flight), their classes, and their root move
// (target state and its psi). A step from state s:
//
//  1. the children of the states on s's suffix chain (s, link(s), ..., the
//     root excluded) override the root move of their class, the deepest state
//     first: a per-class tag table in LDS points the overridden classes at a
//     short list of (target state, psi) built level by level;
//  2. every thread forms key[v] = z[v] + psi[delta(s, class v)] for its tokens
//     (blank: z[V] + phi[s], which keeps the state), its best (key, index)
//     and its part of the log-sum-exp (its own max and sum of exponentials);
//  3. one workgroup reduction gives the lowest-index maximum, the state it
//     moves to, and lse.
#include <climits>

#include "device.hpp"
#include "launch.hpp"

namespace tbias {
namespace wide {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
constexpr float kNegInf = -__builtin_huge_valf();

// Read-only load through the scalar cache (uniform address).
template <class T>
__device__ __forceinline__ T sld(const T* p) {
  return *(const __attribute__((address_space(4))) T*)(p);
}

// The row length passes through an empty asm each time it is used, so that
// the compiler keeps the per-slot bounds tests where they are used instead of
// hoisting 2*TPV lane masks out of the row loop (they would not fit in SGPRs).
__device__ __forceinline__ int32_t opaque(int32_t x) {
  asm volatile("" : "+s"(x));
  return x;
}

// The workgroup's view of one stream's model: arena and the LDS tag table.
struct Ctx {
  const ArenaView* A;
  int32_t off;       // first global state of the model
  int mode;          // 1 biased, 0 model -1, -1 invalid model or state
  int32_t fixed;     // state written for unbiased streams
  int32_t cap;       // override list capacity
  uint32_t* omark;   // [V]: tag << 16 | list slot of an overridden class
  int32_t* olist_y;  // [cap] target state of an override
  float* olist_psi;  // [cap] its psi
  int32_t* nlist;    // list fill counter (LDS)
  const float* gpsi; // the model's root moves
  const int32_t* gdst;
  uint32_t tag;
};

// Bytes of dynamic LDS a workgroup needs: the tag table and the override list.
__host__ __device__ inline size_t lds_bytes(const ArenaView& A) {
  const int32_t cap = A.max_override > 0 ? A.max_override : 1;
  return 4 * (size_t)(A.V1 - 1) + 8 * (size_t)cap;
}

// Per-thread registers of its tokens v = tid + kThreads * j. The blank and the
// positions past the row have root psi -inf, so they never win as tokens; the
// blank is scored on its own (zb, held by the thread that owns it).
template <int TPV>
struct Own {
  float z[TPV];
  float zb;          // the blank's logit (thread V mod kThreads only)
  int32_t cls[TPV];  // class of v (-1: none, blank or past the row)
  float rps[TPV];    // psi of v's root move (0 when unbiased; -inf: blank, past the row)
  int32_t rds[TPV];  // target of v's root move (the fixed state when unbiased)
};

template <class Ld, int TPV>
__device__ __forceinline__ void load_row(float (&z)[TPV], float& zb, const typename Ld::T* row,
                                         int32_t V1x) {
  const int32_t V1 = opaque(V1x);
  const int32_t V = V1 - 1;
#pragma unroll
  for (int j = 0; j < TPV; ++j) {
    const int32_t v = (int32_t)threadIdx.x + kThreads * j;
    z[j] = (v < V1) ? Ld::get(row, v) : kNegInf;
  }
  zb = ((int32_t)threadIdx.x == V % kThreads) ? Ld::get(row, V) : kNegInf;
}

template <int TPV>
__device__ __forceinline__ void own_tables(Own<TPV>& o, const Ctx& C) {
  const int32_t V = C.A->V1 - 1;
#pragma unroll
  for (int j = 0; j < TPV; ++j) {
    const int32_t v = (int32_t)threadIdx.x + kThreads * j;
    const bool tok = v < V;
    o.cls[j] = tok ? C.A->class_map[v] : -1;
    o.rps[j] = tok ? (C.mode == 1 ? C.gpsi[v] : 0.f) : kNegInf;
    o.rds[j] = (C.mode == 1) ? (tok ? C.gdst[v] : 0) : C.fixed;
  }
}

// The classes overridden in state s: the children of the states on s's
// suffix chain (s, link(s), ..., the root excluded), the deepest state first,
// go to the tag table and the override list, level by level. Returns whether
// any chain was walked (s != 0 for a biased stream); phi_s gets phi[s].
// Contains workgroup barriers (uniform s): all threads must call it.
__device__ __forceinline__ bool build_overrides(Ctx& C, int32_t s, float& phi_s) {
  const ArenaView& A = *C.A;
  const int tid = threadIdx.x;
  phi_s = 0.f;
  if (C.mode != 1) return false;
  phi_s = sld(A.phi + C.off + s);
  if (s == 0) return false;
  ++C.tag;  // a call has far fewer steps than tags
  if (tid == 0) *C.nlist = 0;
  __syncthreads();
  for (int32_t x = s; x != 0;) {
    const int32_t fc = sld(A.first_child + C.off + x);
    const int32_t nc = sld(A.n_child + C.off + x);
    const int32_t lk = sld(A.link + C.off + x);
    for (int32_t j = tid; j < nc; j += kThreads) {
      const int32_t y = fc + j;
      const int32_t c = A.label[C.off + y];
      // a class already listed by a deeper chain state keeps that move
      if ((C.omark[c] >> 16) != C.tag) {
        const int32_t slot = atomicAdd(C.nlist, 1);
        if (slot < C.cap) {
          C.olist_y[slot] = y;
          C.olist_psi[slot] = A.psi[C.off + y];
          C.omark[c] = (C.tag << 16) | (uint32_t)slot;
        }
      }
    }
    __syncthreads();
    x = lk;
  }
  return true;
}

// Calls visit(j, p, ns) for every token slot j of this thread with the psi p
// of its move and the state ns it moves to: the override when its class is in
// the table (chain), else its root move. Tag reads of 8 tokens are issued
// together, then their list entries (slot 0 when not overridden).
template <int TPV, class F>
__device__ __forceinline__ void for_each_move(const Ctx& C, const Own<TPV>& o, bool chain,
                                              F&& visit) {
  if (chain) {
    constexpr int kG = 8;
#pragma unroll
    for (int g0 = 0; g0 < TPV; g0 += kG) {
      uint32_t e[kG];
#pragma unroll
      for (int i = 0; i < kG; ++i)
        if (g0 + i < TPV) e[i] = C.omark[o.cls[g0 + i] > 0 ? o.cls[g0 + i] : 0];
      float po[kG];
      int32_t yo[kG];
#pragma unroll
      for (int i = 0; i < kG; ++i) {
        if (g0 + i < TPV) {
          const bool ov = o.cls[g0 + i] >= 0 && (e[i] >> 16) == C.tag;
          const int32_t slot = ov ? (int32_t)(e[i] & 0xffffu) : 0;
          po[i] = C.olist_psi[slot];
          yo[i] = C.olist_y[slot];
          e[i] = ov ? 1u : 0u;
        }
      }
#pragma unroll
      for (int i = 0; i < kG; ++i) {
        if (g0 + i < TPV) {
          const int j = g0 + i;
          visit(j, e[i] ? po[i] : o.rps[j], e[i] ? yo[i] : o.rds[j]);
        }
      }
    }
  } else {
#pragma unroll
    for (int j = 0; j < TPV; ++j) visit(j, o.rps[j], o.rds[j]);
  }
}

struct Red {
  float k, z, psi, m, s;
  int32_t v, ns;
};

// (key, index) argmax carrying the target state, psi and logit of the winner,
// together with a log-sum-exp (max m, sum s of exp(z - m)) merge.
__device__ __forceinline__ void merge(Red& a, const Red& b) {
  if (better(b.k, b.v, a.k, a.v)) {
    a.k = b.k;
    a.v = b.v;
    a.ns = b.ns;
    a.psi = b.psi;
    a.z = b.z;
  }
  const float M = fmaxf(a.m, b.m);
  const float sa = (a.m == M) ? a.s : a.s * __expf(a.m - M);
  const float sb = (b.m == M) ? b.s : b.s * __expf(b.m - M);
  a.m = M;
  a.s = sa + sb;
}

// One step from state s on the row in o.z; returns the winner and lse in
// every thread. Contains workgroup barriers: all threads must call it.
template <class Ld, int TPV>
__device__ __forceinline__ Red step(Ctx& C, const Own<TPV>& o, const typename Ld::T* row, int32_t s,
                                    int32_t V1, Red* red) {
  const int32_t V = V1 - 1;
  const int tid = threadIdx.x;
  float phi_s;
  const bool chain = build_overrides(C, s, phi_s);

  float bk = kNegInf, bpsi = 0.f, bz = 0.f;
  int32_t bv = INT_MAX, bns = 0;
  float m = kNegInf;
#pragma unroll
  for (int j = 0; j < TPV; ++j) m = fmaxf(m, o.z[j]);
  float se = 0.f;  // the blank's logit is also in its slot of o.z: counted once there
#pragma unroll
  for (int j = 0; j < TPV; ++j) se += (o.z[j] == kNegInf) ? 0.f : __expf(o.z[j] - m);
  for_each_move<TPV>(C, o, chain, [&](int j, float p, int32_t ns) {
    const float key = o.z[j] + p;
    const bool gt = key > bk;  // tokens ascend: strict > keeps the lowest index on ties
    bk = gt ? key : bk;
    bv = gt ? tid + kThreads * j : bv;
    bns = gt ? ns : bns;
    bpsi = gt ? p : bpsi;
    bz = gt ? o.z[j] : bz;
  });
  if (tid == V % kThreads) {  // the blank keeps the state; phi[s] in its key, no boost
    const float key = o.zb + phi_s;
    if (better(key, V, bk, bv)) {
      bk = key;
      bv = V;
      bns = (C.mode == 1) ? s : C.fixed;
      bpsi = phi_s;
      bz = o.zb;
    }
  }
  // wave reductions (DPP): the winner's fields from its lane, and the
  // log-sum-exp as the wave max of the thread maxima and the rescaled sums
  Red r;
  const int32_t wl = wave_argmax_dpp(bk, bv, r.k, r.v);
  r.ns = __builtin_amdgcn_readlane(bns, wl);
  r.psi = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(bpsi), wl));
  r.z = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(bz), wl));
  r.m = wave_max_dpp(m);
  r.s = wave_sum_dpp((m == r.m) ? se : se * __expf(m - r.m));
  if ((tid & 63) == 0) red[tid >> 6] = r;
  __syncthreads();
  Red f = red[0];
#pragma unroll
  for (int w = 1; w < kWaves; ++w) merge(f, red[w]);
  __syncthreads();  // red is rewritten by the next step
  if (__builtin_amdgcn_readfirstlane((int32_t)(f.k == kNegInf))) {
    // no key is above -inf: the lowest that is no nan (the first token when all
    // are), at its own move
    int32_t v0 = INT_MAX;
    for (int32_t v = tid; v < V1 && v0 == INT_MAX; v += kThreads) {
      const float z = Ld::get(row, v);
      if (z == z) v0 = v;
    }
    v0 = wave_min_i32_dpp(v0);
    if ((tid & 63) == 0) red[tid >> 6].v = v0;
    __syncthreads();
    v0 = red[0].v;
#pragma unroll
    for (int w = 1; w < kWaves; ++w) v0 = min(v0, red[w].v);
    __syncthreads();
    f.v = v0 < V1 ? v0 : 0;
    f.z = Ld::get(row, f.v);
    f.psi = phi_s;
    f.ns = (C.mode == 1) ? s : C.fixed;
    if (f.v < V && C.mode == 1) {
      const int32_t c = C.A->class_map[f.v];
      const bool ov = chain && c >= 0 && (C.omark[c] >> 16) == C.tag;
      const int32_t slot = ov ? (int32_t)(C.omark[c] & 0xffffu) : 0;
      f.ns = ov ? C.olist_y[slot] : C.gdst[f.v];
      f.psi = ov ? C.olist_psi[slot] : C.gpsi[f.v];
    }
  }
  f.psi -= phi_s;  // the boost: psi[next] - phi[s] (0 for the blank)
  return f;
}

struct Shared {
  Red red[kWaves];
  int32_t nlist;
};

template <class Ld, int TPV>
__global__ __launch_bounds__(kThreads) void greedy_wide_kernel(
    ArenaView A, const typename Ld::T* __restrict__ logits, int32_t T, int32_t B, int64_t stride,
    const int32_t* __restrict__ model_ids, int32_t* __restrict__ states,
    int32_t* __restrict__ out_tok, int32_t* __restrict__ out_state,
    float* __restrict__ out_score) {
  extern __shared__ __align__(16) unsigned char dyn[];
  __shared__ Shared sh;
  lds_poison(&sh, sizeof(sh));
  lds_poison(dyn, wide::lds_bytes(A));
  const int32_t V1 = A.V1, V = V1 - 1;
  const int32_t b = blockIdx.x;
  const typename Ld::T* col = logits + (int64_t)b * stride;
  const int64_t tstride = (int64_t)B * stride;
  const int32_t m = model_ids[b];
  const int32_t s0 = states[b];
  int32_t off = 0, n = 0;
  const int mode = resolve_stream(A, m, s0, off, n);

  Own<TPV> o;
  float zn[TPV], zbn = kNegInf;
  load_row<Ld, TPV>(o.z, o.zb, col, V1);
  Ctx C;
  C.A = &A;
  C.off = off;
  C.mode = mode;
  C.fixed = unbiased_state(mode, s0 == TB_STATE_TIMEOUT);
  C.cap = A.max_override > 0 ? A.max_override : 1;
  C.omark = reinterpret_cast<uint32_t*>(dyn);
  C.olist_y = reinterpret_cast<int32_t*>(dyn + 4 * (size_t)V);
  C.olist_psi = reinterpret_cast<float*>(dyn + 4 * (size_t)V + 4 * (size_t)C.cap);
  C.nlist = &sh.nlist;
  C.gpsi = A.root_psi + (int64_t)(mode == 1 ? m : 0) * V1;
  C.gdst = A.root_dst + (int64_t)(mode == 1 ? m : 0) * V1;
  C.tag = 0u;
  for (int32_t c = threadIdx.x; c < V; c += kThreads) C.omark[c] = 0u;
  own_tables<TPV>(o, C);
  __syncthreads();

  int32_t s = (mode == 1) ? s0 : C.fixed;
  for (int32_t t = 0; t < T; ++t) {
    const typename Ld::T* row = col + (int64_t)t * tstride;
    if (t + 1 < T) load_row<Ld, TPV>(zn, zbn, row + tstride, V1);
    const Red f = step<Ld, TPV>(C, o, row, s, V1, sh.red);
    if (threadIdx.x == 0) {
      const int64_t oi = (int64_t)t * B + b;
      out_tok[oi] = f.v;
      out_state[oi] = f.ns;
      out_score[oi] = (f.z - (f.m + __logf(f.s))) + f.psi;
    }
    s = f.ns;
    if (t + 1 < T) {
#pragma unroll
      for (int j = 0; j < TPV; ++j) o.z[j] = zn[j];
      o.zb = zbn;
    }
  }
  if (threadIdx.x == 0) states[b] = s;
}

// The most steps of a call this kernel is the faster one for, 0 for none. Times
// of one call in a row of calls, each with rows of its own and 1000 phrases a
// list, this kernel / row summaries and walk, in us:
//
//   float32    V   1 stream               128 streams            256 streams
//            3000  4: 16 / 17  6: 22 / 20  4: 22 / 24  6: 31 / 29  6: 31 / 31  8: 38 / 37
//            4096  2: 13 / 13  4: 22 / 17  3: 22 / 22  4: 28 / 25  4: 28 / 29  6: 39 / 34
//            6000  2: 13 / 14  3: 18 / 16  3: 22 / 23  5: 33 / 31  4: 30 / 31  6: 42 / 41
//            8192  1: 10 / 11  2: 15 / 13  2: 19 / 20  4: 33 / 28  3: 27 / 28  4: 36 / 35
//           10400  1: 13 / 12              1: 16 / 15              1: 16 / 18
//   bfloat16 (2-byte loads)
//            3000  3: 16 / 17  4: 20 / 18  3: 19 / 22  4: 26 / 25  3: 24 / 25  4: 32 / 26
//            6000  1: 10 / 12  2: 17 / 15  1: 16 / 17  2: 27 / 22  1: 16 / 20  2: 27 / 24
//            8192  1: 13 / 11              1: 19 / 17              1: 20 / 16
inline int32_t most_steps(int32_t V1, int32_t B, int32_t dtype) {
  if (dtype != TB_F32) return V1 <= 12 * kThreads ? 3 : (V1 <= 24 * kThreads ? 1 : 0);
  const int32_t base = V1 <= 12 * kThreads ? 4
                       : V1 <= 24 * kThreads ? 2
                       : V1 <= 33 * kThreads ? 1
                       : V1 <= 41 * kThreads ? -1 : -2;
  return base + (B >= 256 ? 2 : (B >= 128 ? 1 : 0));
}

template <class Ld, int TPV>
hipError_t launch_t(const ArenaView& A, const void* logits, int32_t T, int32_t B, int64_t stride,
                    const int32_t* model_ids, int32_t* states, int32_t* out_tok,
                    int32_t* out_state, float* out_score, hipStream_t st) {
  hipLaunchKernelGGL((greedy_wide_kernel<Ld, TPV>), dim3(B), dim3(kThreads), lds_bytes(A), st, A,
                     static_cast<const typename Ld::T*>(logits), T, B, stride, model_ids, states,
                     out_tok, out_state, out_score);
  return hipGetLastError();
}

}  // namespace wide

// hipErrorNotSupported for calls that row summaries and walk serve better, or
// whose tables do not fit LDS.
hipError_t launch_greedy_wide(const ArenaView& A, const void* logits, int32_t dtype, int32_t T,
                              int32_t B, int64_t row_stride, const int32_t* model_ids,
                              int32_t* states, int32_t* out_tok, int32_t* out_state,
                              float* out_score, hipStream_t st) {
  if (T > wide::most_steps(A.V1, B, dtype) || wide::lds_bytes(A) > 60 * 1024 ||
      B > most_groups(wide::kThreads))
    return hipErrorNotSupported;
  const int tpv = (A.V1 + wide::kThreads - 1) / wide::kThreads;
#define TB_WIDE(L, N)                                                                       \
  if (tpv <= N)                                                                             \
    return wide::launch_t<L, N>(A, logits, T, B, row_stride, model_ids, states, out_tok,    \
                                out_state, out_score, st);
  if (dtype == TB_F32) {
    TB_WIDE(LoadF32, 12)
    TB_WIDE(LoadF32, 16)
    TB_WIDE(LoadF32, 24)
    TB_WIDE(LoadF32, 33)
    TB_WIDE(LoadF32, 41)
  } else {
    TB_WIDE(LoadBF16, 12)
    TB_WIDE(LoadBF16, 16)
    TB_WIDE(LoadBF16, 24)
  }
#undef TB_WIDE
  return hipErrorNotSupported;
}

}  // namespace tbias
