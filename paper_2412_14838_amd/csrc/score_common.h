// Device helpers shared by the matrix-core scoring kernels.
#pragma once
#include "dkv_internal.h"

namespace dkv {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr float kLog2e = 1.4426950408889634f;
constexpr int kMaxHalo = 64;          // >= 2 * half

__device__ inline float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Workgroup barrier that orders LDS traffic only. __syncthreads() also waits for every global load the wavefront
// has in flight (its release fence covers global memory), which would cut the prefetch of the key tiles down to
// what fits between two barriers; the wavefronts of a score kernel talk to each other through LDS alone.
__device__ inline void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// ---- Merging of partial row statistics (max, sum of exp2), log2 domain
__device__ inline void merge_pair(float& M, float& Lsum, const float2 v) {
  const float Mn = fmaxf(M, v.x);
  const float Mu = Mn == -INFINITY ? 0.0f : Mn;
  Lsum = fmaf(Lsum, fast_exp2(M - Mu), v.y * fast_exp2(v.x - Mu));   // spelled out: every call site rounds alike
  M = Mn;
}

// The caller's row normalisers of a multi-layer call (natural log, [n_seqs][Hq][w] per layer) into the layout and the
// log2 domain the emit kernels read: lse_rows [layer][seq][head][rows_pad].
void launch_import_lse(const Params& p, int n_layers, const float* const* lse_layers, float* lse_rows, hipStream_t st);

}  // namespace dkv
