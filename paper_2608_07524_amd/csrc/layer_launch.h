// Host-side launch interface of the layer kernels (layer.hip, layer_gemm.hip, layer_proj.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dcp {

// y = x * rstd * g per row (bf16 [rows, h], h a multiple of 8); rstd fp32 [rows].
hipError_t launch_rmsnorm_fwd(const void* x, const void* g, void* y, float* rstd, int64_t rows, int h, float eps,
                              hipStream_t s);
// dx = res + RMSNorm backward of dy (fp32 [rows, h]); dg (fp32 [h]) += the
// gain gradient, reduced through `partial` (fp32 [rmsnorm_bwd_blocks(rows), h]).
hipError_t launch_rmsnorm_bwd(const float* dy, const void* x, const void* g, const float* rstd, const void* res,
                              void* dx, float* partial, float* dg, int64_t rows, int h, hipStream_t s);
int64_t rmsnorm_bwd_blocks(int64_t rows);
// Weight gradients c[m, n] (fp32) += a^T b over the batch's tokens, a [tokens,
// m] and b [tokens, n] bf16 row-major (m, n multiples of 8); scratch holds
// partial sums (256-byte aligned).
constexpr int kWgradMax = 6;  // a layer's weight matrices
struct WgradProblem {
  const void* a;
  const void* b;
  float* c;
  int m, n;
  int tile0;  // (set by the launch)
};
struct WgradBatch {
  WgradProblem p[kWgradMax];
  int64_t tokens;
  int n_tiles, splits;  // (set by the launch)
};
hipError_t launch_wgrad(WgradBatch b, void* scratch, size_t scratch_bytes, hipStream_t s);

// Projections C[tokens, n] = sum_s a[s] w[s] (w [k, n]) or a[s] w[s]^T (w [n,
// k]); a [tokens, k] and w bf16 row-major, n and k multiples of 8.  outs == 1:
// one sum over `pairs` operand pairs; outs > 1: pair s gives out[s] (pairs == 1).
enum class ProjEpilogue {
  kStore,     // a w, bf16
  kResidual,  // a w + aux, bf16
  kGelu,      // a w, bf16, and GELU of it to out2
  kGeluGrad,  // a w^T times GELU'(aux), bf16
  kStoreT,    // a w^T, bf16
  kSumF32,    // sum of a w^T, fp32
};
constexpr int kProjMax = 3;
struct Proj {
  const void* a[kProjMax];
  const void* w[kProjMax];
  void* out[kProjMax];
  const void* aux;  // bf16 [tokens, n]
  void* out2;
  int64_t tokens;
  int n, k, pairs, outs;
  int n_tiles;  // (set by the launch)
};
hipError_t launch_proj(const Proj& p, ProjEpilogue epi, hipStream_t s);

// a = GELU(u) and du = da * GELU'(u), n elements (a multiple of 8), bf16.
hipError_t launch_gelu_fwd(const void* u, void* a, int64_t n, hipStream_t s);
hipError_t launch_gelu_bwd(const void* u, const void* da, void* du, int64_t n, hipStream_t s);

}  // namespace dcp
