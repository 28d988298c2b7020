// Projections of the transformer layer: C[T, N] = sum_s A_s W_s (or A_s W_s^T)
// over up to three operand pairs of the same shape, A [T, K] and W ([K, N], or
// [N, K] when transposed) bf16 row-major, with what follows a projection in the
// layer done on the accumulators: the residual, GELU and its derivative, or the
// plain fp32 sum the RMSNorm backward reads.  Q, K and V are one launch (three
// outputs), and so is dY1 = dQ Wq^T + dK Wk^T + dV Wv^T (one sum).
//
// Tiles of 192 features x 64 * TB tokens, four wavefronts in 2 x 2, each with
// 96 features x 32 * TB tokens.  The features are the rows of the products, so
// a lane ends with four consecutive features of one token.  Slices of 64 of the
// contraction (a whole cache line of every row) arrive through a two-stage ring
// of direct global-to-LDS copies; at TB = 2 the 80 KB let two workgroups share a
// CU, one computing while the other waits at its barrier.  Bound by the matrix
// cores and the LDS reads that feed them (3 % of the LDS cycles are bank conflicts)
// at 0.87-0.95 PFLOP/s where the tiles fill the chip: hidden 1,152, 16,381 tokens, Q,
// K and V 145 us, W_up with GELU 201, dY1 137 (eight wavefronts with 256 x 256
// tiles, 192 x 256 tiles, and reading the next slice's first operands across the
// barrier: 1-40 % slower); library and fused times at the layer's sizes stand at
// the rules in layer_api.cpp.
#include <type_traits>

#include "attn_common.h"
#include "layer_launch.h"

namespace dcp {
namespace {

constexpr int kFT = 192;      // features per tile
constexpr int kBK = 64;       // contraction per ring stage
constexpr int kThreads = 256;
constexpr int kWChunks = kFT / 8;  // 16-byte chunks per LDS row of a [K, N] slice

__device__ __attribute__((aligned(16))) const uint32_t zero_chunk[4] = {0, 0, 0, 0};

// A slice of ROWS rows x 64 contiguous contraction elements.  LDS rows are 128
// bytes, chunk c of row r in slot c ^ (r / 2 % 8): 16 consecutive rows read at
// one chunk then cover all banks.
template <int ROWS>
struct RowSlice {
  static constexpr int N = ROWS * 8 / kThreads;  // copies per wavefront
  static constexpr int ELEMS = ROWS * kBK;
  uint32_t off[N];  // byte offsets of this lane's chunks from the slice's first row
  int chunk;        // the chunk of a row this lane copies

  __device__ __forceinline__ void init(int rows_left, int64_t ld, int wave, int lane) {
    chunk = (lane & 7) ^ ((4 * wave + (lane >> 4)) & 7);
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int r = min(8 * (wave + 4 * i) + (lane >> 3), rows_left - 1);  // (rows past the end are not stored)
      off[i] = uint32_t((r * ld + 8 * chunk) * 2);
    }
  }
  __device__ __forceinline__ void issue(__bf16* lds, const __bf16* src, int k_left, int wave) const {
    const uint64_t base = copy_base(src);
    if (k_left >= kBK) {
#pragma unroll
      for (int i = 0; i < N; ++i) lds_copy16(lds_addr(lds + 512 * (wave + 4 * i)), off[i], base);
    } else {
#pragma unroll
      for (int i = 0; i < N; ++i)
        lds_copy16(lds_addr(lds + 512 * (wave + 4 * i)),
               8 * chunk < k_left ? base + off[i] : reinterpret_cast<uint64_t>(zero_chunk));
    }
  }
};

// A slice of 64 contraction rows x 192 features.  LDS row r holds chunk c in
// slot c ^ 4 * (r / 2 % 2), which spreads a transposing read's four rows over
// all banks.
struct ColSlice {
  static constexpr int N = kBK * kWChunks / kThreads;
  static constexpr int ELEMS = kBK * kFT;
  uint32_t off[N];

  __device__ __forceinline__ static int row_of(int i, int wave, int lane, int& chunk) {
    const int slot = 64 * (wave + 4 * i) + lane, r = slot / kWChunks;
    chunk = (slot % kWChunks) ^ (4 * ((r >> 1) & 1));
    return r;
  }
  __device__ __forceinline__ void init(int cols_left, int64_t ld, int wave, int lane) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      int c;
      const int r = row_of(i, wave, lane, c);
      if (8 * c >= cols_left) c = 0;  // past the matrix: such features are not stored
      off[i] = uint32_t((r * ld + 8 * c) * 2);
    }
  }
  __device__ __forceinline__ void issue(__bf16* lds, const __bf16* src, int k_left, int wave, int lane) const {
    const uint64_t base = copy_base(src);
    if (k_left >= kBK) {
#pragma unroll
      for (int i = 0; i < N; ++i) lds_copy16(lds_addr(lds + 512 * (wave + 4 * i)), off[i], base);
    } else {
#pragma unroll
      for (int i = 0; i < N; ++i) {
        int c;
        const int r = row_of(i, wave, lane, c);
        lds_copy16(lds_addr(lds + 512 * (wave + 4 * i)),
               r < k_left ? base + off[i] : reinterpret_cast<uint64_t>(zero_chunk));
      }
    }
  }
};

// A tile's output, first token and first feature.  Tiles are numbered in bands
// of kBand feature tiles, so that the tiles a die runs at one time form a block
// and share their operands' slices in its L2.
constexpr int kBand = 8;
struct Place {
  int out, t0, f0;
};
__device__ __forceinline__ Place place(int tile, int tt, int tf, int nf, int tokens_per_tile) {
  const int band = tile / (tt * kBand), width = min(kBand, nf - band * kBand), x = tile - band * tt * kBand;
  const int f = band * kBand + x % width;
  return {f / tf, x / width * tokens_per_tile, f % tf * kFT};
}

constexpr float kGeluK0 = 0.7978845608028654f;  // sqrt(2 / pi)
constexpr float kGeluK1 = 0.044715f;

// GELU, tanh form, as u * s with s = (1 + tanh(z)) / 2 = 1 / (1 + exp(-2 z)),
// z = k0 (u + k1 u^3); its derivative is s + u * s (1 - s) * 2 k0 (1 + 3 k1 u^2).
__device__ __forceinline__ float gelu_gate(float u) {
  const float z = kGeluK0 * (u + kGeluK1 * u * u * u);
  return __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-2.f * kLog2e * z));
}
__device__ __forceinline__ float gelu(float u) { return u * gelu_gate(u); }
__device__ __forceinline__ float gelu_grad(float u) {
  const float s = gelu_gate(u);
  return fmaf(u * (s * (1.f - s)), 2.f * kGeluK0 * fmaf(3.f * kGeluK1 * u, u, 1.f), s);
}

template <bool WT, int TB, ProjEpilogue EPI>
__global__ __launch_bounds__(kThreads, 2) void proj_kernel(Proj p) {
  constexpr int TT = 64 * TB;  // tokens per tile
  using XS = RowSlice<TT>;
  using WS = std::conditional_t<WT, RowSlice<kFT>, ColSlice>;
  constexpr int STAGE = XS::ELEMS + WS::ELEMS;
  constexpr int HALF = 32 * TB;  // tokens of the output staged at once
  constexpr int RING = 2 * STAGE > HALF * kFT * 2 ? 2 * STAGE : HALF * kFT * 2;
  __shared__ __attribute__((aligned(16))) __bf16 ring[RING];

  const int per_xcd = gridDim.x / kNumXcd;
  const int id = (blockIdx.x % kNumXcd) * per_xcd + blockIdx.x / kNumXcd;
  if (id >= p.n_tiles) return;
  const int T = int(p.tokens), N = p.n, K = p.k;
  const int tf = (N + kFT - 1) / kFT;
  const Place pl = place(id, (T + TT - 1) / TT, tf, tf * p.outs, TT);
  const int t0 = pl.t0, f0 = pl.f0;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wf = wave >> 1, wt = wave & 1;
  const int g = lane >> 5, j = lane & 31;
  XS xs;
  WS ws;
  xs.init(T - t0, K, wave, lane);
  if constexpr (WT)
    ws.init(N - f0, K, wave, lane);
  else
    ws.init(N - f0, N, wave, lane);

  // The slices: all of pair `pair`, then (one sum) all of the next one.
  const int per_pair = (K + kBK - 1) / kBK;
  const int n_it = per_pair * p.pairs;
  int pair = pl.out, k0 = 0;  // of the next slice copied
  auto issue = [&](int stage) DCP_INLINE {
    const __bf16* a = static_cast<const __bf16*>(p.a[pair]);
    const __bf16* w = static_cast<const __bf16*>(p.w[pair]);
    __bf16* buf = ring + stage * STAGE;
    xs.issue(buf, a + int64_t(t0) * K + k0, K - k0, wave);
    if constexpr (WT)
      ws.issue(buf + XS::ELEMS, w + int64_t(f0) * K + k0, K - k0, wave);
    else
      ws.issue(buf + XS::ELEMS, w + int64_t(k0) * N + f0, K - k0, wave, lane);
    k0 += kBK;
    if (k0 >= K) {
      k0 = 0;
      ++pair;
    }
  };

  // Operand reads: lane (g, j) takes row 32 * blk + j, contraction 16 * ks + 8 *
  // g + {0 .. 7}.
  const int sw = (j >> 1) & 7;
  unsigned xo[4], wo[4];  // per 16-wide step (row slices)
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    const unsigned slot = 8 * ((2 * ks + g) ^ sw);
    xo[ks] = (32 * TB * wt + j) * kBK + slot;
    wo[ks] = XS::ELEMS + (96 * wf + j) * kBK + slot;
  }
  const int swt = (lane >> 3) & 1;  // (transposing reads)
  unsigned wtr[3];
#pragma unroll
  for (int i = 0; i < 3; ++i)
    wtr[i] = XS::ELEMS + (8 * g + ((lane & 15) >> 2)) * kFT + 16 * ((lane >> 4) & 1) + 4 * (lane & 3) +
             32 * ((3 * wf + i) ^ swt);
  const lds_bf16* ring3 = lds_ptr(ring);

  f32x16 acc[3][TB];
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int k = 0; k < TB; ++k) acc[i][k] = f32x16{};

  // Half the tokens of the output at a time, eight features per thread and item;
  // what the epilogue reads (GELU's argument, the residual) is fetched before the products.
  constexpr int kItems = HALF * kWChunks / kThreads;
  constexpr bool kAux = EPI == ProjEpilogue::kGeluGrad || EPI == ProjEpilogue::kResidual;
  bf16x8 aux[kAux ? 2 : 1][kItems];
  if constexpr (kAux) {
#pragma unroll
    for (int hm = 0; hm < 2; ++hm)
#pragma unroll
      for (int n = 0; n < kItems; ++n) {
        const int x = tid + kThreads * n, row = t0 + HALF * hm + x / kWChunks, col = f0 + 8 * (x % kWChunks);
        aux[hm][n] = bf16x8{};
        if (row < T && col < N)
          aux[hm][n] = *reinterpret_cast<const bf16x8*>(static_cast<const __bf16*>(p.aux) + int64_t(row) * N + col);
      }
  }
  issue(0);
  for (int it = 0; it < n_it; ++it) {
    wait_vmcnt<0>();
    __syncthreads();  // slice `it` is there, and its predecessor's stage is free
    if (it + 1 < n_it) issue((it + 1) & 1);
    const unsigned st = (it & 1) * STAGE;
    bf16x8 x[4][TB], w[4][3];
    unsigned rt[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      rt[i] = wtr[i] + st;
      asm("" : "+v"(rt[i]));  // keeps the constant terms below in the offset fields
    }
    auto fetch = [&](int ks) DCP_INLINE {
      unsigned rx = xo[ks] + st, rw = wo[ks] + st;
      asm("" : "+v"(rx), "+v"(rw));
#pragma unroll
      for (int k = 0; k < TB; ++k) x[ks][k] = lds_read_b128(ring3 + rx + 32 * k * kBK);
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        if constexpr (WT) {
          w[ks][i] = lds_read_b128(ring3 + rw + 32 * i * kBK);
        } else {
          const lds_bf16* pw = ring3 + rt[i] + 16 * ks * kFT;
          w[ks][i] = cat(lds_read_tr(pw), lds_read_tr(pw + 4 * kFT));
        }
      }
    };
    fetch(0);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      if (ks + 1 < 4) fetch(ks + 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int k = 0; k < TB; ++k) acc[i][k] = mfma32(w[ks][i], x[ks][k], acc[i][k]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  // Lane (g, j), register r of acc[i][k]: feature 96 wf + 32 i + 8 (r / 4) + 4 g
  // + r % 4, token 32 TB wt + 32 k + j.  Half the tokens at a time go through
  // LDS (rows of 48 16-byte chunks, chunk c of row t in slot c ^ (t % 16), which
  // spreads 16 rows over the banks) and leave as whole rows.
  f32x4* stage = reinterpret_cast<f32x4*>(ring);
#pragma unroll
  for (int hm = 0; hm < 2; ++hm) {
    const int th = t0 + HALF * hm;
    if (th >= T) break;
    __syncthreads();
    if (wt == hm) {
#pragma unroll
      for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int k = 0; k < TB; ++k)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int t = 32 * k + j, c = 24 * wf + 8 * i + 2 * q + g;
            stage[t * 48 + (c ^ (t & 15))] =
                f32x4{acc[i][k][4 * q], acc[i][k][4 * q + 1], acc[i][k][4 * q + 2], acc[i][k][4 * q + 3]};
          }
    }
    __syncthreads();
#pragma unroll
    for (int n = 0; n < kItems; ++n) {
      const int x = tid + kThreads * n, t = x / kWChunks, c = x % kWChunks;
      const int row = th + t, col = f0 + 8 * c;
      if (row >= T || col >= N) continue;
      const f32x4 lo = stage[t * 48 + ((2 * c) ^ (t & 15))], hi = stage[t * 48 + ((2 * c + 1) ^ (t & 15))];
      const int64_t at = int64_t(row) * N + col;
      if constexpr (EPI == ProjEpilogue::kSumF32) {
        f32x4* out = reinterpret_cast<f32x4*>(static_cast<float*>(p.out[0]) + at);
        out[0] = lo;
        out[1] = hi;
      } else {
        bf16x8 r;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          float v = e < 4 ? lo[e] : hi[e - 4];
          if constexpr (EPI == ProjEpilogue::kResidual) v += float(aux[hm][n][e]);
          if constexpr (EPI == ProjEpilogue::kGeluGrad) v *= gelu_grad(float(aux[hm][n][e]));
          r[e] = __bf16(v);
        }
        *reinterpret_cast<bf16x8*>(static_cast<__bf16*>(p.out[pl.out]) + at) = r;
        if constexpr (EPI == ProjEpilogue::kGelu) {
          bf16x8 a;
#pragma unroll
          for (int e = 0; e < 8; ++e) a[e] = __bf16(gelu(float(r[e])));
          *reinterpret_cast<bf16x8*>(static_cast<__bf16*>(p.out2) + at) = a;
        }
      }
    }
  }
}

template <bool WT, ProjEpilogue EPI>
hipError_t launch(Proj p, hipStream_t s) {
  // Tiles of 128 tokens, unless they leave CUs without one.  Three outputs,
  // hidden 1,152, tiles of 128 / 64 tokens: 1,000 tokens (144 tiles of 128)
  // 20.6 / 17.2 us, 2,500 (360) 29 / 34; one sum of three, 2,500 (120) 49 / 42,
  // 6,000 (282) 65 / 85.
  const int feature_tiles = (p.n + kFT - 1) / kFT * p.outs;
  auto tiles = [&](int tb) { return int((p.tokens + 64 * tb - 1) / (64 * tb)) * feature_tiles; };
  const bool small = tiles(2) <= kNumCU;
  p.n_tiles = tiles(small ? 1 : 2);
  const dim3 grid((p.n_tiles + kNumXcd - 1) / kNumXcd * kNumXcd);
  if (small)
    hipLaunchKernelGGL((proj_kernel<WT, 1, EPI>), grid, dim3(kThreads), 0, s, p);
  else
    hipLaunchKernelGGL((proj_kernel<WT, 2, EPI>), grid, dim3(kThreads), 0, s, p);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_proj(const Proj& p, ProjEpilogue epi, hipStream_t s) {
  if (p.tokens == 0) return hipSuccess;
  switch (epi) {
    case ProjEpilogue::kStore: return launch<false, ProjEpilogue::kStore>(p, s);
    case ProjEpilogue::kResidual: return launch<false, ProjEpilogue::kResidual>(p, s);
    case ProjEpilogue::kStoreT: return launch<true, ProjEpilogue::kStoreT>(p, s);
    case ProjEpilogue::kGelu: return launch<false, ProjEpilogue::kGelu>(p, s);
    case ProjEpilogue::kGeluGrad: return launch<true, ProjEpilogue::kGeluGrad>(p, s);
    default: return launch<true, ProjEpilogue::kSumF32>(p, s);
  }
}

}  // namespace dcp
