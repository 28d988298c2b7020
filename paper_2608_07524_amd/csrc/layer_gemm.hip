// Weight gradients of the transformer layer: C[M, N] += A^T B with A [T, M]
// and B [T, N] bf16 row-major (activations and upstream gradients, one row per
// token) and C fp32, for all six matrices of a layer in one launch.
//
// The contraction runs over the tokens, the slow index of both operands, and
// the outputs are small next to it (1,152 x 1,152 from 16k tokens), so what
// counts is to keep every CU on matrix products with few output tiles: tiles
// of 192 x 192 (the model widths are multiples of it), the six products
// launched together, and, when even those are too few, the tokens split over
// workgroups whose partial tiles a second kernel adds in a fixed order.
//
// A workgroup is four wavefronts in 2 x 2, each with 96 x 96 of the tile in 3 x
// 3 accumulators.  Token slices of 32 rows arrive through a three-stage ring
// of direct global-to-LDS copies, and both operands are read by transposing LDS
// reads.  74 KB of LDS and at most 256 registers: two workgroups share a CU, so
// one computes while the other waits at its barrier (one workgroup of eight
// wavefronts with a 192 x 384 tile and a four-stage ring: 8-14 % slower).
// Bound by the matrix cores at the clock the card holds under them (counted 1.9
// GHz at hidden 1,152, 1.7 at 3,072; no bank conflicts, 3 TB/s from memory); at
// few tokens, by reading and writing C.  Measured, all six gradients, as library
// GEMMs and here: hidden 1,152, 300 / 4,000 / 16,381 tokens 81 / 324 / 1,185 ->
// 34 / 143 / 481 us (1,084 TFLOP/s); hidden 3,072, 300 / 2,000 / 8,192 tokens
// 315 / 737 / 1,994 -> 272 / 536 / 1,541 us (1,204 TFLOP/s).
#include <algorithm>

#include "attn_common.h"
#include "layer_launch.h"

namespace dcp {
namespace {

constexpr int kTile = 192;   // rows and columns of an output tile
constexpr int kBK = 32;      // tokens per ring stage
constexpr int kStages = 3;
constexpr int kThreads = 256;
constexpr int kCh = kTile / 8;            // 16-byte chunks per LDS row
constexpr int kBuf = kBK * kTile;         // elements of one operand's stage
constexpr int kCopies = kBK * kCh / kThreads;  // copies per wavefront, operand and stage
constexpr int kTileElems = kTile * kTile;
static_assert(kBK * kCh % kThreads == 0 && kCh % 8 == 0, "whole copies, swizzled in groups of 8 chunks");

__device__ __attribute__((aligned(16))) const uint32_t zero_chunk[4] = {0, 0, 0, 0};

// One operand's slice: LDS row r (a token) holds the tile's 24 chunks with
// chunk c in slot c ^ 4 * (r / 2 % 2).  Rows are 384 bytes apart, so rows r and
// r + 2 would start on the same bank; a half-wavefront's transposing read takes
// 64-byte runs of 4 consecutive rows, which this spreads over all banks.
struct Operand {
  const __bf16* src;     // the tile's first column
  uint32_t off[kCopies];  // byte offsets of this lane's chunks from the slice's first row
  int ld;

  __device__ __forceinline__ void init(const __bf16* p, int dim, int col0, int wave, int lane) {
    src = p + col0;
    ld = dim;
#pragma unroll
    for (int i = 0; i < kCopies; ++i) {
      int c;
      const int r = row_of(i, wave, lane, c);
      if (col0 + 8 * c >= dim) c = 0;  // past the matrix: such columns are not stored
      off[i] = uint32_t(r * dim + 8 * c) * 2;
    }
  }
  __device__ __forceinline__ static int row_of(int i, int wave, int lane, int& chunk) {
    const int slot = 64 * (wave + 4 * i) + lane, r = slot / kCh;
    chunk = (slot % kCh) ^ (4 * ((r >> 1) & 1));
    return r;
  }
  // Copies the slice starting at token t0, all of whose rows exist.
  __device__ __forceinline__ void issue_full(__bf16* lds, int64_t t0, int wave) const {
    const uint64_t base = copy_base(src + t0 * ld);
#pragma unroll
    for (int i = 0; i < kCopies; ++i) {
      lds_copy16(lds_at(lds, i, wave), off[i], base);
    }
  }
  // The same with rows from `tokens` on read as zero.
  __device__ __forceinline__ void issue_tail(__bf16* lds, int64_t t0, int64_t tokens, int wave, int lane) const {
    const uint64_t base = copy_base(src + t0 * ld);
#pragma unroll
    for (int i = 0; i < kCopies; ++i) {
      int c;
      const int r = row_of(i, wave, lane, c);
      const uint64_t g = t0 + r < tokens ? base + off[i] : reinterpret_cast<uint64_t>(zero_chunk);
      lds_copy16(lds_at(lds, i, wave), g);
    }
  }
  __device__ __forceinline__ static uint32_t lds_at(__bf16* lds, int i, int wave) {
    return lds_addr(lds + 512 * (wave + 4 * i));
  }
};

// A tile's matrix and first row and column.  Tiles are numbered in bands of
// kBand tile columns, so that the tiles a die runs at one time form a block
// and share their operands' slices in its L2.
constexpr int kBand = 8;
struct Place {
  int problem, m0, n0;
};
__device__ __forceinline__ Place place(const WgradBatch& batch, int tile) {
  int p = 0;
  while (p + 1 < kWgradMax && tile >= batch.p[p + 1].tile0) ++p;
  const int t = tile - batch.p[p].tile0;
  const int tm = (batch.p[p].m + kTile - 1) / kTile, tn = (batch.p[p].n + kTile - 1) / kTile;
  const int band = t / (tm * kBand), width = min(kBand, tn - band * kBand), x = t - band * tm * kBand;
  return {p, x / width * kTile, (band * kBand + x % width) * kTile};
}

__global__ __launch_bounds__(kThreads, 2) void wgrad_kernel(WgradBatch batch, float* __restrict__ partial) {
  __shared__ __attribute__((aligned(16))) __bf16 ring[2 * kStages * kBuf];
  __bf16* As = ring;
  __bf16* Bs = ring + kStages * kBuf;
  // consecutive tiles (sharing rows of A) run on one die
  const int per_xcd = gridDim.x / kNumXcd;
  const int id = (blockIdx.x % kNumXcd) * per_xcd + blockIdx.x / kNumXcd;
  if (id >= batch.n_tiles * batch.splits) return;
  const int split = id / batch.n_tiles, tile = id % batch.n_tiles;
  const Place pl = place(batch, tile);
  const WgradProblem& pr = batch.p[pl.problem];
  const int M = pr.m, N = pr.n, m0 = pl.m0, n0 = pl.n0;
  const int64_t slices = (batch.tokens + kBK - 1) / kBK;
  const int64_t s0 = slices * split / batch.splits;
  const int n_it = int(slices * (split + 1) / batch.splits - s0);

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int g = lane >> 5, j = lane & 31;
  Operand oa, ob;
  oa.init(static_cast<const __bf16*>(pr.a), M, m0, wave, lane);
  ob.init(static_cast<const __bf16*>(pr.b), N, n0, wave, lane);
  auto issue = [&](int it, unsigned ring) DCP_INLINE {  // ring: element offset of the stage
    const int64_t t0 = (s0 + it) * kBK;
    if (t0 + kBK <= batch.tokens) {
      oa.issue_full(&As[ring], t0, wave);
      ob.issue_full(&Bs[ring], t0, wave);
    } else {
      oa.issue_tail(&As[ring], t0, batch.tokens, wave, lane);
      ob.issue_tail(&Bs[ring], t0, batch.tokens, wave, lane);
    }
  };
  auto next = [](unsigned ring) DCP_INLINE { return ring == (kStages - 1) * kBuf ? 0u : ring + kBuf; };

  // Transposing reads (see lds_read_tr): lane (g, j) takes column 32 * blk + j,
  // tokens 16 * ks + 8 * g + {0 .. 7}; the swizzle bit of its rows is fixed.
  const int sw = (lane >> 3) & 1;
  unsigned ao[3], bo[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const unsigned lane_off = (8 * g + ((lane & 15) >> 2)) * kTile + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
    ao[i] = lane_off + 32 * ((3 * wm + i) ^ sw);
    bo[i] = lane_off + 32 * ((3 * wn + i) ^ sw);
  }
  const lds_bf16* As3 = lds_ptr(As);
  const lds_bf16* Bs3 = lds_ptr(Bs);

  f32x16 acc[3][3];
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int k = 0; k < 3; ++k) acc[i][k] = f32x16{};

  unsigned rd = 0, wr = 0;  // ring offsets of the slice being read and of the next one copied
  for (int i = 0; i < kStages - 1; ++i, wr = next(wr))
    if (i < n_it) issue(i, wr);
  if (n_it > 1)
    wait_vmcnt<2 * kCopies>();
  else
    wait_vmcnt<0>();
  __syncthreads();
  for (int it = 0; it < n_it; ++it, rd = next(rd), wr = next(wr)) {
    if (it + kStages - 1 < n_it) issue(it + kStages - 1, wr);
    unsigned ra[3], rb[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      ra[i] = ao[i] + rd;
      rb[i] = bo[i] + rd;
      asm("" : "+v"(ra[i]), "+v"(rb[i]));  // keeps the constant terms below in the offset fields
    }
    bf16x8 a[2][3], b[2][3];
    auto fetch = [&](int ks) DCP_INLINE {
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        const lds_bf16* pa = As3 + ra[i] + 16 * ks * kTile;
        const lds_bf16* pb = Bs3 + rb[i] + 16 * ks * kTile;
        a[ks][i] = cat(lds_read_tr(pa), lds_read_tr(pa + 4 * kTile));
        b[ks][i] = cat(lds_read_tr(pb), lds_read_tr(pb + 4 * kTile));
      }
    };
    auto products = [&](int ks) DCP_INLINE {
#pragma unroll
      for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int k = 0; k < 3; ++k) acc[i][k] = mfma32(a[ks][i], b[ks][k], acc[i][k]);
    };
    // (all 24 reads, then the products, the CU's other workgroup filling the
    // gaps: interleaving the two, or reading half a slice ahead across the
    // barrier, was 3 % slower at hidden 1,152)
    fetch(0);
    fetch(1);
    __builtin_amdgcn_sched_barrier(0);
    products(0);
    __builtin_amdgcn_sched_barrier(0);
    products(1);
    if (it + 2 < n_it)
      wait_vmcnt<2 * kCopies>();
    else
      wait_vmcnt<0>();
    __syncthreads();
  }

  // Lane (g, j), register r of acc[i][k]: row 96 wm + 32 i + 8 (r / 4) + 4 g +
  // r % 4, column 96 wn + 32 k + j of the tile.
  if (batch.splits > 1) {
    f32x4* out = reinterpret_cast<f32x4*>(partial + int64_t(id) * kTileElems);
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          out[((i * 3 + k) * 4 + q) * kThreads + tid] =
              f32x4{acc[i][k][4 * q], acc[i][k][4 * q + 1], acc[i][k][4 * q + 2], acc[i][k][4 * q + 3]};
    return;
  }
  // C += tile, half the rows at a time through LDS, so that C is read and
  // written in 16-byte pieces of whole tile rows.  (Added straight from the
  // accumulators, 4 bytes per lane, the 0.9 GB at hidden 3,072 moved at 2.1
  // TB/s: 1,853 us against 1,541 at 8,192 tokens, 542 against 272 at 300.)
  constexpr int kPieces = kTile / 4;  // 16-byte pieces per row
  static_assert(sizeof(ring) >= kTileElems / 2 * sizeof(float) && kTileElems / 2 % (4 * kThreads) == 0, "half a tile");
  float* half = reinterpret_cast<float*>(ring);
  for (int hm = 0; hm < 2; ++hm) {
    if (wm == hm) {
#pragma unroll
      for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            half[(32 * i + 8 * (r >> 2) + 4 * g + (r & 3)) * kTile + 96 * wn + 32 * k + j] = acc[i][k][r];
    }
    __syncthreads();
#pragma unroll 6
    for (int x = tid; x < kTileElems / 8; x += kThreads) {
      const int row = m0 + kTile / 2 * hm + x / kPieces, col = n0 + 4 * (x % kPieces);
      if (row < M && col < N) {
        f32x4* c = reinterpret_cast<f32x4*>(pr.c + int64_t(row) * N + col);
        *c += reinterpret_cast<const f32x4*>(half)[x];
      }
    }
    __syncthreads();
  }
}

// C += the splits' partial tiles, in split order; a workgroup takes one of a
// tile's 36 register pieces.
__global__ __launch_bounds__(kThreads) void wgrad_reduce_kernel(WgradBatch batch, const float* __restrict__ partial) {
  const int tile = blockIdx.x / 36, x = blockIdx.x % 36;
  const Place pl = place(batch, tile);
  const WgradProblem& pr = batch.p[pl.problem];
  const int m0 = pl.m0, n0 = pl.n0;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int i = x / 12, k = x / 4 % 3, q = x % 4;
  f32x4 sum = {};
  for (int s = 0; s < batch.splits; ++s)
    sum += reinterpret_cast<const f32x4*>(partial + (int64_t(s) * batch.n_tiles + tile) * kTileElems)[x * kThreads + tid];
  const int col = n0 + 96 * (wave & 1) + 32 * k + (lane & 31);
  const int row0 = m0 + 96 * (wave >> 1) + 32 * i + 8 * q + 4 * (lane >> 5);
  if (col >= pr.n) return;
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (row0 + e < pr.m) pr.c[int64_t(row0 + e) * pr.n + col] += sum[e];
}

// Whether two problems add into the same memory (weights that share a gradient).
bool share_output(const WgradBatch& b) {
  for (const WgradProblem& p : b.p)
    for (const WgradProblem* q = b.p; q != &p; ++q) {
      const uintptr_t x = reinterpret_cast<uintptr_t>(p.c), y = reinterpret_cast<uintptr_t>(q->c);
      if (x < y + sizeof(float) * size_t(q->m) * size_t(q->n) && y < x + sizeof(float) * size_t(p.m) * size_t(p.n))
        return true;
    }
  return false;
}

}  // namespace

hipError_t launch_wgrad(WgradBatch b, void* scratch, size_t scratch_bytes, hipStream_t s) {
  if (b.tokens == 0) return hipSuccess;
  // Workgroups of one launch add to C without atomics, so problems with a common
  // C run one after another (problems without rows or columns have no tiles).
  if (share_output(b)) {
    for (const WgradProblem& p : b.p) {
      WgradBatch one{};
      one.p[0] = p;
      one.tokens = b.tokens;
      const hipError_t e = launch_wgrad(one, scratch, scratch_bytes, s);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  b.n_tiles = 0;
  for (WgradProblem& p : b.p) {
    p.tile0 = b.n_tiles;
    b.n_tiles += ((p.m + kTile - 1) / kTile) * ((p.n + kTile - 1) / kTile);
  }
  // Enough tiles for every CU need no split; fewer split the tokens until the
  // 512 workgroups that fit the chip are busy, in slices of at least 256 tokens
  // and as far as the scratch holds their partial tiles.
  const int64_t slices = (b.tokens + kBK - 1) / kBK;
  const int64_t fit = int64_t(scratch_bytes / (size_t(kTileElems) * sizeof(float)));
  int64_t splits = b.n_tiles >= kNumCU ? 1 : 2 * kNumCU / b.n_tiles;
  splits = std::max<int64_t>(1, std::min(std::min(splits, slices / 8), fit / b.n_tiles));
  b.splits = int(splits);
  const int grid = (b.n_tiles * b.splits + kNumXcd - 1) / kNumXcd * kNumXcd;
  hipLaunchKernelGGL(wgrad_kernel, dim3(grid), dim3(kThreads), 0, s, b, static_cast<float*>(scratch));
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || b.splits == 1) return e;
  hipLaunchKernelGGL(wgrad_reduce_kernel, dim3(b.n_tiles * 36), dim3(kThreads), 0, s, b,
                     static_cast<const float*>(scratch));
  return hipGetLastError();
}

}  // namespace dcp
