// Tile shapes and the work-unit record shared by the host code that builds
// work lists and the HIP kernels that consume them.  Plain C++ (no HIP
// headers), so the host-side list builder also compiles on its own.
#pragma once

#include <stdint.h>

namespace dcp {

// One tile of work: rows [row0, row0 + rows) of the packed tensor for head
// `head`, all in the sequence that occupies rows [seq0, seq0 + seqlen).
// rows == 0 marks padding (the workgroup exits at once).
// A negative seqlen marks a packed window instead: consecutive sequences,
// each shorter than a tile, sharing one tile of `rows` rows that starts at
// row0 == seq0.  Row i of the window attends only to rows of its own
// sequence; -seqlen - 1 indexes the window's mask of sequence starts (four
// 64-bit words, bit x set where a sequence starts at window offset x).
struct WorkUnit {
  int32_t row0;
  int32_t seq0;
  int32_t seqlen;
  uint16_t rows;  // at most one tile (256)
  uint16_t head;  // head counts are limited to 65535 by the C ABI
};
static_assert(sizeof(WorkUnit) == 16, "16 bytes per tile");
constexpr int kWindowWords = 4;  // 64-bit words per window mask: windows hold at most 256 rows

constexpr int kNumXcd = 8;  // MI355X: 8 accelerator dies, each with its own L2
constexpr int kNumCU = 256;  // and 32 compute units per die

// How many workgroups share one unit of a sequence-tile list of n_units
// (padding included) whose longest sequence has `longest` rows: 8 / parts of
// its rows each, the 8 (or, for 8 parts, 4) wavefronts then splitting the other
// side of the score matrix as well, so a workgroup's walk is `parts` (at 8: 4)
// times shorter.  A workgroup takes most of a CU's LDS, so the chip runs one per
// CU: parts pay as long as they find idle CUs, and cost where they do not (a
// barrier per shorter step, and every part streams the same rows).  Forward, 2
// heads of width 128, 1 / 2 / 4 / 8 parts: 1,000 tokens (32 units) 32 / 21 / 16 /
// 15 us; 8,192 (64) 197 / 120 / 92 / 167; 16,384 (128) 399 / 270 / 348 / 636;
// 20,000 (158) 499 / 580.
// Causal units hold half the work on average and come longest first, so up to
// two rounds of workgroups still fill the chip, if the walks are long: 5,003
// tokens (40 units) 121 / 75 / 54 / 53; 20,000 (158) 476 / 285 / 288.  Short ones
// are mostly a workgroup's start and end, and a second round doubles that.  Two
// rounds against one, forward, 48 to 256 units of one length, widths 64 to 128:
// 300 to 700 tokens 1.02-1.6 x the time, 1,000 1.05-1.3, 1,500 0.68-0.98 with the
// second round at most half full and 0.97-1.17 fuller, 2,000 0.78 and 0.91-1.13,
// 3,000 0.77-0.96, 5,000 and more 0.65-1.02; dK/dV and dQ alike.
// A walk of one or two key tiles is not worth a cut: at most 64 tokens, any parts
// 1.1-1.4 x the forward and 1.1-1.3 x the backward, 80 to 127 tokens 8 parts
// 0.78-1.03 and 0.93-1.04, 4 or 2 parts 0.90-1.18 and 0.96-1.18.  From 129 tokens
// on 8 and 4 parts always pay (forward 0.73-0.86, backward with both passes cut
// 0.82-0.98); 2 parts in the forward (0.79-1.00), in the backward from about 200
// (dK/dV and dQ: 129 tokens 1.02-1.06 and 0.94-1.16, 180 0.97-1.02 and 0.92-1.10,
// 200 0.95-1.01 and 0.85-1.03, 256 0.93-0.98 and 0.91-0.95).
constexpr int parts_within(int n_units, int workgroups) {
  return n_units <= workgroups / 8 ? 8 : n_units <= workgroups / 4 ? 4 : n_units <= workgroups / 2 ? 2 : 1;
}
constexpr int tile_parts(int n_units, bool causal, int longest, bool backward) {
  int parts = parts_within(n_units, kNumCU);
  if (causal && longest >= 1408) {
    const int more = parts_within(n_units, 2 * kNumCU);
    if (longest >= 2560 || n_units * more <= kNumCU + kNumCU / 2) parts = more;
  }
  if (longest <= 128 && (backward || parts < 8 || longest <= 64)) parts = 1;
  if (backward && parts == 2 && longest < 192) parts = 1;
  return parts;
}

// Offsets (bf16 elements) of the 16-byte constant chunks every attention
// workspace starts with.
constexpr int kConstZero = 0;   // [0, 0, 0, 0, 0, 0, 0, 0]
constexpr int kConstOnes = 8;   // [1, 0, 0, 0, 0, 0, 0, 0]
constexpr int kConstInf = 16;   // fp32 +inf (a query past its sequence end)
constexpr int kConstBytes = 256;

// Query rows per forward workgroup: kFwdWaves wavefronts x 32.
constexpr int kFwdWaves = 8;
// Backward, dK/dV pass: `waves` wavefronts per workgroup, each owning
// 32*kb keys whose K, V fragments and dK, dV accumulators stay resident,
// stepping over `bm` queries at a time through a `stages`-deep LDS ring;
// waves_per_eu is the occupancy the register allocation must allow.
// Head widths up to 72 run two wavefronts of 32 keys per SIMD, with Q and
// dO held once per ring stage (the transposing reads of dV and dK use the
// row-read copy, at the cost of some bank conflicts), which leaves LDS for
// a four-stage ring of 64-query tiles.  At head width 128, K and V
// fragments plus the dK, dV accumulators would need more than the 256
// registers two wavefronts per SIMD can each have; V is therefore read from
// an LDS copy of the tile's 256 V rows (68 KB), which leaves K, the
// accumulators and one 16-column step of operands in registers (249-256),
// and the ring holds Q and dO once in two stages of 64-query tiles (76 KB).
// dQ pass: kBwdDqWaves wavefronts of 32 queries, 64 keys per step,
// K held once per ring stage (its transposing reads share the row-read
// copy; at head width 128 this also frees the registers the second copy's
// offsets took).
struct DkdvShape {
  int kb, waves, bm, stages, waves_per_eu;
  bool onecopy;  // the ring holds Q and dO once (row-read stride) instead of twice
  bool vlds;     // V fragments read from an LDS copy of the tile's V rows instead of held in registers
};
constexpr DkdvShape bwd_dkdv_shape(int head_dim) {
  return head_dim > 96 ? DkdvShape{1, 8, 64, 2, 2, true, true} : DkdvShape{1, 8, 64, 4, 2, true, false};
}
// The dK/dV pass with `qs` query streams among `waves` wavefronts (waves / qs
// groups of 32 keys): a ring tile is one 32-query block per stream, in as many
// stages as the LDS beside the (smaller) V copy holds.
constexpr DkdvShape bwd_dkdv_split_shape(int head_dim, int waves, int qs) {
  return head_dim > 96 ? DkdvShape{1, waves, 32 * qs, qs == 2 ? 3 : 2, 2, true, true}
                       : DkdvShape{1, waves, 32 * qs, qs == 2 ? 4 : 3, 2, true, false};
}
constexpr int kBwdDqWaves = 8;
constexpr int kBwdDqStages = 3;
constexpr int kBwdDqStagesD128 = 2;
constexpr bool kBwdDqOneCopy = true;

// Packed windows (runs of short sequences sharing one tile) launch with
// their own shape: fewer wavefronts per workgroup (smaller tiles) and a
// shallower ring -- for the dK/dV pass also 32-query ring tiles -- so that
// two workgroups share a CU; a window then spans at most that many rows.
constexpr int kWinFwdWaves = 4;
constexpr int kWinFwdStages = 2;  // the whole window at once, three workgroups per CU
constexpr int kWinDqWaves = 4;
constexpr int kWinDqStages = 2;
constexpr int kWinDkdvWaves = 4;
constexpr int kWinDkdvStages = 3;
constexpr int kWinDkdvBM = 32;
constexpr DkdvShape bwd_dkdv_window_shape(int head_dim) {
  return head_dim > 96 ? bwd_dkdv_shape(head_dim)
                       : DkdvShape{1, kWinDkdvWaves, kWinDkdvBM, kWinDkdvStages, bwd_dkdv_shape(head_dim).waves_per_eu,
                                   false, false};
}
// Every query and key of a packed window lies inside the window, so at head
// widths up to 96 one workgroup computes dQ of its window as well as dK and
// dV (dS goes through LDS instead of being recomputed by the dQ pass), and
// the dQ pass skips the windows.  This needs the two passes to cut the same
// windows (equal window sizes).
constexpr bool bwd_window_fused(int head_dim) {
  return head_dim <= 96 && kWinDkdvBM == 32 && kWinDkdvWaves == kWinDqWaves;
}

// Rows per tile of each pass, and the most rows a packed window of each pass
// may span.
constexpr int fwd_tile_rows(int) { return kFwdWaves * 32; }
constexpr int fwd_window_rows(int) { return kWinFwdWaves * 32; }
constexpr int bwd_key_tile_rows(int head_dim) {
  return 32 * bwd_dkdv_shape(head_dim).kb * bwd_dkdv_shape(head_dim).waves;
}
constexpr int bwd_query_tile_rows(int) { return 32 * kBwdDqWaves; }
constexpr int bwd_key_window_rows(int head_dim) {
  return 32 * bwd_dkdv_window_shape(head_dim).kb * bwd_dkdv_window_shape(head_dim).waves;
}
constexpr int bwd_query_window_rows(int) { return 32 * kWinDqWaves; }

}  // namespace dcp
