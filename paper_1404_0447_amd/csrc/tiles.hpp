// Tile shapes shared by the scheduler (task lists) and the kernels.
#pragma once
#include <cstddef>

namespace selinv {
constexpr int kThreads = 256;    // work-group size of every tiled kernel (4 waves)
constexpr int kMaxS = 256;       // widest supported block (cap)
constexpr int kTileM = 64;       // rows of an MFMA output tile (gather-GEMM, panel, Schur)
constexpr int kSchurTile = 64;   // edge of a Schur-update tile (lower c x c)
constexpr int kDiagTile = 32;    // edge of a diagonal-block tile (pairs (I,J), I >= J)
constexpr int kDiagTile64 = 64;  // the same on the per-level path (pipelined MFMA tile)
constexpr int kLdsDiagMax = 128; // diagonal blocks inverted in LDS and registers up to this width
constexpr int kZMaxS = 64;       // widest block of the complex path (one 64-wide tile per diagonal step)
// Complex gather-GEMM and diagonal step: a level with fewer than
// kZSplitFill / 2 tasks cuts each task's contraction over C into pieces of
// at least kZSplitRows rows, about kZSplitFill work-groups in all; a piece
// writes its 64 x 64 complex partial product to a scratch slot of
// kZSlotDoubles doubles.
constexpr int kZSplitFill = 2048;
constexpr int kZSplitRows = 128;
// levels with fewer tasks than this (those of a single pole) cut shorter
// pieces and fewer of them: there a piece's length is its time, while in the
// larger levels of a batch the pieces' sums cost more than they gain.
// Measured, ms, these constants against 64 rows (32 below 64 tasks) and a fill
// of 2,048 everywhere: n = 8,000, 1 pole 3.34 and 3.43, 2 4.49 and 4.48, 4 6.44
// and 6.43, 8 10.17 and 10.17, 16 17.19 and 17.30, 32 29.93 and 30.10; n = 1,728,
// 1 pole 1.02 and 1.02, 4 1.18 and 1.30, 8 1.60 and 1.58, 16 2.18 and 2.12, 32
// 3.17 and 3.13; n = 1,372, 1 pole 0.71 and 0.70, 4 0.77 and 0.81, 8 0.94 and
// 0.97, 16 1.28 and 1.30, 32 1.89 and 1.96.
constexpr int kZSplitFewTasks = 128;
constexpr int kZSplitFewRows = 32;
constexpr int kZSplitFewFill = 768;
constexpr size_t kZSlotDoubles = 2 * (size_t)kZMaxS * kZMaxS;

// small blocks run whole on one wave (all phases, 16 x 16 MFMA tiles)
constexpr int kSbS = 16;          // widest small block
constexpr int kSbC = 256;         // largest |C| of a small block
constexpr int kSbPerTask = 4;     // small blocks per work-group task (one per wave)
inline bool is_small(int s, int c, int smax) { return s <= smax && c <= kSbC; }
// per-level path: a wave per block only where |C| is small.  Blocks with a
// larger |C| sit in few, nearly empty levels near the leaves, where the tiled
// kernels spread them over many more work-groups (swept over 0..256: 32
// fastest at 40^3, 64^3 and molecular 16^3)
constexpr int kSbCLevel = 32;
// A level with few panel tiles (a Schur colour group with few tiles) gives
// each 16 x 16 tile to a wave, which loads its whole contraction (s <= 128)
// before its first product: there the tiles' latency, not the device's
// throughput, sets the level time.  Measured, us, few-tile kernel < or >
// tiled kernel at the same number of 64-wide tiles (a: batches of dense chains
// of that s; b: the 40^3 grid, c: the molecular 16^3 matrix, where s is mostly
// 128):
//   Schur  s = 16  144 6.5 = 6.5, 192 7.1 > 6.6, 240 8.2 > 7.0 (a)
//          s = 32  132 7.1 = 7.2, 168 8.5 > 8.2, 224 10.2 > 8.6 (a)
//          s = 64  120 6.4 < 8.6, 168 9.7 < 10.7, 192 10.2 > 9.3 (a)
//          s = 128 120 9.0 < 11.8, 144 12.3 > 11.6, 224 16.1 > 13.1 (a);
//                  120 10.8 < 12.6, 153 13.7 = 13.6, 231 16.4 > 14.6 (b);
//                  136 12.5 = 12.4, 171 13.5 > 13.2, 253 16.6 > 13.3 (c)
//   panel  s = 16  96 3.8 = 3.6, 160 4.3 > 3.7; s = 32  144 4.6 = 4.8, 192 5.4
//          > 4.9; s = 64  144 7.1 < 7.4, 192 7.6 < 8.2, 220 8.8 > 8.5 (a)
//          s = 128, against tiles of 128 columns: 128 9.3 < 16.7, 230 15.1 <
//          17.3, 298 17.8 = 17.8, 326 19.9 > 17.8 (b); 247 10.8 < 16.3 (c)
constexpr int kFewSchurTiles = 160;
constexpr int kFewPanelTiles = 160;      // of blocks at most 64 wide
constexpr int kFewPanelTilesWide = 256;  // of wider ones
constexpr int kDeepK = 128;  // longest contraction of the kernels of few tiles
constexpr int kZeroCols = 8;  // columns of Ainv(:, B) a task of the set-up kernel clears
// A level's Schur update runs in colour groups (read-modify-write, one launch
// each) only when its blocks need at most this many colours; more launches
// cost more than the atomics they save (molecular 16^3: 10.3 -> 9.5 ms).
constexpr int kMaxSchurColours = 3;
inline bool is_small_level(int s, int c) { return s <= kSbS && c <= kSbCLevel; }

// reverse sweep: split the contraction when a level has fewer tiles than this
// (swept over 256..2048: 1024 fastest at 64^3 and molecular 16^3)
constexpr int kFillTiles = 1024;
// resident work-groups of the gather-GEMM and diagonal-tile kernels on the
// target (256 CUs x 2); the per-level split is sized for them
constexpr long kGemmSlots = 512;
// fixed cost of one work-group of the split contractions, in 16-deep chunks
// (swept over 3, 6, 10 at 64^3: gather-GEMM 18.3, 18.1, 18.2 ms)
constexpr double kGemmTaskOvh = 6.0;
constexpr double kSdiagTaskOvh = 8.0;  // smaller epilogue (half a 64 x 64 tile)
constexpr int kMinSplitK = 128;  // rows of C per split piece, at least
// the same in a level that even so has at most a work-group per CU (kGemmSlots
// / 2), where a piece's length is its time: gather-GEMM of a 301 x 257 grid
// 202 -> 164 us, of the indefinite 12^3 matrix 820 -> 777, of 40^3 1.82 ->
// 1.78 ms; 32 rows 181, 771 us, 1.78 ms.  With 64 everywhere 40^3 took 1.83.
constexpr int kMinSplitKFew = 64;
constexpr int kMinSplitKDiag = 64;  // the same for the diagonal tile pairs

// output-column tile of a block of width s: 16, 32, 64 or 128
inline int tile_bn(int s) { return s <= 16 ? 16 : s <= 32 ? 32 : s <= 64 ? 64 : 128; }
}  // namespace selinv
