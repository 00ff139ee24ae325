// Device kernels for the supernodal LDL^T and the selected inversion.
//
// Data layout (all FP64, in one caller-bound workspace):
//   Lp  panels of the factor: block B is an (s+c) x s column-major panel,
//       ld = s+c; rows = cols(B) then C(B).  The s x s block holds L_BB
//       (unit diagonal implied, D on the diagonal; with 2x2 pivots it keeps
//       the assembled F_BB, whose inverse goes to Tp alone); the C rows hold
//       F(C,B), the assembled and updated entries of A (L(C,B) is
//       F(C,B) L_BB^{-T} D^{-1} and is formed only on export).
//   Ap  same layout, holds the selected entries of A^{-1}.
//   Hp  L_hat(C,B) = L(C,B) L_BB^{-1} = F(C,B) T, c x s column-major (ld c).
//   Tp  T = F_BB^{-1} (s x s); Wp  scratch (s x s): L_BB^{-1} of a block wider
//       than 128 columns while its T is formed, not written for the others.
// Block index maps: for position r of C(B), cbase[r] is the arena offset of
// column C[r] inside its owning block J, and rel[rbase[r] + i] the row of
// C[i] (i >= r's segment start) inside rows(J).  So the entry
// A^{-1}(C[i], C[k]), i >= k, lives at cbase[k] + rel[rbase[k] + i].
//
// Dense products use v_mfma_f64_16x16x4f64: lane l holds A[l%16][l/16] and
// B[l/16][l%16]; the 16x16 result element (l/16 + 4v, l%16) sits in
// register v of lane l.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "kernels.hpp"
#include "lanes.hpp"
#include "plan.hpp"
#include "tiles.hpp"

namespace selinv {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef double d2 __attribute__((ext_vector_type(2)));
// two doubles read with one load from an 8-byte aligned address
typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));
// (cbase, rbase) of one position, one 16-byte load
typedef int64_t i64x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ d4 mfma(double a, double b, d4 c)
{
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Wait states after the last MFMA of a loop, before its accumulators are
// read by ordinary vector instructions (the scheduler may not move anything
// across the barrier).
__device__ __forceinline__ void mfma_drain()
{
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 15\n\ts_nop 15" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

__global__ void k_fill(double* __restrict__ p, int64_t n, double v)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// status[0]: smallest failing pivot column (~0 = none); status[1]: error
// flags of the persistent work queues (0 = none)
__global__ void k_status_reset(unsigned long long* status)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) {
        status[0] = ~0ull;
        status[1] = 0ull;
    }
}

__global__ void k_scatter_set(const double* __restrict__ src, const int64_t* __restrict__ off, int64_t n,
                              double* __restrict__ dst)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        dst[off[i]] = src[i];
}

__global__ void k_gather(const double* __restrict__ src, const int64_t* __restrict__ off, int64_t n,
                         double* __restrict__ dst)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        dst[i] = src[off[i]];
}

// Blocks whose products accumulate over several work-groups start from
// the lower triangle of Ainv(B,B) := T and, when the gather-GEMM is split
// (zx), X = Ainv(C,B) := 0.  One wave per column, lanes along its rows.
__device__ __forceinline__ void zero_task(const BlockDesc d, double* __restrict__ Ap, const double* __restrict__ Tp,
                                          bool zx = true, int j0 = 0, int j1 = 1 << 30)
{
    const int64_t ld = (int64_t)d.s + d.c;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    j1 = min(j1, d.s);
    for (int j = j0 + wave; j < j1; j += kThreads / 64) {
        double* col = Ap + d.poff + (int64_t)j * ld;
        const double* tcol = Tp + d.woff + (int64_t)j * d.s;
        for (int i = j + lane; i < d.s; i += 64) col[i] = tcol[i];
        if (zx)
            for (int i = lane; i < d.c; i += 64) col[d.s + i] = 0.0;
    }
}

__global__ __launch_bounds__(kThreads) void k_zero_x(const Task* __restrict__ tasks,
                                                     const BlockDesc* __restrict__ blk, double* __restrict__ Ap,
                                                     const double* __restrict__ Tp)
{
    const Task t = tasks[blockIdx.x];
    zero_task(blk[t.b], Ap, Tp, t.flags & 1, t.kb, t.ke);  // columns [kb, ke)
}

// Checkpoint copy of whole inverse panels ((s + c) x s, contiguous): dir 0
// panel -> store, dir 1 store -> panel; blocks without a slot are skipped.
// Up to 32 work-groups per block (fewer where a plan has more than 8,000
// blocks): one alone took as long as the widest panel needs at one CU's
// bandwidth, 121 us for the molecular 9^3 matrix, now 8 us.
__global__ __launch_bounds__(kThreads) void k_ck_copy(const Task* __restrict__ tasks,
                                                      const BlockDesc* __restrict__ blk,
                                                      const int64_t* __restrict__ ck_off, double* __restrict__ Ap,
                                                      double* __restrict__ ck, int dir)
{
    const int b = tasks[blockIdx.x].b;
    const int64_t o = ck_off[b];
    if (o < 0) return;
    const BlockDesc d = blk[b];
    const int64_t n = ((int64_t)d.s + d.c) * d.s;
    double* panel = Ap + d.poff;
    double* slot = ck + o;
    const double* from = dir == 0 ? panel : slot;
    double* to = dir == 0 ? slot : panel;
    for (int64_t i = threadIdx.x + (int64_t)blockIdx.y * kThreads; i < n; i += (int64_t)gridDim.y * kThreads)
        to[i] = from[i];
}

// L on the canonical pattern: diagonal-block entries are stored; an entry in
// C(B) rows is L(r,j) = sum_{k>=j} L_hat(r,k) L_BB(k,j).  One thread per column.
__global__ void k_export_L(const BlockDesc* __restrict__ blk, const int32_t* __restrict__ colblk,
                           const int64_t* __restrict__ colptrL, const int64_t* __restrict__ off, int64_t n,
                           const double* __restrict__ Lp, const double* __restrict__ Hp, double* __restrict__ out)
{
    for (int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; j < n; j += (int64_t)gridDim.x * blockDim.x) {
        const BlockDesc d = blk[colblk[j]];
        const int64_t ld = (int64_t)d.s + d.c;
        for (int64_t q = colptrL[j]; q < colptrL[j + 1]; ++q) {
            const int64_t o = off[q] - d.poff;
            const int row = (int)(o % ld), col = (int)(o / ld);
            double v;
            if (row < d.s) {
                v = Lp[off[q]];
            } else {
                const int r = row - d.s;
                v = Hp[d.hoff + r + (int64_t)col * d.c];
                for (int k = col + 1; k < d.s; ++k)
                    v += Hp[d.hoff + r + (int64_t)k * d.c] * Lp[d.poff + k + (int64_t)col * ld];
            }
            out[q] = v;
        }
    }
}

// ---------------------------------------------------------------------------
// 64 x BN MFMA tiles, four waves: BN >= 64 -> 2 x 2 waves of 32 x BN/2, else
// 4 x 1 waves of 16 x BN; contractions in chunks of 16.
// ---------------------------------------------------------------------------
constexpr int TBM = 64, TBK = 16;

template <int BN>
struct TileShape {
    static constexpr int WM = BN >= 64 ? 2 : 4;
    static constexpr int WN = 4 / WM;
    static constexpr int MT = TBM / WM / 16;
    static constexpr int NT = BN / WN / 16;
};

// Visit every element f(i, j, value) (tile-local i, j) of a tile whose
// MFMAs ran with their operands swapped: mfma(b, a) forms the transposed
// 16 x 16 product, and register v of lane l holds row l / 16 + 4 v, column
// l % 16 of whatever product it forms, so here lane l holds row i = l % 16.
// Sixteen lanes then cover sixteen consecutive rows of one column, which
// makes the stores (and atomics) into a column-major output contiguous.
template <int BN, class F>
__device__ __forceinline__ void tile_epilogue_t(const d4 (&acc)[2][4], F f)
{
    using SH = TileShape<BN>;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm0 = (wave % SH::WM) * (TBM / SH::WM), wn0 = (wave / SH::WM) * (BN / SH::WN);
#pragma unroll
    for (int mt = 0; mt < SH::MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < SH::NT; ++nt)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                f(wm0 + mt * 16 + (lane & 15), wn0 + nt * 16 + (lane >> 4) + 4 * v, acc[mt][nt][v]);
}

#define SELINV_BN_DISPATCH(bn, CALL) \
    switch (bn) {                    \
        case 16: CALL(16); break;    \
        case 32: CALL(32); break;    \
        case 64: CALL(64); break;    \
        default: CALL(128); break;   \
    }

// ---------------------------------------------------------------------------
// Selected inversion, step 3: X = Ainv(C,B) = -Ainv(C,C) L_hat(C,B) for rows
// [i0, i0+64) and columns [j0, j0+BN) of X.  Ainv(C,C) is gathered from the
// ancestors' panels: entries with i >= k directly, the others by symmetry.
// ---------------------------------------------------------------------------
// The pipelined gather-GEMM loop, shared by the forward gather-GEMM and the
// reverse sweep: acc += A B over the contraction [Kb, Ke) for tile rows
// [r0, r0+64) and columns [n0, n0+BN), accumulated transposed, with
//   A(i, k) = S[cbase[p] + rel[rbase[p] + q]],  p = min(i, k), q = max(i, k)
// (an arena gathered through the block index maps; kTri = 1 keeps k <= i
// only, 2 keeps k >= i only, 0 all) and B(k, j) = Bm[k + (n0 + j) ldb].
//
// What bounds it: the FP64 MFMAs and the vector instructions beside them.
// The two share the SIMD's FP64 hardware on this part: a vector instruction
// next to an FP64 MFMA costs its four issue cycles (measured: 77 TFLOP/s with
// none, 54 with five per MFMA).  So the loop is built to issue few:
//  * Chunks of the contraction come in three modes.  Below the diagonal band
//    (k < i for the whole tile) p = k: the lanes of a wave run along i, so
//    the map entry is one address per wave and the rel entries and values are
//    contiguous.  Above it p = i, and the lanes run along k.  Only the chunks
//    of the band, and a ragged last chunk, form min and max per element and
//    carry masks.  In the other modes every per-lane offset is a constant of
//    the tile, and the chunk's position sits in the scalar base.
//  * Rows past c read row c - 1 (their products are never stored), columns
//    past s read column s - 1, and chunks past the end read the last chunk
//    again, so no load needs a mask.
//  * Both operands lie in LDS as rows of 16 contraction entries (128 bytes):
//    a 16-byte slot holds entries k and k + 4, what a lane needs for two
//    consecutive MFMAs, and slots are exclusive-or'ed with row / 2 mod 8,
//    which makes these reads conflict-free without padding.
// Vector instructions per 32 MFMAs: 154 -> 21.  Gather-GEMM of the 64^3
// matrix: 22.0 -> 18.4 ms (11.2 ms of it MFMA at the rate above, padding
// included; without the loads of A it takes 15.3).
//
// The software pipeline: while the MFMAs consume chunk n from one LDS buffer,
// the values of chunk n+1 are stored to the other, and the loads of A of
// chunk n+3, of B of chunk n+2, of the rel entries of chunk n+4 and of the
// (cbase, rbase) pairs of chunk n+5 are issued: A, which comes from HBM, has
// two iterations of MFMAs to arrive, the others one.  One barrier per chunk.
// Byte offsets inside a block's panel and C's maps are 32-bit, here and at the
// buffer descriptors below, so s (s + |C|) doubles have to stay below 4 GiB.
// With s <= 256 that holds to |C| of 2.09 million.  No plan gets there: C x C
// lies in the ancestors' panels, |C|^2 / 2 doubles, 17.6 TB at that size, and
// the 288 GB of a card end at a |C| of 270,000.
constexpr int kGatherRow = 16 * (int)sizeof(double);  // bytes of one LDS row
// byte offset of contraction entry k of a row: entries 8 t + g and 8 t + 4 + g
// (g < 4) share slot 4 t + g
__device__ __forceinline__ int lds_at(int row, int k)
{
    const int slot = ((k >> 3) << 2) | (k & 3);
    return row * kGatherRow + ((slot ^ ((row >> 1) & 7)) << 4) + ((k >> 2) & 1) * 8;
}
template <int BNMAX>
struct alignas(16) GatherLdsN {
    char A[2][TBM * kGatherRow];
    char B[2][BNMAX * kGatherRow];
};
using GatherLds = GatherLdsN<128>;

template <int BN, int kTri, class LDS>
__device__ __forceinline__ void gather_mma(LDS& L, const BlockDesc d, const int r0, const int n0, const int Kb,
                                           const int Ke, const double* __restrict__ S, const double* __restrict__ Bm,
                                           const int64_t ldb, const int64_t* __restrict__ cr2,
                                           const int32_t* __restrict__ rel, d4 (&acc)[2][4])
{
    using SH = TileShape<BN>;
    static_assert(sizeof(L.B[0]) >= BN * kGatherRow, "the LDS tile holds BN columns");
    constexpr int NP = BN >= 32 ? BN / 32 : 1;  // pairs (k, k + 1) of B per thread per chunk
    const int c = d.c;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm0 = (wave % SH::WM) * (TBM / SH::WM), wn0 = (wave / SH::WM) * (BN / SH::WN);
    const int nch = Ke > Kb ? (Ke - Kb + TBK - 1) / TBK : 0;
    if (nch == 0) return;
    enum { kBelow = 0, kAbove = 1, kBand = 2 };
    auto k_of = [&](int ch) { return Kb + min(ch, nch - 1) * TBK; };
    auto mode_of = [&](int k0) {
        if (k0 + TBK > Ke) return (int)kBand;
        if (kTri != 2 && k0 + TBK <= r0) return (int)kBelow;
        if (kTri != 1 && k0 >= r0 + TBM) return (int)kAbove;
        return (int)kBand;
    };
    // element q of this thread: below the band (kk, ii) = (4 q + wave, lane),
    // else (tid & 15, tid / 16 + 16 q)
    const int ak = tid & 15, ai = tid >> 4;
    const int iBelow = min(r0 + lane, c - 1);
    const int64_t* map = cr2 + 2 * d.coff;
    // Stages, each for one chunk; M: the chunk's mode where it is known, -1
    // in the general form (which finds the mode out, a uniform branch).
    i64x2 m_cr[4];          // stage MAP: (cbase[p], rbase[p])
    const double* r_at[4];  // stage REL: S + cbase[p]
    uint32_t r_rel[4];      //            rel entry
    double v_a[2][4];       // stage VAL: A of two chunks (by the chunk's parity), B of one
    d2u v_b[NP];
    // the band's (i, k) of element q, clamped into C and the contraction
    auto band_ik = [&](int k0, int q, int& i, int& k) {
        i = min(r0 + ai + 16 * q, c - 1);
        k = min(k0 + ak, Ke - 1);
    };
    auto load_map = [&](auto M, int ch) {
        constexpr int kM = decltype(M)::value;
        const int k0 = k_of(ch), md = kM >= 0 ? kM : mode_of(k0);
        uint32_t off[4];
        const int64_t* base = map;
        if (md == kBelow) {
            base += 2 * k0;
#pragma unroll
            for (int q = 0; q < 4; ++q) off[q] = (uint32_t)(4 * q + wave) * 16u;
        } else if (md == kAbove) {
            // row ai + 16 q of the tile (all rows are inside C here)
            base += 2 * r0;
#pragma unroll
            for (int q = 0; q < 4; ++q) off[q] = (uint32_t)(ai + 16 * q) * 16u;
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                int i, k;
                band_ik(k0, q, i, k);
                off[q] = (uint32_t)min(i, k) * 16u;
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
            m_cr[q] = *reinterpret_cast<const i64x2*>(reinterpret_cast<const char*>(base) + off[q]);
    };
    auto load_rel = [&](auto M, int ch) {
        constexpr int kM = decltype(M)::value;
        const int k0 = k_of(ch), md = kM >= 0 ? kM : mode_of(k0);
        if (md == kBand) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                int i, k;
                band_ik(k0, q, i, k);
                r_rel[q] = (uint32_t)rel[m_cr[q].y + max(i, k)];
            }
        } else {  // one second index for all four elements
            const int32_t* rq = rel + (md == kBelow ? iBelow : k0 + ak);
#pragma unroll
            for (int q = 0; q < 4; ++q) r_rel[q] = (uint32_t)rq[m_cr[q].y];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) r_at[q] = S + m_cr[q].x;
    };
    // B: pair bk of columns bj + 32 q, through a buffer descriptor (the
    // chunk's offset is scalar; columns past s are out of its range and read 0)
    const int bk = tid & 7, bj = tid >> 3;
    const int64_t bytes = ((int64_t)(d.s - 1 - n0) * ldb + c) * (int64_t)sizeof(double);
    const double* Bt = Bm + (int64_t)n0 * ldb;
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)Bt, 0, (int)(uint32_t)bytes, 0x00020000);
    uint32_t boff[NP];
#pragma unroll
    for (int q = 0; q < NP; ++q)
        boff[q] = (uint32_t)(((int64_t)(bj + 32 * q) * ldb + 2 * bk) * (int64_t)sizeof(double));
    auto load_b = [&](auto M, int ch) {
        constexpr int kM = decltype(M)::value;
        const int k0 = k_of(ch);
        if (kM >= 0 || k0 + TBK <= Ke) {
#pragma unroll
            for (int q = 0; q < NP; ++q)
                v_b[q] = __builtin_bit_cast(
                    d2u, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)boff[q], k0 * (int)sizeof(double), 0));
        } else {  // ragged end: rows past Ke - 1 read that row (A is zero there)
#pragma unroll
            for (int q = 0; q < NP; ++q) {
                const double* col = Bm + (int64_t)min(n0 + bj + 32 * q, d.s - 1) * ldb;
                v_b[q].x = col[min(k0 + 2 * bk, Ke - 1)];
                v_b[q].y = col[min(k0 + 2 * bk + 1, Ke - 1)];
            }
        }
    };
    const int wAbove = lds_at(ai, ak), wB = lds_at(bj, 2 * bk), wB1 = lds_at(bj, 2 * bk + 1);
    int wBelow[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) wBelow[q] = lds_at(lane, 4 * q + wave);
    auto store = [&](auto M, const double (&va)[4], int ch, int buf) {
        constexpr int kM = decltype(M)::value;
        const int k0 = k_of(ch), md = kM >= 0 ? kM : mode_of(k0);
        char* A = L.A[buf];
        if (md == kBelow) {
#pragma unroll
            for (int q = 0; q < 4; ++q) *reinterpret_cast<double*>(A + wBelow[q]) = va[q];
        } else if (md == kAbove) {
#pragma unroll
            for (int q = 0; q < 4; ++q) *reinterpret_cast<double*>(A + wAbove + q * 16 * kGatherRow) = va[q];
        } else {
            const int kr = k0 + ak;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int ir = r0 + ai + 16 * q;
                const bool ok = kr < Ke && (kTri == 0 || (kTri == 1 ? kr <= ir : kr >= ir));
                *reinterpret_cast<double*>(A + wAbove + q * 16 * kGatherRow) = ok ? va[q] : 0.0;
            }
        }
        char* B = L.B[buf];
        if (BN >= 32 || wave < 2) {
#pragma unroll
            for (int q = 0; q < NP; ++q) {
                *reinterpret_cast<double*>(B + wB + q * 32 * kGatherRow) = v_b[q].x;
                *reinterpret_cast<double*>(B + wB1 + q * 32 * kGatherRow) = v_b[q].y;
            }
        }
    };
    // fragment rows: wm0, wn0 and 16 mt are multiples of 16, so one slot per
    // lane and half chunk serves every fragment
    const int fr = lane & 15, fg = lane >> 4;
    const int f0 = lds_at(fr, fg), f1 = lds_at(fr, 8 + fg);
    auto body = [&](auto M, auto X, int ch) {  // X: the parity of ch
        constexpr int buf = decltype(X)::value;
        const char *A = L.A[buf] + wm0 * kGatherRow, *B = L.B[buf] + wn0 * kGatherRow;
        d2 a[SH::MT], b[SH::NT];
        auto frags = [&](int f) {
#pragma unroll
            for (int mt = 0; mt < SH::MT; ++mt) a[mt] = *reinterpret_cast<const d2*>(A + f + mt * 16 * kGatherRow);
#pragma unroll
            for (int nt = 0; nt < SH::NT; ++nt) b[nt] = *reinterpret_cast<const d2*>(B + f + nt * 16 * kGatherRow);
        };
        auto products = [&]() {
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int mt = 0; mt < SH::MT; ++mt)
#pragma unroll
                    for (int nt = 0; nt < SH::NT; ++nt) acc[mt][nt] = mfma(b[nt][h], a[mt][h], acc[mt][nt]);
        };
        frags(f0);
        store(M, v_a[buf ^ 1], ch + 1, buf ^ 1);
        // The loads stay ahead of the products (the scheduler would sink them
        // to the end, in front of their own waits), and in this order: they
        // return in order, so a wait on one waits for all before it, and the
        // values of A, whose use is two iterations away, come last.
        const double* at[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) at[q] = r_at[q] + r_rel[q];
        load_rel(M, ch + 4);
        load_map(M, ch + 5);
        __builtin_amdgcn_sched_barrier(0);
        load_b(M, ch + 2);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < 4; ++q) v_a[buf ^ 1][q] = *at[q];  // chunk ch + 3
        __builtin_amdgcn_sched_barrier(0);
        products();
        frags(f1);
        products();
        __syncthreads();
    };
    using Any = std::integral_constant<int, -1>;
    using Below = std::integral_constant<int, kBelow>;
    using Above = std::integral_constant<int, kAbove>;
    using X0 = std::integral_constant<int, 0>;
    using X1 = std::integral_constant<int, 1>;
    {
        // chunk 0 in LDS, A of chunks 1 and 2 and B of chunk 1, rel entries of
        // chunk 3, pairs of chunk 4.  The first chunks' chains of loads run
        // side by side, and the loads that stay in flight are issued in the
        // loop's order (its waits count the loads behind the one they need).
        i64x2 c[4][4];
#pragma unroll
        for (int n = 0; n < 4; ++n) {
            load_map(Any{}, n);
#pragma unroll
            for (int q = 0; q < 4; ++q) c[n][q] = m_cr[q];
        }
        const double* at3[3][4];
        uint32_t re[3][4];
#pragma unroll
        for (int n = 0; n < 3; ++n) {
#pragma unroll
            for (int q = 0; q < 4; ++q) m_cr[q] = c[n][q];
            load_rel(Any{}, n);
#pragma unroll
            for (int q = 0; q < 4; ++q) at3[n][q] = r_at[q], re[n][q] = r_rel[q];
        }
        double a0[4];
        d2u b0[NP];
        load_b(Any{}, 0);
#pragma unroll
        for (int q = 0; q < NP; ++q) b0[q] = v_b[q];
#pragma unroll
        for (int q = 0; q < 4; ++q) a0[q] = at3[0][q][re[0][q]];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < 4; ++q) v_a[1][q] = at3[1][q][re[1][q]];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < 4; ++q) m_cr[q] = c[3][q];
        load_rel(Any{}, 3);
        load_map(Any{}, 4);
        __builtin_amdgcn_sched_barrier(0);
        load_b(Any{}, 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < 4; ++q) v_a[0][q] = at3[2][q][re[2][q]];
        __builtin_amdgcn_sched_barrier(0);
        d2u b1[NP];
#pragma unroll
        for (int q = 0; q < NP; ++q) b1[q] = v_b[q], v_b[q] = b0[q];
        store(Any{}, a0, 0, 0);
#pragma unroll
        for (int q = 0; q < NP; ++q) v_b[q] = b1[q];
    }
    __syncthreads();
    // Iteration ch handles chunks ch + 1 (store) to ch + 5 (map): the mode is
    // known where all of them lie on one side of the band and the last chunk,
    // which is read again past the end, is whole.
    const bool whole = ((Ke - Kb) & (TBK - 1)) == 0;
    const int nb0 = max(0, min(r0 - Kb, Ke - Kb) / TBK);  // whole chunks below the band
    const int belowEnd = kTri == 2 ? 0 : (whole && nb0 == nch ? nch : max(0, nb0 - 5));
    const bool above = kTri != 1 && Kb + (nch - 1) * TBK >= r0 + TBM;  // the last chunk is
    const int aboveBegin = above ? max(0, (r0 + TBM - Kb + TBK - 1) / TBK - 1) : nch;
    const int aboveEnd = whole ? nch : max(0, (Ke - Kb) / TBK - 5);
    int ch = 0;
    auto run = [&](auto M, int end) {
        if ((ch & 1) && ch < end) body(M, X1{}, ch++);
        for (; ch + 1 < end; ch += 2) {
            body(M, X0{}, ch);
            body(M, X1{}, ch + 1);
        }
        if (ch < end) body(M, X0{}, ch++);
    };
    run(Below{}, belowEnd);
    run(Any{}, aboveBegin);
    run(Above{}, aboveEnd);
    run(Any{}, nch);
    mfma_drain();
}

template <int BN, class LDS>
__device__ __forceinline__ void gemm_task(LDS& L, const Task t, const BlockDesc d, double* __restrict__ Ap,
                          const double* __restrict__ Hp, const int64_t* __restrict__ cr2, const int32_t* __restrict__ rel)
{
    const int s = d.s, c = d.c;
    const int64_t ld = (int64_t)s + c;
    const int r0 = t.i0, n0 = t.j0;
    d4 acc[2][4] = {};
    gather_mma<BN, 0>(L, d, r0, n0, t.kb, t.ke, Ap, Hp + d.hoff, c, cr2, rel, acc);
    // transposed accumulation: stores and atomics run down the columns of X
    tile_epilogue_t<BN>(acc, [&](int i, int j, double v) {
        const int ii = r0 + i, jj = n0 + j;
        if (ii < c && jj < s) {
            double* x = Ap + d.poff + s + ii + (int64_t)jj * ld;
            if (t.flags & 1) unsafeAtomicAdd(x, -v); else *x = -v;
        }
    });
}

__global__ __launch_bounds__(kThreads, 2) void k_gemm(const Task* __restrict__ tasks, const BlockDesc* __restrict__ blk,
                                                   double* __restrict__ Ap, const double* __restrict__ Hp,
                                                   const int64_t* __restrict__ cr2,
                                                   const int32_t* __restrict__ rel)
{
    __shared__ GatherLds L;
    const Task t = tasks[blockIdx.x];
    const BlockDesc d = blk[t.b];
#define SELINV_CALL(BN) gemm_task<BN>(L, t, d, Ap, Hp, cr2, rel)
    SELINV_BN_DISPATCH(t.bn, SELINV_CALL)
#undef SELINV_CALL
}

// ---------------------------------------------------------------------------
// The dense counterpart of the gather loop: acc += A B over the contraction
// [Kb, Ke) for a 64 x BN tile, the same LDS rows and fragments, with operands
// that lie in column-major arrays and are read through buffer descriptors, so
// that a chunk's position is a scalar offset and no vector instruction forms
// an address.  An operand row r (of A, or a column of B) holds its
// contraction entry k at p[r + k ld] (kAlongK false: lanes run along the
// rows) or at p[k + r ld] (kAlongK true: lanes take pairs along k).
//  * Rows past the operand's end read what follows in the array; their
//    products are never stored.
//  * Contraction entries past Ke: operands along the rows must end there (the
//    descriptor then returns 0); with operands along k a ragged last chunk
//    reads the last entry again and A is masked.
// Loads are issued two chunks ahead.  kT: accumulate transposed.
// ---------------------------------------------------------------------------
struct Operand {
    __amdgpu_buffer_rsrc_t rsrc;
    const double* p;
    uint32_t ld8;  // bytes between columns
};

// p[0 .. count), columns ld apart
__device__ __forceinline__ Operand operand(const double* p, int64_t count, int64_t ld)
{
    return {__builtin_amdgcn_make_buffer_rsrc((void*)p, 0, (int)(uint32_t)(max(count, (int64_t)0) * 8), 0x00020000), p,
            (uint32_t)(ld * 8)};
}

__device__ __forceinline__ double buffer_f64(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff)
{
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, (int)voff, (int)soff, 0));
}

// One operand of NR rows: what a thread loads of a chunk, and where it goes
template <int NR, bool kAlongK>
struct DenseLoader {
    static constexpr int NQ = kAlongK ? (NR >= 32 ? NR / 32 : 1) : NR / 16;  // loads per thread
    static constexpr int KS = kAlongK ? 0 : 16 / NQ;                         // k step between them
    static constexpr int NV = kAlongK ? 2 * NQ : NQ;                         // values
    Operand o;
    uint32_t voff;
    int wpart, kp, wr[kAlongK ? 2 : NQ];
    bool on;

    __device__ __forceinline__ DenseLoader(const Operand& op, int wave) : o(op)
    {
        const int tid = threadIdx.x, lane = tid & 63;
        if constexpr (kAlongK) {
            kp = tid & 7;
            const int row = tid >> 3;
            voff = (uint32_t)row * o.ld8 + (uint32_t)kp * 16u;
            wr[0] = lds_at(row, 2 * kp);
            wr[1] = lds_at(row, 2 * kp + 1);
            on = NR >= 32 || wave < 2;
            wpart = 0;
        } else {
            constexpr int RW = NR < 64 ? NR : 64;  // rows a wave covers
            const int row = NR == 128 ? (wave & 1) * 64 + lane : lane % RW;
            const int kl = lane / RW;  // k within the wave
            wpart = NR == 128 ? wave >> 1 : wave * (64 / RW);
            voff = (uint32_t)row * 8u + (uint32_t)kl * o.ld8;
#pragma unroll
            for (int q = 0; q < NQ; ++q) wr[q] = lds_at(row, q * KS + wpart + kl);
            kp = 0;
            on = true;
        }
    }
    // the chunk at k0; ragged: it passes Ke (along k only)
    __device__ __forceinline__ void load(double (&v)[NV], int k0, bool ragged, int Ke) const
    {
        if constexpr (kAlongK) {
            if (!ragged) {
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    const d2u x = __builtin_bit_cast(
                        d2u, __builtin_amdgcn_raw_buffer_load_b128(o.rsrc, (int)(voff + q * 32 * o.ld8), k0 * 8, 0));
                    v[2 * q] = x.x;
                    v[2 * q + 1] = x.y;
                }
            } else {
                const int e = Ke - 1 - k0, x0 = (min(2 * kp, e) - 2 * kp) * 8, x1 = (min(2 * kp + 1, e) - 2 * kp) * 8;
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    v[2 * q] = buffer_f64(o.rsrc, voff + q * 32 * o.ld8 + k0 * 8 + x0, 0);
                    v[2 * q + 1] = buffer_f64(o.rsrc, voff + q * 32 * o.ld8 + k0 * 8 + x1, 0);
                }
            }
        } else {
#pragma unroll
            for (int q = 0; q < NQ; ++q) v[q] = buffer_f64(o.rsrc, voff, (uint32_t)(k0 + q * KS + wpart) * o.ld8);
        }
    }
    // mask: zero the entries past Ke (A of a ragged chunk along k)
    __device__ __forceinline__ void store(char* lds, const double (&v)[NV], int k0, bool mask, int Ke) const
    {
        if constexpr (kAlongK) {
            if (on) {
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    d2 x = {v[2 * q], v[2 * q + 1]};
                    if (mask) {
                        x.x = k0 + 2 * kp < Ke ? x.x : 0.0;
                        x.y = k0 + 2 * kp + 1 < Ke ? x.y : 0.0;
                    }
                    *reinterpret_cast<double*>(lds + wr[0] + q * 32 * kGatherRow) = x.x;
                    *reinterpret_cast<double*>(lds + wr[1] + q * 32 * kGatherRow) = x.y;
                }
            }
        } else {
#pragma unroll
            for (int q = 0; q < NQ; ++q) *reinterpret_cast<double*>(lds + wr[q]) = v[q];
        }
    }
};

template <int BN, bool kAk, bool kBk, bool kT, class LDS, class FH>
__device__ __forceinline__ void dense_mma(LDS& L, const Operand& opA, const Operand& opB, int Kb, int Ke,
                                          d4 (&acc)[2][4], FH afterPrologue)
{
    using SH = TileShape<BN>;
    static_assert(sizeof(L.B[0]) >= BN * kGatherRow, "the LDS tile holds BN columns");
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int wm0 = (wave % SH::WM) * (TBM / SH::WM), wn0 = (wave / SH::WM) * (BN / SH::WN);
    const int nch = Ke > Kb ? (Ke - Kb + TBK - 1) / TBK : 0;
    const DenseLoader<TBM, kAk> la(opA, wave);
    const DenseLoader<BN, kBk> lb(opB, wave);
    using LA = DenseLoader<TBM, kAk>;
    using LB = DenseLoader<BN, kBk>;
    double va[2][LA::NV], vb[2][LB::NV];  // by the chunk's parity
    auto k_of = [&](int ch) { return Kb + min(ch, nch - 1) * TBK; };
    auto load = [&](double (&a)[LA::NV], double (&b)[LB::NV], int ch) {
        const int k0 = k_of(ch);
        const bool ragged = (kAk || kBk) && k0 + TBK > Ke;
        la.load(a, k0, ragged, Ke);
        lb.load(b, k0, ragged, Ke);
    };
    auto store = [&](const double (&a)[LA::NV], const double (&b)[LB::NV], int ch, int buf) {
        const int k0 = k_of(ch);
        la.store(L.A[buf], a, k0, kAk && k0 + TBK > Ke, Ke);
        lb.store(L.B[buf], b, k0, false, Ke);
    };
    const int f0 = lds_at(lane & 15, lane >> 4), f1 = lds_at(lane & 15, 8 + (lane >> 4));
    if (nch > 0) {
        double a0[LA::NV], b0[LB::NV];
        load(a0, b0, 0);
        __builtin_amdgcn_sched_barrier(0);
        load(va[1], vb[1], 1);
        __builtin_amdgcn_sched_barrier(0);
        load(va[0], vb[0], 2);
        __builtin_amdgcn_sched_barrier(0);
        store(a0, b0, 0, 0);
    }
    afterPrologue();  // loads of the caller's own that may run under the main loop
    __syncthreads();
    auto body = [&](auto X, int ch) {  // X: the parity of ch
        constexpr int buf = decltype(X)::value;
        const char *A = L.A[buf] + wm0 * kGatherRow, *B = L.B[buf] + wn0 * kGatherRow;
        d2 a[SH::MT], b[SH::NT];
        auto frags = [&](int f) {
#pragma unroll
            for (int mt = 0; mt < SH::MT; ++mt) a[mt] = *reinterpret_cast<const d2*>(A + f + mt * 16 * kGatherRow);
#pragma unroll
            for (int nt = 0; nt < SH::NT; ++nt) b[nt] = *reinterpret_cast<const d2*>(B + f + nt * 16 * kGatherRow);
        };
        auto products = [&]() {
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int mt = 0; mt < SH::MT; ++mt)
#pragma unroll
                    for (int nt = 0; nt < SH::NT; ++nt)
                        acc[mt][nt] = kT ? mfma(b[nt][h], a[mt][h], acc[mt][nt]) : mfma(a[mt][h], b[nt][h], acc[mt][nt]);
        };
        frags(f0);
        store(va[buf ^ 1], vb[buf ^ 1], ch + 1, buf ^ 1);
        load(va[buf ^ 1], vb[buf ^ 1], ch + 3);
        __builtin_amdgcn_sched_barrier(0);
        products();
        frags(f1);
        products();
        __syncthreads();
    };
    int ch = 0;
    for (; ch + 1 < nch; ch += 2) {
        body(std::integral_constant<int, 0>{}, ch);
        body(std::integral_constant<int, 1>{}, ch + 1);
    }
    if (ch < nch) body(std::integral_constant<int, 0>{}, ch);
    mfma_drain();
}

// ---------------------------------------------------------------------------
// Factor panel (Algorithm 1 step 2, fused into the factorization):
// L_hat(C,B) = F(C,B) T for rows [i0, i0+64), columns [j0, j0+BN).
// ---------------------------------------------------------------------------
// L_hat(i, j) = sum over k of F(i, k) T(j, k): T is symmetric, so both
// operands lie along their rows
template <int BN, class LDS>
__device__ __forceinline__ void panel_product(LDS& L, const Task& t, const BlockDesc& d, const double* F,
                                              const double* T, d4 (&acc)[2][4])
{
    const int s = d.s, c = d.c;
    const int64_t ld = (int64_t)s + c;
    dense_mma<BN, false, false, true>(L, operand(F + t.i0, (int64_t)(s - 1) * ld + c - t.i0, ld),
                                      operand(T + t.j0, (int64_t)s * s - t.j0, s), 0, s, acc, [] {});
}

template <int BN, class LDS>
__device__ __forceinline__ void panel_task(LDS& L, const Task t, const BlockDesc d, const double* __restrict__ Lp,
                           double* __restrict__ Hp, const double* __restrict__ Tp)
{
    const int s = d.s, c = d.c;
    const int r0 = t.i0, n0 = t.j0;
    d4 acc[2][4] = {};
    panel_product<BN>(L, t, d, Lp + d.poff + s, Tp + d.woff, acc);
    tile_epilogue_t<BN>(acc, [&](int i, int j, double v) {
        const int ii = r0 + i, jj = n0 + j;
        if (ii < c && jj < s) Hp[d.hoff + ii + (int64_t)jj * c] = v;
    });
}

__global__ __launch_bounds__(kThreads) void k_panel(const Task* __restrict__ tasks,
                                                    const BlockDesc* __restrict__ blk, const double* __restrict__ Lp,
                                                    double* __restrict__ Hp, const double* __restrict__ Tp)
{
    __shared__ GatherLds L;
    const Task t = tasks[blockIdx.x];
    const BlockDesc d = blk[t.b];
#define SELINV_CALL(BN) panel_task<BN>(L, t, d, Lp, Hp, Tp)
    SELINV_BN_DISPATCH(t.bn, SELINV_CALL)
#undef SELINV_CALL
}

// ---------------------------------------------------------------------------
// Levels of few tiles, where a tile's time is its latency: one 16 x 16 tile
// per wave, with every operand load of the contraction (s <= kDeepK) in
// flight at once, straight into MFMA form; no LDS and no barrier.  Rows ra..
// of a and rb.. of b (entry k of row r at p[r + k ld], 0 past the
// contraction); element (g + 4 v, m) in register v.  `under` runs between
// the loads and the products.  With a 64 x 64 tile per work-group, its chunks
// through LDS (4 us on the matrix unit of one CU at s = 128, and eight
// barriers), the panel and Schur launches of a 301 x 257 grid took 8.2 and
// 9.3 us on average, now 5.4 and 6.0; of a 40^3 grid 12.2 and 11.2, now 8.0
// and 8.9.
// ---------------------------------------------------------------------------
template <int NS, class AF>
__device__ __forceinline__ d4 wave_mma_n(const Operand& a, int ra, const Operand& b, int rb, AF& under)
{
    const int lane = threadIdx.x & 63, m = lane & 15, g = lane >> 4;
    double x[NS], y[NS];
#pragma unroll
    for (int t = 0; t < NS; ++t) {
        x[t] = buffer_f64(a.rsrc, (uint32_t)(ra + m) * 8u + (uint32_t)(4 * t + g) * a.ld8, 0);
        y[t] = buffer_f64(b.rsrc, (uint32_t)(rb + m) * 8u + (uint32_t)(4 * t + g) * b.ld8, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    under();
    d4 acc = {0, 0, 0, 0};
#pragma unroll
    for (int t = 0; t < NS; ++t) acc = mfma(x[t], y[t], acc);
    mfma_drain();
    return acc;
}
template <class AF>
__device__ __forceinline__ d4 wave_mma(const Operand& a, int ra, const Operand& b, int rb, int s, AF under)
{
    if (s <= 16) return wave_mma_n<4>(a, ra, b, rb, under);
    if (s <= 32) return wave_mma_n<8>(a, ra, b, rb, under);
    if (s <= 64) return wave_mma_n<16>(a, ra, b, rb, under);
    return wave_mma_n<kDeepK / 4>(a, ra, b, rb, under);
}

// four work-groups per task, each 16 columns; a wave 16 rows
__global__ __launch_bounds__(kThreads, 2) void k_panel_few(const Task* __restrict__ tasks,
                                                           const BlockDesc* __restrict__ blk,
                                                           const double* __restrict__ Lp, double* __restrict__ Hp,
                                                           const double* __restrict__ Tp)
{
    const Task t = tasks[blockIdx.x >> 2];
    const BlockDesc d = blk[t.b];
    const int s = d.s, c = d.c, lane = threadIdx.x & 63, jq = 16 * (blockIdx.x & 3);
    const int i0 = t.i0 + 16 * __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), j0 = t.j0 + jq;
    if (i0 >= c || j0 >= s || jq >= t.bn) return;
    const int64_t ld = (int64_t)s + c;
    const d4 acc = wave_mma(operand(Tp + d.woff, (int64_t)s * s, s), j0,
                            operand(Lp + d.poff + s, (int64_t)(s - 1) * ld + c, ld), i0, s, [] {});
    const int i = i0 + (lane & 15);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int j = j0 + (lane >> 4) + 4 * v;
        if (i < c && j < s) Hp[d.hoff + i + (int64_t)j * c] = acc[v];
    }
}

// ---------------------------------------------------------------------------
// Factor, Schur update: F(C,C) -= L(C,B) D_B L(C,B)^T = L_hat(C,B) F(C,B)^T,
// lower half, tile rows [i0, i0+64) x columns [k0, k0+64), added into the
// ancestor panels through the block index maps.  FP64 atomics where sibling
// blocks of the level may update the same ancestor entry; plain
// read-modify-write for blocks the host found exclusive (flags bit 2).
//
// The tile is formed transposed, as F(k0.., :) L_hat(i0.., :)^T, so that the
// sixteen lanes of an MFMA output row hold sixteen consecutive rows ii of one
// target column kk: rows of one ancestor column are contiguous in its panel,
// so each group of sixteen lanes updates one run of memory instead of
// sixteen columns.  The scatter targets do not depend on the product: their
// (cbase, rbase) pairs are loaded before the main loop and the rel entries
// right after its prologue, so the epilogue issues only the updates.
//
// Bounds at 64^3: the products (padding included) 5.7 ms of MFMA, the
// read-modify-write of the targets 27 GB, 6 ms at the copy rate; without the
// update of the targets the kernel takes 8.6 ms.  With about ten vector
// instructions per MFMA (addresses and masks, which share the SIMD with FP64
// MFMAs) it took 16.0 ms; the loop of dense_mma has none: 15.5, and 14.5
// with three work-groups on a CU (four spill: 18.8).
// ---------------------------------------------------------------------------
// The scatter of a 64 x 64 tile of updates: product(acc, prefetch) forms the
// tile (target columns k0.. along its rows, rows i0.. along its columns) and
// calls prefetch once its own first loads are issued; value(ii, kk, x) is
// what entry (ii, kk) of C x C adds to its place in the arena Z.
template <class FP, class FV>
__device__ __forceinline__ void scatter_update(const Task& t, const BlockDesc& d, double* __restrict__ Z,
                                               const int64_t* __restrict__ cr2, const int32_t* __restrict__ rel,
                                               FP product, FV value)
{
    using SH = TileShape<64>;
    const int c = d.c, i0 = t.i0, k0c = t.j0;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm0 = (wave % SH::WM) * (TBM / SH::WM), wn0 = (wave / SH::WM) * (64 / SH::WN);
    // this thread's outputs (mt, nt, v): target column kk = k0 + wm0 + 16 mt +
    // lane / 16 + 4 v, row ii = i0 + wn0 + 16 nt + lane % 16; past C's end and
    // above the diagonal (never stored) the map is read at a valid place
    auto col_of = [&](int mt, int v) { return k0c + wm0 + mt * 16 + (lane >> 4) + 4 * v; };
    auto row_of = [&](int nt) { return i0 + wn0 + nt * 16 + (lane & 15); };
    // a tile strictly below the diagonal and inside C has every entry live
    const bool full = i0 > k0c && i0 + TBM <= c;
    i64x2 cr[SH::MT][4];  // (cbase, rbase) of the column
#pragma unroll
    for (int mt = 0; mt < SH::MT; ++mt)
#pragma unroll
        for (int v = 0; v < 4; ++v)
            cr[mt][v] = *reinterpret_cast<const i64x2*>(cr2 + 2 * (d.coff + min(col_of(mt, v), c - 1)));
    uint32_t ro[SH::MT][SH::NT][4];
    auto prefetch = [&]() {
        if (full) {
#pragma unroll
            for (int nt = 0; nt < SH::NT; ++nt) {
                const int32_t* rq = rel + row_of(nt);
#pragma unroll
                for (int mt = 0; mt < SH::MT; ++mt)
#pragma unroll
                    for (int v = 0; v < 4; ++v) ro[mt][nt][v] = (uint32_t)rq[cr[mt][v].y];
            }
        } else {
#pragma unroll
            for (int mt = 0; mt < SH::MT; ++mt)
#pragma unroll
                for (int nt = 0; nt < SH::NT; ++nt)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int ii = min(max(row_of(nt), col_of(mt, v)), c - 1);
                        ro[mt][nt][v] = (uint32_t)rel[cr[mt][v].y + ii];
                    }
        }
    };
    d4 acc[2][4] = {};
    product(acc, prefetch);
    double* base[SH::MT][4];
#pragma unroll
    for (int mt = 0; mt < SH::MT; ++mt)
#pragma unroll
        for (int v = 0; v < 4; ++v) base[mt][v] = Z + cr[mt][v].x;
    auto target = [&](int mt, int nt, int v) { return base[mt][v] + ro[mt][nt][v]; };
    auto live = [&](int mt, int nt, int v) {
        const int ii = row_of(nt), kk = col_of(mt, v);
        return ii < c && ii >= kk;  // and so kk < c
    };
    // full tiles: no per-entry branches, which would put a wait on all
    // outstanding memory operations in front of every store
    if (t.flags & 4) {
        // no other block of the level updates these entries: plain
        // read-modify-write, all reads issued before the first write (the
        // targets of one thread are distinct entries; those of entries not
        // live are read, not written)
        double old[SH::MT][SH::NT][4];
#pragma unroll
        for (int mt = 0; mt < SH::MT; ++mt)
#pragma unroll
            for (int nt = 0; nt < SH::NT; ++nt)
#pragma unroll
                for (int v = 0; v < 4; ++v) old[mt][nt][v] = *target(mt, nt, v);
        if (full) {
#pragma unroll
            for (int mt = 0; mt < SH::MT; ++mt)
#pragma unroll
                for (int nt = 0; nt < SH::NT; ++nt)
#pragma unroll
                    for (int v = 0; v < 4; ++v) *target(mt, nt, v) = old[mt][nt][v] + value(row_of(nt), col_of(mt, v), acc[mt][nt][v]);
        } else {
#pragma unroll
            for (int mt = 0; mt < SH::MT; ++mt)
#pragma unroll
                for (int nt = 0; nt < SH::NT; ++nt)
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        if (live(mt, nt, v)) *target(mt, nt, v) = old[mt][nt][v] + value(row_of(nt), col_of(mt, v), acc[mt][nt][v]);
        }
    } else if (full) {
#pragma unroll
        for (int mt = 0; mt < SH::MT; ++mt)
#pragma unroll
            for (int nt = 0; nt < SH::NT; ++nt)
#pragma unroll
                for (int v = 0; v < 4; ++v) unsafeAtomicAdd(target(mt, nt, v), value(row_of(nt), col_of(mt, v), acc[mt][nt][v]));
    } else {
#pragma unroll
        for (int mt = 0; mt < SH::MT; ++mt)
#pragma unroll
            for (int nt = 0; nt < SH::NT; ++nt)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (live(mt, nt, v)) unsafeAtomicAdd(target(mt, nt, v), value(row_of(nt), col_of(mt, v), acc[mt][nt][v]));
    }
}

template <class LDS>
__device__ __forceinline__ void schur_task(LDS& L, const Task t, const BlockDesc d, double* __restrict__ Lp,
                                           const double* __restrict__ Hp, const int64_t* __restrict__ cr2,
                                           const int32_t* __restrict__ rel)
{
    const int s = d.s, c = d.c;
    const int64_t ld = (int64_t)s + c;
    const double *F = Lp + d.poff + s + t.j0, *H = Hp + d.hoff + t.i0;
    scatter_update(
        t, d, Lp, cr2, rel,
        [&](d4(&acc)[2][4], auto prefetch) {
            dense_mma<64, false, false, false>(L, operand(F, (int64_t)(s - 1) * ld + c - t.j0, ld),
                                               operand(H, (int64_t)s * c - t.i0, c), 0, s, acc, prefetch);
        },
        [](int, int, double x) { return -x; });
}

__global__ __launch_bounds__(kThreads, 3) void k_schur(const Task* __restrict__ tasks,
                                                    const BlockDesc* __restrict__ blk, double* __restrict__ Lp,
                                                    const double* __restrict__ Hp,
                                                    const int64_t* __restrict__ cr2,
                                                    const int32_t* __restrict__ rel)
{
    __shared__ GatherLdsN<64> L;
    const Task t = tasks[blockIdx.x];
    schur_task(L, t, blk[t.b], Lp, Hp, cr2, rel);
}

// colour groups of few tiles: four work-groups per task (a 32 x 32 quarter
// each), a wave per 16 x 16 tile
__global__ __launch_bounds__(kThreads, 2) void k_schur_few(const Task* __restrict__ tasks,
                                                           const BlockDesc* __restrict__ blk, double* __restrict__ Lp,
                                                           const double* __restrict__ Hp,
                                                           const int64_t* __restrict__ cr2,
                                                           const int32_t* __restrict__ rel)
{
    const Task t = tasks[blockIdx.x >> 2];
    const BlockDesc d = blk[t.b];
    const int s = d.s, c = d.c, q = blockIdx.x & 3, lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int i0 = t.i0 + 32 * (q >> 1) + 16 * (wave >> 1), k0 = t.j0 + 32 * (q & 1) + 16 * (wave & 1);
    if (i0 >= c || k0 >= c || i0 + 15 < k0) return;
    const int64_t ld = (int64_t)s + c;
    const int row = i0 + (lane & 15);
    const bool alone = t.flags & 4;  // no other block of the level updates these entries
    auto col_of = [&](int v) { return k0 + (lane >> 4) + 4 * v; };
    i64x2 cr[4];
    uint32_t ro[4];
    double old[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) cr[v] = *reinterpret_cast<const i64x2*>(cr2 + 2 * (d.coff + min(col_of(v), c - 1)));
    __builtin_amdgcn_sched_barrier(0);
    const d4 acc = wave_mma(operand(Lp + d.poff + s, (int64_t)(s - 1) * ld + c, ld), k0,
                            operand(Hp + d.hoff, (int64_t)s * c, c), i0, s, [&] {
#pragma unroll
                                for (int v = 0; v < 4; ++v)
                                    ro[v] = (uint32_t)rel[cr[v].y + min(max(row, col_of(v)), c - 1)];
                                if (alone) {
#pragma unroll
                                    for (int v = 0; v < 4; ++v) old[v] = Lp[cr[v].x + ro[v]];
                                }
                            });
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        if (row >= c || row < col_of(v)) continue;
        double* to = Lp + cr[v].x + ro[v];
        if (alone) *to = old[v] - acc[v];
        else unsafeAtomicAdd(to, -acc[v]);
    }
}

// ---------------------------------------------------------------------------
// Selected inversion, step 4 + symmetrisation, one pair of 32 x 32 tiles
// (I, J), I >= J, of the diagonal block per work-group:
//   Y(I,J) = T(I,J) - L_hat(:,I)^T X(:,J),  Y(J,I) = T(J,I) - L_hat(:,J)^T X(:,I)
//   Ainv(I,J) = Ainv(J,I)^T = (Y(I,J) + Y(J,I)^T) / 2.
// ---------------------------------------------------------------------------
constexpr int SDT = 32;

struct SdiagLds {
    double LI[16][SDT + 1], LJ[16][SDT + 1], XI[16][SDT + 1], XJ[16][SDT + 1];
    double Sx[SDT][SDT + 1];
};

__device__ __forceinline__ void sdiag_task(SdiagLds& S, const Task t, const BlockDesc d, double* __restrict__ Ap,
                           const double* __restrict__ Hp, const double* __restrict__ Tp)
{
    auto& LI = S.LI;
    auto& LJ = S.LJ;
    auto& XI = S.XI;
    auto& XJ = S.XJ;
    auto& Sx = S.Sx;
    const int s = d.s, c = d.c;
    const int64_t ld = (int64_t)s + c;
    const int I0 = t.i0, J0 = t.j0;
    double* A = Ap + d.poff;
    const double* H = Hp + d.hoff;
    const double* T = Tp + d.woff;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int fm = (wave & 1) * 16, fn = (wave >> 1) * 16;
    d4 accIJ = {0, 0, 0, 0}, accJI = {0, 0, 0, 0};
    // Branch-free body: a diagonal tile (I == J) simply recomputes its own
    // product as the partner.  Control flow between an FP64 MFMA and a read
    // of its accumulator let the compiler place the read too early.
    const int rend = min(c, t.ke);
    for (int r0 = t.kb; r0 < rend; r0 += 16) {
#pragma unroll
        for (int q = 0; q < (16 * SDT) / kThreads; ++q) {
            const int e = threadIdx.x + q * kThreads;
            const int kk = e & 15, col = e >> 4;
            const int r = r0 + kk;
            const bool okr = r < rend;
            const int ci = I0 + col, cj = J0 + col;
            const double li = (okr && ci < s) ? H[r + (int64_t)ci * c] : 0.0;
            const double lj = (okr && cj < s) ? H[r + (int64_t)cj * c] : 0.0;
            const double xi = (okr && ci < s) ? A[s + r + ci * ld] : 0.0;
            const double xj = (okr && cj < s) ? A[s + r + cj * ld] : 0.0;
            LI[kk][col] = li;
            LJ[kk][col] = lj;
            XI[kk][col] = xi;
            XJ[kk][col] = xj;
        }
        __syncthreads();
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const int kr = ks * 4 + (lane >> 4);
            accIJ = mfma(LI[kr][fm + (lane & 15)], XJ[kr][fn + (lane & 15)], accIJ);
            accJI = mfma(LJ[kr][fm + (lane & 15)], XI[kr][fn + (lane & 15)], accJI);
        }
        __syncthreads();
    }
    mfma_drain();
    // Only the lower triangle of Ainv(B,B) is kept (it is all that the
    // gathers and the export read).  A whole contraction writes
    // (Y(I,J) + Y(J,I)^T)/2 there; a split piece adds its share
    // -(P(I,J) + P(J,I)^T)/2 to the T written beforehand (the average is
    // linear, so the pieces may arrive in any order).
    const bool split = t.flags & 1;
    // Sx[b][a] = element (a, b) of the partner tile
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int i = fm + (lane >> 4) + 4 * v, j = fn + (lane & 15);
        const double tji = (!split && J0 + i < s && I0 + j < s) ? T[(J0 + i) + (I0 + j) * s] : 0.0;
        Sx[j][i] = tji - accJI[v];
    }
    __syncthreads();
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int i = fm + (lane >> 4) + 4 * v, j = fn + (lane & 15);
        const int gi = I0 + i, gj = J0 + j;
        if (gi < s && gj < s && gi >= gj) {
            if (split) {
                unsafeAtomicAdd(A + gi + gj * ld, 0.5 * (Sx[i][j] - accIJ[v]));
            } else {
                A[gi + gj * ld] = 0.5 * ((T[gi + gj * s] - accIJ[v]) + Sx[i][j]);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Selected inversion, step 4 + symmetrisation, per-level path, on 64 x 64
// tiles of the diagonal block, with P = L_hat^T X (so Y = T - P) and
// Ainv(i,j) = T(i,j) - (P(i,j) + P(j,i)) / 2 for i >= j:
//  * diagonal tile I: P(I,I) on the pipelined MFMA tile; the transpose
//    reaches the thread holding P(i,j) through LDS; stored as T - (P + P^T)/2,
//    or with a split contraction added as -(P + P^T)/2 (atomics) to the T
//    written beforehand;
//  * tile (I,J), I > J: two tasks, one per half, each adding -1/2 of its
//    product to Ainv(I,J) with atomics (T written beforehand):
//    L_hat(:,I)^T X(:,J) (flags bit 3 clear) and X(:,I)^T L_hat(:,J) =
//    P(J,I)^T (bit 3 set).  One product per task keeps the longest task of a
//    level short.
// Products accumulate transposed (lane l holds tile row l % 16), so stores
// and atomics run down the columns of the panel.
// ---------------------------------------------------------------------------
// the tile's operands, then the exchange of a diagonal tile's transpose
union SdiagLds64 {
    GatherLdsN<64> d;
    double S[TBM][TBM + 1];
};

__device__ __forceinline__ void sdiag64_task(SdiagLds64& L, const Task t, const BlockDesc d, double* __restrict__ Ap,
                                             const double* __restrict__ Hp, const double* __restrict__ Tp)
{
    using SH = TileShape<64>;
    const int s = d.s, c = d.c;
    const int64_t ld = (int64_t)s + c;
    const int I0 = t.i0, J0 = t.j0;
    const int kb = t.kb, ke = min(t.ke, c);
    const double* H = Hp + d.hoff;       // L_hat(r, j) at H[r + j c]
    const double* X = Ap + d.poff + s;   // X(r, j) at X[r + j ld]
    const bool diag = I0 == J0, second = t.flags & 8;
    // A(i, r) = U(r, I0 + i), B(r, j) = V(r, J0 + j): both contiguous in r
    const double* U = second ? X : H;
    const double* V = second ? H : X;
    const int64_t ldu = second ? ld : c, ldv = second ? c : ld;
    d4 acc[2][4] = {};
    dense_mma<64, true, true, true>(L.d, operand(U + (int64_t)I0 * ldu, (int64_t)(s - 1 - I0) * ldu + c, ldu),
                                    operand(V + (int64_t)J0 * ldv, (int64_t)(s - 1 - J0) * ldv + c, ldv), kb, ke, acc,
                                    [] {});
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm0 = (wave % SH::WM) * (TBM / SH::WM), wn0 = (wave / SH::WM) * (64 / SH::WN);
    const double* T = Tp + d.woff;
    double* A = Ap + d.poff;
    if (!diag) {
#pragma unroll
        for (int mt = 0; mt < SH::MT; ++mt)
#pragma unroll
            for (int nt = 0; nt < SH::NT; ++nt)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int gi = I0 + wm0 + mt * 16 + (lane & 15), gj = J0 + wn0 + nt * 16 + (lane >> 4) + 4 * v;
                    if (gi < s && gj < s) {
                        double* a = A + gi + (int64_t)gj * ld;
                        if (t.flags & 16) *a -= 0.5 * acc[mt][nt][v];  // the only writer of its launch
                        else unsafeAtomicAdd(a, -0.5 * acc[mt][nt][v]);
                    }
                }
        return;
    }
    // diagonal tile: the loop ended on a barrier, the LDS tile is free
    double(*S)[TBM + 1] = L.S;
#pragma unroll
    for (int mt = 0; mt < SH::MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < SH::NT; ++nt)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int i = wm0 + mt * 16 + (lane & 15), j = wn0 + nt * 16 + (lane >> 4) + 4 * v;
                S[j][i] = acc[mt][nt][v];  // S[a][b] = P(b, a)
            }
    __syncthreads();
    const bool split = t.flags & 1;
#pragma unroll
    for (int mt = 0; mt < SH::MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < SH::NT; ++nt)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int i = wm0 + mt * 16 + (lane & 15), j = wn0 + nt * 16 + (lane >> 4) + 4 * v;
                const int gi = I0 + i, gj = J0 + j;
                if (gi < s && gj < s && gi >= gj) {
                    const double p = 0.5 * (acc[mt][nt][v] + S[i][j]);
                    if (split) unsafeAtomicAdd(A + gi + (int64_t)gj * ld, -p);
                    else A[gi + (int64_t)gj * ld] = T[gi + (int64_t)gj * s] - p;
                }
            }
}

__global__ __launch_bounds__(kThreads) void k_sdiag64(const Task* __restrict__ tasks,
                                                      const BlockDesc* __restrict__ blk, double* __restrict__ Ap,
                                                      const double* __restrict__ Hp, const double* __restrict__ Tp)
{
    __shared__ SdiagLds64 L;
    const Task t = tasks[blockIdx.x];
    sdiag64_task(L, t, blk[t.b], Ap, Hp, Tp);
}

// ---------------------------------------------------------------------------
// Factor, diagonal block wider than the kernels below hold (s > 128, only with
// exec_cap above 128), on global memory: right-looking LDL^T without
// pivoting in place of F_BB, then W = L_BB^{-1} column by column (forward
// substitution, one thread a column) and T = W^T D^{-1} W.  A pivot that is
// zero, not finite, or (require_spd) not positive is latched as the smallest
// failing column.
// ---------------------------------------------------------------------------
__device__ void ldlt_global(const BlockDesc d, double* __restrict__ Lp, double* __restrict__ Wp,
                            double* __restrict__ Tp, unsigned long long* __restrict__ status, int require_spd)
{
    const int s = d.s;
    const int64_t ld = (int64_t)d.s + d.c;
    double* F = Lp + d.poff;
    double* W = Wp + d.woff;
    double* T = Tp + d.woff;
    const int tid = threadIdx.x, nthr = blockDim.x;
    for (int j = 0; j < s; ++j) {
        __syncthreads();
        const double dj = F[j + j * ld];
        const bool ok = isfinite(dj) && dj != 0.0 && (!require_spd || dj > 0.0);
        if (!ok && tid == 0) atomicMin(status, (unsigned long long)(d.first + j));
        const int m = s - j - 1;
        for (int e = tid; e < m * m; e += nthr) {
            const int ii = e % m, kk = e / m;
            if (ii >= kk) {
                const int i = j + 1 + ii, k = j + 1 + kk;
                F[i + k * ld] -= F[i + j * ld] * F[k + j * ld] / dj;
            }
        }
        __syncthreads();
        for (int i = j + 1 + tid; i < s; i += nthr) F[i + j * ld] /= dj;
    }
    __syncthreads();
    for (int j = tid; j < s; j += nthr) {
        for (int i = 0; i < j; ++i) W[i + j * s] = 0.0;
        W[j + j * s] = 1.0;
        for (int i = j + 1; i < s; ++i) {
            double v = 0.0;
            for (int k = j; k < i; ++k) v += F[i + k * ld] * W[k + j * s];
            W[i + j * s] = -v;
        }
    }
    __syncthreads();
    for (int e = tid; e < s * s; e += nthr) {
        const int i = e % s, j = e / s;
        const int m = i > j ? i : j;
        double v = 0.0;
        for (int k = m; k < s; ++k) v += W[k + i * s] * W[k + j * s] / F[k + k * ld];
        T[e] = v;
    }
}

// 1 / d: hardware reciprocal (within 2^-24) and two Newton steps, each of which
// squares the relative error
__device__ __forceinline__ double recip(double d)
{
    double inv = __builtin_amdgcn_rcp(d);
    inv = fma(inv, fma(-d, inv, 1.0), inv);
    inv = fma(inv, fma(-d, inv, 1.0), inv);
    return inv;
}

// ---------------------------------------------------------------------------
// Diagonal block, s <= 16 NB (NB = 2, 4, 8): L_BB, D and T = F_BB^{-1} by the
// symmetric sweep of one pivot after the other,
//   M(i, k) -= c_i c_k / d,  M(i, j) = M(j, i) = c_i / d,  M(j, j) = -1 / d
// (pivot j, c = M(:, j), d = c_j), after which M = -F_BB^{-1}, arranged by
// pivot blocks of 16 columns.  Block p is factored in one wave's registers
// (ldl16).  For every block row R, with C(R) = M(R, p), and C(p) = -I,
//   Y(R) = C(R) L_pp^{-T} by substitution, column after column, and
//   l(R) = Y(R) D_p^{-1}: what each pivot finds in the rows and its multipliers;
//   M(I, J) = M'(I, J) - l(I) Y(J)^T for every tile, with M' = M outside row
// and column p and 0 in them.  M's lower 16 x 16 tiles live in the registers of
// the waves that update them, by MFMA; a tile goes to LDS when its column is
// the next step's.
// These are the scalar sweep's operations in its order.  An explicit
// Q = M(p, p)^{-1} (C(R) Q for l(R) L_pp^{-1}) would square the condition
// number of the pivot block; and the pivot blocks have to be exactly
// symmetric, or L D L^T no longer gives F_BB back to rounding.  Largest error
// of T, relative, SPD of condition 1e8, 24 columns (median of 15): the scalar
// sweep 2.0e-10, this 2.3e-10, with Q 5e-6; Gaussian kernel of condition 5e7,
// 128 columns: 7.6e-10, 7.3e-10, no digit.
//
// What bounds it is the chain of s dependent pivots.  So wave 0 does nothing
// but that chain: it updates the next pivot block, factors it (the pivot column
// and row go between lanes by row broadcasts and row swaps, no LDS and no
// barrier) and publishes the factors, while the other waves update the tiles
// and write L_BB.  A block step has two barriers: first all waves form Y(R) and
// l(R) from the published tiles, then the updates run.  (With every tile in
// LDS, its reads and writes took longer than the chain: 33 us for 128 columns.)
// One block of 128 columns: 31.9 us (61 when each pivot's column went through
// LDS behind a barrier), of 64: 14.5 us (20; launch included).
//
// Rows and columns past s hold the identity and are not swept.
// ---------------------------------------------------------------------------
// doubles from row to row: of M's tiles, read and written 8 bytes a lane, and of
// C, N and the pivot block's factors, read 16 bytes a lane (every row aligned
// to that); either is free of bank conflicts
constexpr int kTilePad = 17, kDiagPad = 18;
template <int NB>
struct alignas(16) DiagLds {
    double M[NB * (NB + 1) / 2][16][kTilePad];  // published tile (I, J), I >= J, at I (I + 1) / 2 + J
    double C[16 * NB][kDiagPad];  // Y(R)
    double N[16 * NB][kDiagPad];  // -l(R)
    double Lb[2][16][kDiagPad];   // -L_pp below its diagonal, else 0
    double D[2][16], inv[2][16];  // D_p and its reciprocal
};

// Elimination of a symmetric 16 x 16 block, lane (m, g) holding row m, columns
// g + 4 v.  The part not yet eliminated stays symmetric to the last bit: an
// entry's update c_i c_k / d is formed as (c_i c_k) / d, the same for (k, i),
// and c_i is scaled by d's exponent beforehand so that the product neither
// overflows nor underflows where the update would not.  Rows from n on hold
// the identity and their pivots are skipped (by fours in ldl16).
//
// What bounds it is issue: a lone wave issues an instruction per 4 cycles
// (5 where it is 8 bytes long, 16 for a reciprocal, 8 for a row swap), and no
// result is later than that.

// X(., j): column j as pivot j finds it (d_j in row j), and what has been left
// of the rows above.  P is used up.
__device__ __forceinline__ void ldl16(double (&P)[4], double (&X)[4], const int g, const int n)
{
    double c = row_copy<0>(P[0]);  // column j in every lane (m, .)
    StaticFor<0, 4>::run([&](auto vc) {
        constexpr int vj = decltype(vc)::value;
        if (4 * vj >= n) return;  // uniform
        StaticFor<4 * vj, 4 * vj + 4>::run([&](auto jc) {
            constexpr int j = decltype(jc)::value, j1 = j < 15 ? j + 1 : 15;
            const double d = row_lane<j>(c), s = pow2_scale(d), r = recip3(d * s), u = c * s;
            // the next column, broadcast before its update
            const double next = row_copy<(j1 & 3)>(P[j1 >> 2]);
            const double cn = fma(-(u * row_lane<j1>(c)), r, next);
#pragma unroll
            for (int v = j1 >> 2; v < 4; ++v) P[v] = fma(-(u * row_lane<j>(P[v])), r, P[v]);
            X[vj] = g == (j & 3) ? c : X[vj];
            c = cn;
        });
    });
}

// P becomes its inverse; L: the multipliers (L_pp below the diagonal) and d_j
// in row j.  Symmetric Gauss-Jordan: row j is left unscaled until the end,
// which suffices where only the inverse's lower triangle is used.  Without the
// symmetry, L D L^T was off by 1e-12 of a Gaussian kernel of 16 columns and
// condition 5e7, now by 3e-16.
template <int NV>
__device__ __forceinline__ void gj16(double (&P)[NV], double (&L)[NV], const int m, const int g, const int n)
{
    double im = 1.0;  // 1 / d_m
    StaticFor<0, 4 * NV>::run([&](auto jc) {
        constexpr int j = decltype(jc)::value, gj = j & 3, vj = j >> 2;
        if (j >= n) return;  // uniform
        const double c = row_copy<gj>(P[vj]);
        const double d = row_lane<j>(c), s = pow2_scale(d), r = recip3(d * s), u = m == j ? 0.0 : c * s;
#pragma unroll
        for (int v = 0; v < NV; ++v) P[v] = fma(-(u * row_lane<j>(P[v])), r, P[v]);
        if (g == gj) {
            P[vj] = m == j ? 1.0 : -(u * r);
            L[vj] = m == j ? d : u * r;
        }
        im = m == j ? s * r : im;
    });
#pragma unroll
    for (int v = 0; v < NV; ++v) P[v] *= im;
}

// Y = C L^{-T} for a unit lower triangular L and 16 rows, lane (m, g) holding
// rows g + 4 v, column m: column j, final, leaves the columns right of it.
// lb: -L(m, j), 0 for m <= j.  Each step multiplies a value broadcast within
// the rows of 16 lanes in the instruction itself; four independent ones follow
// each other, which keeps the wait states between a write and its broadcast.
__device__ __forceinline__ void substitute16(double (&x)[4], const double (&lb)[16])
{
#define SELINV_FMAC(V, J) "v_fmac_f64_dpp %" #V ", %" #V ", %[l" #J "] row_newbcast:" #J " row_mask:0xf bank_mask:0xf\n\t"
#define SELINV_STEP(J) SELINV_FMAC(0, J) SELINV_FMAC(1, J) SELINV_FMAC(2, J) SELINV_FMAC(3, J)
    asm volatile("s_nop 1\n\t"
        SELINV_STEP(0) SELINV_STEP(1) SELINV_STEP(2) SELINV_STEP(3) SELINV_STEP(4)
        SELINV_STEP(5) SELINV_STEP(6) SELINV_STEP(7) SELINV_STEP(8) SELINV_STEP(9)
        SELINV_STEP(10) SELINV_STEP(11) SELINV_STEP(12) SELINV_STEP(13) SELINV_STEP(14)
        : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3])
        : [l0] "v"(lb[0]), [l1] "v"(lb[1]), [l2] "v"(lb[2]), [l3] "v"(lb[3]), [l4] "v"(lb[4]), [l5] "v"(lb[5]),
          [l6] "v"(lb[6]), [l7] "v"(lb[7]), [l8] "v"(lb[8]), [l9] "v"(lb[9]), [l10] "v"(lb[10]), [l11] "v"(lb[11]),
          [l12] "v"(lb[12]), [l13] "v"(lb[13]), [l14] "v"(lb[14]));
#undef SELINV_STEP
#undef SELINV_FMAC
}

// NW waves work on the block.  Lane (m, g) = (l % 16, l / 16) holds entry (m, g + 4 v) of a 16 x 16 block in
// register v: the form of both MFMA operands (k = g + 4 v in step v) and,
// with the product formed transposed, of its result.
template <int NB, int NW>
__device__ __forceinline__ void ldlt_blocks(const BlockDesc d, double* __restrict__ Lp, double* __restrict__ Tp,
                                            unsigned long long* __restrict__ status, int require_spd, DiagLds<NB>& S)
{
    // tile waves: all but wave 0, and but wave 4 of 8, which shares its SIMD
    // and writes L_BB.  Every wave substitutes rows, wave 0 one
    constexpr int NK = NW == 8 ? 6 : NW - 1;
    constexpr int NT = NB * (NB + 1) / 2, NL = (NT + NK - 1) / NK;
    constexpr int kRows = (NB - 1 + NW - 2) / (NW - 1);  // rows a wave substitutes, interleaved
    const int s = d.s, nb = (s + 15) >> 4;
    const int64_t ld = (int64_t)d.s + d.c;
    double* F = Lp + d.poff;
    double* T = Tp + d.woff;
    const int lane = threadIdx.x & 63, m = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const bool chain = wave == 0, tiles = wave > 0 && (NW < 8 || wave != 4);
    const int wk = wave - 1 - (NW == 8 && wave > 4);
    const bool lower = NW == 8 ? wave == 4 : tiles;
    const int l0 = NW == 8 ? 0 : wk, lstep = NW == 8 ? 1 : NK;
    auto tile = [](int I, int J) { return (int)((unsigned)(I * (I + 1)) >> 1) + J; };
    // tile (I, J) of index t, row by row: rows 1 .. 7 start at the bits set
    auto tile_of = [&](int t, int& I, int& J) {
        constexpr unsigned long long kStarts = 1ull << 1 | 1ull << 3 | 1ull << 6 | 1ull << 10 | 1ull << 15 |
                                               1ull << 21 | 1ull << 28;
        I = __builtin_popcountll(kStarts & ((2ull << t) - 1));
        J = t - tile(I, 0);
    };
    // factor the pivot block P of step p
    auto pivots = [&](int p, const d4& P) {
        const int buf = p & 1;
        double Q[4], C[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            Q[v] = P[v];
            C[v] = m == g + 4 * v ? 1.0 : 0.0;
        }
        ldl16(Q, C, g, s - 16 * p);
        double dm = C[0];
#pragma unroll
        for (int v = 1; v < 4; ++v) dm = m >> 2 == v ? C[v] : dm;
        const double sc = pow2_scale(dm), im = sc * recip3(dm * sc);
        if (g == (m & 3)) {
            S.D[buf][m] = dm;
            S.inv[buf][m] = im;
        }
        wave_sync();
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int k = g + 4 * v;
            S.Lb[buf][m][k] = m > k ? -C[v] * S.inv[buf][k] : 0.0;
        }
    };
    // F(i, j) of tile (I, J), the identity past s
    auto load_tile = [&](int I, int J) {
        d4 x;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int i = 16 * I + m, j = 16 * J + g + 4 * v;
            const int a = min(max(i, j), s - 1), b = min(min(i, j), s - 1);
            const double f = F[a + (int64_t)b * ld];
            x[v] = i < s && j < s ? f : (i == j ? 1.0 : 0.0);
        }
        return x;
    };
    d4 P = {0, 0, 0, 0};  // the chain's next pivot block
    // this wave's tiles, every NK-th
    const int nt = nb * (nb + 1) / 2;
    d4 x[NL];
    int I[NL], J[NL];
#pragma unroll
    for (int u = 0; u < NL; ++u) {
        tile_of(min(u * NK + wk, nt - 1), I[u], J[u]);
        if (tiles) x[u] = load_tile(I[u], J[u]);
    }
    if (chain) P = load_tile(0, 0);
    // step -1 only factors the first pivot block
    for (int p = -1; p < nb; ++p) {
        const int buf = p & 1;
        const bool more = p + 1 < nb;
        // Y(R) and -l(R), rows R = p + 1 (wave 0), p + 2, .. cyclically to p.
        // Lane (m, g) holds rows g + 4 v, column m, so that a column reaches
        // the lanes right of it by a broadcast within rows of 16 lanes.
        if (p >= 0 && wave < nb) {
            const int step = chain ? nb : NW - 1;
            int R[kRows];
            double x[kRows][4], lb[16];
#pragma unroll
            for (int j = 0; j < 16; j += 2) {
                const d2 q = *reinterpret_cast<const d2*>(&S.Lb[buf][m][j]);
                lb[j] = q.x;
                lb[j + 1] = q.y;
            }
            const double inv = S.inv[buf][m];
#pragma unroll
            for (int e = 0; e < kRows; ++e) {
                const int r = min(wave + e * step, nb - 1);
                R[e] = p + 1 + r < nb ? p + 1 + r : p + 1 + r - nb;
                const double* src = S.M[tile(max(R[e], p), min(R[e], p))][0];
                const int mk = R[e] > p ? 1 : kTilePad, gk = R[e] > p ? kTilePad : 1;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const double c = src[m * mk + (g + 4 * v) * gk];
                    x[e][v] = R[e] != p ? c : m == g + 4 * v ? -1.0 : 0.0;
                }
            }
            StaticFor<0, kRows>::run([&](auto ec) {
                constexpr int e = decltype(ec)::value;
                if (e == 0 || wave + e * step < nb) substitute16(x[e], lb);  // uniform
            });
#pragma unroll
            for (int e = 0; e < kRows; ++e)
                if (wave + e * step < nb) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        S.C[16 * R[e] + g + 4 * v][m] = x[e][v];
                        S.N[16 * R[e] + g + 4 * v][m] = -(x[e][v] * inv);
                    }
                }
        }
        if (chain && more && p >= 0) {
            // the next pivot block: its update needs nothing from the other
            // waves.  Its upper entries are the lower ones: exactly symmetric
            double(*tp)[kTilePad] = S.M[tile(p + 1, p + 1)];
            wave_sync();
            double y[4], n[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                P[v] = tp[m][g + 4 * v];
                y[v] = S.C[16 * (p + 1) + m][g + 4 * v];
                n[v] = S.N[16 * (p + 1) + m][g + 4 * v];
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) P = mfma(y[v], n[v], P);
            mfma_drain();
#pragma unroll
            for (int v = 0; v < 4; ++v) tp[m][g + 4 * v] = P[v];
            wave_sync();
#pragma unroll
            for (int v = 0; v < 4; ++v) P[v] = tp[max(m, g + 4 * v)][min(m, g + 4 * v)];
        }
        __syncthreads();
        if (tiles) {
            // M(I, J) = M'(I, J) - l(I) Y(J)^T
            if (p >= 0) {
#pragma unroll
                for (int u = 0; u < NL; ++u) {
                    if (u * NK + wk >= nt) break;  // uniform
                    d2 a[2], b[2];  // contraction index 4 g + t in step t
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        a[h] = *reinterpret_cast<const d2*>(&S.C[16 * J[u] + m][4 * g + 2 * h]);
                        b[h] = *reinterpret_cast<const d2*>(&S.N[16 * I[u] + m][4 * g + 2 * h]);
                    }
                    if (I[u] == p || J[u] == p) x[u] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
                    for (int h = 0; h < 2; ++h)
#pragma unroll
                        for (int w = 0; w < 2; ++w) x[u] = mfma(a[h][w], b[h][w], x[u]);
                }
                mfma_drain();
            }
            // what the next step reads: the rows' tiles of its column, and
            // for wave 0 the pivot block after it (the next one is its own)
#pragma unroll
            for (int u = 0; u < NL; ++u)
                if (u * NK + wk < nt && ((I[u] == p + 1) != (J[u] == p + 1) || (I[u] == J[u] && I[u] == p + 2))) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) S.M[u * NK + wk][m][g + 4 * v] = x[u][v];
                }
        }
        if (lower && p >= 0) {
            // L_BB(R, p) = l(R) below the pivot block, L_pp and D in it
            double* Fp = F + m + (int64_t)(16 * p + g) * ld;
            if (l0 == 0) {
                const double dm = S.D[buf][m];
                const int row = 16 * p + m;
                if (g == 0 && row < s && !(isfinite(dm) && dm != 0.0 && (!require_spd || dm > 0.0)))
                    atomicMin(status, (unsigned long long)(d.first + row));
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const double x = m == g + 4 * v ? dm : -S.Lb[buf][m][g + 4 * v];
                    if (row < s && m >= g + 4 * v) Fp[16 * p + (int64_t)(4 * v) * ld] = x;
                }
            }
            for (int R = p + 1 + l0; R < nb; R += lstep) {
                double x[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) x[v] = -S.N[16 * R + m][g + 4 * v];
                if (16 * R + m < s) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) Fp[16 * R + (int64_t)(4 * v) * ld] = x[v];
                }
            }
        }
        if (chain && more) pivots(p + 1, P);
        __syncthreads();
    }
    // T = -M, made exactly symmetric from the lower triangle
    if constexpr (NB == 2) {
        // three tiles at most: their transposes straight to their columns
        // (32 columns 8.3 us, through LDS 8.6; 128 columns 34.3 and 31.8)
        if (tiles) {
#pragma unroll
            for (int u = 0; u < NL; ++u) {
                double* Tl = T + 16 * I[u] + m + (int64_t)(16 * J[u] + g) * s;
                double* Tu = T + 16 * J[u] + g + (int64_t)(16 * I[u] + m) * s;
                const bool row = u * NK + wk < nt && 16 * I[u] + m < s;
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (row && (I[u] != J[u] || g + 4 * v <= m)) {
                        Tl[(int64_t)(4 * v) * s] = -x[u][v];
                        Tu[4 * v] = -x[u][v];
                    }
            }
        }
        return;
    }
    if (tiles) {
#pragma unroll
        for (int u = 0; u < NL; ++u)
            if (u * NK + wk < nt) {
#pragma unroll
                for (int v = 0; v < 4; ++v) S.M[u * NK + wk][m][g + 4 * v] = x[u][v];
            }
    }
    __syncthreads();
    for (int t = wave; t < nt; t += NW) {
        int I, J;
        tile_of(t, I, J);
        double lo[4], up[4];  // entries (m, k) and (k, m), k = g + 4 v
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            lo[v] = -S.M[t][m][g + 4 * v];
            up[v] = -S.M[t][g + 4 * v][m];
        }
        double* Tl = T + 16 * I + m + (int64_t)(16 * J + g) * s;
        double* Tu = T + 16 * J + m + (int64_t)(16 * I + g) * s;
        if (I != J && 16 * I + 16 <= s) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                Tl[(int64_t)(4 * v) * s] = lo[v];
                Tu[(int64_t)(4 * v) * s] = up[v];
            }
        } else {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int k = g + 4 * v;
                if (16 * I + m < s && (I != J || k <= m)) Tl[(int64_t)(4 * v) * s] = lo[v];
                if (16 * I + k < s && (I != J || m < k)) Tu[(int64_t)(4 * v) * s] = up[v];
            }
        }
    }
}

// One launch per width class, a work-group per block: two waves for s <= 32,
// four for s <= 64, eight wider; blocks wider than 128 take ldlt_global.
constexpr int diag_waves(int NB) { return NB == 2 ? 2 : NB == 4 ? 4 : 8; }
template <int NB>
__global__ __launch_bounds__(64 * diag_waves(NB)) void k_ldlt_diag(const Task* __restrict__ tasks,
                                                                   const BlockDesc* __restrict__ blk,
                                                                   double* __restrict__ Lp, double* __restrict__ Wp,
                                                                   double* __restrict__ Tp,
                                                                   unsigned long long* __restrict__ status,
                                                                   int require_spd)
{
    __shared__ DiagLds<NB> S;
    const BlockDesc d = blk[tasks[blockIdx.x].b];
    if (NB == 8 && d.s > 16 * NB) ldlt_global(d, Lp, Wp, Tp, status, require_spd);
    else ldlt_blocks<NB, diag_waves(NB)>(d, Lp, Tp, status, require_spd, S);
}

// ---------------------------------------------------------------------------
// Diagonal block of a symmetric indefinite matrix: T_K = F_KK^{-1} with 1x1
// and 2x2 pivots chosen by the Bunch-Kaufman rule (Section 2.1: D may have
// 2x2 blocks; Bunch and Kaufman 1977 for the rule).  The rest of the method
// needs the diagonal block only through T (L_hat = F(C,K) T, the Schur update
// L_hat F(C,K)^T, Algorithm 1 and the adjoint), so the block is inverted
// directly by the symmetric sweep (Gauss-Jordan with diagonal pivots), which
// accepts the pivots in any order: a pivot on index p (d = M(p,p), c = column
// p) sets M(i,j) -= c_i c_j / d, M(i,p) = c_i / d, M(p,p) = -1/d; a 2x2 pivot
// on b = {p, r} does the same with E = M(b,b): M -= M(:,b) E^{-1} M(b,:),
// M(:,b) = M(:,b) E^{-1}, M(b,b) = -E^{-1}.  After every index is swept, M =
// -F_KK^{-1}.  The unswept part of M is the Schur complement the pivoted
// LDL^T would hold, so the rule is applied to it unchanged; an interchange
// only reorders the list of unswept indices (ord[position] = index), and no
// data moves.  The block lives in registers (lower 16 x 16 sub-blocks, thread
// (tx, ty) holds rows tx + 16a, columns ty + 16b); a pivot's column goes
// through LDS, where
// every wave reads it and takes the rule's decisions itself (the same values
// give every wave the same decision, so no decision is broadcast).  One
// work-group per block, NB = 2, 4, 8 for s <= 32, 64, 128.  A singular 1x1 or
// 2x2 pivot latches the block's first column in the status word.
// What bounds it: a chain per pivot of LDS round trips, cross-lane maxima,
// scalar decisions and branches (151 us for 128 columns); neither fewer
// vector instructions in the update nor the update under the search's
// latencies made it faster (159 and 161 us).  Not tried: panels of 16 pivots
// whose columns are brought up to date as they are searched, with the rest of
// the block updated once a panel; the pivots would be the same.
// ---------------------------------------------------------------------------

// a value every lane holds alike, made known to the compiler as uniform
__device__ __forceinline__ double uniform_f64(double x)
{
    const int lo = __builtin_amdgcn_readfirstlane(__double2loint(x));
    const int hi = __builtin_amdgcn_readfirstlane(__double2hiint(x));
    return __hiloint2double(hi, lo);
}

template <int CTRL>
__device__ __forceinline__ double dpp_f64(double x)
{
    const int lo = __builtin_amdgcn_update_dpp(__double2loint(x), __double2loint(x), CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(__double2hiint(x), __double2hiint(x), CTRL, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}

__device__ __forceinline__ double readlane_f64(double x, int l)
{
    const int lo = __builtin_amdgcn_readlane(__double2loint(x), l);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(x), l);
    return __hiloint2double(hi, lo);
}

// largest x over the wave (NaN lanes ignored): within each row of 16 lanes
// by DPP (exchange within quads, then rotations by 4 and 8), then across
// the four rows
__device__ __forceinline__ double wave_max_f64(double x)
{
    x = fmax(x, dpp_f64<0xB1>(x));   // quad_perm [1,0,3,2]
    x = fmax(x, dpp_f64<0x4E>(x));   // quad_perm [2,3,0,1]
    x = fmax(x, dpp_f64<0x124>(x));  // row_ror:4
    x = fmax(x, dpp_f64<0x128>(x));  // row_ror:8
    return fmax(fmax(readlane_f64(x, 0), readlane_f64(x, 16)), fmax(readlane_f64(x, 32), readlane_f64(x, 48)));
}

// f(integral_constant<int, pb>) for the one pb in [0, NB) equal to the
// uniform value v
template <int NB, class Fn>
__device__ __forceinline__ void with_subblock(int v, Fn&& f)
{
    StaticFor<0, NB>::run([&](auto c) {
        if (v == decltype(c)::value) f(c);
    });
}

template <int NB>
__global__ __launch_bounds__(kThreads) void k_ldlt_bk(const Task* __restrict__ tasks, const BlockDesc* __restrict__ blk,
                                                      const double* __restrict__ Lp, double* __restrict__ Tp,
                                                      unsigned long long* __restrict__ status)
{
    constexpr int NS = NB * (NB + 1) / 2;
    constexpr int W = 16 * NB;
    constexpr int NH = (W + 63) / 64;  // positions per lane in a search
    // columns of the pivots: [0], [1] alternate as the next candidate's
    // column, [2] holds the second candidate's (the row searched for sigma)
    __shared__ double cb[3][W];
    const BlockDesc d = blk[tasks[blockIdx.x].b];
    const int s = d.s;
    if (s > W) {  // the launch groups blocks by width, so this does not happen
        if (threadIdx.x == 0) atomicMin(status, (unsigned long long)d.first);
        return;
    }
    const int64_t ld = (int64_t)s + d.c;
    const double* F = Lp + d.poff;
    const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4, lane = tid & 63;
    const double alpha = (1.0 + sqrt(17.0)) / 8.0;
    auto slot = [](int a, int b) { return a * (a + 1) / 2 + b; };
    double M[NS];
#pragma unroll
    for (int a = 0; a < NB; ++a)
#pragma unroll
        for (int b = 0; b <= a; ++b) {
            const int i = tx + 16 * a, k = ty + 16 * b;
            double v = 0.0;
            if (i < s && k < s) v = i >= k ? F[i + k * ld] : F[k + i * ld];
            M[slot(a, b)] = v;
        }
    // ord[q] for the positions q = lane + 64h this lane stands for in searches
    int ordq[NH];
#pragma unroll
    for (int h = 0; h < NH; ++h) ordq[h] = lane + 64 * h;
    auto ord_at = [&](int q) {
        int v = ordq[0];
        if (NH > 1 && q >= 64) v = ordq[NH - 1];
        return __builtin_amdgcn_readlane(v, q & 63);
    };
    auto swap_positions = [&](int q0, int q1) {
        const int v0 = ord_at(q0), v1 = ord_at(q1);
#pragma unroll
        for (int h = 0; h < NH; ++h) {
            const int q = lane + 64 * h;
            ordq[h] = q == q0 ? v1 : (q == q1 ? v0 : ordq[h]);
        }
    };
    // column p of M into col: rows at and below p's sub-block row from the
    // column's owners, rows above it from the owners of row p
    auto publish = [&](int p, double* col) {
        const int pt = p & 15;
        with_subblock<NB>(p >> 4, [&](auto pbc) {
            constexpr int pb = decltype(pbc)::value;
            if (ty == pt) {
#pragma unroll
                for (int a = pb; a < NB; ++a) col[tx + 16 * a] = M[slot(a, pb)];
            }
            if (tx == pt) {
#pragma unroll
                for (int b = 0; b < pb; ++b) col[ty + 16 * b] = M[slot(pb, b)];
            }
        });
    };
    // largest |col[ord[q]]| over positions q in [q0, s), q != skip, and the
    // smallest position holding it (-1 if none): the LDS reads, then the
    // reduction (split so that other reads can be issued in between)
    auto search_load = [&](const double* col, int q0, int skip, double (&v)[NH]) {
#pragma unroll
        for (int h = 0; h < NH; ++h) {
            const int q = lane + 64 * h;
            const bool in = q >= q0 && q < s && q != skip;
            const double x = col[in ? ordq[h] : 0];
            v[h] = in ? fabs(x) : -1.0;
        }
    };
    auto search_reduce = [&](const double (&v)[NH], double& best, int& arg) {
        double m = -1.0;
#pragma unroll
        for (int h = 0; h < NH; ++h) m = fmax(m, v[h]);
        m = wave_max_f64(m);
        int a = -1;
        if (m >= 0.0) {
            const unsigned long long b0 = __ballot(v[0] == m);
            if (b0) a = __builtin_ctzll(b0);
            else if (NH > 1) a = 64 + __builtin_ctzll(__ballot(v[NH - 1] == m));
        }
        best = m;
        arg = a;
    };
    // pivot column values at this thread's rows (ri) and columns (rk)
    auto read_col = [&](const double* col, double (&ri)[NB], double (&rk)[NB]) {
#pragma unroll
        for (int a = 0; a < NB; ++a) ri[a] = col[tx + 16 * a];
#pragma unroll
        for (int b = 0; b < NB; ++b) rk[b] = col[ty + 16 * b];
    };
    // Lanes holding row p (rows tx + 16a) and column p (columns ty + 16b).
    // Row and column p are cleared and the pivot's own entries of the update
    // vectors set (row side at p to -1/d, column side at p to -1); the
    // update M(i,j) -= g_i x_j then writes the new row and column p too:
    // g_i where M(i,p) = 0, x_p = -1; x_j / d where M(p,j) = 0; -1/d at (p,p).
    auto hits = [&](int p, bool (&rz)[NB], bool (&cz)[NB]) {
#pragma unroll
        for (int a = 0; a < NB; ++a) rz[a] = tx + 16 * a == p;
#pragma unroll
        for (int b = 0; b < NB; ++b) cz[b] = ty + 16 * b == p;
    };

    publish(0, cb[0]);
    __syncthreads();
    int cur = 0;
    bool bad = false;
    double ri0[NB], rk0[NB], ri1[NB], rk1[NB];
    for (int k = 0; k < s;) {
        const int pk = ord_at(k);
        // the candidate's diagonal and the search first (they decide the
        // step), then its column for the update
        const double akk_raw = cb[cur][pk];
        double v[NH];
        search_load(cb[cur], k + 1, -1, v);
        read_col(cb[cur], ri0, rk0);
        double lam;
        int rq;
        search_reduce(v, lam, rq);
        const double akk_s = uniform_f64(akk_raw), akk = fabs(akk_s);
        int size = 1, sq = k;
        bool on_r = false;   // 1x1 pivot on the second candidate
        double rr_s = 0.0;   // M(r, r), signed
        double e01 = 0.0;    // M(r, k), signed
        if (rq < 0 || !(lam > 0.0)) {
            bad = akk == 0.0;
        } else if (akk < alpha * lam) {
            const int pr = ord_at(rq);
            const double e01_raw = cb[cur][pr];
            publish(pr, cb[2]);
            __syncthreads();
            const double rr_raw = cb[2][pr];
            search_load(cb[2], k, rq, v);
            double sig;
            int unused;
            search_reduce(v, sig, unused);
            rr_s = uniform_f64(rr_raw);
            e01 = uniform_f64(e01_raw);
            if (akk * sig >= alpha * lam * lam) {
                // 1x1 pivot on the first candidate
            } else if (fabs(rr_s) >= alpha * sig) {
                on_r = true;
                sq = rq;
            } else {
                size = 2;
                sq = rq;
            }
        }
        if (bad) break;
        const int kp = size == 2 ? k + 1 : k;
        if (sq != kp) swap_positions(kp, sq);
        const int p0 = ord_at(k);
        bool rz[NB], cz[NB];
        hits(p0, rz, cz);
        if (size == 1) {
            if (on_r) read_col(cb[2], ri0, rk0);
            const double dd = on_r ? rr_s : akk_s;
            if (dd == 0.0 || !isfinite(dd)) {
                bad = true;
                break;
            }
            const double inv = recip(dd);
            // g = c / d (rows), x = c (columns), the pivot's entries as above
#pragma unroll
            for (int a = 0; a < NB; ++a) ri0[a] = rz[a] ? -inv : ri0[a] * inv;
#pragma unroll
            for (int b = 0; b < NB; ++b) rk0[b] = cz[b] ? -1.0 : rk0[b];
#pragma unroll
            for (int a = 0; a < NB; ++a)
#pragma unroll
                for (int b = 0; b <= a; ++b)
                    M[slot(a, b)] = fma(-ri0[a], rk0[b], (rz[a] || cz[b]) ? 0.0 : M[slot(a, b)]);
        } else {
            const int p1 = ord_at(k + 1);
            bool rz1[NB], cz1[NB];
            hits(p1, rz1, cz1);
            read_col(cb[2], ri1, rk1);
            const double e00 = akk_s, e11 = rr_s;
            const double det = e00 * e11 - e01 * e01;
            if (det == 0.0 || !isfinite(det)) {
                bad = true;
                break;
            }
            const double rdet = recip(det);
            const double i00 = e11 * rdet, i01 = -e01 * rdet, i11 = e00 * rdet;
            // rows: (g0, g1) = M(i, b) E^{-1}, and -E^{-1}'s rows at p0, p1;
            // columns: (x0, x1) = M(b, j), and -(1, 0), -(0, 1) at p0, p1.
            // With rows and columns p0, p1 cleared, M(i,j) -= g0_i x0_j +
            // g1_i x1_j gives M(:,b) E^{-1} in those columns, E^{-1} M(b,:)
            // in those rows and -E^{-1} on the block.
#pragma unroll
            for (int a = 0; a < NB; ++a) {
                const double x = ri0[a], y = ri1[a];
                ri0[a] = rz[a] ? -i00 : (rz1[a] ? -i01 : x * i00 + y * i01);
                ri1[a] = rz[a] ? -i01 : (rz1[a] ? -i11 : x * i01 + y * i11);
                rz[a] = rz[a] || rz1[a];
            }
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                rk0[b] = cz[b] ? -1.0 : (cz1[b] ? 0.0 : rk0[b]);
                rk1[b] = cz[b] ? 0.0 : (cz1[b] ? -1.0 : rk1[b]);
                cz[b] = cz[b] || cz1[b];
            }
#pragma unroll
            for (int a = 0; a < NB; ++a)
#pragma unroll
                for (int b = 0; b <= a; ++b)
                    M[slot(a, b)] = fma(-ri0[a], rk0[b],
                                        fma(-ri1[a], rk1[b], (rz[a] || cz[b]) ? 0.0 : M[slot(a, b)]));
        }
        k += size;
        if (k < s) publish(ord_at(k), cb[cur ^ 1]);
        __syncthreads();
        cur ^= 1;
    }
    if (bad) {  // every thread took the same decisions
        if (tid == 0) atomicMin(status, (unsigned long long)d.first);
        return;
    }
    // T = -M from the lower triangle (exactly symmetric)
    double* T = Tp + d.woff;
#pragma unroll
    for (int a = 0; a < NB; ++a)
#pragma unroll
        for (int b = 0; b <= a; ++b) {
            const int i = tx + 16 * a, j = ty + 16 * b;
            if (i < s && j < s && i >= j) {
                T[i + (int64_t)j * s] = -M[slot(a, b)];
                T[j + (int64_t)i * s] = -M[slot(a, b)];
            }
        }
}

// ===========================================================================
// Small blocks (s <= 16, c <= 256): one wave runs a whole block, every phase
// in turn, on 16 x 16 FP64 MFMA tiles.  Lane (m, g) = (l % 16, l / 16) holds
// entry (m, g + 4 v) of a 16 x 16 block in register v, which is the form of
// both MFMA operands and, with the product formed transposed, of its result:
// every phase feeds the next from registers, with no LDS and no barrier.
//   factor:  F_BB -> L_BB, D, T (gj16); per row group I of C: L_hat(I,:) =
//            F(I,B) T, then for every group K <= I the Schur tile
//            -F(K,:) L_hat(I,:)^T added into the ancestors (lower part);
//   invert:  per row group I: X(I,:) = -G(I,:) L_hat, written to Ainv(C,B),
//            with P += L_hat(I,:)^T X(I,:) and its transpose;
//            then Ainv(B,B) = T - (P + P^T) / 2 on the lower triangle.
// What bounds them is latency (a block is a chain of dependent loads: map,
// rel, value) and, in levels that fill the card, the atomics.  So the loads
// of NG x NG groups of 16 positions of C are issued together, and sixteen
// lanes add into one run of an ancestor column.  NG = 2 (200 registers)
// where a level's launch has a wave to itself, NG = 1 (128 and fewer, for
// residency) in the batched levels; NV and NC cut the registers and the MFMA
// steps to the block's s and c.  Per pass, against a version that kept the
// diagonal block in LDS and loaded each tile's values one at a time: the
// 17 levels of one 32^2 grid 173 -> 80 us; the light levels of a batch
// of 256 grids of 32^2 .. 96^2 (1.2 M unknowns, 49 M atomics) 1.85 -> 1.21 ms.
// ===========================================================================
// s <= 4 NV
template <int NG, int NV>
__device__ __forceinline__ void sb_factor_n(const BlockDesc d, double* __restrict__ Lp, double* __restrict__ Hp,
                                          double* __restrict__ Tp, const int64_t* __restrict__ cr2,
                                          const int32_t* __restrict__ rel, unsigned long long* __restrict__ status,
                                          int require_spd)
{
    const int lane = threadIdx.x & 63, m = lane & 15, g = lane >> 4;
    const int s = d.s, c = d.c;
    const int64_t ld = (int64_t)s + c;
    double* F = Lp + d.poff;
    double* T = Tp + d.woff;
    double* H = Hp + d.hoff;
    const int ng = (c + 15) >> 4;  // groups of C
    // F(C,B): row 16 I + m (past C: the last), columns g + 4 v (past s: 0)
    int64_t fcol[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) fcol[v] = s + (int64_t)min(g + 4 * v, s - 1) * ld;
    auto load_f = [&](int I, double (&f)[NV]) {
        const int row = min(16 * I + m, c - 1);
#pragma unroll
        for (int v = 0; v < NV; ++v) f[v] = F[fcol[v] + row];
    };
    auto mask_f = [&](double (&f)[NV]) {
#pragma unroll
        for (int v = 0; v < NV; ++v) f[v] = g + 4 * v < s ? f[v] : 0.0;
    };
    // the (cbase, rbase) pairs of columns 16 K + g + 4 v of C
    auto load_map = [&](int K, i64x2 (&cr)[4]) {
#pragma unroll
        for (int v = 0; v < 4; ++v)
            cr[v] = *reinterpret_cast<const i64x2*>(cr2 + 2 * (d.coff + min(16 * K + g + 4 * v, c - 1)));
    };
    double P[NV], L[NV];  // L: D on the diagonal
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        const int k = g + 4 * v, a = min(max(m, k), s - 1), b = min(min(m, k), s - 1);
        const double f = F[a + (int64_t)b * ld];
        P[v] = m < s && k < s ? f : (m == k ? 1.0 : 0.0);
    }
    double f[NG][NV];
    i64x2 cr[NG][4];
    if (c > 0) {
#pragma unroll
        for (int e = 0; e < NG; ++e) {
            load_f(min(e, ng - 1), f[e]);
            load_map(min(e, ng - 1), cr[e]);
        }
    }
    gj16(P, L, m, g, s);
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        const int k = g + 4 * v;
        if (m == k && m < s && !(isfinite(L[v]) && L[v] != 0.0 && (!require_spd || L[v] > 0.0)))
            atomicMin(status, (unsigned long long)(d.first + m));
        if (m < s && k <= m) {  // L_BB, D; T made exactly symmetric from the lower triangle
            F[m + (int64_t)k * ld] = L[v];
            T[m + (int64_t)k * s] = P[v];
            T[k + (int64_t)m * s] = P[v];
        }
    }
    for (int K0 = 0; K0 < ng; K0 += NG) {
        if (K0 > 0) {
#pragma unroll
            for (int e = 0; e < NG; ++e) {
                load_f(min(K0 + e, ng - 1), f[e]);
                load_map(min(K0 + e, ng - 1), cr[e]);
            }
        }
#pragma unroll
        for (int e = 0; e < NG; ++e) mask_f(f[e]);
        // row groups from K0 on: the columns' own groups first
        for (int I0 = K0; I0 < ng; I0 += NG) {
            const bool own = I0 == K0;
            double fi[NG][NV];
            uint32_t ro[NG][NG][4];
#pragma unroll
            for (int e = 0; e < NG; ++e) {
                if (!own) load_f(min(I0 + e, ng - 1), fi[e]);
#pragma unroll
                for (int u = 0; u < NG; ++u)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int ii = min(max(16 * (I0 + e) + m, 16 * (K0 + u) + g + 4 * v), c - 1);
                        if (!own || u <= e) ro[e][u][v] = (uint32_t)rel[cr[u][v].y + ii];
                    }
            }
#pragma unroll
            for (int e = 0; e < NG; ++e) {
                if (own) {
#pragma unroll
                    for (int v = 0; v < NV; ++v) fi[e][v] = f[e][v];
                } else {
                    mask_f(fi[e]);
                }
            }
#pragma unroll
            for (int e = 0; e < NG; ++e) {
                const int row = 16 * (I0 + e) + m;
                // L_hat(I,:)^T = T F(I,:)^T
                d4 h = {0, 0, 0, 0};
#pragma unroll
                for (int v = 0; v < NV; ++v) h = mfma(P[v], fi[e][v], h);
                mfma_drain();
                if (K0 == 0) {
#pragma unroll
                    for (int v = 0; v < NV; ++v)
                        if (row < c && g + 4 * v < s) H[row + (int64_t)(g + 4 * v) * c] = h[v];
                }
#pragma unroll
                for (int u = 0; u < NG; ++u) {
                    if (own && u > e) continue;
                    d4 x = {0, 0, 0, 0};
#pragma unroll
                    for (int v = 0; v < NV; ++v) x = mfma(f[u][v], h[v], x);
                    mfma_drain();
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int kk = 16 * (K0 + u) + g + 4 * v;
                        if (row < c && row >= kk) unsafeAtomicAdd(Lp + cr[u][v].x + ro[e][u][v], -x[v]);
                    }
                }
            }
        }
    }
}

template <int NG>
__device__ __forceinline__ void sb_factor(const BlockDesc& d, double* Lp, double* Hp, double* Tp, const int64_t* cr2,
                                          const int32_t* rel, unsigned long long* status, int require_spd)
{
    if (d.s <= 4) sb_factor_n<NG, 1>(d, Lp, Hp, Tp, cr2, rel, status, require_spd);
    else if (d.s <= 8) sb_factor_n<NG, 2>(d, Lp, Hp, Tp, cr2, rel, status, require_spd);
    else sb_factor_n<NG, 4>(d, Lp, Hp, Tp, cr2, rel, status, require_spd);
}

// |C| <= 4 NC, or NC = 4 and any |C|, if kMany
template <int NG, int NC, bool kMany>
__device__ __forceinline__ void sb_invert_n(const BlockDesc d, double* __restrict__ Ap, const double* __restrict__ Hp,
                                          const double* __restrict__ Tp, const int64_t* __restrict__ cr2,
                                          const int32_t* __restrict__ rel)
{
    const int lane = threadIdx.x & 63, m = lane & 15, g = lane >> 4;
    const int s = d.s, c = d.c;
    const int64_t ld = (int64_t)s + c;
    const double* H = Hp + d.hoff;
    const double* T = Tp + d.woff;
    double* A = Ap + d.poff;
    const int ng = kMany ? (c + 15) >> 4 : min(c, 1);
    double t[4];  // T(g + 4 v, m)
#pragma unroll
    for (int v = 0; v < 4; ++v) t[v] = T[min(g + 4 * v, s - 1) + (int64_t)min(m, s - 1) * s];
    // L_hat(16 K + g + 4 v, m), 0 past C and s
    auto load_h = [&](int K, double (&h)[NC]) {
#pragma unroll
        for (int v = 0; v < NC; ++v) h[v] = H[min(16 * K + g + 4 * v, c - 1) + (int64_t)min(m, s - 1) * c];
    };
    auto mask_h = [&](int K, double (&h)[NC]) {
#pragma unroll
        for (int v = 0; v < NC; ++v) h[v] = 16 * K + g + 4 * v < c && m < s ? h[v] : 0.0;
    };
    auto map_at = [&](int p) { return *reinterpret_cast<const i64x2*>(cr2 + 2 * (d.coff + p)); };
    d4 p = {0, 0, 0, 0}, pt = {0, 0, 0, 0};  // P = L_hat^T X and its transpose
    for (int I0 = 0; I0 < ng; I0 += NG) {
        i64x2 ci[NG];  // map entries of rows 16 (I0 + e) + m
#pragma unroll
        for (int e = 0; e < NG; ++e) ci[e] = map_at(min(16 * (I0 + e) + m, c - 1));
        d4 x[NG];
#pragma unroll
        for (int e = 0; e < NG; ++e) x[e] = d4{0, 0, 0, 0};
        double hi[NG][NC];
        for (int K0 = 0; K0 < ng; K0 += NG) {
            i64x2 ck[NG][NC];  // of columns 16 (K0 + u) + g + 4 v
            double h[NG][NC];
#pragma unroll
            for (int u = 0; u < NG; ++u) {
#pragma unroll
                for (int v = 0; v < NC; ++v) ck[u][v] = map_at(min(16 * (K0 + u) + g + 4 * v, c - 1));
                load_h(K0 + u, h[u]);
            }
            // G(i, k) = Ap[cbase[p] + rel[rbase[p] + q]], p = min(i, k), q = max(i, k)
            uint32_t r[NG][NG][NC];
#pragma unroll
            for (int e = 0; e < NG; ++e)
#pragma unroll
                for (int u = 0; u < NG; ++u)
#pragma unroll
                    for (int v = 0; v < NC; ++v) {
                        const int i = min(16 * (I0 + e) + m, c - 1), k = min(16 * (K0 + u) + g + 4 * v, c - 1);
                        r[e][u][v] = (uint32_t)rel[(i >= k ? ck[u][v].y : ci[e].y) + max(i, k)];
                    }
            double a[NG][NG][NC];
#pragma unroll
            for (int e = 0; e < NG; ++e)
#pragma unroll
                for (int u = 0; u < NG; ++u)
#pragma unroll
                    for (int v = 0; v < NC; ++v) {
                        const int i = min(16 * (I0 + e) + m, c - 1), k = min(16 * (K0 + u) + g + 4 * v, c - 1);
                        a[e][u][v] = Ap[(i >= k ? ck[u][v].x : ci[e].x) + r[e][u][v]];
                    }
#pragma unroll
            for (int u = 0; u < NG; ++u) mask_h(K0 + u, h[u]);
            if (I0 == K0) {
#pragma unroll
                for (int u = 0; u < NG; ++u)
#pragma unroll
                    for (int v = 0; v < NC; ++v) hi[u][v] = h[u][v];
            }
#pragma unroll
            for (int u = 0; u < NG; ++u)
#pragma unroll
                for (int v = 0; v < NC; ++v)
#pragma unroll
                    for (int e = 0; e < NG; ++e)
                        x[e] = mfma(16 * (K0 + u) + g + 4 * v < c ? a[e][u][v] : 0.0, h[u][v], x[e]);
        }
        mfma_drain();
        // x[e][v] = (G L_hat)(16 (I0 + e) + g + 4 v, m): X = -x
#pragma unroll
        for (int e = 0; e < NG; ++e) {
#pragma unroll
            for (int v = 0; v < NC; ++v) {
                const int row = 16 * (I0 + e) + g + 4 * v;
                if (row < c && m < s) A[s + row + (int64_t)m * ld] = -x[e][v];
            }
#pragma unroll
            for (int v = 0; v < NC; ++v) {
                p = mfma(hi[e][v], -x[e][v], p);
                pt = mfma(-x[e][v], hi[e][v], pt);
            }
        }
    }
    mfma_drain();
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int ii = g + 4 * v;
        if (ii < s && m <= ii) A[ii + (int64_t)m * ld] = t[v] - 0.5 * (p[v] + pt[v]);
    }
}

template <int NG>
__device__ __forceinline__ void sb_invert(const BlockDesc& d, double* Ap, const double* Hp, const double* Tp,
                                          const int64_t* cr2, const int32_t* rel)
{
    if (d.c <= 8) sb_invert_n<1, 2, false>(d, Ap, Hp, Tp, cr2, rel);
    else if (d.c <= 16) sb_invert_n<1, 4, false>(d, Ap, Hp, Tp, cr2, rel);
    else sb_invert_n<NG, 4, true>(d, Ap, Hp, Tp, cr2, rel);
}

// Per-level launches of the small-block path: task q holds up to four block
// ids (b, i0, j0, bn; -1 = none), one per wave.
__device__ __forceinline__ int sb_block_of(const Task& t)
{
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    return w == 0 ? t.b : w == 1 ? t.i0 : w == 2 ? t.j0 : t.bn;
}

__global__ __launch_bounds__(kThreads) void k_sb_factor(const Task* __restrict__ tasks,
                                                        const BlockDesc* __restrict__ blk, double* __restrict__ Lp,
                                                        double* __restrict__ Hp, double* __restrict__ Tp,
                                                        const int64_t* __restrict__ cr2,
                                                        const int32_t* __restrict__ rel,
                                                        unsigned long long* __restrict__ status, int require_spd)
{
    const int b = sb_block_of(tasks[blockIdx.x]);
    if (b >= 0) sb_factor<2>(blk[b], Lp, Hp, Tp, cr2, rel, status, require_spd);
}

__global__ __launch_bounds__(kThreads) void k_sb_invert(const Task* __restrict__ tasks,
                                                        const BlockDesc* __restrict__ blk, double* __restrict__ Ap,
                                                        const double* __restrict__ Hp, const double* __restrict__ Tp,
                                                        const int64_t* __restrict__ cr2,
                                                        const int32_t* __restrict__ rel)
{
    const int b = sb_block_of(tasks[blockIdx.x]);
    if (b >= 0) sb_invert<2>(blk[b], Ap, Hp, Tp, cr2, rel);
}

// ===========================================================================
// Persistent level kernels (batched form).  One launch per tree level runs
// every task of the level, across all blocks of all matrices of a batch,
// from a work queue: a work-group claims the next index with an atomic add
// on the level's queue head until the queue is empty.  Tasks of one block
// depend on the block's earlier phases (factor: diagonal block -> L_hat
// tiles -> Schur tiles; inversion: zero X -> X tiles -> diagonal tiles); a
// task waits until its block's completion counter reaches task.pad.  Waits
// are on smaller queue indices only, which running work-groups hold, so
// every wait ends; a wait that exceeds spin_limit polls latches status[1]
// and the task proceeds, so the kernel always drains.
// ===========================================================================
template <int NB>  // the widest diagonal block (16 NB; inversion kernels: none, NB = 1)
union PersistLds {
    GatherLds gather;
    SdiagLds sd;
    DiagLds<NB> diag;
};

struct QueueArgs {
    const Task* q;
    int64_t ntasks;
    unsigned* head;   // this level's queue head
    unsigned* done;   // per-block completion counters of this sweep
    unsigned long long* status;
    int require_spd;
    unsigned spin_limit;
};

// The claimed index is the same in every thread; readfirstlane makes it a
// wave-uniform (scalar) value, so the compiler sees a uniform loop whose
// barriers every thread reaches together.
__device__ __forceinline__ int claim(const QueueArgs& a, int* s_idx)
{
    if (threadIdx.x == 0) *s_idx = (int)__hip_atomic_fetch_add(a.head, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const int idx = __builtin_amdgcn_readfirstlane(*s_idx);
    __syncthreads();
    return idx;
}

__device__ __forceinline__ Task uniform_task(const Task* q, int idx)
{
    const Task r = q[idx];
    Task t;
    t.b = __builtin_amdgcn_readfirstlane(r.b);
    t.i0 = __builtin_amdgcn_readfirstlane(r.i0);
    t.j0 = __builtin_amdgcn_readfirstlane(r.j0);
    t.bn = __builtin_amdgcn_readfirstlane(r.bn);
    t.kb = __builtin_amdgcn_readfirstlane(r.kb);
    t.ke = __builtin_amdgcn_readfirstlane(r.ke);
    t.flags = __builtin_amdgcn_readfirstlane(r.flags);
    t.pad = __builtin_amdgcn_readfirstlane(r.pad);
    return t;
}

// Thread 0 polls the block's counter (relaxed loads; one acquire fence for
// the whole work-group once the count is reached).  A wait gives up after
// spin_limit polls, or at once when another wait has already given up, so
// a run ends within about one poll limit whatever happens.
__device__ __forceinline__ void wait_deps(const QueueArgs& a, const Task& t)
{
    if (t.pad > 0 && threadIdx.x == 0) {
        unsigned spins = 0;
        while (__hip_atomic_load(a.done + t.b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < (unsigned)t.pad) {
            const bool gave_up =
                (spins & 255u) == 0 && __hip_atomic_load(a.status + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
            if (gave_up || ++spins > a.spin_limit) {
                atomicOr(a.status + 1, 1ull);
                break;
            }
            __builtin_amdgcn_s_sleep(2);
        }
    }
    __syncthreads();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
}

__device__ __forceinline__ void signal_done(const QueueArgs& a, const Task& t)
{
    __threadfence();  // every thread's results reach device scope first
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_fetch_add(a.done + t.b, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
}

// diagonal block of a tiled level: the host keeps s <= 16 NB, or NB = 8
template <int NB>
__device__ __forceinline__ void diag_block(const BlockDesc& d, double* Lp, double* Wp, double* Tp,
                                           unsigned long long* status, int require_spd, DiagLds<NB>& S)
{
    if constexpr (NB == 8) {
        if (d.s > kLdsDiagMax) {
            ldlt_global(d, Lp, Wp, Tp, status, require_spd);
            return;
        }
    }
    ldlt_blocks<NB, kThreads / 64>(d, Lp, Tp, status, require_spd, S);
}

// L_hat tile; tiles are at most as wide as the level's widest block
template <int NB>
__device__ __forceinline__ void panel_bounded(GatherLds& L, const Task& t, const BlockDesc& d, const double* Lp,
                                              double* Hp, const double* Tp)
{
    if (t.bn <= 16) {
        panel_task<16>(L, t, d, Lp, Hp, Tp);
    } else if (t.bn <= 32) {
        panel_task<32>(L, t, d, Lp, Hp, Tp);
    } else if constexpr (NB >= 4) {
        if (t.bn <= 64) panel_task<64>(L, t, d, Lp, Hp, Tp);
        else if constexpr (NB >= 8) panel_task<128>(L, t, d, Lp, Hp, Tp);
    }
}

// gather-GEMM tile; the host keeps t.bn <= BNMAX in this variant's levels
template <int BNMAX>
__device__ __forceinline__ void gemm_bounded(GatherLds& L, const Task& t, const BlockDesc& d, double* Ap,
                                             const double* Hp, const int64_t* cr2,
                                             const int32_t* rel)
{
    if (t.bn <= 16) {
        gemm_task<16>(L, t, d, Ap, Hp, cr2, rel);
    } else if (t.bn <= 32) {
        gemm_task<32>(L, t, d, Ap, Hp, cr2, rel);
    } else if constexpr (BNMAX >= 64) {
        if (t.bn <= 64) gemm_task<64>(L, t, d, Ap, Hp, cr2, rel);
        else if constexpr (BNMAX >= 128) gemm_task<128>(L, t, d, Ap, Hp, cr2, rel);
    }
}

// Levels with tiled blocks; NB bounds the diagonal sweep (s <= 16 NB, wider
// blocks take ldlt_global) and so the kernel's registers.
template <int NB>
__global__ __launch_bounds__(kThreads, NB < 8 ? 2 : 1) void k_persist_factor(const QueueArgs a, const BlockDesc* __restrict__ blk,
                                                             double* __restrict__ Lp, double* __restrict__ Wp,
                                                             double* __restrict__ Hp, double* __restrict__ Tp,
                                                             const int32_t* __restrict__ rel,
                                                             const int64_t* __restrict__ cr2)
{
    __shared__ PersistLds<NB> sm;
    __shared__ int s_idx;
    // a work-group cannot claim more than ntasks entries: the bound only
    // makes termination evident
    for (int64_t it = 0; it < a.ntasks; ++it) {
        const int idx = claim(a, &s_idx);
        if (idx >= a.ntasks) break;
        const Task t = uniform_task(a.q, idx);
        const int op = t.flags >> 8;
        if (op == qSbFactor) {
            const int b = sb_block_of(t);
            if (b >= 0)
                sb_factor_n<1, 4>(blk[b], Lp, Hp, Tp, cr2, rel, a.status, a.require_spd);
            __syncthreads();  // the LDS union is reused by the next task
            continue;
        }
        const BlockDesc d = blk[t.b];
        // a medium block runs its diagonal block, L_hat tiles and Schur tiles
        // here in turn (one call site per routine keeps registers down)
        const bool whole = op == qMbFactor;
        if (!whole) wait_deps(a, t);
        const int nrow = (d.c + kTileM - 1) / kTileM, ncol = whole ? (d.s + t.bn - 1) / t.bn : 0;
        const int nsc = (d.c + kSchurTile - 1) / kSchurTile;
        const int steps = whole ? 1 + nrow * ncol + nsc * (nsc + 1) / 2 : 1;
        int pr = 0, pj = 0, si = 0, sk = 0;  // next panel tile (row, column), Schur tile (row, column)
        for (int st = 0; st < steps; ++st) {
            int o = op;
            Task u = t;
            if (whole) {
                if (st == 0) {
                    o = qLdlt;
                } else if (st <= nrow * ncol) {
                    o = qPanel;
                    u = Task{t.b, pr * kTileM, pj * t.bn, t.bn, 0, d.s, 0, 0};
                    if (++pr == nrow) pr = 0, ++pj;
                } else {
                    o = qSchur;
                    u = Task{t.b, si * kSchurTile, sk * kSchurTile, kSchurTile, 0, d.s, t.flags & 4, 0};
                    if (++si == nsc) si = ++sk;
                }
            }
            switch (o) {
                case qLdlt:
                    diag_block<NB>(d, Lp, Wp, Tp, a.status, a.require_spd, sm.diag);
                    break;
                case qPanel:
                    panel_bounded<NB>(sm.gather, u, d, Lp, Hp, Tp);
                    break;
                default:
                    schur_task(sm.gather, u, d, Lp, Hp, cr2, rel);
                    break;
            }
            if (whole) __syncthreads();
        }
        if (!whole && (t.flags & 2)) signal_done(a, t);
        else __syncthreads();
    }
}

// Levels with tiled blocks; BNMAX bounds the gather-GEMM tile width and so
// the kernel's registers.
template <int BNMAX>
__global__ __launch_bounds__(kThreads, 2) void k_persist_invert(const QueueArgs a, const BlockDesc* __restrict__ blk,
                                                                double* __restrict__ Ap, const double* __restrict__ Hp,
                                                                const double* __restrict__ Tp,
                                                                const int32_t* __restrict__ rel,
                                                                const int64_t* __restrict__ cr2)
{
    __shared__ PersistLds<1> sm;
    __shared__ int s_idx;
    for (int64_t it = 0; it < a.ntasks; ++it) {
        const int idx = claim(a, &s_idx);
        if (idx >= a.ntasks) break;
        const Task t = uniform_task(a.q, idx);
        const int op = t.flags >> 8;
        if (op == qSbInvert) {
            const int b = sb_block_of(t);
            if (b >= 0) sb_invert_n<1, 4, true>(blk[b], Ap, Hp, Tp, cr2, rel);
            __syncthreads();
            continue;
        }
        const BlockDesc d = blk[t.b];
        // a medium block runs its X tiles (whole contractions) and then its
        // diagonal tiles here in turn
        const bool whole = op == qMbInvert;
        if (!whole) wait_deps(a, t);
        const int nrow = (d.c + kTileM - 1) / kTileM, ncol = whole ? (d.s + t.bn - 1) / t.bn : 0;
        const int nd = (d.s + kDiagTile - 1) / kDiagTile;
        const int steps = whole ? nrow * ncol + nd * (nd + 1) / 2 : 1;
        int gr = 0, gj = 0, di = 0, dj = 0;  // next X tile (row, column), diagonal tile pair (I, J)
        for (int st = 0; st < steps; ++st) {
            int o = op;
            Task u = t;
            if (whole) {
                if (st < nrow * ncol) {
                    o = qGemm;
                    u = Task{t.b, gr * kTileM, gj * t.bn, t.bn, 0, d.c, 0, 0};
                    if (++gr == nrow) gr = 0, ++gj;
                } else {
                    o = qSdiag;
                    u = Task{t.b, di * kDiagTile, dj * kDiagTile, 0, 0, d.c, 0, 0};
                    if (++dj > di) dj = 0, ++di;
                }
            }
            switch (o) {
                case qZero:
                    zero_task(d, Ap, Tp);
                    break;
                case qGemm:
                    gemm_bounded<BNMAX>(sm.gather, u, d, Ap, Hp, cr2, rel);
                    break;
                default:
                    sdiag_task(sm.sd, u, d, Ap, Hp, Tp);
                    break;
            }
            if (whole) __syncthreads();
        }
        if (!whole && (t.flags & 2)) signal_done(a, t);
        else __syncthreads();
    }
}

// Levels made only of small blocks: no dependencies, so no queue head
// either.  Wave g of W takes slots g, g + W, g + 2W, ... (slot = 4 task +
// wave field) of the level's cost-ordered list, so every wave gets a like
// mix; no atomics, no work-group barrier.  (A run of the plan's order per
// XCD, for the locality of the ancestors, was 8 % slower.)  The id of the
// block after the next and the next one's descriptor are loaded while a
// block runs, which takes two of its five dependent loads off the chain.
struct LightQueue {
    const int32_t* ids;
    const BlockDesc* blk;
    int64_t nslots, step, slot;
    int id0, id1;  // of this turn (uniform) and of the next
    BlockDesc next;

    __device__ __forceinline__ LightQueue(const QueueArgs& a, const BlockDesc* b)
        : ids(reinterpret_cast<const int32_t*>(a.q)), blk(b), nslots(a.ntasks * kSbPerTask),
          step((int64_t)gridDim.x * (kThreads / 64))
    {
        slot = (int64_t)blockIdx.x * (kThreads / 64) + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
        id1 = at(slot);
        advance();
    }
    __device__ __forceinline__ int at(int64_t x) const
    {
        x = min(x, nslots - 1);
        return ids[x / kSbPerTask * (int64_t)(sizeof(Task) / sizeof(int32_t)) + x % kSbPerTask];
    }
    __device__ __forceinline__ void advance()
    {
        id0 = __builtin_amdgcn_readfirstlane(id1);
        id1 = at(slot + step);
        next = blk[max(id0, 0)];
    }
    // the block of this turn into d; false: none in this slot
    __device__ __forceinline__ bool take(BlockDesc& d)
    {
        const bool some = id0 >= 0;
        d = next;
        slot += step;
        advance();
        return some;
    }
    __device__ __forceinline__ bool more() const { return slot < nslots; }
};

// Levels of blocks with s <= 4 NV: fewer columns take fewer registers and
// MFMA steps, and more waves per SIMD hide each other's loads (six for
// NV = 1).
template <int NV>
__global__ __launch_bounds__(kThreads, NV == 1 ? 6 : 4) void k_light_factor(const QueueArgs a, const BlockDesc* __restrict__ blk,
                                                           double* __restrict__ Lp, double* __restrict__ Hp,
                                                           double* __restrict__ Tp, const int64_t* __restrict__ cr2,
                                                           const int32_t* __restrict__ rel)
{
    LightQueue queue(a, blk);
    while (queue.more()) {
        BlockDesc d;
        if (queue.take(d)) sb_factor_n<1, NV>(d, Lp, Hp, Tp, cr2, rel, a.status, a.require_spd);
    }
}

// Levels of blocks with |C| <= 4 NC, or any |C| if kMany (NC = 4): one piece
// of G needs no loops and 50 registers instead of 100, eight waves per SIMD
// instead of four (the leaves of the batch above: 168 -> 100 us).
template <int NC, bool kMany>
__global__ __launch_bounds__(kThreads, kMany ? 4 : 8) void k_light_invert(const QueueArgs a, const BlockDesc* __restrict__ blk,
                                                           double* __restrict__ Ap, const double* __restrict__ Hp,
                                                           const double* __restrict__ Tp,
                                                           const int64_t* __restrict__ cr2,
                                                           const int32_t* __restrict__ rel)
{
    LightQueue queue(a, blk);
    while (queue.more()) {
        BlockDesc d;
        if (queue.take(d)) sb_invert_n<1, NC, kMany>(d, Ap, Hp, Tp, cr2, rel);
    }
}

__global__ void k_fill_u32(unsigned* __restrict__ p, int64_t n)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0u;
}

// ===========================================================================
// Reverse sweep: adjoint of the factorization and of the selected inversion.
// Adjoints are those of the stored values: an entry of a diagonal block's
// lower triangle stands for both (i,j) and (j,i), an entry of the C rows for
// itself.  Zb holds the adjoint of Ainv during the reverse selected
// inversion (leaves first) and the adjoint of F during the reverse
// factorization (root first), in the panel layout; Hb is the adjoint of
// L_hat and Tb that of T.  Per block, with Zbar the adjoint of its panel:
//   Ybar = (Zbar_BB + Zbar_BB^T)/2,  Xbar = Zbar(C,B) - L_hat Ybar,
//   Lhat_bar = -X Ybar - G Xbar,  Tbar = Ybar,
//   ancestors' Zbar(C,C) += -(Xbar L_hat^T + L_hat Xbar^T)  (stored lower);
// then, root first, with Ubar(i,k) = -Fbar(C[i],C[k]) (i >= k) from the
// ancestors: Lhat_bar += Ubar F(C,B), Fbar(C,B) = Ubar^T L_hat + Lhat_bar T,
// Tbar += F(C,B)^T Lhat_bar, Fbar_BB = -T (Tbar + Tbar^T) T (stored lower).
// The gradient of A's entries is Fbar at their positions.
// ===========================================================================
__device__ __forceinline__ double ybar_at(const double* __restrict__ Zd, int64_t ld, int t, int j)
{
    if (t == j) return Zd[t + (int64_t)t * ld];
    const int a = t > j ? t : j, b = t > j ? j : t;
    return 0.5 * Zd[a + (int64_t)b * ld];
}

// Tb(B) := Ybar of the level's blocks: the adjoint of T, and the symmetric
// operand of the two products below
__global__ void k_tbar_init(const Task* __restrict__ tasks, const BlockDesc* __restrict__ blk,
                            const double* __restrict__ Zb, double* __restrict__ Tb)
{
    const BlockDesc d = blk[tasks[blockIdx.x].b];
    const int64_t ld = (int64_t)d.s + d.c;
    for (int e = threadIdx.x + blockIdx.y * blockDim.x; e < d.s * d.s; e += blockDim.x * gridDim.y)
        Tb[d.woff + e] = ybar_at(Zb + d.poff, ld, e % d.s, e / d.s);
}

template <int BN>
__device__ __forceinline__ void rs1_task(GatherLds& L, const Task t, const BlockDesc d, double* __restrict__ Zb,
                                         const double* __restrict__ Hp, const double* __restrict__ Tb)
{
    const int s = d.s, c = d.c;
    const int64_t ld = (int64_t)s + c;
    const int r0 = t.i0, n0 = t.j0;
    d4 acc[2][4] = {};
    dense_mma<BN, false, false, true>(L, operand(Hp + d.hoff + r0, (int64_t)s * c - r0, c),
                                      operand(Tb + d.woff + n0, (int64_t)s * s - n0, s), 0, s, acc, [] {});
    tile_epilogue_t<BN>(acc, [&](int i, int j, double v) {
        const int ii = r0 + i, jj = n0 + j;
        if (ii < c && jj < s) Zb[d.poff + s + ii + (int64_t)jj * ld] -= v;
    });
}

__global__ __launch_bounds__(kThreads) void k_rs1(const Task* __restrict__ tasks, const BlockDesc* __restrict__ blk,
                                                  double* __restrict__ Zb, const double* __restrict__ Hp,
                                                  const double* __restrict__ Tb)
{
    __shared__ GatherLds L;
    const Task t = tasks[blockIdx.x];
    const BlockDesc d = blk[t.b];
#define SELINV_CALL(BN) rs1_task<BN>(L, t, d, Zb, Hp, Tb)
    SELINV_BN_DISPATCH(t.bn, SELINV_CALL)
#undef SELINV_CALL
}

template <int BN>
__device__ __forceinline__ void rs2_task(GatherLds& L, const Task t, const BlockDesc d, const double* __restrict__ Ap,
                         const double* __restrict__ Zb, const double* __restrict__ Tb, double* __restrict__ Hb, const int64_t* __restrict__ cr2, const int32_t* __restrict__ rel)
{
    const int s = d.s, c = d.c;
    const int64_t ld = (int64_t)s + c;
    const int r0 = t.i0, n0 = t.j0;
    d4 acc[2][4] = {};
    // G Xbar: G gathered from the inverse panels, Xbar = Zbar(C,B)
    gather_mma<BN, 0>(L, d, r0, n0, t.kb, t.ke, Ap, Zb + d.poff + s, ld, cr2, rel, acc);
    if (t.kb == 0)  // -X Ybar, once per tile
        dense_mma<BN, false, false, true>(L, operand(Ap + d.poff + s + r0, (int64_t)(s - 1) * ld + c - r0, ld),
                                          operand(Tb + d.woff + n0, (int64_t)s * s - n0, s), 0, s, acc, [] {});
    tile_epilogue_t<BN>(acc, [&](int i, int j, double v) {
        const int ii = r0 + i, jj = n0 + j;
        if (ii < c && jj < s) {
            double* p = Hb + d.hoff + ii + (int64_t)jj * c;
            if (t.flags & 1) unsafeAtomicAdd(p, -v); else *p = -v;
        }
    });
}

__global__ __launch_bounds__(kThreads, 2) void k_rs2(const Task* __restrict__ tasks, const BlockDesc* __restrict__ blk,
                                                  const double* __restrict__ Ap, const double* __restrict__ Zb,
                                                  const double* __restrict__ Tb,
                                                  double* __restrict__ Hb, const int64_t* __restrict__ cr2, const int32_t* __restrict__ rel)
{
    __shared__ GatherLds L;
    const Task t = tasks[blockIdx.x];
    const BlockDesc d = blk[t.b];
#define SELINV_CALL(BN) rs2_task<BN>(L, t, d, Ap, Zb, Tb, Hb, cr2, rel)
    SELINV_BN_DISPATCH(t.bn, SELINV_CALL)
#undef SELINV_CALL
}

// ancestors' Zbar += -(Xbar L_hat^T + L_hat Xbar^T): lower tile rows
// [i0, i0+64) x columns [k0, k0+64); a diagonal entry of C x C counts half
__global__ __launch_bounds__(kThreads, 3) void k_rs3(const Task* __restrict__ tasks, const BlockDesc* __restrict__ blk,
                                                     double* __restrict__ Zb, const double* __restrict__ Hp,
                                                     const int64_t* __restrict__ cr2, const int32_t* __restrict__ rel)
{
    __shared__ GatherLdsN<64> L;
    const Task t = tasks[blockIdx.x];
    const BlockDesc d = blk[t.b];
    const int s = d.s, c = d.c;
    const int64_t ld = (int64_t)s + c;
    auto xbar = [&](int r) { return operand(Zb + d.poff + s + r, (int64_t)(s - 1) * ld + c - r, ld); };
    auto lhat = [&](int r) { return operand(Hp + d.hoff + r, (int64_t)s * c - r, c); };
    auto product = [&](d4(&acc)[2][4], auto prefetch) {
        dense_mma<64, false, false, false>(L, xbar(t.j0), lhat(t.i0), 0, s, acc, prefetch);
        dense_mma<64, false, false, false>(L, lhat(t.j0), xbar(t.i0), 0, s, acc, [] {});
    };
    scatter_update(t, d, Zb, cr2, rel, product, [](int ii, int kk, double x) { return ii == kk ? -0.5 * x : -x; });
}

// Lhat_bar += Ubar F(C,B), Ubar(i,k) = -Fbar(C[i],C[k]) for i >= k
template <int BN>
__device__ __forceinline__ void rf1a_task(GatherLds& L, const Task t, const BlockDesc d, const double* __restrict__ Zb,
                          const double* __restrict__ Lp, double* __restrict__ Hb, const int64_t* __restrict__ cr2, const int32_t* __restrict__ rel)
{
    const int s = d.s, c = d.c;
    const int64_t ld = (int64_t)s + c;
    const int r0 = t.i0, n0 = t.j0;
    d4 acc[2][4] = {};
    // Ubar(i,k) = -Fbar(C[i],C[k]) for k <= i, gathered from the adjoint panels; B = F(C,B)
    gather_mma<BN, 1>(L, d, r0, n0, t.kb, t.ke, Zb, Lp + d.poff + s, ld, cr2, rel, acc);
    tile_epilogue_t<BN>(acc, [&](int i, int j, double v) {
        const int ii = r0 + i, jj = n0 + j;
        if (ii < c && jj < s) {
            double* p = Hb + d.hoff + ii + (int64_t)jj * c;
            if (t.flags & 1) unsafeAtomicAdd(p, -v); else *p -= v;
        }
    });
}

__global__ __launch_bounds__(kThreads, 2) void k_rf1a(const Task* __restrict__ tasks, const BlockDesc* __restrict__ blk,
                                                   const double* __restrict__ Zb, const double* __restrict__ Lp,
                                                   double* __restrict__ Hb, const int64_t* __restrict__ cr2,
                                                   const int32_t* __restrict__ rel)
{
    __shared__ GatherLds L;
    const Task t = tasks[blockIdx.x];
    const BlockDesc d = blk[t.b];
#define SELINV_CALL(BN) rf1a_task<BN>(L, t, d, Zb, Lp, Hb, cr2, rel)
    SELINV_BN_DISPATCH(t.bn, SELINV_CALL)
#undef SELINV_CALL
}

// Fbar(C,B) = Ubar^T L_hat (+ Lhat_bar T on piece 0), Ubar^T(i,k) = -Fbar(C[k],C[i]) for k >= i
template <int BN>
__device__ __forceinline__ void rf1b_task(GatherLds& L, const Task t, const BlockDesc d, double* __restrict__ Zb,
                          const double* __restrict__ Hp, const double* __restrict__ Hb, const double* __restrict__ Tp,
                          const int64_t* __restrict__ cr2,
                          const int32_t* __restrict__ rel)
{
    const int s = d.s, c = d.c;
    const int64_t ld = (int64_t)s + c;
    const int r0 = t.i0, n0 = t.j0;
    d4 acc[2][4] = {};
    // -Ubar^T L_hat: Fbar(C[k],C[i]) for k >= i, gathered from the adjoint panels
    gather_mma<BN, 2>(L, d, r0, n0, t.kb, t.ke, Zb, Hp + d.hoff, c, cr2, rel, acc);
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) acc[mt][nt] = -acc[mt][nt];
    if (t.flags & 2)  // T is symmetric
        dense_mma<BN, false, false, true>(L, operand(Hb + d.hoff + r0, (int64_t)s * c - r0, c),
                                          operand(Tp + d.woff + n0, (int64_t)s * s - n0, s), 0, s, acc, [] {});
    tile_epilogue_t<BN>(acc, [&](int i, int j, double v) {
        const int ii = r0 + i, jj = n0 + j;
        if (ii < c && jj < s) {
            double* p = Zb + d.poff + s + ii + (int64_t)jj * ld;
            if (t.flags & 1) unsafeAtomicAdd(p, v); else *p = v;
        }
    });
}

__global__ __launch_bounds__(kThreads, 2) void k_rf1b(const Task* __restrict__ tasks, const BlockDesc* __restrict__ blk,
                                                   double* __restrict__ Zb, const double* __restrict__ Hp,
                                                   const double* __restrict__ Hb, const double* __restrict__ Tp,
                                                   const int64_t* __restrict__ cr2,
                                                   const int32_t* __restrict__ rel)
{
    __shared__ GatherLds L;
    const Task t = tasks[blockIdx.x];
    const BlockDesc d = blk[t.b];
#define SELINV_CALL(BN) rf1b_task<BN>(L, t, d, Zb, Hp, Hb, Tp, cr2, rel)
    SELINV_BN_DISPATCH(t.bn, SELINV_CALL)
#undef SELINV_CALL
}

// Tbar(I,J) += F(C,B)^T Lhat_bar over rows [kb, ke) of C, one 64 x 64 tile
__global__ __launch_bounds__(kThreads) void k_rf2(const Task* __restrict__ tasks, const BlockDesc* __restrict__ blk,
                                                  const double* __restrict__ Lp, const double* __restrict__ Hb,
                                                  double* __restrict__ Tb)
{
    __shared__ GatherLdsN<64> L;
    const Task t = tasks[blockIdx.x];
    const BlockDesc d = blk[t.b];
    const int s = d.s, c = d.c;
    const int64_t ld = (int64_t)s + c;
    const int I0 = t.i0, J0 = t.j0;
    d4 acc[2][4] = {};
    dense_mma<64, true, true, true>(L, operand(Lp + d.poff + s + I0 * ld, (int64_t)(s - 1 - I0) * ld + c, ld),
                                    operand(Hb + d.hoff + (int64_t)J0 * c, (int64_t)(s - 1 - J0) * c + c, c), t.kb,
                                    min(t.ke, c), acc, [] {});
    tile_epilogue_t<64>(acc, [&](int i, int j, double v) {
        const int gi = I0 + i, gj = J0 + j;
        if (gi < s && gj < s) {
            double* p = Tb + d.woff + gi + (int64_t)gj * s;
            if (t.flags & 1) unsafeAtomicAdd(p, v); else *p += v;
        }
    });
}

// Fbar(B,B) stored lower = -T (Tbar + Tbar^T) T with the diagonal halved
// (s <= 128).  A work-group forms 16 columns J of the result: first
// Q = (Tbar + Tbar^T) T(:,J) into LDS, then the tiles of T Q on and below the
// diagonal, a wave per 16 x 16 tile, operands straight from global memory
// (both matrices fit the L2 several times over) with eight steps of loads in
// flight.  The step is a link of the root-first chain, so its time is the
// latency of one block: with one work-group per block 64 tiles of Q shared
// four waves, 155 us at s = 128; eight work-groups take about 15 us (the whole backward and forward of a
// 31 x 29 x 30 grid: 10.7 -> 7.8 ms).
__global__ __launch_bounds__(kThreads) void k_rf3(const Task* __restrict__ tasks, const BlockDesc* __restrict__ blk,
                                                  const double* __restrict__ Tp, const double* __restrict__ Tb,
                                                  double* __restrict__ Zb)
{
    __shared__ double Q[kLdsDiagMax][16 + 1];
    const BlockDesc d = blk[tasks[blockIdx.x].b];
    const int s = d.s, j0 = (int)blockIdx.y * 16;
    if (j0 >= s) return;  // the grid covers the widest block of the level
    const int64_t ld = (int64_t)d.s + d.c;
    const double* T = Tp + d.woff;
    const double* Tbar = Tb + d.woff;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, m16 = lane & 15, q4 = lane >> 4;
    const int nt = (s + 15) / 16;
    // rows, columns and contraction indices past s read the last one instead;
    // what they give is masked (k) or never stored (i, j)
    const double* Tj = T + (int64_t)min(j0 + m16, s - 1) * s;
    for (int p = wave; p < nt; p += kThreads / 64) {
        const int i = min(p * 16 + m16, s - 1);
        d4 acc = {0, 0, 0, 0};
        for (int k0 = 0; k0 < s; k0 += 32)
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const int kt = k0 + 4 * t + q4, k = min(kt, s - 1);
                const double a = Tbar[i + (int64_t)k * s] + Tbar[k + (int64_t)i * s];
                acc = mfma(kt < s ? a : 0.0, Tj[k], acc);
            }
        mfma_drain();
#pragma unroll
        for (int v = 0; v < 4; ++v) Q[p * 16 + q4 + 4 * v][m16] = acc[v];
    }
    __syncthreads();
    for (int p = (j0 >> 4) + wave; p < nt; p += kThreads / 64) {
        const int i = min(p * 16 + m16, s - 1);
        d4 acc = {0, 0, 0, 0};
        for (int k0 = 0; k0 < s; k0 += 32)
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const int kt = k0 + 4 * t + q4, k = min(kt, s - 1);
                const double a = T[i + (int64_t)k * s];
                acc = mfma(kt < s ? a : 0.0, Q[k][m16], acc);
            }
        mfma_drain();
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int ii = p * 16 + q4 + 4 * v, jj = j0 + m16;
            if (ii < s && jj < s && ii >= jj) Zb[d.poff + ii + (int64_t)jj * ld] = ii == jj ? -0.5 * acc[v] : -acc[v];
        }
    }
}

// ---------------------------------------------------------------------------
// host-side launchers
// ---------------------------------------------------------------------------
hipEvent_t Prof::next()
{
    if (used == pool.size()) {
        hipEvent_t e = nullptr;
        if (hipEventCreate(&e) != hipSuccess) return nullptr;
        pool.push_back(e);
    }
    return pool[used++];
}

Prof::~Prof()
{
    for (hipEvent_t e : pool) (void)hipEventDestroy(e);
}

template <class Kern, class... Args>
static void launch_wg(Prof* P, int kind, Kern kern, dim3 grid, int threads, size_t shmem, hipStream_t s, Args... args)
{
    if (P && P->on) {
        hipEvent_t a = P->next(), z = P->next();
        if (a && z) {
            hipExtLaunchKernelGGL(kern, grid, dim3((unsigned)threads), (uint32_t)shmem, s, a, z, 0, args...);
            P->kinds.push_back(kind);
            return;
        }
    }
    hipLaunchKernelGGL(kern, grid, dim3((unsigned)threads), shmem, s, args...);
}

template <class Kern, class... Args>
static void launch(Prof* P, int kind, Kern kern, dim3 grid, size_t shmem, hipStream_t s, Args... args)
{
    launch_wg(P, kind, kern, grid, kThreads, shmem, s, args...);
}

static inline unsigned grid_for(int64_t n)
{
    int64_t g = (n + kThreads - 1) / kThreads;
    if (g > 65536) g = 65536;
    if (g < 1) g = 1;
    return (unsigned)g;
}

hipError_t launch_backward_init(Prof* P, const DevPtrs& D, int64_t arena, int64_t harena, const double* gsel,
                                int64_t nnzL, hipStream_t s)
{
    hipError_t e = launch_fill(P, kRevSel, D.Zb, arena, 0.0, s);
    if (!e) e = launch_fill(P, kRevSel, D.Hb, harena, 0.0, s);
    if (!e) e = launch_scatter_set(P, kRevSel, gsel, D.exp_off, nnzL, D.Zb, s);
    return e;
}

hipError_t launch_revsel_level(Prof* P, const DevPtrs& D, int64_t a0, int64_t na, int64_t b0, int64_t nb,
                               const int64_t* rs3_cuts, int ncuts, int64_t d0, int64_t nd, int smax, hipStream_t s)
{
    if (nd > 0)  // a work-group per 1024 entries of the widest block (per 4096: 8.3 us a level, now 4.7)
        launch(P, kRevSel, k_tbar_init, dim3((unsigned)nd, (unsigned)((smax * smax + 1023) / 1024)), 0, s,
               D.t_diag + d0, D.blocks, (const double*)D.Zb, D.Tb);
    if (na > 0)
        launch(P, kRevSel, k_rs1, dim3((unsigned)na), 0, s, D.t_rs1 + a0, D.blocks, D.Zb, (const double*)D.Hp,
               (const double*)D.Tb);
    if (nb > 0)
        launch(P, kRevSel, k_rs2, dim3((unsigned)nb), 0, s, D.t_rs2 + b0, D.blocks, (const double*)D.Ap,
               (const double*)D.Zb, (const double*)D.Tb, D.Hb, D.cr2, D.rel);
    for (int g = 0; g + 1 < ncuts; g++) {
        const int64_t n = rs3_cuts[g + 1] - rs3_cuts[g];
        if (n > 0)
            launch(P, kRevSel, k_rs3, dim3((unsigned)n), 0, s, D.t_rs3 + rs3_cuts[g], D.blocks, D.Zb,
                   (const double*)D.Hp, D.cr2, D.rel);
    }
    return hipGetLastError();
}

hipError_t launch_revfac_init(Prof* P, const DevPtrs& D, int64_t arena, hipStream_t s)
{
    return launch_fill(P, kRevFac, D.Zb, arena, 0.0, s);
}

hipError_t launch_revfac_level(Prof* P, const DevPtrs& D, int64_t a0, int64_t na, int64_t b0, int64_t nb, int64_t c0,
                               int64_t nc, int64_t d0, int64_t nd, int smax, hipStream_t s)
{
    if (na > 0)
        launch(P, kRevFac, k_rf1a, dim3((unsigned)na), 0, s, D.t_rf1a + a0, D.blocks, (const double*)D.Zb,
               (const double*)D.Lp, D.Hb, D.cr2, D.rel);
    if (nb > 0)
        launch(P, kRevFac, k_rf1b, dim3((unsigned)nb), 0, s, D.t_rf1b + b0, D.blocks, D.Zb, (const double*)D.Hp,
               (const double*)D.Hb, (const double*)D.Tp, D.cr2, D.rel);
    if (nc > 0)
        launch(P, kRevFac, k_rf2, dim3((unsigned)nc), 0, s, D.t_rf2 + c0, D.blocks, (const double*)D.Lp,
               (const double*)D.Hb, D.Tb);
    if (nd > 0)
        launch(P, kRevFac, k_rf3, dim3((unsigned)nd, (unsigned)(smax + 15) / 16), 0, s, D.t_diag + d0, D.blocks, (const double*)D.Tp,
               (const double*)D.Tb, D.Zb);
    return hipGetLastError();
}

hipError_t launch_status_reset(unsigned long long* status, hipStream_t s)
{
    hipLaunchKernelGGL(k_status_reset, dim3(1), dim3(64), 0, s, status);
    return hipGetLastError();
}

hipError_t launch_fill(Prof* P, int kind, double* p, int64_t n, double v, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    launch(P, kind, k_fill, dim3(grid_for(n)), 0, s, p, n, v);
    return hipGetLastError();
}

hipError_t launch_scatter_set(Prof* P, int kind, const double* src, const int64_t* off, int64_t n, double* dst,
                              hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    launch(P, kind, k_scatter_set, dim3(grid_for(n)), 0, s, src, off, n, dst);
    return hipGetLastError();
}

hipError_t launch_gather(Prof* P, int kind, const double* src, const int64_t* off, int64_t n, double* dst,
                         hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    launch(P, kind, k_gather, dim3(grid_for(n)), 0, s, src, off, n, dst);
    return hipGetLastError();
}

hipError_t launch_zero_x(Prof* P, const DevPtrs& D, int64_t t0, int64_t n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    launch(P, kGemm, k_zero_x, dim3((unsigned)n), 0, s, D.t_zero + t0, D.blocks, D.Ap, (const double*)D.Tp);
    return hipGetLastError();
}

hipError_t launch_checkpoint(Prof* P, const DevPtrs& D, int64_t ntasks, int dir, hipStream_t s)
{
    if (ntasks <= 0) return hipSuccess;
    const int64_t parts = std::max<int64_t>(1, std::min<int64_t>(32, (1 << 18) / ntasks));
    launch(P, kCheckpoint, k_ck_copy, dim3((unsigned)ntasks, (unsigned)parts), 0, s, D.t_diag, D.blocks, D.ck_off, D.Ap, D.ck, dir);
    return hipGetLastError();
}

hipError_t launch_export_L(Prof* P, const DevPtrs& D, int64_t n, double* out, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    launch(P, kExport, k_export_L, dim3(grid_for(n)), 0, s, D.blocks, D.colblk, D.colptrL, D.exp_off, n,
           (const double*)D.Lp, (const double*)D.Hp, out);
    return hipGetLastError();
}

hipError_t launch_sb_factor(Prof* P, const DevPtrs& D, int64_t sb0, int64_t nsb, int require_spd, hipStream_t s)
{
    if (nsb > 0)
        launch(P, kSbFactor, k_sb_factor, dim3((unsigned)nsb), 0, s, D.t_sb + sb0, D.blocks, D.Lp, D.Hp, D.Tp, D.cr2,
               D.rel, D.status, require_spd);
    return hipGetLastError();
}

hipError_t launch_sb_invert(Prof* P, const DevPtrs& D, int64_t sb0, int64_t nsb, hipStream_t s)
{
    if (nsb > 0)
        launch(P, kSbInvert, k_sb_invert, dim3((unsigned)nsb), 0, s, D.t_sb + sb0, D.blocks, D.Ap, (const double*)D.Hp,
               (const double*)D.Tp, D.cr2, D.rel);
    return hipGetLastError();
}

hipError_t launch_ldlt_bk(Prof* P, const DevPtrs& D, const int64_t diag[4], hipStream_t s)
{
    // by width class: [diag[0], diag[1]) s <= 32, then <= 64, then <= 128
    if (diag[1] > diag[0])
        launch(P, kLdlt, k_ldlt_bk<2>, dim3((unsigned)(diag[1] - diag[0])), 0, s, D.t_ldlt + diag[0], D.blocks,
               (const double*)D.Lp, D.Tp, D.status);
    if (diag[2] > diag[1])
        launch(P, kLdlt, k_ldlt_bk<4>, dim3((unsigned)(diag[2] - diag[1])), 0, s, D.t_ldlt + diag[1], D.blocks,
               (const double*)D.Lp, D.Tp, D.status);
    if (diag[3] > diag[2])
        launch(P, kLdlt, k_ldlt_bk<8>, dim3((unsigned)(diag[3] - diag[2])), 0, s, D.t_ldlt + diag[2], D.blocks,
               (const double*)D.Lp, D.Tp, D.status);
    return hipGetLastError();
}

hipError_t launch_ldlt_level(Prof* P, const DevPtrs& D, const int64_t diag[4], int require_spd, hipStream_t s)
{
    // diagonal blocks by width class: [diag[0], diag[1]) s <= 32, then <= 64,
    // then wider
    if (diag[1] > diag[0])
        launch_wg(P, kLdlt, k_ldlt_diag<2>, dim3((unsigned)(diag[1] - diag[0])), 64 * diag_waves(2), 0, s, D.t_ldlt + diag[0],
                  D.blocks, D.Lp, D.Wp, D.Tp, D.status, require_spd);
    if (diag[2] > diag[1])
        launch_wg(P, kLdlt, k_ldlt_diag<4>, dim3((unsigned)(diag[2] - diag[1])), 64 * diag_waves(4), 0, s, D.t_ldlt + diag[1],
                  D.blocks, D.Lp, D.Wp, D.Tp, D.status, require_spd);
    if (diag[3] > diag[2])
        launch_wg(P, kLdlt, k_ldlt_diag<8>, dim3((unsigned)(diag[3] - diag[2])), 64 * diag_waves(8), 0, s, D.t_ldlt + diag[2],
                  D.blocks, D.Lp, D.Wp, D.Tp, D.status, require_spd);
    return hipGetLastError();
}

hipError_t launch_panel_level(Prof* P, const DevPtrs& D, int64_t panel0, int64_t npanel, int panel_deep, hipStream_t s)
{
    // panel_deep: bit 0 the level has few panel tiles; bit 1 its blocks are
    // narrow enough for the kernels of few tiles (s <= kDeepK)
    if (npanel > 0 && (panel_deep & 1))
        launch(P, kPanel, k_panel_few, dim3((unsigned)(4 * npanel)), 0, s, D.t_panel + panel0, D.blocks,
               (const double*)D.Lp, D.Hp, (const double*)D.Tp);
    else if (npanel > 0)
        launch(P, kPanel, k_panel, dim3((unsigned)npanel), 0, s, D.t_panel + panel0, D.blocks, (const double*)D.Lp,
               D.Hp, (const double*)D.Tp);
    return hipGetLastError();
}

hipError_t launch_schur_groups(Prof* P, const DevPtrs& D, const int64_t* cuts, int g0, int g1, int panel_deep,
                               hipStream_t s)
{
    // one launch per colour group (groups update disjoint entries)
    for (int g = g0; g < g1; g++) {
        const int64_t n = cuts[g + 1] - cuts[g];
        if (n > 0 && (panel_deep & 2) && n <= kFewSchurTiles)
            launch(P, kSchur, k_schur_few, dim3((unsigned)(4 * n)), 0, s, D.t_schur + cuts[g], D.blocks, D.Lp,
                   (const double*)D.Hp, D.cr2, D.rel);
        else if (n > 0)
            launch(P, kSchur, k_schur, dim3((unsigned)n), 0, s, D.t_schur + cuts[g], D.blocks, D.Lp,
                   (const double*)D.Hp, D.cr2, D.rel);
    }
    return hipGetLastError();
}

hipError_t launch_invert_level(Prof* P, const DevPtrs& D, int64_t gemm0, int64_t ngemm, int64_t sdiag0,
                               int64_t sdiag_cut, int64_t sdiag1, hipStream_t s)
{
    if (ngemm > 0)
        launch(P, kGemm, k_gemm, dim3((unsigned)ngemm), 0, s, D.t_gemm + gemm0, D.blocks, D.Ap,
               (const double*)D.Hp, D.cr2, D.rel);
    if (sdiag_cut > sdiag0)
        launch(P, kSdiag, k_sdiag64, dim3((unsigned)(sdiag_cut - sdiag0)), 0, s, D.t_sdiag + sdiag0, D.blocks, D.Ap,
               (const double*)D.Hp, (const double*)D.Tp);
    if (sdiag1 > sdiag_cut)
        launch(P, kSdiag, k_sdiag64, dim3((unsigned)(sdiag1 - sdiag_cut)), 0, s, D.t_sdiag + sdiag_cut, D.blocks,
               D.Ap, (const double*)D.Hp, (const double*)D.Tp);
    return hipGetLastError();
}


// resident work-groups per CU of each persistent variant, in the order of
// selinv::PersistVariant
hipError_t persist_occupancy(int occ[kNumVariants])
{
    const void* k[kNumVariants] = {(const void*)k_light_factor<1>, (const void*)k_light_factor<2>, (const void*)k_light_factor<4>,       (const void*)k_persist_factor<2>,
                                   (const void*)k_persist_factor<4>,  (const void*)k_persist_factor<8>,
                                   (const void*)k_light_invert<2, false>, (const void*)k_light_invert<4, false>, (const void*)k_light_invert<4, true>,       (const void*)k_persist_invert<32>,
                                   (const void*)k_persist_invert<64>, (const void*)k_persist_invert<128>};
    hipError_t e = hipSuccess;
    for (int v = 0; v < kNumVariants && !e; v++) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(occ + v, k[v], kThreads, 0);
    return e;
}

hipError_t launch_fill_u32(Prof* P, int kind, unsigned* p, int64_t n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    launch(P, kind, k_fill_u32, dim3(grid_for(n)), 0, s, p, n);
    return hipGetLastError();
}

hipError_t launch_persist_factor(Prof* P, const DevPtrs& D, const Task* q, int64_t ntasks, unsigned* head,
                                 unsigned* done, int grid, int variant, int require_spd, unsigned spin_limit,
                                 hipStream_t s)
{
    if (ntasks <= 0) return hipSuccess;
    const QueueArgs a{q, ntasks, head, done, D.status, require_spd, spin_limit};
    const unsigned g = (unsigned)std::max<int64_t>(1, std::min<int64_t>(grid, ntasks));
#define SELINV_PF(K) launch(P, kQFactor, K, dim3(g), 0, s, a, D.blocks, D.Lp, D.Wp, D.Hp, D.Tp, D.rel, D.cr2)
#define SELINV_LF(K) launch(P, kQFactor, K, dim3(g), 0, s, a, D.blocks, D.Lp, D.Hp, D.Tp, D.cr2, D.rel)
    switch (variant) {
        case kLightFactor4: SELINV_LF(k_light_factor<1>); break;
        case kLightFactor8: SELINV_LF(k_light_factor<2>); break;
        case kLightFactor16: SELINV_LF(k_light_factor<4>); break;
        case kFactor32: SELINV_PF(k_persist_factor<2>); break;
        case kFactor64: SELINV_PF(k_persist_factor<4>); break;
        default: SELINV_PF(k_persist_factor<8>); break;
    }
#undef SELINV_LF
#undef SELINV_PF
    return hipGetLastError();
}

hipError_t launch_persist_invert(Prof* P, const DevPtrs& D, const Task* q, int64_t ntasks, unsigned* head,
                                 unsigned* done, int grid, int variant, unsigned spin_limit, hipStream_t s)
{
    if (ntasks <= 0) return hipSuccess;
    const QueueArgs a{q, ntasks, head, done, D.status, 0, spin_limit};
    const unsigned g = (unsigned)std::max<int64_t>(1, std::min<int64_t>(grid, ntasks));
#define SELINV_PI(K) \
    launch(P, kQInvert, K, dim3(g), 0, s, a, D.blocks, D.Ap, (const double*)D.Hp, (const double*)D.Tp, D.rel, D.cr2)
#define SELINV_LI(K) \
    launch(P, kQInvert, K, dim3(g), 0, s, a, D.blocks, D.Ap, (const double*)D.Hp, (const double*)D.Tp, D.cr2, D.rel)
    switch (variant) {
        case kLightInvert8: SELINV_LI((k_light_invert<2, false>)); break;
        case kLightInvert16: SELINV_LI((k_light_invert<4, false>)); break;
        case kLightInvert256: SELINV_LI((k_light_invert<4, true>)); break;
        case kInvert32: SELINV_PI(k_persist_invert<32>); break;
        case kInvert64: SELINV_PI(k_persist_invert<64>); break;
        default: SELINV_PI(k_persist_invert<128>); break;
    }
#undef SELINV_LI
#undef SELINV_PI
    return hipGetLastError();
}

}  // namespace selinv
