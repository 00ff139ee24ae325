// Complex-symmetric path: the same supernodal LDL^T and selected inversion
// (Algorithm 1) for A(z) = H - z S, the matrices of the pole expansion
// (Section 4.3).  Values are complex (re, im interleaved, 16 bytes each);
// every transpose is a plain transpose, never a conjugate.  Blocks are at
// most 64 columns wide; the plan's level schedule is the deterministic one
// (Schur updates in colour groups; a diagonal step's long contraction may be
// cut into pieces, summed afterwards in a fixed order), so no kernel here
// needs atomics.  Products run on FP64 MFMA: a 64 x 64 complex output
// tile per work-group, real and imaginary parts as separate accumulators,
// operands staged through LDS in 8-deep chunks.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "kernels.hpp"
#include "lanes.hpp"
#include "plan.hpp"
#include "tiles.hpp"

namespace selinv {
namespace {

typedef double z2 __attribute__((ext_vector_type(2)));  // (re, im)

__device__ __forceinline__ z2 zmul(z2 a, z2 b) { return z2{a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x}; }

constexpr int kZT = 64;  // output tile edge
constexpr int kZK = 8;   // contraction chunk

// ---------------------------------------------------------------------------
// A 64 x 64 complex product tile on FP64 MFMA: four waves of 32 x 32 (2 x 2
// MFMA tiles each), and per 4-deep step four real products per output tile:
//   C_re += A_re B_re - A_im B_im,  C_im += A_re B_im + A_im B_re.
// v_mfma_f64_16x16x4f64: lane l holds A[l%16][l/16], B[l/16][l%16]; result
// element (l/16 + 4 v, l%16) in register v.
//
// What bounds it: FP64 MFMAs and vector instructions share the SIMD's FP64
// hardware, so the loops issue few of the latter.  Operands go through LDS as
// rows of kZK complex contraction entries (128 bytes), their 16-byte slots
// exclusive-or'ed with row / 2 mod 8 (conflict-free 16-byte reads, no
// padding): one read gives an MFMA step its real and its imaginary operand.
// Two buffers, one barrier per chunk; global operands are read through buffer
// descriptors, a chunk's position being a scalar offset.
// 32 poles of n = 8,000 (factor + inversion): 34.9 -> 31.2 ms.
// ---------------------------------------------------------------------------
typedef double zd4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ zd4 zmfma(double a, double b, zd4 c)
{
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

constexpr int kZRow = kZK * (int)sizeof(z2);

struct alignas(16) ZLds {
    char A[2][kZT * kZRow], B[2][kZT * kZRow];
};

struct ZAcc {
    zd4 re[2][2], im[2][2];
};

struct ZNoHook {
    __device__ void operator()() const {}
};

// LDS byte offset of entry (row, k)
__device__ __forceinline__ int zat(int row, int k) { return row * kZRow + ((k ^ ((row >> 1) & 7)) << 4); }

// The products of one chunk in LDS, `between` run between its two steps'
// fragment reads.  kT: accumulated transposed (lane l % 16 is a row of the
// tile, so that stores run down the columns of a panel).
template <bool kT, class FB>
__device__ __forceinline__ void zproducts(const char* A, const char* B, ZAcc& acc, FB between)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const char *Aw = A + (wave & 1) * 32 * kZRow, *Bw = B + (wave >> 1) * 32 * kZRow;
    const int f[2] = {zat(lane & 15, lane >> 4), zat(lane & 15, 4 + (lane >> 4))};
    z2 x[2], y[2];
    auto frags = [&](int t) {
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            x[m] = *reinterpret_cast<const z2*>(Aw + f[t] + m * 16 * kZRow);
            y[m] = *reinterpret_cast<const z2*>(Bw + f[t] + m * 16 * kZRow);
        }
    };
    auto mma = [&]() {
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int n = 0; n < 2; ++n) {
                const z2 a = kT ? y[n] : x[m], b = kT ? x[m] : y[n];
                acc.re[m][n] = zmfma(a.x, b.x, acc.re[m][n]);
                acc.im[m][n] = zmfma(a.x, b.y, acc.im[m][n]);
                acc.re[m][n] = zmfma(-a.y, b.y, acc.re[m][n]);
                acc.im[m][n] = zmfma(a.y, b.x, acc.im[m][n]);
            }
    };
    frags(0);
    between();
    mma();
    frags(1);
    mma();
}

__device__ __forceinline__ void zdrain()
{
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 15\n\ts_nop 15" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// A column-major complex array p[0 .. count), columns ld apart
struct ZOperand {
    __amdgpu_buffer_rsrc_t rsrc;
    uint32_t ld16;  // bytes between columns
};
__device__ __forceinline__ ZOperand zoperand(const double* p, int64_t off, int64_t count, int64_t ld)
{
    return {__builtin_amdgcn_make_buffer_rsrc((void*)(p + 2 * off), 0,
                                              (int)(uint32_t)((count > 0 ? count : 0) * (int64_t)sizeof(z2)), 0x00020000),
            (uint32_t)(ld * (int64_t)sizeof(z2))};
}
__device__ __forceinline__ z2 zbuffer(const ZOperand& o, uint32_t voff, uint32_t soff)
{
    return __builtin_bit_cast(z2, __builtin_amdgcn_raw_buffer_load_b128(o.rsrc, (int)voff, (int)soff, 0));
}

// One operand of 64 rows; row r holds its contraction entry k at p[r + k ld]
// (lanes along the rows; entries past the contraction are past the array and
// read 0) or, kAlongK, at p[k + r ld] (lanes along k; entries past Ke read
// the last one and are masked where `mask`).
template <bool kAlongK>
struct ZLoader {
    ZOperand o;
    uint32_t voff;
    int kk, wr[2];
    __device__ __forceinline__ ZLoader(const ZOperand& op, int wave) : o(op)
    {
        const int t = threadIdx.x, lane = t & 63;
        if constexpr (kAlongK) {
            kk = t & 7;
            voff = (uint32_t)(t >> 3) * o.ld16 + (uint32_t)kk * 16u;
            wr[0] = zat(t >> 3, kk);
            wr[1] = wr[0] + 32 * kZRow;
        } else {
            kk = wave;
            voff = (uint32_t)lane * 16u;
            wr[0] = zat(lane, wave);
            wr[1] = zat(lane, 4 + wave);
        }
    }
    __device__ __forceinline__ void load(z2 (&v)[2], int k0, int Ke) const
    {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            if constexpr (kAlongK) {
                const uint32_t back = k0 + kZK > Ke ? (uint32_t)(kk - min(kk, Ke - 1 - k0)) * 16u : 0u;
                v[q] = zbuffer(o, voff + (uint32_t)q * 32u * o.ld16 - back, (uint32_t)k0 * 16u);
            } else {
                v[q] = zbuffer(o, voff, (uint32_t)(k0 + 4 * q + kk) * o.ld16);
            }
        }
    }
    __device__ __forceinline__ void store(char* lds, const z2 (&v)[2], int k0, bool mask, int Ke) const
    {
#pragma unroll
        for (int q = 0; q < 2; ++q)
            *reinterpret_cast<z2*>(lds + wr[q]) = kAlongK && mask && k0 + kk >= Ke ? z2{0.0, 0.0} : v[q];
    }
};

// acc += A B over [Kb, Ke); after_first: loads of the caller's own, issued
// once the first chunks' operand loads are in flight (they may then wait
// under the products).  Loads are issued two chunks ahead.
template <bool kAk, bool kBk, bool kT, class AF = ZNoHook>
__device__ __forceinline__ void zdense(ZLds& L, const ZOperand& oa, const ZOperand& ob, int Kb, int Ke, ZAcc& acc,
                                       AF after_first = AF())
{
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int nch = Ke > Kb ? (Ke - Kb + kZK - 1) / kZK : 0;
    const ZLoader<kAk> la(oa, wave);
    const ZLoader<kBk> lb(ob, wave);
    z2 va[2][2], vb[2][2];  // by the chunk's parity
    auto k_of = [&](int ch) { return Kb + min(ch, nch - 1) * kZK; };
    auto load = [&](z2 (&a)[2], z2 (&b)[2], int ch) {
        la.load(a, k_of(ch), Ke);
        lb.load(b, k_of(ch), Ke);
    };
    auto store = [&](const z2 (&a)[2], const z2 (&b)[2], int ch, int buf) {
        la.store(L.A[buf], a, k_of(ch), true, Ke);
        lb.store(L.B[buf], b, k_of(ch), false, Ke);
    };
    if (nch > 0) {
        z2 a0[2], b0[2];
        load(a0, b0, 0);
        __builtin_amdgcn_sched_barrier(0);
        load(va[1], vb[1], 1);
        __builtin_amdgcn_sched_barrier(0);
        load(va[0], vb[0], 2);
        __builtin_amdgcn_sched_barrier(0);
        store(a0, b0, 0, 0);
    }
    after_first();
    __syncthreads();
    auto body = [&](auto X, int ch) {  // X: the parity of ch
        constexpr int buf = decltype(X)::value;
        zproducts<kT>(L.A[buf], L.B[buf], acc, [&] {
            store(va[buf ^ 1], vb[buf ^ 1], ch + 1, buf ^ 1);
            load(va[buf ^ 1], vb[buf ^ 1], ch + 3);
            __builtin_amdgcn_sched_barrier(0);
        });
        __syncthreads();
    };
    int ch = 0;
    for (; ch + 1 < nch; ch += 2) {
        body(std::integral_constant<int, 0>{}, ch);
        body(std::integral_constant<int, 1>{}, ch + 1);
    }
    if (ch < nch) body(std::integral_constant<int, 0>{}, ch);
    zdrain();
}

// f(i, j, value) for every element of a tile accumulated transposed
template <class F>
__device__ __forceinline__ void zvisit(const ZAcc& acc, F f)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm0 = (wave & 1) * 32, wn0 = (wave >> 1) * 32;
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int n = 0; n < 2; ++n)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                f(wm0 + 16 * m + (lane & 15), wn0 + 16 * n + (lane >> 4) + 4 * v, z2{acc.re[m][n][v], acc.im[m][n][v]});
}

__device__ __forceinline__ z2 zload(const double* p, int64_t e) { return *reinterpret_cast<const z2*>(p + 2 * e); }
__device__ __forceinline__ void zstore(double* p, int64_t e, z2 v) { *reinterpret_cast<z2*>(p + 2 * e) = v; }

// 1 / d = s inv: the power of two s is taken from d's larger part, so that
// |d s|^2 is in [1, 32)
__device__ __forceinline__ z2 zrecip(z2 d, double& s)
{
    s = pow2_scale(fmax(fabs(d.x), fabs(d.y)));
    const z2 f = d * s;
    const double r = recip3(fma(f.x, f.x, f.y * f.y));
    return z2{f.x * r, -(f.y * r)};
}

// 1 / d to about half a unit in the last place of its size: a Newton step from
// zrecip, with the residual 1 - f inv of the scaled f from exact products.
// These are D^{-1}'s entries, which a diagonally dominant block's inverse has
// on its diagonal.
__device__ __forceinline__ z2 zrecip_refined(z2 d)
{
#pragma clang fp contract(off)
    double s;
    const z2 i = zrecip(d, s), f = d * s;
    const double p = f.x * i.x, q = f.y * i.x;
    const double ex = fma(f.y, i.y, 1.0 - p) - fma(f.x, i.x, -p);
    const double ey = -(fma(f.x, i.y, q) + fma(f.y, i.x, -q));
    return z2{fma(i.x, ex, fma(-i.y, ey, i.x)), fma(i.x, ey, fma(i.y, ex, i.y))} * s;
}

// ---------------------------------------------------------------------------
// Diagonal block, s <= 64: T_K = F_KK^{-1} by the symmetric sweep of one pivot
// after the other, natural order, plain (not conjugate) products, arranged by
// pivot blocks of 16 columns.  Block p is factored in one wave's registers
// (zldl16: M(p, p) = L_p D_p L_p^T).  For every block row R, with C(R) = M(R, p),
// and C(p) = -I, Y(R) = C(R) L_p^{-T} by substitution, column after column, and
// l(R) = Y(R) D_p^{-1}; then M(I, J) = M'(I, J) - l(I) Y(J)^T for every tile,
// with M' = M outside row and column p and 0 in them.  After the last block
// M = -F_KK^{-1} = -T_K; only T leaves the kernel.
// These are the scalar sweep's operations in its order: no block is inverted on
// the way, so a nearly singular pivot block costs what it costs pivot by pivot.
// Complex symmetric, 64 columns, leading 16 x 16 block with an eigenvalue
// 1e-4 of its diagonal (1e-6), largest relative error of T in the median:
// scalar sweep 1.6e-12 (1.3e-10), this 3.4e-12 (3.7e-10), with the blocks'
// inverses 8e-9 (6e-5).
//
// What bounds it is the chain of s dependent pivots: wave 0 factors the pivot
// blocks in its own registers (lane broadcasts, no LDS, no barrier) while the
// other three waves update the tiles of M, which stay in their registers, with
// MFMA products; the tiles of the next step's column go through LDS.  A block
// of 64 columns: 25 us against 50 us when every pivot's column went through
// LDS behind a barrier.  Rows and columns past s hold the identity.  A zero or
// non-finite pivot latches its column.
// ---------------------------------------------------------------------------
// 16 complex entries a row and 16 bytes: conflict-free operand reads
constexpr int kZDiagPad = 17;
constexpr int kZNB = kZT / 16, kZNT = kZNB * (kZNB + 1) / 2;
struct ZDiagLds {
    z2 M[kZNB][16][kZDiagPad];               // C(R) of the next step
    z2 P[16][kZDiagPad];                     // the pivot block after it
    z2 C[kZT][kZDiagPad], N[kZT][kZDiagPad]; // Y(R), -l(R)
    z2 Lb[2][16][kZDiagPad];                 // -L_p below its diagonal, else 0
    z2 inv[2][16];                           // 1 / D_p
};

// Elimination of a symmetric 16 x 16 block, lane (m, g) holding row m, columns
// g + 4 v; X(., j): column j as pivot j finds it (d_j in row j), and what has
// been left of the rows above.  P is used up.  The part not yet eliminated
// stays symmetric to the last bit: c_i c_k is formed first, its imaginary part
// from two rounded products, alike for (i, k) and (k, i).  Rows from n on hold
// the identity; pivots from the next multiple of 4 on are skipped.
__device__ __forceinline__ void zldl16(z2 (&P)[4], z2 (&X)[4], const int g, const int n)
{
    auto column = [](auto jc, const z2& p) {
        constexpr int G = decltype(jc)::value & 3;
        return z2{row_copy<G>(p.x), row_copy<G>(p.y)};
    };
    z2 c = column(std::integral_constant<int, 0>{}, P[0]);  // column j in every lane (m, .)
    StaticFor<0, 4>::run([&](auto vc) {
        constexpr int vj = decltype(vc)::value;
        if (4 * vj >= n) return;  // uniform
        StaticFor<4 * vj, 4 * vj + 4>::run([&](auto jc) {
            constexpr int j = decltype(jc)::value, j1 = j < 15 ? j + 1 : 15;
            double s;
            const z2 inv = zrecip(z2{row_lane<j>(c.x), row_lane<j>(c.y)}, s), u = c * s;
            auto less = [&](z2 p, z2 b) {  // p - (u b) inv, one rounding at p's size
#pragma clang fp contract(off)
                const double re = fma(-u.y, b.y, u.x * b.x), im = u.x * b.y + u.y * b.x;
                return z2{p.x - fma(-im, inv.y, re * inv.x), p.y - fma(im, inv.x, re * inv.y)};
            };
            // the next column, broadcast before its update
            const z2 next = column(std::integral_constant<int, j1>{}, P[j1 >> 2]);
            const z2 cn = less(next, z2{row_lane<j1>(c.x), row_lane<j1>(c.y)});
#pragma unroll
            for (int v = j1 >> 2; v < 4; ++v) P[v] = less(P[v], z2{row_lane<j>(P[v].x), row_lane<j>(P[v].y)});
            if (g == (j & 3)) X[vj] = c;
            c = cn;
        });
    });
}

// Y = C L^{-T} for a unit lower triangular L and 16 rows, lane (m, g) holding
// rows g + 4 v, column m.  lb: -L(m, j), 0 for m <= j.  Broadcasts within the
// rows of 16 lanes in the instruction itself, at least three other
// instructions after the write of what they read.
__device__ __forceinline__ void zsubstitute16(z2 (&x)[4], const z2 (&lb)[16])
{
    double r[4], i[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) r[v] = x[v].x, i[v] = x[v].y;
#define SELINV_FMAC(D, S, L, J) "v_fmac_f64_dpp %" #D ", " S ", %[" L "] row_newbcast:" #J " row_mask:0xf bank_mask:0xf\n\t"
#define SELINV_STEP(J) \
    SELINV_FMAC(0, "%0", "x" #J, J) SELINV_FMAC(1, "%1", "x" #J, J) SELINV_FMAC(2, "%2", "x" #J, J) SELINV_FMAC(3, "%3", "x" #J, J) \
    SELINV_FMAC(4, "%4", "x" #J, J) SELINV_FMAC(5, "%5", "x" #J, J) SELINV_FMAC(6, "%6", "x" #J, J) SELINV_FMAC(7, "%7", "x" #J, J) \
    SELINV_FMAC(0, "-%4", "y" #J, J) SELINV_FMAC(1, "-%5", "y" #J, J) SELINV_FMAC(2, "-%6", "y" #J, J) SELINV_FMAC(3, "-%7", "y" #J, J) \
    SELINV_FMAC(4, "%0", "y" #J, J) SELINV_FMAC(5, "%1", "y" #J, J) SELINV_FMAC(6, "%2", "y" #J, J) SELINV_FMAC(7, "%3", "y" #J, J)
#define SELINV_ROWS "+v"(r[0]), "+v"(r[1]), "+v"(r[2]), "+v"(r[3]), "+v"(i[0]), "+v"(i[1]), "+v"(i[2]), "+v"(i[3])
#define SELINV_LB(J) [x##J] "v"(lb[J].x), [y##J] "v"(lb[J].y)
    asm volatile("s_nop 1\n\t" SELINV_STEP(0) SELINV_STEP(1) SELINV_STEP(2) SELINV_STEP(3) SELINV_STEP(4) SELINV_STEP(5)
                     SELINV_STEP(6) SELINV_STEP(7)
                 : SELINV_ROWS
                 : SELINV_LB(0), SELINV_LB(1), SELINV_LB(2), SELINV_LB(3), SELINV_LB(4), SELINV_LB(5), SELINV_LB(6),
                   SELINV_LB(7));
    asm volatile("s_nop 1\n\t" SELINV_STEP(8) SELINV_STEP(9) SELINV_STEP(10) SELINV_STEP(11) SELINV_STEP(12) SELINV_STEP(13)
                     SELINV_STEP(14)
                 : SELINV_ROWS
                 : SELINV_LB(8), SELINV_LB(9), SELINV_LB(10), SELINV_LB(11), SELINV_LB(12), SELINV_LB(13),
                   SELINV_LB(14));
#undef SELINV_LB
#undef SELINV_ROWS
#undef SELINV_STEP
#undef SELINV_FMAC
#pragma unroll
    for (int v = 0; v < 4; ++v) x[v] = z2{r[v], i[v]};
}

// (re, im) += a b, 16 x 16 blocks as lane (m, g) holds them: entry
// (m, g + 4 v) of a, and of b transposed, in register v
__device__ __forceinline__ void zblock_mma(const z2 (&a)[4], const z2 (&b)[4], zd4& re, zd4& im)
{
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        re = zmfma(a[v].x, b[v].x, re);
        im = zmfma(a[v].x, b[v].y, im);
        re = zmfma(-a[v].y, b[v].y, re);
        im = zmfma(a[v].y, b[v].x, im);
    }
}

__global__ __launch_bounds__(kThreads) void k_zdiag(const Task* __restrict__ tasks, const BlockDesc* __restrict__ blk,
                                                    double* __restrict__ Lp, double* __restrict__ Tp,
                                                    unsigned long long* __restrict__ status)
{
    __shared__ ZDiagLds S;
    const BlockDesc d = blk[tasks[blockIdx.x].b];
    const int s = d.s, nb = (s + 15) >> 4;
    const int64_t ld = (int64_t)d.s + d.c;
    const int lane = threadIdx.x & 63, m = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const bool chain = wave == 0;
    constexpr int NK = kThreads / 64 - 1, NL = (kZNT + NK - 1) / NK;  // tile waves, tiles of each
    static_assert(kThreads / 64 >= kZNB, "a block row for every wave");
    const int wk = chain ? 0 : wave - 1;
    // factor the pivot block P of step p
    auto pivots = [&](int p, const z2 (&P)[4]) {
        const int buf = p & 1;
        z2 Q[4], C[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            Q[v] = P[v];
            C[v] = z2{m == g + 4 * v ? 1.0 : 0.0, 0.0};
        }
        zldl16(Q, C, g, s - 16 * p);
        z2 dm = C[0];
#pragma unroll
        for (int v = 1; v < 4; ++v)
            if (m >> 2 == v) dm = C[v];
        const z2 im = zrecip_refined(dm);
        if (g == (m & 3)) {
            S.inv[buf][m] = im;
            if (16 * p + m < s && !((dm.x != 0.0 || dm.y != 0.0) && isfinite(dm.x) && isfinite(dm.y)))
                atomicMin(status, (unsigned long long)(d.first + 16 * p + m));
        }
        wave_sync();
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int k = g + 4 * v;
            S.Lb[buf][m][k] = m > k ? -zmul(C[v], S.inv[buf][k]) : z2{0.0, 0.0};
        }
    };
    // F(i, j) of tile (I, J), the identity past s
    auto load_tile = [&](int I, int J, z2 (&x)[4]) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int i = 16 * I + m, j = 16 * J + g + 4 * v;
            const int a = min(max(i, j), s - 1), b = min(min(i, j), s - 1);
            const z2 f = zload(Lp, d.poff + a + (int64_t)b * ld);
            x[v] = i < s && j < s ? f : z2{i == j ? 1.0 : 0.0, 0.0};
        }
    };
    // this wave's tiles, every NK-th, as real and imaginary parts
    const int nt = nb * (nb + 1) / 2;
    zd4 re[NL], im[NL];
    int I[NL], J[NL];
    z2 P[4];  // the chain's next pivot block
#pragma unroll
    for (int u = 0; u < NL; ++u) {
        // row by row: rows 1 .. 3 start at tiles 1, 3, 6
        const int t = min(u * NK + wk, nt - 1);
        I[u] = __builtin_popcount((1u << 1 | 1u << 3 | 1u << 6) & ((2u << t) - 1));
        J[u] = t - (int)((unsigned)(I[u] * (I[u] + 1)) >> 1);
        if (!chain) {
            z2 x[4];
            load_tile(I[u], J[u], x);
#pragma unroll
            for (int v = 0; v < 4; ++v) re[u][v] = x[v].x, im[u][v] = x[v].y;
        }
    }
    if (chain) load_tile(0, 0, P);
    // step -1 only factors the first pivot block
    for (int p = -1; p < nb; ++p) {
        const int buf = p & 1;
        const bool more = p + 1 < nb;
        // Y(R) and -l(R), rows R = p + 1 (wave 0), p + 2, .. cyclically to p;
        // lane (m, g) holds rows g + 4 v, column m
        if (p >= 0 && wave < nb) {
            const int R = p + 1 + wave < nb ? p + 1 + wave : p + 1 + wave - nb;
            z2 x[4], lb[16];
#pragma unroll
            for (int j = 0; j < 15; ++j) lb[j] = S.Lb[buf][m][j];
            const z2 inv = S.inv[buf][m];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const z2 c = S.M[R][g + 4 * v][m];
                x[v] = R != p ? c : z2{m == g + 4 * v ? -1.0 : 0.0, 0.0};
            }
            zsubstitute16(x, lb);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                S.C[16 * R + g + 4 * v][m] = x[v];
                S.N[16 * R + g + 4 * v][m] = -zmul(x[v], inv);
            }
        }
        if (chain && more && p >= 0) {
            // the next pivot block: its update needs nothing from the other
            // waves.  Its upper entries are the lower ones: exactly symmetric
            wave_sync();
            z2 x[4], y[4], n[4];
            zd4 pr = {0, 0, 0, 0}, pi = {0, 0, 0, 0};
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                x[v] = S.P[m][g + 4 * v];
                y[v] = S.C[16 * (p + 1) + m][g + 4 * v];
                n[v] = S.N[16 * (p + 1) + m][g + 4 * v];
            }
            zblock_mma(y, n, pr, pi);
            zdrain();
#pragma unroll
            for (int v = 0; v < 4; ++v) S.P[m][g + 4 * v] = x[v] + z2{pr[v], pi[v]};
            wave_sync();
#pragma unroll
            for (int v = 0; v < 4; ++v) P[v] = S.P[max(m, g + 4 * v)][min(m, g + 4 * v)];
        }
        __syncthreads();
        if (!chain) {
            // M(I, J) = M'(I, J) - l(I) Y(J)^T, the product summed by itself:
            // into M it would round twice a pivot at M's size, where the
            // scalar sweep rounds once (T's error on the blocks of a 4^3-atom
            // pencil 3.8e-16 instead of 1.9e-16; the scalar sweep's 2.9e-16).
            // In row and column p the sum takes the last pivot first: pivots
            // i .. 15 add to a diagonal entry (i, i), and its own, 1 / d_i, is
            // the large one.  The other tiles take the pivots as they come: a
            // small last pivot makes the large term, and comes last.
            if (p >= 0) {
#pragma unroll
                for (int u0 = 0; u0 < NL; u0 += 2) {
                    if (u0 * NK + wk >= nt) break;  // uniform
                    zd4 ar[2] = {}, ai[2] = {};
#pragma unroll
                    for (int u = u0; u < min(u0 + 2, NL); ++u) {
                        z2 a[4], b[4];
                        const int r = I[u] == p || J[u] == p ? 3 : 0;
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            a[v] = S.C[16 * J[u] + m][g + 4 * (v ^ r)];
                            b[v] = S.N[16 * I[u] + m][g + 4 * (v ^ r)];
                        }
                        zblock_mma(a, b, ar[u - u0], ai[u - u0]);
                    }
                    zdrain();
#pragma unroll
                    for (int u = u0; u < min(u0 + 2, NL); ++u) {
                        const bool zero = I[u] == p || J[u] == p;  // uniform
                        re[u] = zero ? ar[u - u0] : re[u] + ar[u - u0];
                        im[u] = zero ? ai[u - u0] : im[u] + ai[u - u0];
                    }
                }
            }
            // what the next step reads: the rows' tiles of its column, and
            // for wave 0 the pivot block after it (the next one is its own)
#pragma unroll
            for (int u = 0; u < NL; ++u) {
                if (u * NK + wk >= nt) break;  // uniform
                const bool col = J[u] == p + 1, row = I[u] == p + 1;
                z2* to = I[u] == J[u] ? S.P[0] : S.M[col ? I[u] : J[u]][0];
                if (I[u] == J[u] ? I[u] == p + 2 : col) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) to[m * kZDiagPad + g + 4 * v] = z2{re[u][v], im[u][v]};
                } else if (I[u] != J[u] && row) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) to[(g + 4 * v) * kZDiagPad + m] = z2{re[u][v], im[u][v]};
                }
            }
        }
        if (chain && more) pivots(p + 1, P);
        __syncthreads();
    }
    // T = -M, made exactly symmetric from the lower triangle
    if (!chain) {
#pragma unroll
        for (int u = 0; u < NL; ++u)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int i = 16 * I[u] + m, j = 16 * J[u] + g + 4 * v;
                if (u * NK + wk < nt && i < s && j <= i) {
                    zstore(Tp, d.woff + i + (int64_t)j * s, -z2{re[u][v], im[u][v]});
                    zstore(Tp, d.woff + j + (int64_t)i * s, -z2{re[u][v], im[u][v]});
                }
            }
    }
}

// One 16 x 16 tile per wave, 4 NS entries of contraction from 0: a wave has
// every operand load in flight at once, straight into MFMA form, and needs no
// LDS and no barrier.  Rows ra.. of a and rb.. of b (entry k of row r at
// p[r + k ld], 0 past the contraction); element (g + 4 v, m) in register v.
// `under` runs between the loads and the products.  For launches of few
// tiles, where a tile's time is its latency: a 64-wide tile spends 7 us on
// the matrix unit of one CU (s = 64), a quarter of it on a CU of its own 1.8.
// The products are those of zdense, in its order.
template <int NS, class AF>
__device__ __forceinline__ void zwave_n(const ZOperand& a, int ra, const ZOperand& b, int rb, zd4& re, zd4& im,
                                        AF& under)
{
    const int lane = threadIdx.x & 63, m = lane & 15, g = lane >> 4;
    z2 x[NS], y[NS];
#pragma unroll
    for (int t = 0; t < NS; ++t) {
        x[t] = zbuffer(a, (uint32_t)(ra + m) * 16u + (uint32_t)(4 * t + g) * a.ld16, 0);
        y[t] = zbuffer(b, (uint32_t)(rb + m) * 16u + (uint32_t)(4 * t + g) * b.ld16, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    under();
#pragma unroll
    for (int t = 0; t < NS; ++t) {
        re = zmfma(x[t].x, y[t].x, re);
        im = zmfma(x[t].x, y[t].y, im);
        re = zmfma(-x[t].y, y[t].y, re);
        im = zmfma(x[t].y, y[t].x, im);
    }
    zdrain();
}
template <class AF>
__device__ __forceinline__ void zwave(const ZOperand& a, int ra, const ZOperand& b, int rb, int s, zd4& re, zd4& im,
                                      AF under)
{
    if (s <= 16) zwave_n<4>(a, ra, b, rb, re, im, under);
    else if (s <= 32) zwave_n<8>(a, ra, b, rb, re, im, under);
    else zwave_n<kZMaxS / 4>(a, ra, b, rb, re, im, under);
}

// L_hat(C,K) rows [r0, r0+64) = F(C,K) T_K: four work-groups per task, a
// wave per 16 x 16 tile
__global__ __launch_bounds__(kThreads, 2) void k_zpanel_few(const Task* __restrict__ tasks,
                                                            const BlockDesc* __restrict__ blk,
                                                            const double* __restrict__ Lp, double* __restrict__ Hp,
                                                            const double* __restrict__ Tp)
{
    const Task tk = tasks[blockIdx.x >> 2];
    const BlockDesc d = blk[tk.b];
    const int s = d.s, c = d.c, lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int i0 = tk.i0 + 16 * wave, j0 = 16 * (blockIdx.x & 3);
    if (i0 >= c || j0 >= s) return;
    const int64_t ld = (int64_t)s + c;
    zd4 re = {0, 0, 0, 0}, im = {0, 0, 0, 0};
    zwave(zoperand(Tp, d.woff, (int64_t)s * s, s), j0, zoperand(Lp, d.poff + s, (int64_t)(s - 1) * ld + c, ld), i0, s,
          re, im, ZNoHook());
    const int i = i0 + (lane & 15);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int j = j0 + (lane >> 4) + 4 * v;
        if (i < c && j < s) zstore(Hp, d.hoff + i + (int64_t)j * c, z2{re[v], im[v]});
    }
}

// L_hat(C,K) rows [r0, r0+64) = F(C,K) T_K
__global__ __launch_bounds__(kThreads) void k_zpanel(const Task* __restrict__ tasks, const BlockDesc* __restrict__ blk,
                                                     const double* __restrict__ Lp, double* __restrict__ Hp,
                                                     const double* __restrict__ Tp)
{
    const Task tk = tasks[blockIdx.x];
    const BlockDesc d = blk[tk.b];
    const int s = d.s, c = d.c, r0 = tk.i0;
    const int64_t ld = (int64_t)s + c;
    auto out = [&](int ti, int j, z2 v) {
        const int i = r0 + ti;
        if (i < c && j < s) zstore(Hp, d.hoff + i + (int64_t)j * c, v);
    };
    __shared__ ZLds L;
    ZAcc acc = {};
    // T is symmetric: both operands along their rows
    zdense<false, false, true>(L, zoperand(Lp, d.poff + s + r0, (int64_t)(s - 1) * ld + c - r0, ld),
                               zoperand(Tp, d.woff, (int64_t)s * s, s), 0, s, acc);
    zvisit(acc, out);
}

// Schur update of one 64 x 64 lower tile (rows i0.., columns k0.. of C):
// F(C[i], C[k]) -= sum_t L_hat(i, t) F(C[k], t), scattered into the owning
// ancestor panels; the tasks of one launch touch disjoint entries.  The tile
// is formed as F(k0.., :) L_hat(i0.., :)^T, so that sixteen lanes hold
// sixteen consecutive rows of one target column, a contiguous run of its
// panel instead of sixteen columns: 11.1 -> 10.0 ms of the 32-pole batch; its
// read-modify-write of the targets alone is about half of that.  The scatter
// targets do not depend on the product: their (cbase, rbase) pairs are loaded
// before the products and the rel entries under them, and the epilogue reads
// every target before it writes the first.
__global__ __launch_bounds__(kThreads, 2) void k_zschur(const Task* __restrict__ tasks, const BlockDesc* __restrict__ blk,
                                                        double* __restrict__ Lp, const double* __restrict__ Hp,
                                                        const int64_t* __restrict__ cr2, const int32_t* __restrict__ rel)
{
    typedef int64_t i64v2 __attribute__((ext_vector_type(2)));
    const Task tk = tasks[blockIdx.x];
    const BlockDesc d = blk[tk.b];
    const int s = d.s, c = d.c, i0 = tk.i0, k0 = tk.j0;
    const int64_t ld = (int64_t)s + c;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm0 = (wave & 1) * 32, wn0 = (wave >> 1) * 32;
    // this thread's outputs: target columns k0 + wm0 + 16 m + lane / 16 + 4 v,
    // rows i0 + wn0 + 16 n + lane % 16; past C's end and above the diagonal
    // (never stored) the map is read at a valid place
    auto col_of = [&](int m, int v) { return k0 + wm0 + 16 * m + (lane >> 4) + 4 * v; };
    auto row_of = [&](int n) { return i0 + wn0 + 16 * n + (lane & 15); };
    i64v2 cr[2][4];
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int v = 0; v < 4; ++v)
            cr[m][v] = *reinterpret_cast<const i64v2*>(cr2 + 2 * (d.coff + min(col_of(m, v), c - 1)));
    uint32_t ro[2][2][4];
    auto prefetch = [&]() {
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int n = 0; n < 2; ++n)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    ro[m][n][v] = (uint32_t)rel[cr[m][v].y + min(max(row_of(n), col_of(m, v)), c - 1)];
    };
    __shared__ ZLds L;
    ZAcc acc = {};
    zdense<false, false, false>(L, zoperand(Lp, d.poff + s + k0, (int64_t)(s - 1) * ld + c - k0, ld),
                                zoperand(Hp, d.hoff + i0, (int64_t)s * c - i0, c), 0, s, acc, prefetch);
    z2 old[2][2][4];
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int n = 0; n < 2; ++n)
#pragma unroll
            for (int v = 0; v < 4; ++v) old[m][n][v] = zload(Lp, cr[m][v].x + ro[m][n][v]);
    const bool full = i0 > k0 && i0 + kZT <= c;  // every entry live: no branches between the stores
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int n = 0; n < 2; ++n)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (full || (row_of(n) < c && row_of(n) >= col_of(m, v)))
                    zstore(Lp, cr[m][v].x + ro[m][n][v], old[m][n][v] - z2{acc.re[m][n][v], acc.im[m][n][v]});
}

// The same update, four work-groups per task (a 32 x 32 quarter each), a wave
// per 16 x 16 tile, with every target read before the products end.
__global__ __launch_bounds__(kThreads, 2) void k_zschur_few(const Task* __restrict__ tasks,
                                                            const BlockDesc* __restrict__ blk, double* __restrict__ Lp,
                                                            const double* __restrict__ Hp,
                                                            const int64_t* __restrict__ cr2,
                                                            const int32_t* __restrict__ rel)
{
    typedef int64_t i64v2 __attribute__((ext_vector_type(2)));
    const Task tk = tasks[blockIdx.x >> 2];
    const BlockDesc d = blk[tk.b];
    const int s = d.s, c = d.c, q = blockIdx.x & 3, lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int i0 = tk.i0 + 32 * (q >> 1) + 16 * (wave >> 1), k0 = tk.j0 + 32 * (q & 1) + 16 * (wave & 1);
    if (i0 >= c || k0 >= c || i0 + 15 < k0) return;
    const int64_t ld = (int64_t)s + c;
    const int row = i0 + (lane & 15);
    auto col_of = [&](int v) { return k0 + (lane >> 4) + 4 * v; };
    i64v2 cr[4];
    uint32_t ro[4];
    z2 old[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) cr[v] = *reinterpret_cast<const i64v2*>(cr2 + 2 * (d.coff + min(col_of(v), c - 1)));
    __builtin_amdgcn_sched_barrier(0);
    auto targets = [&]() {
#pragma unroll
        for (int v = 0; v < 4; ++v) ro[v] = (uint32_t)rel[cr[v].y + min(max(row, col_of(v)), c - 1)];
#pragma unroll
        for (int v = 0; v < 4; ++v) old[v] = zload(Lp, cr[v].x + ro[v]);
    };
    zd4 re = {0, 0, 0, 0}, im = {0, 0, 0, 0};
    zwave(zoperand(Lp, d.poff + s, (int64_t)(s - 1) * ld + c, ld), k0, zoperand(Hp, d.hoff, (int64_t)s * c, c), i0, s,
          re, im, targets);
#pragma unroll
    for (int v = 0; v < 4; ++v)
        if (row < c && row >= col_of(v)) zstore(Lp, cr[v].x + ro[v], old[v] - z2{re[v], im[v]});
}

// Ainv(C,K) rows [r0, r0+64) = -G L_hat with G = Ainv(C,C) gathered from the
// ancestors' inverse panels: G(i,k) = Ainv[cbase[p] + rel[rbase[p] + q]] with
// p = min(i,k), q = max(i,k) (lower entries; the upper ones by symmetry).
// Chunks of the contraction come in three modes.  Below the diagonal band
// (k < i for the whole tile) p = k: the lanes of a wave run along i, so the
// map entry is one address per wave.  Above it p = i, and the lanes run
// along k.  Only the chunks of the band, and a ragged last chunk, form min
// and max per element and carry masks; in the other modes every per-lane
// offset is a constant of the tile and the chunk's position sits in the
// scalar base.  Rows past c read row c - 1 (their products are never stored)
// and chunks past the end read the last chunk again, so no load needs a mask.
// Each element's address is a chain of three dependent loads, so the loop is
// a pipeline: while the products of chunk n run, the values of chunk n+1 are
// stored to LDS and the loads of A of chunk n+3, L_hat of chunk n+2, rel
// entries of chunk n+4 and (cbase, rbase) pairs of chunk n+5 are issued.
// The 32-pole batch's gather-GEMM: 16.3 -> 13.6 ms.
// kPiece (kernel k_zgemm_piece): the contraction runs over rows [kb, ke) of C
// (kb on a 16-row boundary) and the tile's G L_hat goes to scratch slot `pad`
// (column-major 64 x 64 complex), for k_zgemm_sum to complete.
template <bool kPiece>
__device__ __forceinline__ void zgemm_body(const Task* __restrict__ tasks, const BlockDesc* __restrict__ blk,
                                                    double* __restrict__ Ap, const double* __restrict__ Hp,
                                                    const int64_t* __restrict__ cr2, const int32_t* __restrict__ rel,
                                                    double* __restrict__ Zs)
{
    typedef int64_t i64v2 __attribute__((ext_vector_type(2)));
    const Task tk = tasks[blockIdx.x];
    const BlockDesc d = blk[tk.b];
    const int s = d.s, c = d.c, r0 = tk.i0;
    const int64_t ld = (int64_t)s + c;
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int Kb = kPiece ? tk.kb : 0, Ke = kPiece ? tk.ke : c;
    const int nch = Ke > Kb ? (Ke - Kb + kZK - 1) / kZK : 0;
    enum { kBelow = 0, kAbove = 1, kBand = 2 };
    auto k_of = [&](int ch) { return Kb + min(ch, nch - 1) * kZK; };
    auto mode_of = [&](int k0) {
        if (k0 + kZK > Ke) return (int)kBand;
        return k0 + kZK <= r0 ? (int)kBelow : k0 >= r0 + kZT ? (int)kAbove : (int)kBand;
    };
    // element q of this thread: below the band (kk, ii) = (4 q + wave, lane),
    // else (t % 8, t / 8 + 32 q)
    const int ak = t & 7, ai = t >> 3;
    const int iBelow = min(r0 + lane, c - 1);
    const int64_t* map = cr2 + 2 * d.coff;
    i64v2 m_cr[2];
    const z2* r_at[2];
    uint32_t r_rel[2];
    z2 v_a[2][2], v_b[2];  // A by the chunk's parity
    const z2* G = reinterpret_cast<const z2*>(Ap);
    auto band_ik = [&](int k0, int q, int& i, int& k) {
        i = min(r0 + ai + 32 * q, c - 1);
        k = min(k0 + ak, Ke - 1);
    };
    auto load_map = [&](auto M, int ch) {
        constexpr int kM = decltype(M)::value;
        const int k0 = k_of(ch), md = kM >= 0 ? kM : mode_of(k0);
        uint32_t off[2];
        const int64_t* base = map;
        if (md == kBelow) {
            base += 2 * k0;
#pragma unroll
            for (int q = 0; q < 2; ++q) off[q] = (uint32_t)(4 * q + wave) * 16u;
        } else if (md == kAbove) {
            base += 2 * r0;
#pragma unroll
            for (int q = 0; q < 2; ++q) off[q] = (uint32_t)(ai + 32 * q) * 16u;
        } else {
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                int i, k;
                band_ik(k0, q, i, k);
                off[q] = (uint32_t)min(i, k) * 16u;
            }
        }
#pragma unroll
        for (int q = 0; q < 2; ++q)
            m_cr[q] = *reinterpret_cast<const i64v2*>(reinterpret_cast<const char*>(base) + off[q]);
    };
    auto load_rel = [&](auto M, int ch) {
        constexpr int kM = decltype(M)::value;
        const int k0 = k_of(ch), md = kM >= 0 ? kM : mode_of(k0);
        if (md == kBand) {
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                int i, k;
                band_ik(k0, q, i, k);
                r_rel[q] = (uint32_t)rel[m_cr[q].y + max(i, k)];
            }
        } else {
            const int32_t* rq = rel + (md == kBelow ? iBelow : k0 + ak);
#pragma unroll
            for (int q = 0; q < 2; ++q) r_rel[q] = (uint32_t)rq[m_cr[q].y];
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) r_at[q] = G + m_cr[q].x;
    };
    const ZLoader<true> lb(zoperand(Hp, d.hoff, (int64_t)s * c, c), wave);
    int wBelow[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) wBelow[q] = zat(lane, 4 * q + wave);
    const int wAbove = zat(ai, ak);
    __shared__ ZLds L;
    auto store = [&](auto M, const z2 (&va)[2], int ch, int buf) {
        constexpr int kM = decltype(M)::value;
        const int k0 = k_of(ch), md = kM >= 0 ? kM : mode_of(k0);
        char* A = L.A[buf];
        if (md == kBelow) {
#pragma unroll
            for (int q = 0; q < 2; ++q) *reinterpret_cast<z2*>(A + wBelow[q]) = va[q];
        } else {
#pragma unroll
            for (int q = 0; q < 2; ++q)
                *reinterpret_cast<z2*>(A + wAbove + q * 32 * kZRow) =
                    md == kAbove || k0 + ak < Ke ? va[q] : z2{0.0, 0.0};
        }
        lb.store(L.B[buf], v_b, k0, false, Ke);
    };
    auto load_b = [&](auto M, int ch) { lb.load(v_b, k_of(ch), decltype(M)::value >= 0 ? 1 << 30 : Ke); };
    ZAcc acc = {};
    auto body = [&](auto M, auto X, int ch) {  // X: the parity of ch
        constexpr int buf = decltype(X)::value;
        zproducts<true>(L.A[buf], L.B[buf], acc, [&] {
            store(M, v_a[buf ^ 1], ch + 1, buf ^ 1);
            // in this order, ahead of the products: loads return in order, and
            // the values of A, whose use is two iterations away, come last
            const z2* at[2] = {r_at[0] + r_rel[0], r_at[1] + r_rel[1]};
            load_rel(M, ch + 4);
            load_map(M, ch + 5);
            __builtin_amdgcn_sched_barrier(0);
            load_b(M, ch + 2);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int q = 0; q < 2; ++q) v_a[buf ^ 1][q] = *at[q];  // chunk ch + 3
            __builtin_amdgcn_sched_barrier(0);
        });
        __syncthreads();
    };
    using Any = std::integral_constant<int, -1>;
    using Below = std::integral_constant<int, kBelow>;
    using Above = std::integral_constant<int, kAbove>;
    using X0 = std::integral_constant<int, 0>;
    using X1 = std::integral_constant<int, 1>;
    if (nch > 0) {
        // chunk 0 in LDS, A of chunks 1 and 2 and L_hat of chunk 1, rel entries
        // of chunk 3, pairs of chunk 4: the first chunks' chains of loads side
        // by side, what stays in flight in the loop's order
        i64v2 cm[4][2];
#pragma unroll
        for (int n = 0; n < 4; ++n) {
            load_map(Any{}, n);
#pragma unroll
            for (int q = 0; q < 2; ++q) cm[n][q] = m_cr[q];
        }
        const z2* at3[3][2];
#pragma unroll
        for (int n = 0; n < 3; ++n) {
#pragma unroll
            for (int q = 0; q < 2; ++q) m_cr[q] = cm[n][q];
            load_rel(Any{}, n);
#pragma unroll
            for (int q = 0; q < 2; ++q) at3[n][q] = r_at[q] + r_rel[q];
        }
        load_b(Any{}, 0);
        z2 a0[2], b0[2], b1[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            b0[q] = v_b[q];
            a0[q] = *at3[0][q];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < 2; ++q) v_a[1][q] = *at3[1][q];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < 2; ++q) m_cr[q] = cm[3][q];
        load_rel(Any{}, 3);
        load_map(Any{}, 4);
        __builtin_amdgcn_sched_barrier(0);
        load_b(Any{}, 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < 2; ++q) v_a[0][q] = *at3[2][q];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            b1[q] = v_b[q];
            v_b[q] = b0[q];
        }
        store(Any{}, a0, 0, 0);
#pragma unroll
        for (int q = 0; q < 2; ++q) v_b[q] = b1[q];
    }
    __syncthreads();
    // iteration ch handles chunks ch + 1 (store) to ch + 5 (map): the mode is
    // known where all of them lie on one side of the band and the last chunk,
    // which is read again past the end, is whole
    const bool whole = ((Ke - Kb) & (kZK - 1)) == 0;
    const int nb0 = max(0, min(r0 - Kb, Ke - Kb) / kZK);  // whole chunks below the band
    const int belowEnd = whole && nb0 == nch ? nch : max(0, nb0 - 5);
    const bool above = Kb + (nch - 1) * kZK >= r0 + kZT;  // the last chunk is
    const int aboveBegin = above ? max(0, (r0 + kZT - Kb + kZK - 1) / kZK - 1) : nch;
    const int aboveEnd = whole ? nch : max(0, (Ke - Kb) / kZK - 5);
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
    zdrain();
    if constexpr (kPiece) {
        double* z = Zs + (int64_t)tk.pad * kZSlotDoubles;
        zvisit(acc, [&](int ti, int j, z2 v) { zstore(z, (int64_t)j * kZT + ti, v); });
    } else {
        zvisit(acc, [&](int ti, int j, z2 v) {
            const int i = r0 + ti;
            if (i < c && j < s) zstore(Ap, d.poff + s + i + (int64_t)j * ld, -v);
        });
    }
}

__global__ __launch_bounds__(kThreads, 3) void k_zgemm(const Task* __restrict__ tasks, const BlockDesc* __restrict__ blk,
                                                    double* __restrict__ Ap, const double* __restrict__ Hp,
                                                    const int64_t* __restrict__ cr2, const int32_t* __restrict__ rel)
{
    zgemm_body<false>(tasks, blk, Ap, Hp, cr2, rel, nullptr);
}
__global__ __launch_bounds__(kThreads, 3) void k_zgemm_piece(const Task* __restrict__ tasks, const BlockDesc* __restrict__ blk,
                                                    double* __restrict__ Ap, const double* __restrict__ Hp,
                                                    const int64_t* __restrict__ cr2, const int32_t* __restrict__ rel,
                                                    double* __restrict__ Zs)
{
    zgemm_body<true>(tasks, blk, Ap, Hp, cr2, rel, Zs);
}

// The sum of a split task's pieces (slots kb .. kb + bn - 1) at element e of
// the column-major 64 x 64 tile: four running sums over the pieces q = 4m + r,
// combined in a fixed order, so that four loads are in flight at a time.
__device__ __forceinline__ z2 zslot_sum(const double* __restrict__ z0, int np, int e)
{
    z2 a[4] = {{0, 0}, {0, 0}, {0, 0}, {0, 0}};
    int q = 0;
    for (; q + 4 <= np; q += 4) {
#pragma unroll
        for (int r = 0; r < 4; ++r) a[r] += zload(z0 + (int64_t)(q + r) * kZSlotDoubles, e);
    }
#pragma unroll
    for (int r = 0; r < 3; ++r)
        if (q + r < np) a[r] += zload(z0 + (int64_t)(q + r) * kZSlotDoubles, e);
    return (a[0] + a[1]) + (a[2] + a[3]);
}

// Columns of a 64 x 64 summing tile one work-group handles (one element per
// thread); a summing task takes kZT / kZSumCols work-groups (blockIdx.y), so
// the reads of its pieces spread over that many CUs.
constexpr int kZSumCols = kThreads / kZT;

// A split gather-GEMM tile: the sum of its pieces' G L_hat, stored negated
// as Ainv(C,K) rows [r0, r0+64); this work-group's columns j0 .. j0 + 3.
__global__ __launch_bounds__(kThreads) void k_zgemm_sum(const Task* __restrict__ tasks,
                                                        const BlockDesc* __restrict__ blk, double* __restrict__ Ap,
                                                        const double* __restrict__ Zs)
{
    const Task tk = tasks[blockIdx.x];
    const BlockDesc d = blk[tk.b];
    const int s = d.s, c = d.c;
    const int64_t ld = (int64_t)s + c;
    const int j = blockIdx.y * kZSumCols + threadIdx.x / kZT, ti = threadIdx.x % kZT, i = tk.i0 + ti;
    if (i >= c || j >= s) return;
    const z2 x = zslot_sum(Zs + (int64_t)tk.kb * kZSlotDoubles, tk.bn, j * kZT + ti);
    zstore(Ap, d.poff + s + i + (int64_t)j * ld, -x);
}

// Ainv(K,K) = T - (P + P^T) / 2 with P = L_hat^T Ainv(C,K) (lower triangle),
// the contraction over rows [kb, ke) of C.  A piece of a split block (flags
// bit 5) stores its P to scratch slot `pad` (column-major, kZMaxS x kZMaxS
// complex) instead; k_zsdiag_sum completes the block.
static_assert(kZT == kZMaxS, "one output tile holds a whole diagonal block");
__global__ __launch_bounds__(kThreads) void k_zsdiag(const Task* __restrict__ tasks, const BlockDesc* __restrict__ blk,
                                                     double* __restrict__ Ap, const double* __restrict__ Hp,
                                                     const double* __restrict__ Tp, double* __restrict__ Zs)
{
    // the product's operands, then P for the transpose (the tile loop ends
    // with a barrier, so P may reuse the space)
    __shared__ union {
        ZLds L;
        z2 P[kZT][kZT + 1];
    } U;
    auto& P = U.P;
    const Task tk = tasks[blockIdx.x];
    const BlockDesc d = blk[tk.b];
    const int s = d.s, c = d.c;
    const int64_t ld = (int64_t)s + c;
    ZAcc acc = {};
    zdense<true, true, true>(U.L, zoperand(Hp, d.hoff, (int64_t)s * c, c),
                             zoperand(Ap, d.poff + s, (int64_t)(s - 1) * ld + c, ld), tk.kb, tk.ke, acc);
    if (tk.flags & 32) {
        double* z = Zs + (int64_t)tk.pad * kZSlotDoubles;
        zvisit(acc, [&](int i, int j, z2 v) { zstore(z, (int64_t)j * kZT + i, v); });
        return;
    }
    zvisit(acc, [&](int i, int j, z2 v) { P[i][j] = v; });
    __syncthreads();
    const int i = threadIdx.x & 63;
    for (int j = threadIdx.x >> 6; j < s; j += kThreads / 64)
        if (i < s && i >= j) {
            const z2 p = 0.5 * (P[i][j] + P[j][i]);
            zstore(Ap, d.poff + i + (int64_t)j * ld, zload(Tp, d.woff + i + (int64_t)j * s) - p);
        }
}

// A split block's diagonal step: P = the sum of its pieces' partial
// products, then Ainv(K,K) = T - (P + P^T) / 2 on the lower triangle; this
// work-group's columns j0 .. j0 + 3 (P(i,j) and P(j,i) summed separately, each
// in the fixed order of zslot_sum).
__global__ __launch_bounds__(kThreads) void k_zsdiag_sum(const Task* __restrict__ tasks,
                                                         const BlockDesc* __restrict__ blk, double* __restrict__ Ap,
                                                         const double* __restrict__ Tp, const double* __restrict__ Zs)
{
    const Task tk = tasks[blockIdx.x];
    const BlockDesc d = blk[tk.b];
    const int s = d.s;
    const int64_t ld = (int64_t)s + d.c;
    const int j = blockIdx.y * kZSumCols + threadIdx.x / kZT, i = threadIdx.x % kZT;
    if (i >= s || j > i) return;
    const double* z0 = Zs + (int64_t)tk.kb * kZSlotDoubles;
    const z2 pij = zslot_sum(z0, tk.bn, j * kZT + i), pji = zslot_sum(z0, tk.bn, i * kZT + j);
    zstore(Ap, d.poff + i + (int64_t)j * ld, zload(Tp, d.woff + i + (int64_t)j * s) - 0.5 * (pij + pji));
}

// assemble: panel entry off[q] (a complex element) := value q; export: out
// entry q := panel entry off[q]
__global__ void k_zscatter(const double* __restrict__ src, const int64_t* __restrict__ off, int64_t n,
                           double* __restrict__ dst)
{
    for (int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; q < n; q += (int64_t)gridDim.x * blockDim.x)
        zstore(dst, off[q], zload(src, q));
}

__global__ void k_zgather(const double* __restrict__ src, const int64_t* __restrict__ off, int64_t n,
                          double* __restrict__ dst)
{
    for (int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; q < n; q += (int64_t)gridDim.x * blockDim.x)
        zstore(dst, q, zload(src, off[q]));
}

unsigned zgrid(int64_t n)
{
    int64_t g = (n + kThreads - 1) / kThreads;
    return (unsigned)(g < 1 ? 1 : g > 65536 ? 65536 : g);
}
}  // namespace

hipError_t launch_zassemble(const double* vals, const int64_t* off, int64_t n, double* Lp, hipStream_t s)
{
    if (n > 0) hipLaunchKernelGGL(k_zscatter, dim3(zgrid(n)), dim3(kThreads), 0, s, vals, off, n, Lp);
    return hipGetLastError();
}

hipError_t launch_zexport(const double* Ap, const int64_t* off, int64_t n, double* out, hipStream_t s)
{
    if (n > 0) hipLaunchKernelGGL(k_zgather, dim3(zgrid(n)), dim3(kThreads), 0, s, Ap, off, n, out);
    return hipGetLastError();
}

// Launches of at most this many tiles take the wave-per-16 x 16 kernels (they
// load each operand four times as often).  Measured, us, these < or > the
// 64-wide tiles at the same number of tiles (a: batches of dense chains of
// that s; b: poles of n = 8,000, s mostly 64):
//   panel  s = 16  144 5.1 < 5.5, 192 6.1 = 6.0, 220 7.7 > 6.2; s = 32  160
//          8.6 = 8.8, 192 9.1 < 9.4, 220 11.2 > 9.7; s = 64  160 14.4 < 14.9,
//          192 15.2 < 15.7, 220 18.6 > 16.4 (a); 132 12.8 < 13.5, 168 13.5 =
//          13.5, 212 16.0 > 15.1 (b); past 256, where the 64-wide tiles no
//          longer have a CU each, 264 18.1 < 22.1, 384 22.8 = 23.1 (b)
//   Schur  s = 16  360 13.1 < 14.5, 480 15.3 = 15.5; s = 32  360 15.1 < 18.2,
//          480 19.4 < 20.3; s = 64  360 23.8 < 26.2, 440 27.8 = 28.1, 480 30.5
//          > 29.1 (a); 376 21.4 < 25.0, 476 26.9 < 28.7 (b)
// Without a limit 8 poles take 9.8 ms instead of 10.2, but 32 poles 30.5
// instead of 29.9.  One pole with 64-wide tiles alone: 4.36 instead of 3.49.
constexpr int64_t kZFewPanel = 160, kZFewSchur = 384;

hipError_t launch_zfactor_level(const DevPtrs& D, int64_t diag0, int64_t ndiag, int64_t panel0, int64_t npanel,
                                const int64_t* schur_cuts, int ncuts, hipStream_t s)
{
    if (ndiag > 0)
        hipLaunchKernelGGL(k_zdiag, dim3((unsigned)ndiag), dim3(kThreads), 0, s, D.t_ldlt + diag0, D.blocks, D.Lp,
                           D.Tp, D.status);
    if (npanel > 0 && npanel <= kZFewPanel)
        hipLaunchKernelGGL(k_zpanel_few, dim3((unsigned)(4 * npanel)), dim3(kThreads), 0, s, D.t_panel + panel0,
                           D.blocks, (const double*)D.Lp, D.Hp, (const double*)D.Tp);
    else if (npanel > 0)
        hipLaunchKernelGGL(k_zpanel, dim3((unsigned)npanel), dim3(kThreads), 0, s, D.t_panel + panel0, D.blocks,
                           (const double*)D.Lp, D.Hp, (const double*)D.Tp);
    for (int g = 0; g + 1 < ncuts; g++) {
        const int64_t n = schur_cuts[g + 1] - schur_cuts[g];
        if (n > 0 && n <= kZFewSchur)
            hipLaunchKernelGGL(k_zschur_few, dim3((unsigned)(4 * n)), dim3(kThreads), 0, s, D.t_schur + schur_cuts[g],
                               D.blocks, D.Lp, (const double*)D.Hp, D.cr2, D.rel);
        else if (n > 0)
            hipLaunchKernelGGL(k_zschur, dim3((unsigned)n), dim3(kThreads), 0, s, D.t_schur + schur_cuts[g], D.blocks,
                               D.Lp, (const double*)D.Hp, D.cr2, D.rel);
    }
    return hipGetLastError();
}

hipError_t launch_zinvert_level(const DevPtrs& D, const int64_t gemm[4], int64_t sdiag0, int64_t sdiag_cut,
                                int64_t sdiag1, hipStream_t s)
{
    if (gemm[1] > gemm[0])
        hipLaunchKernelGGL(k_zgemm, dim3((unsigned)(gemm[1] - gemm[0])), dim3(kThreads), 0, s,
                           D.t_gemm + gemm[0], D.blocks, D.Ap, (const double*)D.Hp, D.cr2, D.rel);
    if (gemm[2] > gemm[1])
        hipLaunchKernelGGL(k_zgemm_piece, dim3((unsigned)(gemm[2] - gemm[1])), dim3(kThreads), 0, s,
                           D.t_gemm + gemm[1], D.blocks, D.Ap, (const double*)D.Hp, D.cr2, D.rel, D.Zs);
    if (gemm[3] > gemm[2])
        hipLaunchKernelGGL(k_zgemm_sum, dim3((unsigned)(gemm[3] - gemm[2]), kZT / kZSumCols), dim3(kThreads), 0, s,
                           D.t_gemm + gemm[2], D.blocks, D.Ap, (const double*)D.Zs);
    if (sdiag_cut > sdiag0)
        hipLaunchKernelGGL(k_zsdiag, dim3((unsigned)(sdiag_cut - sdiag0)), dim3(kThreads), 0, s, D.t_sdiag + sdiag0,
                           D.blocks, D.Ap, (const double*)D.Hp, (const double*)D.Tp, D.Zs);
    if (sdiag1 > sdiag_cut)
        hipLaunchKernelGGL(k_zsdiag_sum, dim3((unsigned)(sdiag1 - sdiag_cut), kZT / kZSumCols), dim3(kThreads), 0, s,
                           D.t_sdiag + sdiag_cut, D.blocks, D.Ap, (const double*)D.Tp, (const double*)D.Zs);
    return hipGetLastError();
}

}  // namespace selinv
