// Stage 1, one block reflector for a whole panel (paper Section 3.1, Algorithm 1 lines 2/4, without the
// tree of domain QRs): Cholesky QR in 64-bit arithmetic and the Householder vectors rebuilt from Q.
//
//   G = A^T A                     panel_gram_kernel: partial sums over ranges of 128 rows, f64 matrix instructions
//   G = R^T R                     panel_recon_kernel (one workgroup)
//   A_1 - S R = L U               the same: LU of the top block without pivoting; the sign S_k is that which keeps
//                                 the k-th pivot from cancelling (its magnitude is R_kk or more)
//   V = [L; A_2 U^-1]             panel_apply_kernel
//   T = -U R^-1 S L^-T, H = I - V T V^T, H^T A = [S R; 0]
//
// (The reconstruction: Ballard, Demmel, Grigori, Jacquelin, Nguyen, Solomonik, "Reconstructing Householder
// vectors from tall-skinny QR", 2014; Cholesky QR applied twice: Yamamoto, Nakatsukasa, Yanagisawa, Fukaya,
// 2015.)  How far Q = A R^-1 is from orthonormal is 2^-53 times the square of the panel's condition number, with its
// columns brought to norm 1 first (their lengths D do not matter); no pivot shows that number (unit upper triangular with
// -a above the diagonal: pivots near 1, condition number (1 + a)^nb).
//   f32 arithmetic: everything above is formed in 64 bits and rounded once, one pass.  ||D R^-1||_F^2 (nb times it bounds the
//     squared condition number) is formed from R^-T, and at most kMaxInv is accepted: Q is orthonormal to about 2^-26 there
//     (in a model on the host the deviation of H rose above f32's own rounding from 2^30 on).
//   f64: the pass is repeated on Q: G' = I + E, R' = I + N, N = E's upper triangle with half its diagonal.  What that
//     leaves out is N^T N, so E itself is looked at, and at most kMaxE is accepted (nb E^2 at most 2^-52).
// A panel that is refused, that has a pivot below kMinRho times its diagonal entry of G, or whose sums of squares leave the
// range, sets *stop: the block_sub_kernel of this and of every later half-sweep then leaves the matrix as it is, and the
// host goes on with the tree of domain QRs, which takes any panel, from this half-sweep on.  What was launched behind it
// ends early: the kernels of a panel read the flag at their start and look at it once their first operands have come, so
// that it is not waited for alone; the sums and small products in between run on what there is.
// Trailing columns of zeros (padding) are allowed: their reflectors are identities.
#include "svb_internal.h"
#include "lane_ops.h"
#include "mfma_frag.h"

namespace svb {

namespace {

constexpr double kMinRho = 0x1p-22;
constexpr double kMaxInv = 0x1p26;   // of ||D R^-1||_F^2, one pass
constexpr double kMaxE = 0x1p-29;    // of max |E|, the first of two passes
constexpr int kGramRows = 128;

using F64 = Frag<double>;
typedef F64::acc_t d4;

__device__ __forceinline__ int ublk(int bi, int bj) { return bj * (bj + 1) / 2 + bi; }

// ---- G = A^T A over 128 rows; the panel goes to P (leading dimension ldp) in the compute type on the way ---
// Panel element (p, c): QR A[p + c lda], LQ A[c + p lda].  Gp: per workgroup the 16 x 16 blocks of the upper
// block triangle, row-major.
template <typename C, int NBP, bool LQ>
__global__ __launch_bounds__(256) void panel_gram_kernel(const C* __restrict__ A, int64_t lda, int len, C* P, int64_t ldp,
                                                         double* __restrict__ Gp, const int* __restrict__ stop)
{
    constexpr int RB = kGramRows, NBK = NBP / 16, NT = NBK * (NBK + 1) / 2;
    constexpr int LDC = RB + (sizeof(C) == 4 ? 4 : 2);   // QR: [c][p]
    constexpr int LDP = NBP + 1;                         // LQ: [p][c]
    constexpr int VK = 16 / (int)sizeof(C);
    __shared__ __align__(16) C Ps[LQ ? RB * LDP : NBP * LDC];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int i = lane & 15, g = lane >> 4;
    const int p0 = blockIdx.x * RB, np = min(RB, len - p0);
    const int halt = *stop;
    if constexpr (LQ) {
        for (int idx = tid; idx < RB * NBP / VK; idx += 256) {
            const int p = idx / (NBP / VK), c = idx % (NBP / VK) * VK;
            C v[VK];
#pragma unroll
            for (int q = 0; q < VK; ++q) v[q] = 0;
            if (p < np) VecIO<C, C>::ld(&A[(int64_t)(p0 + p) * lda + c], v);
#pragma unroll
            for (int q = 0; q < VK; ++q) Ps[p * LDP + c + q] = v[q];
        }
        __syncthreads();
        for (int idx = tid; idx < RB * NBP; idx += 256) {
            const int p = idx % RB, c = idx / RB;
            if (p < np) P[p0 + p + c * ldp] = Ps[p * LDP + c];
        }
    } else {
        for (int idx = tid; idx < RB * NBP / VK; idx += 256) {
            const int c = idx / (RB / VK), p = idx % (RB / VK) * VK;
            C v[VK];
#pragma unroll
            for (int q = 0; q < VK; ++q) v[q] = 0;
            if (p < np) {
                VecIO<C, C>::ld(&A[p0 + p + (int64_t)c * lda], v);
                if (P) VecIO<C, C>::st(&P[p0 + p + c * ldp], v);
            }
            VecIO<C, C>::st(&Ps[c * LDC + p], v);
        }
        __syncthreads();
    }
    if (halt) return;
    double* out = Gp + (int64_t)blockIdx.x * NT * 256;
    constexpr int NTW = (NT + 3) / 4;
    d4 acc[NTW];
#pragma unroll
    for (int u = 0; u < NTW; ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[u][r] = 0;
    int bi[NTW], bj[NTW];
#pragma unroll
    for (int u = 0; u < NTW; ++u) {
        int t = wave + 4 * u, j = 0;
        while ((j + 1) * (j + 2) / 2 <= t) ++j;
        bj[u] = j < NBK ? j : NBK - 1;
        bi[u] = j < NBK ? t - j * (j + 1) / 2 : 0;
    }
#pragma unroll 4
    for (int k = 0; k < RB / 4; ++k) {
        const int p = 4 * k + g;
#pragma unroll
        for (int u = 0; u < NTW; ++u) {
            const double a = (double)(LQ ? Ps[p * LDP + bi[u] * 16 + i] : Ps[(bi[u] * 16 + i) * LDC + p]);
            const double b = (double)(LQ ? Ps[p * LDP + bj[u] * 16 + i] : Ps[(bj[u] * 16 + i) * LDC + p]);
            acc[u] = F64::mma(a, b, acc[u]);
        }
    }
#pragma unroll
    for (int u = 0; u < NTW; ++u)
        if (wave + 4 * u < NT)
#pragma unroll
            for (int r = 0; r < 4; ++r) out[(wave + 4 * u) * 256 + (4 * r + g) * 16 + i] = acc[u][r];
}

// the partial sums of many workgroups, 32 at a time, in a fixed order
__global__ __launch_bounds__(256) void gram_sum_kernel(const double* __restrict__ Gp, int n, int blocks, double* __restrict__ out)
{
    const int b = blockIdx.x, z0 = blockIdx.y * 32, z1 = min(n, z0 + 32);
    double s = 0;
#pragma unroll 8
    for (int z = z0; z < z1; ++z) s += Gp[((int64_t)z * blocks + b) * 256 + threadIdx.x];
    out[((int64_t)blockIdx.y * blocks + b) * 256 + threadIdx.x] = s;
}

// ---- 16 x 16 pieces of the one-workgroup kernel -----------------------------------------------------------
// acc += A B: A(i, k) at a[i * ars + k * acs], B(k, j) at b[k * brs + j * bcs]
__device__ __forceinline__ d4 mm16(d4 acc, const double* a, int ars, int acs, const double* b, int brs, int bcs, int i, int g)
{
    double x[4], y[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        x[s] = a[i * ars + (4 * s + g) * acs];
        y[s] = b[(4 * s + g) * brs + i * bcs];
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) acc = F64::mma(x[s], y[s], acc);
    return acc;
}
__device__ __forceinline__ d4 zero4() { d4 z; z[0] = z[1] = z[2] = z[3] = 0; return z; }
__device__ __forceinline__ d4 get16(const double* m, int ld, int i, int g)
{
    d4 v;
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = m[(4 * r + g) * ld + i];
    return v;
}
__device__ __forceinline__ void put16(double* m, int ld, int i, int g, const d4& v)
{
#pragma unroll
    for (int r = 0; r < 4; ++r) m[(4 * r + g) * ld + i] = v[r];
}
// reciprocal and reciprocal square root from the hardware's (about 2^-23) by one step of third order
__device__ __forceinline__ double rcp64(double x)
{
    const double r = __builtin_amdgcn_rcp(x), e = fma(-x, r, 1.0);
    return fma(r, fma(e, e, e), r);
}
__device__ __forceinline__ double rsqrt64(double d)
{
    const double y = __builtin_amdgcn_rsq(d), e = fma(-d * y, y, 1.0);
    return fma(y * e, fma(e, 0.375, 0.5), y);
}

// Multiply-adds whose first factor is lane K's value of the lane's row of sixteen, taken as the operand is read.
// (An operand read across lanes may not have been written by the last two vector instructions, and the compiler does
// not see what these write: two wait states in front of each.)
#define SVB_BC " row_newbcast:%c[K] row_mask:0xf bank_mask:0xf"
// value of lane K
template <int K> __device__ __forceinline__ double lane_bc(double v)
{
    double r;
    asm("s_nop 1\n\tv_mov_b64_dpp %[r], %[v]" SVB_BC : [r] "=v"(r) : [v] "v"(v), [K] "n"(K));
    return r;
}
// a += bc(x) p, e += bc(x) q
template <int K> __device__ __forceinline__ void bc_fma2(double& a, double& e, double x, double p, double q)
{
    asm("s_nop 1\n\tv_fmac_f64_dpp %[a], %[x], %[p]" SVB_BC "\n\tv_fmac_f64_dpp %[e], %[x], %[q]" SVB_BC
        : [a] "+&v"(a), [e] "+&v"(e) : [x] "v"(x), [p] "v"(p), [q] "v"(q), [K] "n"(K));
}
// x += bc(a) q
template <int K> __device__ __forceinline__ void bc_fma(double& x, double a, double q)
{
    asm("s_nop 1\n\tv_fmac_f64_dpp %[x], %[a], %[q]" SVB_BC : [x] "+&v"(x) : [a] "v"(a), [q] "v"(q), [K] "n"(K));
}
#undef SVB_BC

// the values of the four rows of lanes, in all of them
__device__ __forceinline__ void gather4(double v, double (&o)[4])
{
    const Words u = __builtin_bit_cast(Words, v);
    const auto tl = __builtin_amdgcn_permlane16_swap(u.lo, u.lo, false, false);
    const auto th = __builtin_amdgcn_permlane16_swap(u.hi, u.hi, false, false);
    const unsigned l0 = tl[0], l1 = tl[1], h0 = th[0], h1 = th[1];   // rows 0 0 2 2 and 1 1 3 3
    const auto al = __builtin_amdgcn_permlane32_swap(l0, l0, false, false);
    const auto ah = __builtin_amdgcn_permlane32_swap(h0, h0, false, false);
    const auto bl = __builtin_amdgcn_permlane32_swap(l1, l1, false, false);
    const auto bh = __builtin_amdgcn_permlane32_swap(h1, h1, false, false);
    o[0] = __builtin_bit_cast(double, Words{al[0], ah[0]});
    o[1] = __builtin_bit_cast(double, Words{bl[0], bh[0]});
    o[2] = __builtin_bit_cast(double, Words{al[1], ah[1]});
    o[3] = __builtin_bit_cast(double, Words{bl[1], bh[1]});
}
__device__ __forceinline__ double own_row(const double (&o)[4], int g)
{
    const double a = g & 1 ? o[1] : o[0], b = g & 1 ? o[3] : o[2];
    return g & 2 ? b : a;
}

// The two 16 x 16 factorisations work on four rows at a time: the four rows, handed to all four rows of lanes
// (column i in lane i), are factored there; the rest of the block, in accumulator layout, gets their update as one
// matrix instruction.  (One row at a time with every row of lanes holding the whole block: 340 cycles a row against
// 150, of which 30 f64 multiply-adds a row with a broadcast operand were the larger part.)

// Cholesky factor of a 16 x 16 block (upper triangle given) in place, and the inverse of its transpose (lower
// triangular).  False where a pivot is below kMinRho times g0, the diagonal entry it began as.
__device__ __forceinline__ bool chol16(double* m, int ld, double* inv, int ldi, const double* g0, int i, int g)
{
    d4 av, ev;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int row = 4 * r + g;
        av[r] = row <= i ? m[row * ld + i] : m[i * ld + row];
        ev[r] = row == i ? 1.0 : 0.0;
    }
    const double lim = kMinRho * g0[i];
    double piv = 0;   // lane k: the k-th pivot
    unroll<4>([&](auto sc) {
        constexpr int s = decltype(sc)::value;
        double a[4], e[4];
        gather4(av[s], a);
        gather4(ev[s], e);
        unroll<4>([&](auto qc) {
            constexpr int q = decltype(qc)::value, k = 4 * s + q;
            const double d = lane_bc<k>(a[q]);
            piv = i == k ? d : piv;
            const double y = rsqrt64(d);
            a[q] *= y;
            e[q] *= y;
            const double nx = -a[q], nz = -e[q];
            unroll<3 - q>([&](auto rc) {
                constexpr int r = q + 1 + decltype(rc)::value;
                bc_fma2<4 * s + r>(a[r], e[r], a[q], nx, nz);
            });
        });
        const double x = own_row(a, g), z = own_row(e, g);
        const int row = 4 * s + g;
        m[row * ld + i] = row <= i ? x : 0.0;
        inv[row * ldi + i] = row >= i ? z : 0.0;
        if constexpr (s < 3) {
            av = F64::mma(-x, x, av);
            ev = F64::mma(-x, z, ev);
        }
    });
    return !__any(!(piv > lim));
}

// x[j] in row q of lanes <-> x[q] in row j
__device__ __forceinline__ void transpose4(double (&x)[4])
{
    swap_rows(x[0], x[1]);
    swap_rows(x[2], x[3]);
    swap_halves(x[0], x[2]);
    swap_halves(x[1], x[3]);
}

// LU of a 16 x 16 block M - S R, R upper triangular with positive diagonal, the signs S chosen on the way: L (unit,
// strictly below the diagonal) and U in place of M, the inverses of both, the signs.  M is kept by rows and by columns
// (rows of U, columns of L); L^-1 and U^-T arise in the same steps.  Of the four rows being worked on, the rows of
// lanes hold those of M, of M^T, of L^-1 and of U^-T: one multiply-add brings all four on.
__device__ __forceinline__ void lu16(double* m, const double* rm, int ld, double* linv, double* uinv, int ldi, double* sgn,
                                     int i, int g)
{
    d4 av, tv, ev, fv;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int row = 4 * r + g;
        av[r] = m[row * ld + i];
        tv[r] = m[i * ld + row];
        ev[r] = fv[r] = row == i ? 1.0 : 0.0;
    }
    double rr[16], rd[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const double v = rm[r * ld + i];
        rr[r] = g == 0 ? v : 0.0;
        rd[r] = rm[r * ld + r];
    }
    const bool odd = g & 1;
    double my_s = 0;
    unroll<4>([&](auto sc) {
        constexpr int s = decltype(sc)::value;
        double x[4] = {av[s], tv[s], ev[s], fv[s]};
        transpose4(x);
        unroll<4>([&](auto qc) {
            constexpr int q = decltype(qc)::value, k = 4 * s + q;
            const double alpha = lane_value(x[q], k);
            const double sg = copysign(1.0, -alpha), rc = rcp64(fma(-sg, rd[k], alpha));
            my_s = i == k ? sg : my_s;
            x[q] = fma(-sg, rr[k], x[q]) * (odd ? rc : 1.0);   // u, l, L^-1's row, U^-T's row
            if constexpr (q < 3) {
                double a = x[q], b = x[q];
                swap_rows(a, b);                               // u u . . and l l . .
                double y = odd ? a : b, z = y;                 // l u . .
                swap_halves(y, z);                             // l u l u
                const double n = -x[q];
                unroll<3 - q>([&](auto rr_) {
                    constexpr int r = q + 1 + decltype(rr_)::value;
                    bc_fma<4 * s + r>(x[r], y, n);
                });
            }
        });
        transpose4(x);
        const int row = 4 * s + g;
        if constexpr (s < 3) {
            av = F64::mma(-x[1], x[0], av);
            tv = F64::mma(-x[0], x[1], tv);
            ev = F64::mma(-x[1], x[2], ev);
            fv = F64::mma(-x[0], x[3], fv);
        }
        if (i >= row) m[row * ld + i] = x[0];
        if (i > row) m[i * ld + row] = x[1];
        linv[row * ldi + i] = i <= row ? x[2] : 0.0;
        uinv[i * ldi + row] = i <= row ? x[3] : 0.0;
    });
    sgn[i] = my_s;
}

template <int NBP> struct ReconGeom {
    static constexpr int NBK = NBP / 16, LD = NBP + 2, LDD = 18;
    static constexpr int oG = 0, oE = oG + NBP * LD, oB = oE + NBP * LD, oL = oB + NBP * LD;
    static constexpr int oLd = oL + NBP * LD, oUd = oLd + NBK * 16 * LDD, oG0 = oUd + NBK * 16 * LDD, oS = oG0 + NBP;
    static constexpr int kElems = oS + NBP;
    static constexpr size_t kBytes = (size_t)kElems * 8;
};

// The one-workgroup step.
//   kFull (f32 arithmetic): G -> R; L, U, S; V's top, X = U^-1 (V's rest is A X), T, S R.
//   kFirst (f64): G -> R, X = R^-1 (Q = A X).
//   kSecond (f64): G' = Q^T Q -> N, R' = I + N; L, U, S of Q_1 - S R'; V's top, X, T, S R' R.
// Blocks of sixteen: a diagonal block in the registers of one wave, the rest of a step on f64 matrix instructions by
// all; the next diagonal block is updated by the wave that factors it, so the others' share of the update runs beside
// its factorisation.  The LU factorisation follows the Cholesky factorisation one block behind, by another wave: what
// stands on the chain is one Cholesky block and the LU blocks.  Bound by latency: 62k cycles
// (28 us) at NBP = 64, of which each LU block 6900 and each Cholesky block 3600; 107k with one row at a time, Q formed,
// the two factorisations one after the other and full barriers.  At NBP = 64 nine (f32) and fourteen (f64, second
// pass) registers a lane are spilled (three waves a SIMD leave 168): the panel's top rows, fetched with the partial sums and
// needed behind them.
enum { kFull, kFirst, kSecond };
template <typename C> struct ReconArgs {
    const double* Gp; int np;        // partial sums of G
    const C* P; int64_t ldp;         // the panel (Q in the second pass), top rows
    double* X;                       // NBP x NBP, X(k, c) at c * NBP + k
    double* R1;                      // the first pass's R (row-major) between the passes
    C* V; int64_t ldv; C* Vt; int64_t ldvt;   // the sub-panel's top block in both orders
    C* T; int64_t ldt;
    C* band; int64_t ldab, row0, col0; int lq, nb;   // where S R goes: the sub-panel's corner of the band
    int* stop; int* host_stop; int hs;   // half-sweep number, from 0
    int above;                       // rows of V above the sub-panel (zeros there; R's block above it comes from P)
};
template <int NBP> constexpr int kReconThreads = NBP == 64 ? 768 : 512;
template <typename C, int NBP, int MODE>
__global__ __launch_bounds__(kReconThreads<NBP>) void panel_recon_kernel(ReconArgs<C> a)
{
    using Gm = ReconGeom<NBP>;
    constexpr int NBK = Gm::NBK, LD = Gm::LD, LDD = Gm::LDD, NT = NBK * (NBK + 1) / 2, NTH = kReconThreads<NBP>, NWV = NTH / 64;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    double* sm = reinterpret_cast<double*>(smem_raw);
    double *G = sm + Gm::oG, *E = sm + Gm::oE, *B = sm + Gm::oB, *L = sm + Gm::oL, *Ld = sm + Gm::oLd, *Ud = sm + Gm::oUd;
    double *g0 = sm + Gm::oG0, *S = sm + Gm::oS;
    __shared__ int sh_bad, sh_nz;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = lane & 15, g = lane >> 4;
    const int halted = *a.stop;
    int bi = 0, bj = 0;   // this wave's block of T, by falling length of its sums
    {
        int dist = NBK - 1, left = wave < NT ? wave : 0;
        while (left >= NBK - dist) {
            left -= NBK - dist;
            --dist;
        }
        bi = left;
        bj = left + dist;
    }
    auto blk = [](double* m, int bi, int bj) { return m + bi * 16 * LD + bj * 16; };

    auto refuse = [&] {
        *a.stop = a.hs + 1;
        __hip_atomic_store(a.host_stop, a.hs + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    };

    // ---- G (every 256 threads take a share of the partial sums); E = 0; the panel's top rows in B
    if (tid == 0) sh_bad = 0;
    {
        constexpr int NE = (NBP * NBP + NTH - 1) / NTH, NS = NTH / 256;   // (every 256 threads: a share)
        C top[NE];
        if constexpr (MODE != kFirst) {
#pragma unroll
            for (int u = 0; u < NE; ++u) {
                const int idx = min(tid + u * NTH, NBP * NBP - 1);
                top[u] = a.P[idx % NBP + (int64_t)(idx / NBP) * a.ldp];
            }
        }
        const int el = tid & 255, share = tid >> 8, r = el >> 4, c = el & 15;
        double s[NT];
#pragma unroll
        for (int b = 0; b < NT; ++b) s[b] = 0;
        if (MODE == kSecond && !share && r == c) {
#pragma unroll
            for (int bj = 0; bj < NBK; ++bj) s[ublk(bj, bj)] = -1.0;
        }
        for (int z = share; z < a.np; z += NS)
#pragma unroll
            for (int b = 0; b < NT; ++b) s[b] += a.Gp[((int64_t)z * NT + b) * 256 + el];
        for (int idx = tid; idx < NBP * LD; idx += NTH) E[idx] = 0.0;
        if (share) {
            double* o = share == 1 ? L : B;
#pragma unroll
            for (int b = 0; b < NT; ++b) o[b * 256 + el] = s[b];
        }
        lds_barrier();
        if (halted) return;
        if (!share) {
#pragma unroll
            for (int bj = 0; bj < NBK; ++bj)
#pragma unroll
                for (int bi = 0; bi <= bj; ++bi) {
                    const int at = ublk(bi, bj) * 256 + el;
                    const double v = s[ublk(bi, bj)] + L[at] + (NS == 3 ? B[at] : 0.0);
                    blk(G, bi, bj)[r * LD + c] = v;
                    if (bi == bj && r == c) g0[bi * 16 + r] = MODE == kSecond ? v + 1.0 : v;
                }
        }
        lds_barrier();
        if constexpr (MODE != kFirst) {
#pragma unroll
            for (int u = 0; u < NE; ++u) {
                const int idx = tid + u * NTH;
                if (idx < NBP * NBP) B[idx % NBP * LD + idx / NBP] = (double)top[u];
            }
        }
        for (int idx = tid; idx < NBP * LD; idx += NTH) L[idx] = 0.0;
    }
    if (wave == 0) {
        // columns of zeros: allowed at the end only; sums of squares outside the range or not finite: not
        const double d = lane < NBP ? g0[lane] : 1.0;
        const unsigned long long zero = __ballot(d == 0.0);
        const int nz = zero ? __builtin_ctzll(zero) : NBP;
        const unsigned long long want = nz >= NBP ? 0ull : (~0ull << nz) & (NBP == 64 ? ~0ull : (1ull << NBP) - 1);
        const bool range = d == 0.0 || (d > 0x1p-800 && d < 0x1p900);
        if (__any(!range) || zero != want) {
            if (lane == 0) sh_bad = 1;
        }
        if (lane == 0) sh_nz = nz;
        if (lane < NBP && d == 0.0) {
            g0[lane] = 1.0;
            G[lane * LD + lane] = MODE == kSecond ? 0.0 : 1.0;
        }
    }
    d4 rr = zero4();   // second pass: a block of R' R in each of the waves from 2 on
    int ri = 0, rj = 0;
    if constexpr (MODE == kSecond) {
        while ((rj + 1) * (rj + 2) / 2 <= wave - 2) ++rj;
        ri = wave - 2 - rj * (rj + 1) / 2;
    }
    if constexpr (MODE == kSecond) {
        // N: E's upper triangle with half its diagonal; I + N in the place of G, N^T in E.  (N is about 2^-53: in I + N the
        // most of it is lost, and more of it above 1 than below, where numbers are twice as close.  With the sum of squares
        // formed around 1 and T from U (I - N), all singular values came out smaller by 7e-17 of themselves on average.)
        lds_barrier();
        for (int idx = tid; idx < NBP * NBP; idx += NTH) {
            const int c = idx % NBP, r = idx / NBP;
            const double dev = r <= c ? G[r * LD + c] : 0.0;
            if (!(fabs(dev) <= kMaxE)) sh_bad = 1;   // (a NaN as well)
            const double v = r == c ? 0.5 * dev : dev;
            G[r * LD + c] = r == c ? 1.0 + v : v;
            if (r <= c) E[c * LD + r] = v;
        }
    }
    lds_barrier();

    // ---- step t: block t of G -> R, E = R^-T; block t - 1 of B - S R = L U.  L's inverse arises below the diagonal of
    //      the array L, U's above it (their diagonal blocks in Ld, Ud).
    constexpr bool kChol = MODE != kSecond, kLu = MODE != kFirst;
    for (int t = kChol ? 0 : 1; t <= (kLu ? NBK : NBK - 1); ++t) {
        const int kb = t - 1;
        const bool chol = kChol && t < NBK, lu = kLu && t > 0;
        double *Lkk = Ld + kb * 16 * LDD, *Ukk = Ud + kb * 16 * LDD;
        if (chol && wave == 0) {
            if (!chol16(blk(G, t, t), LD, blk(E, t, t), LD, g0 + t * 16, i, g) && lane == 0) sh_bad = 1;
        }
        if (MODE == kFull && t == NBK && wave == 0) {
            // ||D R^-1||_F^2 beside the last LU block (R^-T is whole by now), eight entries a lane at a time: one by one the
            // reads' latency made this longer than that block, 2.4 us a panel at NBP = 64
            constexpr int CS = 64 / NBP;
            const int k = lane % NBP, c0 = lane / NBP;
            double s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll 1
            for (int c = c0; c < NBP; c += 8 * CS)
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    double x = E[(c + u * CS) * LD + k];
                    x = k <= c + u * CS ? x : 0.0;
                    s[u] = fma(x, x, s[u]);
                }
            double f = (((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]))) * g0[k];
            for (int off = 32; off > 0; off >>= 1) f += __shfl_xor(f, off, kWave);
            if (!(f <= kMaxInv) && lane == 0) sh_bad = 1;
        }
        if (lu && wave == 1) lu16(blk(B, kb, kb), blk(G, kb, kb), LD, Lkk, Ukk, LDD, S + kb * 16, i, g);
        if (MODE == kSecond && kb == 0 && wave >= 2 && wave < NT + 2) {   // R' R = R + N R, a block a wave
            rr = get16(a.R1 + ri * 16 * NBP + rj * 16, NBP, i, g);
            for (int k = ri; k <= rj; ++k) rr = mm16(rr, blk(E, k, ri), 1, LD, a.R1 + k * 16 * NBP + rj * 16, NBP, 1, i, g);
        }
        lds_barrier();
        if (chol && wave >= 2 && wave < NBK + 1) {
            const int j0 = wave - 2, j = j0 + (j0 >= t ? 1 : 0);
            double* m = blk(j > t ? G : E, t, j);
            put16(m, LD, i, g, mm16(zero4(), blk(E, t, t), LD, 1, m, LD, 1, i, g));
        }
        if (lu && wave >= NWV - 2 * (NBK - 1)) {
            const int job = wave - (NWV - 2 * (NBK - 1)), j0 = job % (NBK - 1), j = j0 + (j0 >= kb ? 1 : 0);
            if (job < NBK - 1) {
                // rows of U: L(kb, kb)^-1 (B - S R); rows of L's inverse
                double* m = blk(j > kb ? B : L, kb, j);
                const double* rm = blk(G, kb, j);
                double x[4], y[4];
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    x[s] = Lkk[i * LDD + 4 * s + g];
                    y[s] = m[(4 * s + g) * LD + i];
                    if (j > kb) y[s] = fma(-S[kb * 16 + 4 * s + g], rm[(4 * s + g) * LD + i], y[s]);
                }
                d4 v = zero4();
#pragma unroll
                for (int s = 0; s < 4; ++s) v = F64::mma(x[s], y[s], v);
                put16(m, LD, i, g, v);
            } else {
                // columns of L; U's column times the inverse of its diagonal block
                double* m = blk(B, j, kb);
                put16(j > kb ? m : blk(L, j, kb), LD, i, g, mm16(zero4(), m, LD, 1, Ukk, LDD, 1, i, g));
            }
        }
        lds_barrier();
        // m -= A B, A(i, k) at la[i * rs + k * cs]
        auto less = [&](double* m, const double* la, int rs, int cs, const double* rb, int ldb) {
            const d4 p = mm16(zero4(), la, rs, cs, rb, ldb, 1, i, g);
            d4 v = get16(m, LD, i, g);
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] -= p[r];
            put16(m, LD, i, g, v);
        };
        // column kb of U's inverse: -sum_k U^-1(bi, k) (U(k, kb) U(kb, kb)^-1)
        auto ucol = [&](int bi) {
            d4 v = zero4();
            for (int k = bi; k < kb; ++k)
                v = mm16(v, k == bi ? Ud + bi * 16 * LDD : blk(L, bi, k), k == bi ? LDD : LD, 1, blk(L, k, kb), LD, 1, i, g);
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = -v[r];
            return v;
        };
        if (lu && kb == NBK - 1) {
            d4 v = zero4();
            if (wave < kb) v = ucol(wave);
            lds_barrier();
            if (wave < kb) put16(blk(L, wave, kb), LD, i, g, v);
        } else if (wave == 0) {
            if (chol && t + 1 < NBK) less(blk(G, t + 1, t + 1), blk(G, t, t + 1), 1, LD, blk(G, t, t + 1), LD);
        } else if (wave == 1) {
            if (lu) less(blk(B, t, t), blk(B, t, kb), LD, 1, blk(B, kb, t), LD);
        } else if (wave == NWV - 1) {
            if (lu)
                for (int bi = 0; bi < kb; ++bi) put16(blk(L, bi, kb), LD, i, g, ucol(bi));
        } else {
            for (int q = wave - 2; q < 2 * NBK * NBK; q += NWV - 3) {
                const int ib = q / NBK % NBK, j = q % NBK;
                if (q < NBK * NBK) {
                    if (!chol || ib <= t || (j > t && j < ib) || (ib == t + 1 && j == ib)) continue;
                    double* src = j > t ? G : E;
                    less(blk(src, ib, j), blk(G, t, ib), 1, LD, blk(src, t, j), LD);
                } else {
                    if (!lu || ib <= kb || (ib == t && j == t)) continue;
                    double* src = j > kb ? B : L;
                    less(blk(src, ib, j), blk(B, ib, kb), LD, 1, j == kb ? Lkk : blk(src, kb, j), j == kb ? LDD : LD);
                }
            }
        }
    }
    if constexpr (MODE == kFirst) {
        // X = R^-1 = E^T; R stays for the second pass
        lds_barrier();
        for (int idx = tid; idx < NBP * NBP; idx += NTH) {
            const int k = idx % NBP, c = idx / NBP;
            a.X[idx] = k <= c ? E[c * LD + k] : 0.0;
            a.R1[idx] = c <= k ? G[c * LD + k] : 0.0;   // row c, column k
        }
        if (tid == 0 && sh_bad) refuse();
        return;
    }
    lds_barrier();
    // ---- T = -(U R^-1) S L^-T, a block a wave; in the second pass U R'^-1 = U - U N
    static_assert(NT <= NWV, "a block a wave");
    d4 ur = zero4();
    if (MODE == kSecond && wave < NT) {
        ur = get16(blk(B, bi, bj), LD, i, g);
        if (bi == bj)
#pragma unroll
            for (int r = 0; r < 4; ++r) ur[r] = 4 * r + g <= i ? ur[r] : 0.0;
    }
    if (wave < NT)
        for (int k = bi; k <= bj; ++k)
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int c = 4 * s + g;
                double u = blk(B, bi, k)[i * LD + c];
                if (k == bi) u = i <= c ? u : 0.0;
                if (MODE == kSecond) u = -u;
                ur = F64::mma(u, blk(E, bj, k)[i * LD + c], ur);
            }
    // (X, and V's top block, unit lower triangular, in both orders, while U is still in the array with L)
    constexpr int NE = (NBP * NBP + NTH - 1) / NTH;
#pragma unroll
    for (int u = 0; u < NE; ++u) {
        const int idx = tid + u * NTH, k = idx % NBP, c = idx / NBP;
        if (NBP * NBP % NTH && idx >= NBP * NBP) break;
        const double x = k / 16 == c / 16 ? Ud[(c / 16 * 16 + k % 16) * LDD + c % 16] : L[k * LD + c];
        a.X[idx] = k <= c ? x : 0.0;
        const double lo = B[k * LD + c], up = B[c * LD + k];
        a.V[k + (int64_t)c * a.ldv] = (C)(k > c ? lo : (k == c ? 1.0 : 0.0));
        a.Vt[(int64_t)c * a.ldvt + k] = (C)(c > k ? up : (k == c ? 1.0 : 0.0));
    }
    lds_barrier();
    if (wave < NT) put16(blk(B, bi, bj), LD, i, g, ur);
    lds_barrier();
    const int nz = sh_nz;
    if (wave < NT) {
        d4 x = zero4();
        for (int k = bi; k <= bj; ++k) {
            const bool dg = k == bj;
            const double* lm = dg ? Ld + k * 16 * LDD : blk(L, bj, k);
            const int ll = dg ? LDD : LD;
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int c = 4 * s + g;
                x = F64::mma(blk(B, bi, k)[i * LD + c] * S[k * 16 + c], lm[i * ll + c], x);
            }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = bi * 16 + 4 * r + g, col = bj * 16 + i;
            a.T[(int64_t)col * a.ldt + row] = (C)(row <= col && col < nz ? -x[r] : 0.0);
            if (bi != bj) a.T[(int64_t)row * a.ldt + col] = 0;
        }
    }
    for (int idx = tid; idx < a.above * NBP; idx += NTH) {
        const int p = idx % NBP, c = idx / NBP;   // zeros above the sub-panel (above is NBP)
        a.V[p - a.above + (int64_t)c * a.ldv] = 0;
        a.Vt[(int64_t)(p - a.above) * a.ldvt + c] = 0;
    }
    // ---- S R to the band
    if (sh_bad && tid == 0) refuse();
    if (sh_bad) return;
    // entry (ri, ci) of R: band entry (row0 + ri, col0 + ci) in a QR sweep, (row0 + ci, col0 + ri) in an LQ sweep
    C* const base = a.band + (a.row0 - a.col0 + 2 * a.nb - 1) + a.col0 * a.ldab;
    const int64_t sr = a.lq ? a.ldab - 1 : 1, sc = a.lq ? 1 : a.ldab - 1;
    if constexpr (MODE == kSecond) {
        if (wave >= 2 && wave < NT + 2) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = ri * 16 + 4 * r + g, col = rj * 16 + i;
                if (row <= col) base[row * sr + col * sc] = (C)(col < nz ? S[row] * rr[r] : 0.0);
            }
        }
    } else {
#pragma unroll
        for (int u = 0; u < NE; ++u) {
            const int idx = tid + u * NTH, ri = idx % NBP, ci = idx / NBP;
            if (NBP * NBP % NTH && idx >= NBP * NBP) break;
            if (ri <= ci) base[ri * sr + ci * sc] = (C)(ci < nz ? S[ri] * G[ri * LD + ci] : 0.0);
        }
    }
    for (int idx = tid; idx < a.above * NBP; idx += NTH) {
        const int ri = idx % NBP, ci = idx / NBP;
        base[(ri - a.above) * sr + ci * sc] = a.P[ri - a.above + (int64_t)ci * a.ldp];
    }
}

// ---- Out(p, c) = sum_k A(p, k) X(k, c), X upper triangular, in 64 bits; to out (leading dimension ldo, may be A
// itself) and, where given, to outt with c running fastest.  16 rows a wave.
// FIRST (f64, first pass: X = R^-1, R1 = R row-major): Out = Q + (A - Q R) X with Q = A X.  A product with the inverse
// leaves a residual of |A| |R^-1| |R| roundings, where a substitution leaves |Q| |R|; what of A is not Q R is missing from
// the band (relative residual 2^-42 for the panel Q (I - 0.15 triu), nb = 64, singular values off by 1.6e-15 of their
// norm; 2^-49 and 3e-16 with the correction).  An accumulator entry of Q is the next product's operand as it lies.
template <typename C, int NBP, bool FIRST>
__global__ __launch_bounds__(256) void panel_apply_kernel(const C* A, int64_t lda, int len, const double* __restrict__ X,
                                                          const double* __restrict__ R1, C* out, int64_t ldo, C* outt,
                                                          int64_t ldt, const int* __restrict__ stop)
{
    constexpr int NBK = NBP / 16, LDX = NBP + 2;
    __shared__ __align__(16) double Xs[NBP * LDX];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int i = lane & 15, g = lane >> 4;
    const int p0 = blockIdx.x * 64 + wave * 16;
    const int halt = *stop;
    C b[NBP / 4];
    if (p0 < len) {
#pragma unroll
        for (int k = 0; k < NBP / 4; ++k) b[k] = A[p0 + i + (int64_t)(4 * k + g) * lda];
    }
    for (int idx = tid; idx < NBP * NBP; idx += 256) Xs[idx / NBP * LDX + idx % NBP] = X[idx];
    __syncthreads();
    if (halt || p0 >= len) return;
    d4 acc[NBK];
#pragma unroll
    for (int c = 0; c < NBK; ++c) acc[c] = zero4();
#pragma unroll
    for (int k = 0; k < NBP / 4; ++k) {
        const double y = (double)b[k];
#pragma unroll
        for (int c = 0; c < NBK; ++c)
            if (c >= k / 4) acc[c] = F64::mma(Xs[(c * 16 + i) * LDX + 4 * k + g], y, acc[c]);
    }
    if constexpr (FIRST) {
        d4 res[NBK];
#pragma unroll
        for (int k = 0; k < NBP / 4; ++k) res[k / 4][k % 4] = (double)b[k];
#pragma unroll
        for (int k = 0; k < NBP / 4; ++k) {
            const double y = -acc[k / 4][k % 4];
#pragma unroll
            for (int c = 0; c < NBK; ++c)
                if (c >= k / 4) res[c] = F64::mma(R1[(4 * k + g) * NBP + c * 16 + i], y, res[c]);
        }
#pragma unroll
        for (int k = 0; k < NBP / 4; ++k) {
            const double y = res[k / 4][k % 4];
#pragma unroll
            for (int c = 0; c < NBK; ++c)
                if (c >= k / 4) acc[c] = F64::mma(Xs[(c * 16 + i) * LDX + 4 * k + g], y, acc[c]);
        }
    }
#pragma unroll
    for (int c = 0; c < NBK; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int64_t p = p0 + i, cc = c * 16 + 4 * r + g;
            const C v = (C)acc[c][r];
            out[p + cc * ldo] = v;
            if (outt) outt[p * ldt + cc] = v;
        }
}

// ---- T's block above the diagonal of two sub-panels: T12 = -T11 (V1^T V2) T22; the block below it is zero
// Wp: partial sums of V1^T V2 (block_wt_kernel: element (c, q) at q * 64 + c).  There are up to 64 of them of 4096
// elements, too much for the one workgroup of the products (one after the other in its threads they took 231 us of
// every half-sweep at n = 32768, 9 % of the call), so they are added up by the whole chip first: 16 elements a
// workgroup, 16 threads an element, in a fixed order.
template <typename C>
__global__ __launch_bounds__(256) void join_sum_kernel(const C* __restrict__ Wp, int ns, double* __restrict__ M)
{
    __shared__ double red[16][17];
    const int e = threadIdx.x & 15, z0 = threadIdx.x >> 4, idx = blockIdx.x * 16 + e;
    double s = 0;
#pragma unroll 4
    for (int z = z0; z < ns; z += 16) s += (double)Wp[(int64_t)z * 4096 + idx];
    red[z0][e] = s;
    __syncthreads();
    if (z0 != 0) return;
#pragma unroll
    for (int z = 1; z < 16; ++z) s += red[z][e];
    M[idx] = s;
}

// one wave a 16 x 16 block; the three factors are held as they are stored, columns apart
template <typename C>
__global__ __launch_bounds__(1024) void panel_join_kernel(const double* __restrict__ M12, C* __restrict__ T, int64_t ldt)
{
    constexpr int NB = 64, LD = NB + 2;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    double* M = reinterpret_cast<double*>(smem_raw);
    double *A = M + NB * LD, *B = A + NB * LD, *Z = B + NB * LD;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int i = lane & 15, g = lane >> 4;
#pragma unroll
    for (int idx = tid; idx < NB * NB; idx += 1024) {
        const int r = idx % NB, c = idx / NB;
        M[c * LD + r] = M12[idx];
        A[c * LD + r] = (double)T[r + c * ldt];
        B[c * LD + r] = (double)T[NB + r + (NB + c) * ldt];
    }
    __syncthreads();
    const int bi = wave / 4, bj = wave % 4;
    d4 v = zero4();
    for (int k = bi; k < 4; ++k) v = mm16(v, A + k * 16 * LD + bi * 16, 1, LD, M + bj * 16 * LD + k * 16, 1, LD, i, g);
    put16(Z + bi * 16 * LD + bj * 16, LD, i, g, v);
    __syncthreads();
    v = zero4();
    for (int k = 0; k <= bj; ++k) v = mm16(v, Z + bi * 16 * LD + k * 16, LD, 1, B + bj * 16 * LD + k * 16, 1, LD, i, g);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int row = bi * 16 + 4 * r + g, col = bj * 16 + i;
        T[row + (int64_t)(NB + col) * ldt] = (C)-v[r];
        T[NB + row + (int64_t)col * ldt] = 0;
    }
}

template <typename C, int NBP, int MODE> void recon_launch(const ReconArgs<C>& a, hipStream_t s)
{
    auto kern = panel_recon_kernel<C, NBP, MODE>;
    static bool attr_set = false;
    if (!attr_set) {
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)ReconGeom<NBP>::kBytes);
        attr_set = true;
    }
    hipLaunchKernelGGL(kern, dim3(1), dim3(kReconThreads<NBP>), ReconGeom<NBP>::kBytes, s, a);
}

template <typename C, int NBP, bool LQ>
int gram(const C* A, int64_t lda, int64_t len, C* P, int64_t ldp, double* Gp, double** sum, const int* stop, hipStream_t s)
{
    constexpr int NT = NBP / 16 * (NBP / 16 + 1) / 2;
    const int n = (int)((len + kGramRows - 1) / kGramRows);
    hipLaunchKernelGGL((panel_gram_kernel<C, NBP, LQ>), dim3(n), dim3(256), 0, s, A, lda, (int)len, P, ldp, Gp, stop);
    *sum = Gp;
    if (n <= 16) return n;
    const int m = (n + 31) / 32;
    *sum = Gp + (int64_t)n * NT * 256;
    hipLaunchKernelGGL(gram_sum_kernel, dim3(NT, m), dim3(256), 0, s, Gp, n, NT, *sum);
    return m;
}

// Cholesky QR and reconstruction of one sub-panel of NBP columns that lies in the work panel (or, first_src, still
// in the matrix)
template <typename C, int NBP>
void subpanel(const ReconPanel<C>& a, int64_t off, int64_t sub0, hipStream_t s)
{
    const int64_t len = a.len - off;
    C* P = a.P + off + sub0 * a.ldv;
    double* Gs = nullptr;
    int np;
    if (a.src && a.lq) np = gram<C, NBP, true>(a.src, a.lda, len, P, a.ldv, a.Gp, &Gs, a.stop, s);
    else if (a.src) np = gram<C, NBP, false>(a.src, a.lda, len, P, a.ldv, a.Gp, &Gs, a.stop, s);
    else np = gram<C, NBP, false>(P, a.ldv, len, (C*)nullptr, 0, a.Gp, &Gs, a.stop, s);
    ReconArgs<C> r{};
    r.Gp = Gs; r.np = np; r.P = P; r.ldp = a.ldv; r.X = a.X; r.R1 = a.X + NBP * NBP;
    r.V = a.V + off + sub0 * a.ldv; r.ldv = a.ldv; r.Vt = a.Vt + off * a.nb + sub0; r.ldvt = a.nb;
    r.T = a.Tf + sub0 * a.nb + sub0; r.ldt = a.nb;
    r.band = a.band; r.ldab = a.ldab;
    r.row0 = a.row0 + off; r.col0 = a.col0 + off;   // (off = sub0: rows and columns of the sub-panel's corner of R)
    r.lq = a.lq; r.nb = a.nb; r.stop = a.stop; r.host_stop = a.host_stop; r.hs = a.hs; r.above = (int)off;
    const dim3 rest((unsigned)((len - NBP + 63) / 64));
    if constexpr (sizeof(C) == 8) {
        recon_launch<C, NBP, kFirst>(r, s);
        hipLaunchKernelGGL((panel_apply_kernel<C, NBP, true>), dim3((unsigned)((len + 63) / 64)), dim3(256), 0, s, P, a.ldv,
                           (int)len, a.X, r.R1, P, a.ldv, (C*)nullptr, (int64_t)0, a.stop);
        r.np = gram<C, NBP, false>(P, a.ldv, len, (C*)nullptr, 0, a.Gp, &Gs, a.stop, s);
        r.Gp = Gs;
        recon_launch<C, NBP, kSecond>(r, s);
    } else {
        recon_launch<C, NBP, kFull>(r, s);
    }
    if (len > NBP)
        hipLaunchKernelGGL((panel_apply_kernel<C, NBP, false>), rest, dim3(256), 0, s, P + NBP, a.ldv, (int)(len - NBP), a.X,
                           (const double*)nullptr, r.V + NBP, a.ldv, r.Vt + (int64_t)NBP * a.nb, (int64_t)a.nb, a.stop);
}

}  // namespace

// doubles of the partial Gram sums and of X, R1
size_t recon_scratch_doubles(int64_t rows, int nb)
{
    const int nbp = nb < 64 ? nb : 64;
    const size_t nt = (size_t)(nbp / 16) * (nbp / 16 + 1) / 2;
    const size_t n = (size_t)((rows + kGramRows - 1) / kGramRows);
    return (n + n / 32 + 2) * nt * 256 + 2 * (size_t)nbp * nbp;
}

template <typename C> void launch_panel_recon(const ReconPanel<C>& in, hipStream_t s)
{
    if (in.nb == 32) { subpanel<C, 32>(in, 0, 0, s); return; }
    if (in.nb == 64) { subpanel<C, 64>(in, 0, 0, s); return; }
    // nb = 128: two sub-panels of 64 columns, the second one updated with the first one's reflector in the work panel
    ReconPanel<C> a = in;
    launch_panel_gather<C, C>(in.A, in.lda, in.arow, in.acol, in.lq != 0, in.len, 128, in.P, in.ldv, s);
    a.src = nullptr;
    subpanel<C, 64>(a, 0, 0, s);
    C* right = a.P + 64 * a.ldv;
    int ns = launch_block_wt<C>(64, false, right, a.ldv, a.len, 64, a.wp_cols, a.V, a.ldv, a.Wp, a.stop, s);
    launch_block_tw<C>(64, a.Wp, ns, 64, a.Tf, a.nb, a.W2, s);
    launch_block_sub<C>(false, right, a.ldv, a.len, 64, 64, a.Vt, a.nb, a.W2, 64, a.stop, s);
    subpanel<C, 64>(a, 64, 64, s);
    ns = launch_block_wt<C>(64, false, a.V + 64 * a.ldv, a.ldv, a.len, 64, a.wp_cols, a.V, a.ldv, a.Wp, a.stop, s);
    static bool attr_set = false;
    const size_t bytes = 4 * 64 * 66 * sizeof(double);
    if (!attr_set) {
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(panel_join_kernel<C>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
        attr_set = true;
    }
    // (X, 64 x 64 doubles, is free between the sub-panel's panel_apply_kernel and the next panel)
    hipLaunchKernelGGL((join_sum_kernel<C>), dim3(256), dim3(256), 0, s, a.Wp, ns, a.X);
    hipLaunchKernelGGL((panel_join_kernel<C>), dim3(1), dim3(1024), bytes, s, a.X, a.Tf, (int64_t)a.nb);
}

template void launch_panel_recon<float>(const ReconPanel<float>&, hipStream_t);
template void launch_panel_recon<double>(const ReconPanel<double>&, hipStream_t);

}  // namespace svb
