// Stage 1, products of a half-sweep with one block reflector for the whole panel (paper Section 3.1,
// Algorithm 1): with the panel's H = I - V T V^T (stage1_recon.hip) the trailing matrix C goes to H^T C in
// a QR sweep and to C H in an LQ sweep.  In panel orientation (p along the panel, q across it, C(p, q)
// at p + q lda or q + p lda) both are
//     W(c, q) = sum_p V(p, c) C(p, q),   W2 = -T^T W,   C(p, q) += sum_c V(p, c) W2(c, q),
// two matrix products of 2 rows cols nb flops each and nothing else: 8/3 n^3 in all.
//   block_wt_kernel    partial sums of W over ranges of p (C is read once)
//   block_tw_kernel    W2: the partial sums added up in a fixed order, multiplied by T^T and negated
//   block_sub_kernel   C += V W2 (C is read and written once)
// W and W2 are stored with c running fastest; V in both orders (Vt: c fastest), so that every operand but
// C is contiguous along the contraction and C is always touched along its contiguous direction.
#include <algorithm>

#include "svb_internal.h"
#include "lane_ops.h"
#include "mfma_gemm.h"

namespace svb {

namespace {

// one matrix instruction: D (TM x TM) += A (TM x G) B (G x TM); lane i + TM g supplies A[i][g] and B[g][i]
// and holds NR entries of column i of D, in the rows row(r, g).  VK consecutive elements of the contraction
// (16 bytes) from each lane group make VK instructions.
template <typename C> struct Mm;
template <> struct Mm<float> {
    typedef float acc_t __attribute__((ext_vector_type(16)));
    static constexpr int TM = 32, G = 2, VK = 4, NR = 16;
    static __device__ __forceinline__ acc_t mma(float a, float b, acc_t c)
    {
        return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int r, int g) { return 8 * (r >> 2) + 4 * g + (r & 3); }
};
template <> struct Mm<double> {
    typedef double acc_t __attribute__((ext_vector_type(4)));
    static constexpr int TM = 16, G = 4, VK = 2, NR = 4;
    static __device__ __forceinline__ acc_t mma(double a, double b, acc_t c)
    {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int r, int g) { return 4 * r + g; }
};

// a staged operand: rows of KC contraction elements (128 bytes), 16 bytes of padding behind each (sixteen
// rows read 16 bytes each without a bank conflict)
template <typename C> constexpr int kKC = 128 / (int)sizeof(C);
template <typename C> constexpr int kLD = 144 / (int)sizeof(C);
// lengths, ranges and tile sizes are multiples of this many lines (wt_plan; svb_svdvals pads to whole tiles), and whole
// chunks are read
constexpr int kUnit = 32;
static_assert(kUnit % kKC<float> == 0 && kUnit % kKC<double> == 0, "a chunk does not reach past the end of a range");

// Global memory goes through buffer instructions: a wave-uniform base, one 32-bit byte offset a lane, wave-uniform
// byte offsets (the host keeps 128 lines of the matrix below 2^32 bytes).
typedef __amdgpu_buffer_rsrc_t rsrc_t;
__device__ __forceinline__ rsrc_t make_rsrc(const void* base)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, 0xffffffff, 0x00020000);
}
template <typename C> struct Buf1;
template <> struct Buf1<float> {
    static __device__ __forceinline__ float ld(rsrc_t r, unsigned v, unsigned s)
    {
        return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, v, s, 0));
    }
    static __device__ __forceinline__ void st(rsrc_t r, unsigned v, unsigned s, float x)
    {
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, x), r, v, s, 0);
    }
};
template <> struct Buf1<double> {
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    static __device__ __forceinline__ double ld(rsrc_t r, unsigned v, unsigned s)
    {
        return __builtin_bit_cast(double, (u2)__builtin_amdgcn_raw_buffer_load_b64(r, v, s, 0));
    }
    static __device__ __forceinline__ void st(rsrc_t r, unsigned v, unsigned s, double x)
    {
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, x), r, v, s, 0);
    }
};

// ---- C += A B^T on tiles of BR x BJ -------------------------------------------------------------------
// C(r, j) at r * lda + j (j contiguous), A(r, k) at r * lda_r + k, B(j, k) at j * ldb_j + k; K a multiple of
// 32; nr and nj multiples of 32.  Nothing is done where *stop is set.  (Looked at behind the first chunk, where the flag
// would have come by itself: f32 32768, nb = 128 1185 ms a call against 1168; without: 1167.)
// Four waves in a square.  A lane's column of an accumulator tile is j, so C moves along its contiguous
// direction.  Tiles are numbered so that an XCD works on a contiguous range of them, eight columns of tiles
// at a time (their operands stay in its L2).
template <typename C, int BR, int BJ>
__global__ __launch_bounds__(256, sizeof(C) == 4 ? 3 : 2) void block_sub_kernel(C* __restrict__ Cm, int64_t lda, int nr, int nj,
                                                           const C* __restrict__ Ar, int64_t lda_r,
                                                           const C* __restrict__ Bj, int64_t ldb_j, int K,
                                                           const int* __restrict__ stop)
{
    using M = Mm<C>;
    typedef typename M::acc_t acc_t;
    constexpr int KC = kKC<C>, LD = kLD<C>, VK = M::VK, TM = M::TM;
    constexpr int WR = BR / 2, WJ = BJ / 2, NR = WR / TM, NJ = WJ / TM;   // tiles of a wave per direction
    constexpr int NPA = BR * 8 / 256, NPB = BJ * 8 / 256;                 // 16-byte pieces a thread stages per chunk
    __shared__ __align__(16) C As[BR * LD];
    __shared__ __align__(16) C Bs[BJ * LD];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = lane % TM, g = lane / TM;
    if (*stop) return;

    const int ntr = (nr + BR - 1) / BR, ntj = (nj + BJ - 1) / BJ, nt = ntr * ntj;
    const int per = (nt + 7) / 8;
    const int t = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per || t >= nt) return;
    const int grp = t / (8 * ntr), in = t - grp * 8 * ntr;
    const int gs = min(8, ntj - grp * 8);
    const int r0 = in / gs * BR, j0 = (grp * 8 + in % gs) * BJ;

    C ra[NPA][VK], rb[NPB][VK];
    auto fetch = [&](int k0) {
        // (a row beyond the edge repeats the last one: its products are not stored)
#pragma unroll
        for (int e = 0; e < NPA; ++e) {
            const int idx = tid + e * 256, row = idx >> 3, kk = (idx & 7) * VK;
            VecIO<C, C>::ld(&Ar[(int64_t)min(r0 + row, nr - 1) * lda_r + k0 + kk], ra[e]);
        }
#pragma unroll
        for (int e = 0; e < NPB; ++e) {
            const int idx = tid + e * 256, row = idx >> 3, kk = (idx & 7) * VK;
            VecIO<C, C>::ld(&Bj[(int64_t)min(j0 + row, nj - 1) * ldb_j + k0 + kk], rb[e]);
        }
    };
    fetch(0);

    const int rw = r0 + (wave >> 1) * WR, jw = j0 + (wave & 1) * WJ;
    const unsigned line = (unsigned)(lda * sizeof(C));
    const unsigned voff = (unsigned)M::row(0, g) * line + (unsigned)(i * sizeof(C));
    const bool edge = rw + WR > nr || jw + WJ > nj;
    acc_t acc[NR][NJ];
    auto tile_on = [&](int a, int b) { return !edge || (rw + a * TM < nr && jw + b * TM < nj); };
#pragma unroll
    for (int a = 0; a < NR; ++a)
#pragma unroll
        for (int b = 0; b < NJ; ++b) {
            if (tile_on(a, b)) {
                const rsrc_t rs = make_rsrc(Cm + (int64_t)(rw + a * TM) * lda + jw + b * TM);
#pragma unroll
                for (int r = 0; r < M::NR; ++r) acc[a][b][r] = Buf1<C>::ld(rs, voff, (unsigned)M::row(r, 0) * line);
            } else {
#pragma unroll
                for (int r = 0; r < M::NR; ++r) acc[a][b][r] = 0;
            }
        }
    for (int k0 = 0; k0 < K; k0 += KC) {
        if (k0) lds_barrier();
#pragma unroll
        for (int e = 0; e < NPA; ++e) {
            const int idx = tid + e * 256;
            VecIO<C, C>::st(&As[(idx >> 3) * LD + (idx & 7) * VK], ra[e]);
        }
#pragma unroll
        for (int e = 0; e < NPB; ++e) {
            const int idx = tid + e * 256;
            VecIO<C, C>::st(&Bs[(idx >> 3) * LD + (idx & 7) * VK], rb[e]);
        }
        lds_barrier();
        if (k0 + KC < K) fetch(k0 + KC);
#pragma unroll
        for (int kk = 0; kk < KC; kk += M::G * VK) {
            C fa[NR][VK], fb[NJ][VK];
#pragma unroll
            for (int a = 0; a < NR; ++a) VecIO<C, C>::ld(&As[((wave >> 1) * WR + a * TM + i) * LD + kk + g * VK], fa[a]);
#pragma unroll
            for (int b = 0; b < NJ; ++b) VecIO<C, C>::ld(&Bs[((wave & 1) * WJ + b * TM + i) * LD + kk + g * VK], fb[b]);
#pragma unroll
            for (int q = 0; q < VK; ++q)
#pragma unroll
                for (int a = 0; a < NR; ++a)
#pragma unroll
                    for (int b = 0; b < NJ; ++b) acc[a][b] = M::mma(fa[a][q], fb[b][q], acc[a][b]);
        }
    }
#pragma unroll
    for (int a = 0; a < NR; ++a)
#pragma unroll
        for (int b = 0; b < NJ; ++b) {
            if (tile_on(a, b)) {
                const rsrc_t rs = make_rsrc(Cm + (int64_t)(rw + a * TM) * lda + jw + b * TM);
#pragma unroll
                for (int r = 0; r < M::NR; ++r) Buf1<C>::st(rs, voff, (unsigned)M::row(r, 0) * line, acc[a][b][r]);
            }
        }
}

// ---- partial sums of W ---------------------------------------------------------------------------------
// Wp(s, q, c) at (s * nq + q) * NBW + c: the sum over p in [s * chunk, (s + 1) * chunk) of V(p, c) C(p, q),
// V(p, c) at p + c * ldv.  len and chunk multiples of 32, nq a multiple of 32.
// QR orientation: C's tile is staged as it lies, p fastest; LQ: q fastest, its operand read element by element.
// *stop as in block_sub_kernel.
template <typename C, int NBW, int QT, bool LQ>
__global__ __launch_bounds__(256, 2) void block_wt_kernel(const C* __restrict__ Cm, int64_t lda, int len, int nq,
                                                       const C* __restrict__ V, int64_t ldv, int chunk,
                                                       C* __restrict__ Wp, const int* __restrict__ stop)
{
    using M = Mm<C>;
    typedef typename M::acc_t acc_t;
    constexpr int KC = kKC<C>, LD = kLD<C>, VK = M::VK, TM = M::TM;
    constexpr int WQN = NBW == 32 ? 4 : 2, WCN = 4 / WQN;   // waves across q and c
    constexpr int WQ = QT / WQN, WC = NBW / WCN;
    constexpr int NTQ = WQ / TM, NTC = WC / TM;
    static_assert(NTQ >= 1 && NTC >= 1, "a wave has a tile");
    constexpr int LDQ = QT + (sizeof(C) == 4 ? 4 : 8);      // LQ: rows of q
    constexpr int NPV = (NBW * 8 + 255) / 256, NPC = QT * 8 / 256;
    constexpr int kV = NBW * LD, kC = LQ ? KC * LDQ : QT * LD;
    __shared__ __align__(16) C Vs[kV];
    __shared__ __align__(16) C Cs[kC];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int i = lane % TM, g = lane / TM;
    const int q0 = blockIdx.x * QT;
    const int pbeg = blockIdx.y * chunk, pend = min(len, pbeg + chunk);
    if (*stop) return;

    C rv[NPV][VK], rc[NPC][VK];
    auto fetch = [&](int p0) {   // (beyond nq the last one again: those sums are not stored)
#pragma unroll
        for (int e = 0; e < NPV; ++e) {
            const int idx = tid + e * 256, row = idx >> 3, kk = (idx & 7) * VK;
            VecIO<C, C>::ld(&V[(int64_t)row * ldv + p0 + kk], rv[e]);
        }
#pragma unroll
        for (int e = 0; e < NPC; ++e) {
            const int idx = tid + e * 256;
            if constexpr (LQ) {
                const int p = idx / (QT / VK), qq = idx % (QT / VK) * VK;
                VecIO<C, C>::ld(&Cm[(int64_t)(p0 + p) * lda + min(q0 + qq, nq - VK)], rc[e]);
            } else {
                const int row = idx >> 3, kk = (idx & 7) * VK;
                VecIO<C, C>::ld(&Cm[(int64_t)min(q0 + row, nq - 1) * lda + p0 + kk], rc[e]);
            }
        }
    };
    fetch(pbeg);
    const int cw = wave / WQN * WC, qw = wave % WQN * WQ;
    acc_t acc[NTC][NTQ];
#pragma unroll
    for (int a = 0; a < NTC; ++a)
#pragma unroll
        for (int b = 0; b < NTQ; ++b)
#pragma unroll
            for (int r = 0; r < M::NR; ++r) acc[a][b][r] = 0;
    for (int p0 = pbeg; p0 < pend; p0 += KC) {
        if (p0 > pbeg) lds_barrier();
#pragma unroll
        for (int e = 0; e < NPV; ++e) {
            const int idx = tid + e * 256, row = idx >> 3, kk = (idx & 7) * VK;
            VecIO<C, C>::st(&Vs[row * LD + kk], rv[e]);
        }
#pragma unroll
        for (int e = 0; e < NPC; ++e) {
            const int idx = tid + e * 256;
            if constexpr (LQ) VecIO<C, C>::st(&Cs[idx / (QT / VK) * LDQ + idx % (QT / VK) * VK], rc[e]);
            else VecIO<C, C>::st(&Cs[(idx >> 3) * LD + (idx & 7) * VK], rc[e]);
        }
        lds_barrier();
        if (p0 + KC < pend) fetch(p0 + KC);
#pragma unroll
        for (int kk = 0; kk < KC; kk += M::G * VK) {
            C fa[NTC][VK], fb[NTQ][VK];
#pragma unroll
            for (int a = 0; a < NTC; ++a) VecIO<C, C>::ld(&Vs[(cw + a * TM + i) * LD + kk + g * VK], fa[a]);
#pragma unroll
            for (int b = 0; b < NTQ; ++b) {
                if constexpr (LQ) {
#pragma unroll
                    for (int q = 0; q < VK; ++q) fb[b][q] = Cs[(kk + g * VK + q) * LDQ + qw + b * TM + i];
                } else {
                    VecIO<C, C>::ld(&Cs[(qw + b * TM + i) * LD + kk + g * VK], fb[b]);
                }
            }
#pragma unroll
            for (int q = 0; q < VK; ++q)
#pragma unroll
                for (int a = 0; a < NTC; ++a)
#pragma unroll
                    for (int b = 0; b < NTQ; ++b) acc[a][b] = M::mma(fa[a][q], fb[b][q], acc[a][b]);
        }
    }
#pragma unroll
    for (int a = 0; a < NTC; ++a)
#pragma unroll
        for (int b = 0; b < NTQ; ++b) {
            const int q = q0 + qw + b * TM + i;
            if (q < nq) {
                C* o = Wp + ((int64_t)blockIdx.y * nq + q) * NBW + cw + a * TM;
                if constexpr (sizeof(C) == 4) {
#pragma unroll
                    for (int r = 0; r < M::NR; r += 4) {
                        const C v[4] = {acc[a][b][r], acc[a][b][r + 1], acc[a][b][r + 2], acc[a][b][r + 3]};
                        VecIO<C, C>::st(o + M::row(r, g), v);
                    }
                } else {
#pragma unroll
                    for (int r = 0; r < M::NR; ++r) o[M::row(r, g)] = acc[a][b][r];
                }
            }
        }
}

// ---- W2 = -T^T sum_s Wp(s) -----------------------------------------------------------------------------
// T(c', c) at c * ldt + c', zero below the diagonal; W2(c, q) at q * NBW + c.  32 columns a workgroup.
template <typename C, int NBW>
__global__ __launch_bounds__(256) void block_tw_kernel(const C* __restrict__ Wp, int ns, int nq,
                                                       const C* __restrict__ T, int64_t ldt, C* __restrict__ W2)
{
    using M = Mm<C>;
    typedef typename M::acc_t acc_t;
    constexpr int VK = M::VK, TM = M::TM, LD = NBW + VK;
    __shared__ __align__(16) C Ws[32 * LD];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int i = lane % TM, g = lane / TM;
    const int64_t q0 = (int64_t)blockIdx.x * 32;
    const int64_t plane = (int64_t)nq * NBW;
    for (int idx = tid; idx < 32 * NBW / VK; idx += 256) {
        const C* p = Wp + q0 * NBW + (int64_t)idx * VK;
        C s[VK];
        VecIO<C, C>::ld(p, s);
        int z = 1;
        auto batch = [&](auto n) {
            constexpr int N = decltype(n)::value;
            C x[N][VK];
#pragma unroll
            for (int u = 0; u < N; ++u) VecIO<C, C>::ld(p + (z + u) * plane, x[u]);
#pragma unroll
            for (int u = 0; u < N; ++u)
#pragma unroll
                for (int q = 0; q < VK; ++q) s[q] += x[u][q];
        };
        for (; z + 16 <= ns; z += 16) batch(std::integral_constant<int, 16>{});
        for (; z + 4 <= ns; z += 4) batch(std::integral_constant<int, 4>{});
        for (; z < ns; ++z) {
            C x[VK];
            VecIO<C, C>::ld(p + z * plane, x);
#pragma unroll
            for (int q = 0; q < VK; ++q) s[q] += x[q];
        }
        VecIO<C, C>::st(&Ws[idx * VK / NBW * LD + idx * VK % NBW], s);
    }
    __syncthreads();
    constexpr int NQ = 32 / TM, NC = NBW / TM;
    for (int t = wave; t < NQ * NC; t += 4) {
        const int ct = NC - 1 - t / NQ, qt = t % NQ;   // the longest sums first
        acc_t acc;
#pragma unroll
        for (int r = 0; r < M::NR; ++r) acc[r] = 0;
        const C* ta = T + (ct * TM + i) * ldt + g * VK;
        const C* wb = &Ws[(qt * TM + i) * LD + g * VK];
#pragma unroll 4
        for (int k = 0; k < (ct + 1) * TM; k += M::G * VK) {
            C a[VK], b[VK];
            VecIO<C, C>::ld(ta + k, a);
            VecIO<C, C>::ld(wb + k, b);
#pragma unroll
            for (int q = 0; q < VK; ++q) acc = M::mma(a[q], b[q], acc);
        }
        C* o = W2 + (q0 + qt * TM + i) * NBW + ct * TM;
        if constexpr (sizeof(C) == 4) {
#pragma unroll
            for (int r = 0; r < M::NR; r += 4) {
                const C v[4] = {-acc[r], -acc[r + 1], -acc[r + 2], -acc[r + 3]};
                VecIO<C, C>::st(o + M::row(r, g), v);
            }
        } else {
#pragma unroll
            for (int r = 0; r < M::NR; ++r) o[M::row(r, g)] = -acc[r];
        }
    }
}

template <typename C, int NBW, int QT>
void wt_launch(bool lq, const C* Cm, int64_t lda, int len, int nq, const C* V, int64_t ldv, int chunk, int ns, C* Wp,
               const int* stop, hipStream_t s)
{
    const dim3 grid((unsigned)((nq + QT - 1) / QT), (unsigned)ns);
    if (lq) hipLaunchKernelGGL((block_wt_kernel<C, NBW, QT, true>), grid, dim3(256), 0, s, Cm, lda, len, nq, V, ldv, chunk, Wp, stop);
    else hipLaunchKernelGGL((block_wt_kernel<C, NBW, QT, false>), grid, dim3(256), 0, s, Cm, lda, len, nq, V, ldv, chunk, Wp, stop);
}

}  // namespace

// how the contraction over p is split: enough workgroups for the chip, at least 64 elements each, and
// partial sums within the workspace (block_wp_cols).  1024 workgroups where the size allows: two to four fit on
// a compute unit, and with 512 they all begin and end together (ms a call with 512 and 1024: f32 32768, nb = 128 1209, 1172;
// 16384, nb = 64 231, 225.5; f64 16384, nb = 128 510.5, 504).  Room for four times the longer side's columns makes 1024 the
// most that the large sizes can have, and eight and four ranges, about 500 workgroups, at the first sweeps of order 4096 and
// 8192.  With four times that room 1024 are reached there too, and are slower (4096 24.0 against 23.85, 8192 61.2 against 60.5:
// more partial sums, shorter ranges); 2048 at 32768 would be 0.9 % faster (1162), for 192 MiB.
// The order in which W is summed is no matter for the error: folding the accumulators every 512 terms left it where it is
// (mean over random matrices, f32: 8192 1.13e-7, folded 1.11e-7; 32768 1.25e-7, 1.29e-7; the tree of domain QRs 1.17e-7, 1.26e-7).
constexpr int64_t kMaxRanges = 64;   // (block_tw_kernel adds them up one after the other)
static int64_t max_ranges(int64_t len) { return std::max<int64_t>(1, std::min(len / 64, kMaxRanges)); }
int64_t block_wp_cols(int64_t rows, int64_t cols)
{
    const int64_t most = std::max(cols * max_ranges(rows), rows * max_ranges(cols));   // (a QR and an LQ sweep)
    return std::min(most, std::max<int64_t>(4 * rows, 32768));
}

struct WtPlan { int qt, ns, chunk; };
static WtPlan wt_plan(int nbw, int64_t len, int64_t nq, int64_t wp_cols)
{
    WtPlan p;
    p.qt = nbw == 32 ? 128 : (nq >= 128 * 128 ? 128 : 64);
    const int64_t strips = (nq + p.qt - 1) / p.qt;
    int64_t ns = (1024 + strips - 1) / strips;
    const int64_t room = wp_cols / nq;
    if (ns > room) ns = room;
    if (ns > max_ranges(len)) ns = max_ranges(len);
    if (ns < 1) ns = 1;
    int64_t chunk = ((len + ns - 1) / ns + kUnit - 1) / kUnit * kUnit;
    p.chunk = (int)chunk;
    p.ns = (int)((len + chunk - 1) / chunk);
    return p;
}

template <typename C>
int launch_block_wt(int nbw, bool lq, const C* Cm, int64_t lda, int64_t len, int64_t nq, int64_t wp_cols, const C* V,
                    int64_t ldv, C* Wp, const int* stop, hipStream_t s)
{
    const WtPlan p = wt_plan(nbw, len, nq, wp_cols);
    const int l = (int)len, q = (int)nq;
    if (nbw == 32) wt_launch<C, 32, 128>(lq, Cm, lda, l, q, V, ldv, p.chunk, p.ns, Wp, stop, s);
    else if (nbw == 64 && p.qt == 64) wt_launch<C, 64, 64>(lq, Cm, lda, l, q, V, ldv, p.chunk, p.ns, Wp, stop, s);
    else if (nbw == 64) wt_launch<C, 64, 128>(lq, Cm, lda, l, q, V, ldv, p.chunk, p.ns, Wp, stop, s);
    else if (p.qt == 64) wt_launch<C, 128, 64>(lq, Cm, lda, l, q, V, ldv, p.chunk, p.ns, Wp, stop, s);
    else wt_launch<C, 128, 128>(lq, Cm, lda, l, q, V, ldv, p.chunk, p.ns, Wp, stop, s);
    return p.ns;
}

template <typename C>
void launch_block_tw(int nbw, const C* Wp, int ns, int64_t nq, const C* T, int64_t ldt, C* W2, hipStream_t s)
{
    const dim3 grid((unsigned)(nq / 32)), blk(256);
    switch (nbw) {
    case 32: hipLaunchKernelGGL((block_tw_kernel<C, 32>), grid, blk, 0, s, Wp, ns, (int)nq, T, ldt, W2); break;
    case 64: hipLaunchKernelGGL((block_tw_kernel<C, 64>), grid, blk, 0, s, Wp, ns, (int)nq, T, ldt, W2); break;
    default: hipLaunchKernelGGL((block_tw_kernel<C, 128>), grid, blk, 0, s, Wp, ns, (int)nq, T, ldt, W2); break;
    }
}

// (the operands' order follows the orientation: a lane's direction is the contiguous one of C)
template <typename C>
void launch_block_sub(bool lq, C* Cm, int64_t lda, int64_t len, int64_t nq, int K, const C* Vt, int64_t ldvt,
                      const C* W2, int64_t ldw, const int* stop, hipStream_t s)
{
    const int nr = (int)(lq ? len : nq), nj = (int)(lq ? nq : len);
    const C* ar = lq ? Vt : W2;
    const C* bj_ = lq ? W2 : Vt;
    const int64_t la = lq ? ldvt : ldw, lb = lq ? ldw : ldvt;
    auto go = [&](auto kern, int br, int bj) {
        const int64_t nt = (int64_t)((nr + br - 1) / br) * ((nj + bj - 1) / bj);
        hipLaunchKernelGGL(kern, dim3((unsigned)((nt + 7) / 8 * 8)), dim3(256), 0, s, Cm, lda, nr, nj, ar, la, bj_, lb, K, stop);
    };
    const int64_t big = (int64_t)((nr + 127) / 128) * ((nj + 127) / 128);
    if (big >= 1024) go(block_sub_kernel<C, 128, 128>, 128, 128);
    else go(block_sub_kernel<C, 64, 64>, 64, 64);
}

#define SVB_INST(C)                                                                                                 \
    template int launch_block_wt<C>(int, bool, const C*, int64_t, int64_t, int64_t, int64_t, const C*, int64_t, C*, const int*, hipStream_t); \
    template void launch_block_tw<C>(int, const C*, int, int64_t, const C*, int64_t, C*, hipStream_t);              \
    template void launch_block_sub<C>(bool, C*, int64_t, int64_t, int64_t, int, const C*, int64_t, const C*, int64_t, const int*, hipStream_t)
SVB_INST(float);
SVB_INST(double);
#undef SVB_INST

}  // namespace svb
