// Small matrices (both dimensions up to 256): one workgroup takes the matrix to bidiagonal form directly, in registers.
//
// The two-stage method is a chain of launches at this size (256 x 256 in f64: 15 panels, 15 updates, two chases and half
// a dozen small kernels, 1.4 ms of dependent work in front of stage 3).  Here a column costs three barriers:
//   the column, in LDS -> left reflector (every wave forms it for itself) -> products with the wave's columns, summed
//   over its lanes -> update; the row, to LDS -> right reflector -> products with the rows, summed over the waves
//   through LDS -> update; the next column to LDS.
// Eight waves.  Lane l of every wave holds rows l, l + 64, ..; wave w columns w, w + 8, ..: both directions shrink evenly.
// The matrix is 4 x 32 elements a thread at 256 x 256.  In f64 that is more than the registers hold, so the first 64
// columns, which are the first to be finished, lie in LDS (each thread's own elements, 128 KB).
// Bound by instruction issue at the larger sizes (two waves a SIMD; the multiply-adds are two thirds of it in f32 at 256)
// and by the chain of the two reflectors at the small ones, about 2000 cycles a column.  The columns go in phases of 64,
// in which the finished row and column slots are left out by compilation; a wave's elements are taken a column at a time
// where they lie in LDS (four columns at a time, 32 more registers, were spilled: f64 256 1.48 ms a call against 1.15).
// In f64 with four row slots the registers do not suffice all the same: of the two runs below 53 (129 to 192 columns) and 136
// (193 to 256) registers are spilled; every other form keeps everything.
// H = I - g u u^T with u not normalised.  The matrix is scaled by a power of two so that its largest entry is in [0.5, 1),
// and the bidiagonal scaled back.  A line whose sum of squares is so small that subnormal squares can be a part of it
// (SmallRange::kLow) has to be moved up by a power of two first, or its reflector is not orthogonal, and it also hits
// lines of order one.  That is left to a second run from the start, which only a matrix with such a line pays for: with the
// branch in every column of the one run a call took up to 5 % longer.  A tail whose squares all underflow gives H = I, and so
// does, in the second run, one below 2^-96 (f32) or 2^-850 (f64).
#include "svb_internal.h"
#include "lane_ops.h"

namespace svb {

namespace {

// a's sum in the lanes where `up` is clear, b's in the others, over pairs of lanes that a data-parallel move brings together
template <int CTRL, typename C> __device__ __forceinline__ C pair_sum(C a, C b, bool up)
{
    const C keep = up ? b : a, give = up ? a : b;
    return keep + dpp<CTRL>(give);
}
// Sums of x[0 .. N-1] over the wave's 64 lanes, N a power of two from 4 to 32: every exchange halves the number of
// values a lane carries.  Lane l holds the sum of x[sum_index<N>(l)] on return.
template <int N> __device__ __forceinline__ int sum_index(int l)
{
    int c = 0, n = N;
    c += (l & 32) ? n / 2 : 0; n /= 2;
    if (n > 1) { c += (l & 16) ? n / 2 : 0; n /= 2; }
    if (n > 1) { c += (l & 8) ? n / 2 : 0; n /= 2; }
    if (n > 1) { c += (l & 4) ? n / 2 : 0; n /= 2; }
    if (n > 1) { c += (l & 2) ? n / 2 : 0; n /= 2; }
    return c;
}
template <int N, typename C> __device__ __forceinline__ C wave_sums(C (&x)[N], int lane)
{
    static_assert(N >= 4 && N <= 32, "range");
#pragma unroll
    for (int c = 0; c < N / 2; ++c) {
        swap_halves(x[c], x[c + N / 2]);
        x[c] += x[c + N / 2];
    }
#pragma unroll
    for (int c = 0; c < N / 4; ++c) {
        swap_rows(x[c], x[c + N / 4]);
        x[c] += x[c + N / 4];
    }
    if constexpr (N >= 8) {
#pragma unroll
        for (int c = 0; c < N / 8; ++c) x[c] = pair_sum<kRor8>(x[c], x[c + N / 8], lane & 8);
    } else x[0] += dpp<kRor8>(x[0]);
    if constexpr (N >= 16) {
#pragma unroll
        for (int c = 0; c < N / 16; ++c) x[c] = pair_sum<kHalfMirror>(x[c], x[c + N / 16], lane & 4);
    } else x[0] += dpp<kHalfMirror>(x[0]);
    if constexpr (N >= 32) x[0] = pair_sum<kSwap2>(x[0], x[1], lane & 2);
    else x[0] += dpp<kSwap2>(x[0]);
    return x[0] + dpp<kSwap1>(x[0]);
}
__device__ __forceinline__ float ldexp_of(float x, int e) { return __builtin_amdgcn_ldexpf(x, e); }
__device__ __forceinline__ double ldexp_of(double x, int e) { return __builtin_amdgcn_ldexp(x, e); }

// sums of squares below kLow are formed again from the line times 2^kUp (an entry is at most 2^8, the matrix's norm)
template <typename C> struct SmallRange;
template <> struct SmallRange<float> { static constexpr float kLow = 0x1p-96f; static constexpr int kUp = 48; };
template <> struct SmallRange<double> { static constexpr double kLow = 0x1p-900; static constexpr int kUp = 400; };

// The reflector of a line with first entry alpha and tail of squared norm ss: H = I - g u u^T, u = (alpha - beta, tail)
template <typename C> __device__ __forceinline__ void reflector(C alpha, C ss, C& beta, C& u0, C& g)
{
    const bool ident = ss < SmallRange<C>::kLow;
    const C b = copysign(newton_sqrt(fma(alpha, alpha, ss)), -alpha);
    u0 = ident ? (C)0 : alpha - b;   // (b is not a number where everything is zero)
    g = ident ? (C)0 : newton_rcp(-b * u0);
    beta = ident ? alpha : b;
}

// RJ, CJ: rows and columns in units of 64
template <typename C, int RJ, int CJ> struct SmallGeom {
    static constexpr int NC = 8 * CJ;                                          // columns a wave
    static constexpr int LC = sizeof(C) == 8 && RJ == 4 && CJ == 4 ? 8 : 0;    // of them in LDS
    static constexpr int NR = 64 * RJ;
    static constexpr int oCol = 0, oU = oCol + NR, oW = oU + 8 * NC, oZ = oW + 8 * NC, oS = oZ + 8 * NR, oD = oS + 8, oE = oD + NR,
                         oA = oE + NR;
    static constexpr size_t kBytes = (size_t)(oA + LC * RJ * 512) * sizeof(C);
    static_assert(kBytes <= 160 * 1024, "LDS");
};

// One run.  True, and nothing written, where a line would have to be moved up (never with CAREFUL, which moves them).
template <bool CAREFUL, typename T, typename C, int RJ, int CJ>
__device__ __forceinline__ bool small_run(const T* A, int64_t lda, int m, int n, int transpose, C* __restrict__ d,
                                          C* __restrict__ e, C* sm, double* sh_big)
{
    using Gm = SmallGeom<C, RJ, CJ>;
    constexpr int NC = Gm::NC, LC = Gm::LC, RC = NC - LC, NR = Gm::NR, NG = NC / 4, LG = LC / 4;
    C *col = sm + Gm::oCol, *ub = sm + Gm::oU, *wb = sm + Gm::oW, *zb = sm + Gm::oZ, *sq = sm + Gm::oS, *la = sm + Gm::oA;
    C *dl = sm + Gm::oD, *el = sm + Gm::oE;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // this thread's slots in LDS: two bases, so that a slot is within an instruction's 16-bit offset of one of them
    int la0 = tid, la1 = tid + 16 * 512;
    asm volatile("" : "+v"(la0), "+v"(la1));
    auto la_at = [=](int slot) -> C& { return slot < 16 ? la[la0 + slot * 512] : la[la1 + (slot - 16) * 512]; };

    // ---- the matrix (m rows, n <= m columns; A is its transpose where asked), zero outside; largest magnitude
    C a[RJ][RC];
    double big = 0.0;
    bool bad = false;
    auto load = [&](int c, int j) -> C {
        const int r = lane + 64 * j, q = 8 * c + wave;
        C v = 0;
        if (r < m && q < n) v = ld_as<C, T>(transpose ? A + q + r * lda : A + r + q * lda);
        const double x = fabs((double)v);
        bad |= !(x <= (sizeof(C) == 8 ? 1.7976931348623157e308 : 3.4028234663852886e38));
        big = fmax(big, x);
        return v;
    };
#pragma unroll
    for (int c = 0; c < LC; ++c)
#pragma unroll
        for (int j = 0; j < RJ; ++j) la_at(c * RJ + j) = load(c, j);
#pragma unroll
    for (int c = 0; c < RC; ++c)
#pragma unroll
        for (int j = 0; j < RJ; ++j) a[j][c] = load(LC + c, j);
    for (int off = 32; off > 0; off >>= 1) big = fmax(big, __shfl_xor(big, off, kWave));
    if (__any(bad)) big = NAN;
    if (lane == 0) sh_big[wave] = big;
    __syncthreads();
    big = 0.0;
#pragma unroll
    for (int w = 0; w < 8; ++w) {
        const double x = sh_big[w];
        bad |= x != x;
        big = fmax(big, x);
    }
    if (bad) {
        for (int i = tid; i < n; i += 512) {
            d[i] = (C)NAN;
            e[i] = 0;
        }
        return false;
    }
    const int ex = big > 0.0 ? __builtin_amdgcn_frexp_exp(big) : 0;
#pragma unroll
    for (int c = 0; c < LC; ++c)
#pragma unroll
        for (int j = 0; j < RJ; ++j) la_at(c * RJ + j) = ldexp_of(la_at(c * RJ + j), -ex);
#pragma unroll
    for (int c = 0; c < RC; ++c)
#pragma unroll
        for (int j = 0; j < RJ; ++j) a[j][c] = ldexp_of(a[j][c], -ex);

    if (wave == 0) {
#pragma unroll
        for (int j = 0; j < RJ; ++j) {
            if constexpr (LC > 0) {
                col[lane + 64 * j] = la_at(j);
                la_at(j) = 0;
            } else {
                col[lane + 64 * j] = a[j][0];
                a[j][0] = 0;
            }
        }
    }
    lds_barrier();
    bool again = false;
    // Columns 64 J0 .. 64 J0 + 63 as one phase: the rows of the slots below J0 and the columns of the groups below 2 J0
    // are finished, and only the first two groups of a phase can be finished within it.
    unroll<CJ>([&](auto phase) {
        constexpr int J0 = decltype(phase)::value, G0 = 2 * J0;
        // f(group, column of the group, its elements, pre's value for it) over the columns of COUNT groups of four from
        // FIRST on; store: the elements go back
        auto groups = [&](auto first, auto count, int k, auto store, auto&& pre, auto&& f) {
            unroll<decltype(count)::value>([&](auto ic) {
                constexpr int q = decltype(first)::value + decltype(ic)::value;
                const std::integral_constant<int, q> qc{};
                if (q < G0 + 2 && 8 * (4 * q + 3) + wave <= k) return;
                C y[4];
                pre(qc, y);
                unroll<4>([&](auto uc) {
                    constexpr int u = decltype(uc)::value;
                    C x[RJ];
#pragma unroll
                    for (int j = J0; j < RJ; ++j) {
                        if constexpr (q < LG) x[j] = la_at((4 * q + u) * RJ + j);
                        else x[j] = a[j][4 * (q - LG) + u];
                    }
                    f(qc, uc, x, y[u]);
                    if constexpr (decltype(store)::value) {
#pragma unroll
                        for (int j = J0; j < RJ; ++j) {
                            if constexpr (q < LG) la_at((4 * q + u) * RJ + j) = x[j];
                            else a[j][4 * (q - LG) + u] = x[j];
                        }
                    }
                });
            });
        };
        auto none = [](auto, C (&)[4]) {};
        constexpr std::integral_constant<int, G0> kFirst{};
        constexpr std::integral_constant<int, NG - G0> kAll{};
        constexpr std::integral_constant<bool, true> kStore{};
        constexpr std::integral_constant<bool, false> kRead{};
        const int kend = min(n, 64 * (J0 + 1));
        for (int k = 64 * J0; k < kend; ++k) {
            // ---- left reflector from column k
            C alpha = col[k];
            C v[RJ], s4 = 0;
#pragma unroll
            for (int j = J0; j < RJ; ++j) {
                const C t = col[lane + 64 * j];
                v[j] = j > J0 || lane + 64 * j > k ? t : (C)0;
                s4 = fma(v[j], v[j], s4);
            }
            s4 = wave_sum(s4);
            bool low = s4 < SmallRange<C>::kLow;   // (the same in every lane and wave)
            again |= low && s4 > (C)0;
            low = CAREFUL && __any(low);
            if (low) {
                alpha = ldexp_of(alpha, SmallRange<C>::kUp);
                s4 = 0;
#pragma unroll
                for (int j = J0; j < RJ; ++j) {
                    v[j] = ldexp_of(v[j], SmallRange<C>::kUp);
                    s4 = fma(v[j], v[j], s4);
                }
                s4 = wave_sum(s4);
            }
            C hb, hu, hg;
            reflector(alpha, s4, hb, hu, hg);
            dl[k] = low ? ldexp_of(hb, -SmallRange<C>::kUp) : hb;
            if (k == n - 1) break;
            v[J0] = lane + 64 * J0 == k ? hu : v[J0];
            // products with the columns, CH columns of a wave at a time: sums over the lanes, times g, to the wave's part of LDS
            constexpr int NL = NC - 8 * J0, CH = LC && J0 == 0 ? 4 : (NL % 16 || LC ? 8 : 16);   // (registers are short in the LDS form)
            unroll<NL / CH>([&](auto hc) {
                constexpr int c0 = 8 * J0 + decltype(hc)::value * CH;
                C w[CH];
#pragma unroll
                for (int c = 0; c < CH; ++c) w[c] = 0;
                groups(std::integral_constant<int, c0 / 4>{}, std::integral_constant<int, CH / 4>{}, k, kRead, none,
                       [&](auto qc, auto uc, const C (&x)[RJ], C) {
                    constexpr int c = 4 * decltype(qc)::value + decltype(uc)::value - c0;
#pragma unroll
                    for (int j = J0; j < RJ; ++j) w[c] = fma(v[j], x[j], w[c]);
                });
                const C t = wave_sums<CH>(w, lane);
                wb[wave * NC + c0 + sum_index<CH>(lane)] = hg * t;
            });
            // ---- update; the squared norm of row k's tail (finished columns are zero; column k + 1 is left out)
            const int k1 = k + 1, q1 = k1 >> 5, u1 = (k1 >> 3) & 3;
            const bool mine = (k1 & 7) == wave;
            const bool row = lane == (k & 63);
            groups(kFirst, kAll, k, kStore, [&](auto qc, C (&y)[4]) {
#pragma unroll
                for (int u = 0; u < 4; ++u) y[u] = wb[wave * NC + 4 * decltype(qc)::value + u];
            }, [&](auto, auto, C (&x)[RJ], C w) {
#pragma unroll
                for (int j = J0; j < RJ; ++j) x[j] = fma(-v[j], w, x[j]);
            });
            C ss[4] = {0, 0, 0, 0};
            groups(kFirst, kAll, k, kRead, none, [&](auto qc, auto uc, const C (&x)[RJ], C) {
                constexpr int q = decltype(qc)::value, u = decltype(uc)::value;
                C y = x[J0];
                if (q <= G0 + 2) y = mine && q1 == q && u1 == u ? (C)0 : y;   // (k + 1 may be the next phase's first column)
                ss[u] = fma(y, y, ss[u]);
            });
            if (row) {
                groups(kFirst, kAll, k, kRead, none, [&](auto qc, auto uc, const C (&x)[RJ], C) {
                    ub[wave * NC + 4 * decltype(qc)::value + decltype(uc)::value] = x[J0];
                });
                sq[wave] = (ss[0] + ss[1]) + (ss[2] + ss[3]);
            }
            lds_barrier();
            // ---- right reflector from row k
            C alpha2 = ub[(k1 & 7) * NC + (k1 >> 3)], s8;
            if constexpr (LC > 0) {
                s8 = lane < 8 ? sq[lane & 7] : (C)0;
                s8 += dpp<kHalfMirror>(s8);
                s8 += dpp<kSwap2>(s8);
                s8 += dpp<kSwap1>(s8);
                s8 = lane_value(s8, 0);
            } else {
                C t[8];
#pragma unroll
                for (int w = 0; w < 8; ++w) t[w] = sq[w];
                s8 = ((t[0] + t[1]) + (t[2] + t[3])) + ((t[4] + t[5]) + (t[6] + t[7]));
            }
            bool low2 = s8 < SmallRange<C>::kLow;
            again |= low2 && s8 > (C)0;
            low2 = CAREFUL && __any(low2);
            if (low2) {   // (the row stays as it is in LDS: only the sum, u's first entry and z are moved)
                alpha2 = ldexp_of(alpha2, SmallRange<C>::kUp);
                s8 = 0;
                for (int q = k1 + 1 + lane; q < 8 * NC; q += 64) {
                    const C y = ldexp_of(ub[(q & 7) * NC + (q >> 3)], SmallRange<C>::kUp);
                    s8 = fma(y, y, s8);
                }
                s8 = wave_sum(s8);
            }
            C fb, fu, fg;
            reflector(alpha2, s8, fb, fu, fg);
            if (low2) {
                fb = ldexp_of(fb, -SmallRange<C>::kUp);
                fu = ldexp_of(fu, -SmallRange<C>::kUp);
            }
            el[k] = fb;
            C z[RJ];
#pragma unroll
            for (int j = J0; j < RJ; ++j) z[j] = 0;
            // (the entry of column k + 1 stays in LDS for the waves that have yet to read it: u's first entry is put in its
            // place as it is read)
            auto entries = [&](auto qc, C (&y)[4]) {
                constexpr int q = decltype(qc)::value;
#pragma unroll
                for (int u = 0; u < 4; ++u) y[u] = ub[wave * NC + 4 * q + u];
                if (q <= G0 + 2 && mine && q1 == q) {
#pragma unroll
                    for (int u = 0; u < 4; ++u) y[u] = u1 == u ? fu : y[u];
                }
            };
            groups(kFirst, kAll, k, kRead, entries, [&](auto, auto, const C (&x)[RJ], C y) {
#pragma unroll
                for (int j = J0; j < RJ; ++j) z[j] = fma(x[j], y, z[j]);
            });
#pragma unroll
            for (int j = J0; j < RJ; ++j) zb[wave * NR + lane + 64 * j] = z[j];
            lds_barrier();
#pragma unroll
            for (int j = J0; j < RJ; ++j) {
                C p[8];
#pragma unroll
                for (int w = 0; w < 8; ++w) p[w] = zb[w * NR + lane + 64 * j];
                z[j] = -fg * (((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7])));
                if constexpr (LC > 0) __builtin_amdgcn_sched_barrier(0);
            }
            if (low2) {   // (fg is at most 2^96 or 2^900, an entry of z above as small as the row's)
#pragma unroll
                for (int j = J0; j < RJ; ++j) z[j] = ldexp_of(z[j], 2 * SmallRange<C>::kUp);
            }
            // ---- update; column k + 1 to LDS and, finished, zero in the registers
            groups(kFirst, kAll, k, kStore, entries, [&](auto qc, auto uc, C (&x)[RJ], C y) {
                constexpr int q = decltype(qc)::value, u = decltype(uc)::value;
#pragma unroll
                for (int j = J0; j < RJ; ++j) x[j] = fma(z[j], y, x[j]);
                if (q <= G0 + 2 && mine && q1 == q && u1 == u) {
#pragma unroll
                    for (int j = J0; j < RJ; ++j) {
                        col[lane + 64 * j] = x[j];
                        x[j] = 0;
                    }
                }
            });
            lds_barrier();
        }
    });
    lds_barrier();
    if (!CAREFUL && __any(again)) return true;
    for (int i = tid; i < n; i += 512) {
        d[i] = ldexp_of(dl[i], ex);
        e[i] = i < n - 1 ? ldexp_of(el[i], ex) : (C)0;
    }
    return false;
}

template <typename T, typename C, int RJ, int CJ>
__global__ __launch_bounds__(512) void small_bidiag_kernel(const T* A, int64_t lda, int m, int n, int transpose,
                                                           C* __restrict__ d, C* __restrict__ e)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    __shared__ double sh_big[8];
    C* sm = reinterpret_cast<C*>(smem_raw);
    if (small_run<false, T, C, RJ, CJ>(A, lda, m, n, transpose, d, e, sm, sh_big)) {
        __syncthreads();
        small_run<true, T, C, RJ, CJ>(A, lda, m, n, transpose, d, e, sm, sh_big);
    }
}

template <typename T, typename C, int RJ, int CJ>
void small_launch(const T* A, int64_t lda, int m, int n, bool transpose, C* d, C* e, hipStream_t s)
{
    if constexpr (CJ > 1) {
        if (n <= 64 * (CJ - 1)) {
            small_launch<T, C, RJ, CJ - 1>(A, lda, m, n, transpose, d, e, s);
            return;
        }
    }
    using Gm = SmallGeom<C, RJ, CJ>;
    auto kern = small_bidiag_kernel<T, C, RJ, CJ>;
    static bool attr_set = false;
    if (!attr_set) {
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)Gm::kBytes);
        attr_set = true;
    }
    hipLaunchKernelGGL(kern, dim3(1), dim3(512), Gm::kBytes, s, A, lda, m, n, transpose ? 1 : 0, d, e);
}

}  // namespace

// d, e (min(m, n) entries each) of the m x n matrix, both dimensions at most kSmallMax
template <typename T, typename C>
void launch_small_bidiag(const T* A, int64_t lda, int64_t m, int64_t n, C* d, C* e, hipStream_t s)
{
    const bool tr = m < n;
    const int r = (int)(tr ? n : m), c = (int)(tr ? m : n);
    switch ((r + 63) / 64) {
    case 1: small_launch<T, C, 1, 1>(A, lda, r, c, tr, d, e, s); break;
    case 2: small_launch<T, C, 2, 2>(A, lda, r, c, tr, d, e, s); break;
    case 3: small_launch<T, C, 3, 3>(A, lda, r, c, tr, d, e, s); break;
    default: small_launch<T, C, 4, 4>(A, lda, r, c, tr, d, e, s); break;
    }
}
template void launch_small_bidiag<float, float>(const float*, int64_t, int64_t, int64_t, float*, float*, hipStream_t);
template void launch_small_bidiag<double, double>(const double*, int64_t, int64_t, int64_t, double*, double*, hipStream_t);
template void launch_small_bidiag<__half, float>(const __half*, int64_t, int64_t, int64_t, float*, float*, hipStream_t);
template void launch_small_bidiag<bf16_t, float>(const bf16_t*, int64_t, int64_t, int64_t, float*, float*, hipStream_t);

}  // namespace svb
