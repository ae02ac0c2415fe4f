// Stage 2, first phase: band of B super-diagonals -> band of D = 8 super-diagonals
// (paper Section 3, second stage; the paper names a band-to-bidiagonal reduction without
// giving the algorithm, so this is a blocked bulge chase in the spirit of the successive
// band reduction literature; the second phase, D -> 1, is in stage2_narrow.hip).
//
// Block sweep s makes rows s*D .. s*D+D-1 final (at most D super-diagonals) and chases the
// fill down the band in steps of B columns.  Step t of sweep s works at c0 = (s+1)*D + t*B:
//   right: LQ of the D x B block X (rows rho .. rho+D-1, columns c0 .. c0+B-1; rho = s*D for
//          t = 0, rho = c0 - B otherwise); its D reflectors are applied from the right, as one
//          compact-WY block, to all other rows that have entries in those columns
//          (down to row c0+B-1), which fills the diagonal block Z (rows and columns c0 ..);
//   left:  QR of the first D columns of Z; the reflectors are applied from the left to the
//          other columns of Z and to the block right of it (A3), which becomes the next
//          step's upper block.
// Only D rows / columns of every bulge are annihilated per step; the rest moves down the band
// with the following sweeps.  Sweeps are pipelined: one workgroup per sweep, sweeps drawn from a
// ticket counter, a progress counter per sweep, bounded waits (as in stage2_chase.hip).  Of the
// blocks step (s+1, t) brings in, Z needs of step (s, t+1) its upper block and the D x D corner its left panel
// leaves, A3 the rest of that step's Z and the corner the right panel of step (s, t+2) leaves; the corners are
// stored and published ahead of their blocks, so that a sweep can follow its predecessor two steps behind.
//
// The whole reduction is one chain: what a sweep costs is the two steps its successor waits.  So of a
// step only the two panels and what the next panel needs of a block reflector (the first sixteen columns of Z,
// the first sixteen rows of A3) stand one behind the other; the rest of both block reflectors, and
// all traffic with the band, run beside the next panel.  Per step the workgroup holds the upper block U (rows
// c0-B .., the previous step's A3) and Z in LDS; every block is read once and written once per sweep.
// us per eight columns (one sweep), n = 8192, before (each block reflector in one piece between the panels,
// applied from LDS line by line; whole blocks published) -> now: f32 13.5 -> 8.3 (nb = 32), 20.8 -> 12.4 (64),
// 50 -> 32.0 (128); f64 16.5 -> 11.1 (32), 29.3 -> 18.3 (64).
//
// Packed band: entry (i,j) at band[(i - j + ku) + j*ldab], ku = 2B-1, ldab >= 3B.
#include <type_traits>
#include <utility>

#include "svb_internal.h"
#include "lane_ops.h"
#include "mfma_frag.h"

namespace svb {

namespace {

constexpr int kSweepDone = 0x7fffffff;
// Progress counters of consecutive sweeps are 32 bytes apart: their lines are polled by one workgroup and written
// by another all the time (with 4 bytes between them the reduction at n = 8192, nb = 32 took 10.8 ms in f32, 8.8 so).
constexpr int kProgressStride = 8;

// Barriers inside a workgroup are lds_barrier(): __syncthreads() would also wait for every outstanding
// global load and store, i.e. for the block prefetches that are meant to stay in flight across the
// phases of a step; visibility of global data between workgroups is handled separately (stores_done
// below, fences at the ends of a sweep).
// Every band access of this kernel is a device-scope atomic (written through to, and read
// from, the level all compute dies share), so publishing a step needs no cache write-back and
// consuming one no invalidate: the writer only waits until its stores have been acknowledged
// (s_waitcnt vmcnt(0)) before the barrier that precedes the progress store, and the reader
// issues its loads after the barrier that follows the progress load.
__device__ __forceinline__ void stores_done()
{
    __builtin_amdgcn_s_waitcnt(0x0f70);
}

template <typename C> __device__ __forceinline__ C rgld(const C* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename C> __device__ __forceinline__ void rgst(C* p, C v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// value of lane (l ^ pattern) through the data-parallel-primitive path (no LDS traffic)
template <int CTRL> __device__ __forceinline__ double dpp_get(double v)
{
    const long long b = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffll), CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xF, 0xF, true);
    return __builtin_bit_cast(double, ((long long)hi << 32) | (long long)(unsigned)lo);
}
constexpr int kDppXor1 = 0xB1;        // quad_perm [1,0,3,2]
constexpr int kDppXor2 = 0x4E;        // quad_perm [2,3,0,1]
constexpr int kDppHalfMirror = 0x141; // lane i <-> 7-i inside groups of 8

constexpr int kDppRor8 = 0x128;       // lane i <-> i^8 inside rows of 16 (rotate by 8)

// hardware reciprocal refined by Newton steps: a biased tau or scale makes every reflector slightly non-orthogonal in
// the same direction, which adds up
__device__ __forceinline__ double rrcp(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    r = fma(r, fma(-x, r, 1.0), r);
    return fma(r, fma(-x, r, 1.0), r);
}

// f(0), f(1), .. with the index as a compile-time constant
template <typename Fn, int... K> __device__ __forceinline__ void static_steps(Fn&& f, std::integer_sequence<int, K...>)
{
    (f(std::integral_constant<int, K>{}), ...);
}

// position of reflector-vector element e inside the V buffer (D values per element); the
// four segments of the long direction are shifted against each other so that the four
// parts of a line read different LDS banks
template <int B, int D> __device__ __forceinline__ int vidx(int e) { return e * D + (e / (B / 4)) * D; }

// The panels form sums of squares, so a line whose entries are all below 2 is moved up by a power of two
// first and its part of the triangular factor back (H depends on a line's direction only, and is
// linear in every line by itself).  A tail is given up (H = I) where its sum of squares is
// below `least`: 2^-47 (f32) or 2^-477 (f64) beside an entry of 2 or more, 2^-106 / 2^-980 of a line that was
// moved.  Without the move, bands of entries near 2^-65 (f32) or 2^-515 (f64) lost their tails
// altogether; with squares below the normal range used as they are, tiny lines beside large ones gave
// reflectors that were not orthogonal.  The other lines are moved down by 8: u^T u is up to four times the sum of
// squares, which may lie at the end of the range.  `least` also keeps the entries of T, up to 4 / least, finite.
template <typename C> struct LineRange;
template <> struct LineRange<float> { static constexpr float up = 0x1p56f, down = 0x1p-56f, least = 0x1p-100f, floor = 0x1p-126f; };
template <> struct LineRange<double> { static constexpr double up = 0x1p500, down = 0x1p-500, least = 0x1p-960, floor = 0x1p-1022; };
// the upper words of a line's entries, or-ed: bit 30 is set if and only if one of them is 2 or larger (or a NaN)
template <int N> __device__ __forceinline__ unsigned exponent_bits(const float (&x)[N])
{
    unsigned u = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) u |= __builtin_bit_cast(unsigned, x[i]);
    return u;
}
template <int N> __device__ __forceinline__ unsigned exponent_bits(const double (&x)[N])
{
    unsigned u = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) u |= (unsigned)(__builtin_bit_cast(unsigned long long, x[i]) >> 32);
    return u;
}

// m / d, and 1 / d, with the Newton step of the reciprocal beside the product where it is the last
__device__ __forceinline__ float panel_ratio(float m, float d, float& r)
{
    const float r0 = __builtin_amdgcn_rcpf(d), e = fmaf(-d, r0, 1.0f), w = m * r0;
    r = fmaf(r0, e, r0);
    return fmaf(w, e, w);
}
__device__ __forceinline__ double panel_ratio(double m, double d, double& r)
{
    double r0 = __builtin_amdgcn_rcp(d);
    r0 = fma(r0, fma(-d, r0, 1.0), r0);
    const double e = fma(-d, r0, 1.0), w = m * r0;
    r = fma(r0, e, r0);
    return fma(w, e, w);
}

// What is left to do once a panel's vectors are known: for T, this lane's line's products c with the vectors and
// the factors g; for the triangular factor, the line's entries f before its diagonal, and the sum of squares of its tail
// and the element before it as its own reflector found them.
template <typename C> struct PanelTail { C c[8], g[8], f[8], ss, alpha, down; };

// One reflector (number K) of the panel factorisation below.  This lane holds elements QN rw + i, i < QN, of line
// ln; row0: rw = 0, where the panel's first eight elements are, and first = ln there, -1 elsewhere.  (Conditions are
// compared by themselves and not combined: a scalar instruction on a comparison's result costs some 50 cycles.)
template <typename C, int QN, int K>
__device__ __forceinline__ void panel_reflector(C (&x)[QN], PanelTail<C>& tail, int ln, int first, bool row0)
{
    // products of the pivot line's tail with this line's (its elements before K are zero), and the line's element
    // K; summed over the four rows of lanes
    C a = row0 ? x[K] : (C)0;
    x[K] = row0 ? (C)0 : x[K];
    C p4[4], ss, alpha;
    row_lane_dot<K>(x, p4);
    C f = (p4[0] + p4[1]) + (p4[2] + p4[3]);
    const C xk = a;
    rows_sum2<K>(f, a, ss, alpha);
    const bool ident = ss < LineRange<C>::least;   // (H = I: a zero tail leaves every line as it is)
    // u = (alpha + sign(alpha) norm, tail), H = I - g u u^T, g = 2 / u^T u
    const C u0 = alpha + copysign(newton_sqrt(fma(alpha, alpha, ss) + LineRange<C>::floor), alpha);
    const C c = fma(u0, a, f);               // u^T line
    C m = ln > K ? (C)-2 * c : (C)0;
    asm("" : "+v"(m));
    m = ident ? (C)0 : m;
    C r;
    const C w = panel_ratio(m, fma(u0, u0, ss), r);   // m / (u^T u); r = 1 / (u^T u)
    // (element K: the pivot line's becomes u's, those of the lines behind it entries of the factor)
    x[K] = row0 ? xk : x[K];
    x[K] = first == K ? u0 : x[K];
    row_lane_axpy<K>(x, w);
    tail.c[K] = c;
    tail.g[K] = ident ? (C)0 : r + r;
    tail.f[K] = x[K];
    tail.ss = ln == K ? ss : tail.ss;
    tail.alpha = ln == K ? alpha : tail.alpha;
    x[K] = first > K ? (C)0 : x[K];
}

// Householder factorisation of a D x B panel held in LDS, by one wave: panel element (k, e),
// k < D along the short and e < B along the long direction, lives at P[k + e*LD] (RIGHT: a block's rows) or
// P[k*LD + e].  Reflector k is built from line k, elements k .. B-1, and applied to lines k+1 .. D-1.  On exit
// Vs holds the vectors u (Vs[k*LDV + e], zeros before element k); P is left as it was.  panel_rest forms, while
// the other waves are at V^T C, the D x D upper triangular T of H_0 H_1 .. H_{D-1} = I - V T V^T
// (row-major) and the panel's triangular factor, element (k, e), e <= k, in Fs[k*8 + e].  D = 8.
// The panels are the longest part of a step and one dependent chain; what they cost is instructions
// (4 to 5 cycles each from a lone wave) and latencies (8 cycles a dependent one, 70 a shuffle through LDS,
// 55 a branch on a vector comparison).  So: a row of sixteen lanes holds a quarter of the long direction of
// all eight lines (lanes 8 .. 15 a copy), the pivot line's elements being operands of the multiply-adds by
// row broadcast; two sums over the four rows share their swaps of lane groups; the vectors are not
// normalised; nothing branches.  Cycles a panel alone (f32 32, 64, 128; f64 32, 64): 2940, 3780, 5390; 3990,
// 4850; a lane with every eighth element of a line, the pivot line copied by two moves an element, normalised
// vectors and T on the chain took 1.65, 2.2, 2.5; 2.4, 3.2 us.
template <typename C, int B, int D, int LD, int LDV, bool RIGHT>
__device__ __forceinline__ void panel_wave(const C* P, C* Vs, PanelTail<C>& tail)
{
    static_assert(D == 8, "eight lines, one per lane of a group of eight");
    constexpr int QN = B / 4, NV = 16 / (int)sizeof(C);
    int lane = threadIdx.x & (kWave - 1);
    asm volatile("" : "+v"(lane));   // (addresses are formed here and not held by the caller's loop)
    const int ln = lane & 7, e0 = (lane >> 4) * QN;
    const bool row0 = lane < 16;
    int first = row0 ? ln : -1;
    asm volatile("" : "+v"(first));
    C x[QN];
    if constexpr (RIGHT) {
#pragma unroll
        for (int i = 0; i < QN; ++i) x[i] = P[ln + (e0 + i) * LD];
    } else {
#pragma unroll
        for (int i = 0; i < QN; i += NV) {
            C v[NV];
            VecIO<C, C>::ld(P + ln * LD + e0 + i, v);
#pragma unroll
            for (int j = 0; j < NV; ++j) x[i + j] = v[j];
        }
    }
    const bool large = rows_or(exponent_bits(x)) & 0x40000000u;
    const C up = large ? (C)0.125 : LineRange<C>::up;
    tail.down = large ? (C)8 : LineRange<C>::down;
    tail.ss = tail.alpha = 0;
#pragma unroll
    for (int i = 0; i < QN; ++i) x[i] *= up;
    static_steps([&](auto kc) {
        panel_reflector<C, QN, decltype(kc)::value>(x, tail, ln, first, row0);
    }, std::make_integer_sequence<int, 8>{});
    // each of two copies of a line stores half of it
    const bool second = lane & 8;
    C* const vs = Vs + ln * LDV + e0 + (second ? QN / 2 : 0);
#pragma unroll
    for (int i = 0; i < QN / 2; i += NV) {
        C v[NV];
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            C lo = x[i + j], hi = x[QN / 2 + i + j];
            asm("" : "+v"(lo), "+v"(hi));   // (two values: of two places the compiler would make an array in scratch memory)
            v[j] = second ? hi : lo;
        }
        VecIO<C, C>::st(vs + i, v);
    }
}
// T(0:K, K) = -g_K T(0:K, 0:K) (V^T u_K), T(K, K) = g_K; a lane builds the row of its line
template <typename C> __device__ __forceinline__ void panel_rest(const PanelTail<C>& tail, C* Ts, C* Fs)
{
    const int lane = threadIdx.x & (kWave - 1), ln = lane & 7;
    constexpr int NV = 16 / (int)sizeof(C);
    C t[8], acc[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) acc[k] = 0;
    static_steps([&](auto kc) {
        constexpr int K = decltype(kc)::value;
        t[K] = fma(-tail.g[K], acc[K], ln == K ? tail.g[K] : (C)0);   // (acc is zero in lines K and on)
        if constexpr (K < 7) row_lane_columns<K>(acc, tail.c, t[K]);
    }, std::make_integer_sequence<int, 8>{});
    // (times 16 under the root: where u^T u, up to four times this, may be beyond the quarter of the range that the
    // reciprocal instruction does not answer with zero, the factor becomes a NaN.  Lines of entries whose squares do not sum
    // up inside the type's range get there; with a zero the reflector was left out and finite, wrong values came out.)
    const C x2 = (fma(tail.alpha, tail.alpha, tail.ss) + LineRange<C>::floor) * 16;
    const C beta = tail.ss < LineRange<C>::least ? tail.alpha : -copysign((C)0.25 * newton_sqrt(x2), tail.alpha);
    if (lane < 8) {
#pragma unroll
        for (int k = 0; k < 8; k += NV) {
            C v[NV], w[NV];
#pragma unroll
            for (int j = 0; j < NV; ++j) {
                v[j] = t[k + j];
                w[j] = tail.f[k + j] * tail.down;
            }
            VecIO<C, C>::st(Ts + ln * 8 + k, v);
            VecIO<C, C>::st(Fs + ln * 8 + k, w);
        }
        Fs[ln * 9] = beta * tail.down;
    }
}

// The same factorisation with a lane per element (every 64th of all eight lines): eight sums over the
// wave per reflector.  Kept for the in-band form of the kernel (two blocks do not fit in LDS: f64 at
// B = 128), which has 128 registers a lane: an earlier form of the factorisation above did not fit beside the lines that the
// apply waves then held (16.9 against 15.4 us a column for the whole reduction, before the tiles of apply_tile_g; it is at
// 10.5 now and the present form has not been tried in it).  It does not move tiny lines either (every form of it that
// did spilled more: 15.7 to 17.0 then): its reflectors are orthogonal to 2^-1075 / ss, so lines of entries below
// about 2^-515 (f64) are reduced to the accuracy of their own squares, and so is what they are applied to.
// Sums of eight per-lane values over the 64 lanes of a wave, as wave-uniform scalars.
// The first three stages halve the number of values while doubling the lanes summed
// (each lane keeps the half selected by one of its index bits and hands the other half to
// its partner: partners i^7 with bit 2, i^1 with bit 0, i^2 with bit 1), so that after them
// lane i holds, summed over its group of eight lanes, the value with index
// 4*bit1(i) + 2*bit0(i) + bit2(i); two more stages sum over the row of 16 and over the four rows.
template <typename C> __device__ __forceinline__ void wave_sum8(const C (&a)[8], C (&out)[8])
{
    const int lane = threadIdx.x & (kWave - 1);
    const bool b0 = lane & 1, b1 = lane & 2, b2 = lane & 4;
    C b[4], c[2];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const C keep = b2 ? a[2 * j + 1] : a[2 * j], send = b2 ? a[2 * j] : a[2 * j + 1];
        b[j] = keep + dpp_get<kDppHalfMirror>(send);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const C keep = b0 ? b[2 * j + 1] : b[2 * j], send = b0 ? b[2 * j] : b[2 * j + 1];
        c[j] = keep + dpp_get<kDppXor1>(send);
    }
    const C keep = b1 ? c[1] : c[0], send = b1 ? c[0] : c[1];
    C v = keep + dpp_get<kDppXor2>(send);
    v += dpp_get<kDppRor8>(v);
    v += __shfl_xor(v, 16, kWave);
    v += __shfl_xor(v, 32, kWave);
#pragma unroll
    for (int i = 0; i < 8; ++i) out[i] = lane_value(v, ((i >> 1) & 1) + 2 * ((i >> 2) & 1) + 4 * (i & 1));
}

template <typename C, int B, int D, bool G>
__device__ __forceinline__ void panel_wave_spread(C* P, int64_t sk, int64_t se, C* Vs, C* Ts, int ne)
{
    constexpr int QN = (B + kWave - 1) / kWave;
    const int lane = threadIdx.x & (kWave - 1);
    C x[D][QN];
#pragma unroll
    for (int k = 0; k < D; ++k)
#pragma unroll
        for (int q = 0; q < QN; ++q) {
            const int e = lane + kWave * q;
            if (G) x[k][q] = (e < ne) ? rgld(P + k * sk + e * se) : (C)0;
            else x[k][q] = (e < B) ? P[k * sk + e * se] : (C)0;
        }
    const int tj = lane & (D - 1);   // this lane builds row tj of T as the reflectors appear
    C trow[D];
#pragma unroll
    for (int k = 0; k < D; ++k) {
        C part[D], p[D], colk[D];
#pragma unroll
        for (int j = 0; j < D; ++j) {
            C acc = 0;
#pragma unroll
            for (int q = 0; q < QN; ++q) {
                const int e = lane + kWave * q;
                acc += (e > k) ? x[j][q] * x[k][q] : (C)0;
            }
            part[j] = acc;
            colk[j] = lane_value(x[j][0], k);   // element k of every line
        }
        wave_sum8(part, p);
        const C alpha = colk[k], ss = p[k];
        C beta, inv, tau;
        if (ss == (C)0) {
            beta = alpha; tau = 0; inv = 0;
        } else {
            // (alpha and ss are the same in every lane: a uniform branch.  The refined hardware
            // square root wants a normal argument; sums near the underflow threshold take the
            // library routine.)
            const C x2 = alpha * alpha + ss;
            const C nrm = x2 < (sizeof(C) == 8 ? (C)1e-290 : (C)1e-30f) ? sqrt(x2) : newton_sqrt(x2);
            beta = alpha >= (C)0 ? -nrm : nrm;
            tau = (beta - alpha) * rrcp(beta);
            inv = rrcp(alpha - beta);
        }
        // T(0:k,k) = -tau_k T(0:k,0:k) (V^T v_k), T(k,k) = tau_k; v_j^T v_k = v_j(k) + inv * p_j for j < k
        {
            C acc = 0;
#pragma unroll
            for (int i = 0; i < k; ++i) acc += trow[i] * (colk[i] + inv * p[i]);
            trow[k] = (k == tj) ? tau : (k > tj ? -tau * acc : (C)0);
        }
#pragma unroll
        for (int j = k + 1; j < D; ++j) {
            const C sj = tau * (colk[j] + inv * p[j]);
#pragma unroll
            for (int q = 0; q < QN; ++q) {
                const int e = lane + kWave * q;
                const C vk = (e == k) ? (C)1 : (e > k ? x[k][q] * inv : (C)0);
                x[j][q] -= sj * vk;
            }
        }
#pragma unroll
        for (int q = 0; q < QN; ++q) {
            const int e = lane + kWave * q;
            if (e > k) x[k][q] *= inv;
            else if (e == k) x[k][q] = beta;
        }
    }
    // factor back into the panel, vectors to Vs
#pragma unroll
    for (int q = 0; q < QN; ++q) {
        const int e = lane + kWave * q;
        if (e < B) {
#pragma unroll
            for (int k = 0; k < D; ++k) {
                if (G) {
                    if (e < ne) rgst(P + k * sk + e * se, (e <= k) ? x[k][q] : (C)0);
                } else {
                    P[k * sk + e * se] = (e <= k) ? x[k][q] : (C)0;
                }
                Vs[vidx<B, D>(e) + k] = (e < k) ? (C)0 : (e == k ? (C)1 : x[k][q]);
            }
        }
    }
    if (lane < D) {
#pragma unroll
        for (int k = 0; k < D; ++k) Ts[tj * D + k] = trow[k];
    }
}

// The block reflector (Vs, Ts) applied to SIXTEEN lines at once on MFMA, by one wave: element e
// of line n of the tile lives at base[e*es + n*ls] (LDS), e < B, lines n >= nvalid are left
// alone.  With Y(e, n) the tile's elements:
//     P = V^T Y  (16 x 16, rows 8.. zero),  Z = -T^T P,  Y += V Z
// (line <- line - ((line . V) T) V^T for every line).  The
// first product contracts over e with Y as the B operand straight from LDS; the second and
// third use the accumulator registers of the previous one as their B operand (Frag).
template <typename C, int B, int D>
__device__ __forceinline__ void apply_tile(C* base, int es, int ls, int nvalid, const C* Vs, const C* Ts)
{
    using F = Frag<C>;
    typedef typename F::acc_t acc_t;
    const int lane = threadIdx.x & 63, i = lane & 15, gq = lane >> 4;
    const bool valid = i < nvalid;
    C* mine = base + i * ls;   // this lane's line (B / accumulator operands)
    acc_t p0, p1;
#pragma unroll
    for (int r = 0; r < 4; ++r) { p0[r] = 0; p1[r] = 0; }
#pragma unroll 8
    for (int s4 = 0; s4 < B / 4; ++s4) {
        const int k = 4 * s4 + gq;
        const C a = (i < D) ? Vs[vidx<B, D>(k) + i] : (C)0;   // A[m = i][k] = V(k, i)
        const C b = valid ? mine[k * es] : (C)0;              // B[k][n = i] = Y(k, i)
        if (s4 & 1) p1 = F::mma(a, b, p1);
        else p0 = F::mma(a, b, p0);
    }
    acc_t z;
#pragma unroll
    for (int r = 0; r < 4; ++r) { p0[r] += p1[r]; z[r] = 0; }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int kk = F::roff(r, gq);
        const C a = (i < D && kk < D) ? Ts[kk * D + i] : (C)0;   // A[m = i][kk] = T(kk, i)
        z = F::mma(a, p0[r], z);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) z[r] = -z[r];
#pragma unroll 2
    for (int e0 = 0; e0 < B; e0 += 16) {
        acc_t y;
#pragma unroll
        for (int r = 0; r < 4; ++r) y[r] = valid ? mine[(e0 + F::roff(r, gq)) * es] : (C)0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int j = F::roff(r, gq);
            if (F::roff(r, 0) < D) {   // some lane group still has a reflector index below D in this slot
                const C a = (j < D) ? Vs[vidx<B, D>(e0 + i) + j] : (C)0;   // A[m = i][j] = V(e0 + i, j)
                y = F::mma(a, z[r], y);
            }
        }
        if (valid) {
#pragma unroll
            for (int r = 0; r < 4; ++r) mine[(e0 + F::roff(r, gq)) * es] = y[r];
        }
    }
}

// The same for sixteen lines of the packed band in device memory (device-scope accesses), held in registers
// between the two products: element e of line n at p + n*ls + e*es, e < ne, lines n < nvalid.  All loads go out
// together, without a predicate where the tile is whole.  What bounds it are the pieces of 128 (rows) and 32 bytes
// (columns) the lanes of an access fall into.  Eight lanes per line, two rounds of eight lines, V re-read from LDS for
// every line, took 35 us for the rows of a step of the in-band kernel (f64, B = 128), 10 so; the columns are at 14 in
// both.  The reduction at n = 8192: 124 -> 86 ms.
// Two partial sums in the first product: against one 101.6 -> 99.9 ms (both phases, n = 8192) and 2 % less error; four
// 102.3 ms.
template <typename C, int B, int D>
__device__ __forceinline__ void apply_tile_g(C* p, int64_t es, int64_t ls, int nvalid, int ne, const C* Vs, const C* Ts)
{
    using F = Frag<C>;
    typedef typename F::acc_t acc_t;
    constexpr int NTL = B / 16, NP = 2;   // partial sums of the first product
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));
    const int i = lane & 15, gq = lane >> 4, j = i & 7;
    const bool valid = i < nvalid, full = nvalid >= 16 && ne >= B;
    const int64_t off = i * ls + F::roff(0, gq) * es;
    const int64_t e1 = F::roff(1, 0) * es, e2 = 16 * es - 3 * e1;   // to the next register / tile
    ne = valid ? ne - F::roff(0, gq) : 0;
    acc_t y[NTL];
    if (full) {
        const C* q = p;
#pragma unroll
        for (int a = 0; a < NTL; ++a)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                y[a][r] = rgld(q + off);
                q += r < 3 ? e1 : e2;
            }
    } else {
        const C* q = p;
#pragma unroll
        for (int a = 0; a < NTL; ++a)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                C v = 0;
                if (16 * a + F::roff(r, 0) < ne) v = rgld(q + off);
                y[a][r] = v;
                q += r < 3 ? e1 : e2;
            }
    }
    acc_t w, z, part[NP];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        z[r] = 0;
#pragma unroll
        for (int q = 0; q < NP; ++q) part[q][r] = 0;
    }
#pragma unroll
    for (int a = 0; a < NTL; ++a)
#pragma unroll
        for (int r = 0; r < 4; ++r) part[r % NP] = F::mma(Vs[vidx<B, D>(16 * a + F::roff(r, gq)) + j], y[a][r], part[r % NP]);
#pragma unroll
    for (int r = 0; r < 4; ++r) w[r] = part[0][r] + part[1][r];
#pragma unroll
    for (int r = 0; r < 2; ++r) z = F::mma(-Ts[F::roff(r, gq) * D + j], w[r], z);
#pragma unroll
    for (int a = 0; a < NTL; ++a)
#pragma unroll
        for (int r = 0; r < 2; ++r) y[a] = F::mma(Vs[vidx<B, D>(16 * a + i) + F::roff(r, gq)], z[r], y[a]);
    if (full) {
#pragma unroll
        for (int a = 0; a < NTL; ++a)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                rgst(p + off, y[a][r]);
                p += r < 3 ? e1 : e2;
            }
    } else {
#pragma unroll
        for (int a = 0; a < NTL; ++a)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if (16 * a + F::roff(r, 0) < ne) rgst(p + off, y[a][r]);
                p += r < 3 ? e1 : e2;
            }
    }
}

// ---- block reflectors on MFMA.  A wave takes sixteen lines (rows under a right transformation, columns
// under a left one) at a time, all B elements of a line in registers: accumulator tile a, register r
// of lane (gq, i) is element 16 a + roff(r, gq) of line i.  With Y(e, n) the elements of line n
//     P = V^T Y,  Z = -T^T P,  Y += V Z
// (line <- line - ((line . V) T) V^T).  Every product contracts over an index that runs through the
// accumulator registers of its right operand, so nothing moves between them (Frag); the eight
// reflectors are spread over the sixteen rows of P and Z so that they fill registers 0 and 1 of every
// lane, and the last two products take two instructions a tile.
// What bounds this is the issue of the matrix instructions: B / 4 + 2 + B / 8 a tile, of which half the
// first product's work is on empty rows; between two panels stand B / 4 + 4 of them.  The form before it (a quad of
// lanes per line, V re-read from LDS for every line) was bound by LDS: 2.05 us a block pair at nb = 64 in
// f32, 7.3 at nb = 128, all of it between the panels.
template <typename C> struct Refl;   // row of P / Z <-> reflector
template <> struct Refl<float> {
    static __device__ __forceinline__ int of_slot(int r, int gq) { return 2 * gq + r; }
    static __device__ __forceinline__ int of_row(int i) { return 2 * (i >> 2) + (i & 1); }   // (rows with bit 1 set: a copy nobody reads)
};
template <> struct Refl<double> {
    static __device__ __forceinline__ int of_slot(int r, int gq) { return 4 * r + gq; }
    static __device__ __forceinline__ int of_row(int i) { return i & 7; }
};

// Where a lane finds its operands of a block reflector: V (line k of V, LDV apart, is vector k) and T (row-major,
// 8 x 8).
template <typename C, int B, int LDV> struct BlockRefl {
    static constexpr int NTL = B / 16;
    typedef typename Frag<C>::acc_t acc_t;
    int o1, t0, t1, v0, v1;   // offsets of its elements of V^T (first product), of T, of V (last product)
    __device__ __forceinline__ void init(int i, int gq)
    {
        const int j = Refl<C>::of_row(i), s0 = Refl<C>::of_slot(0, gq), s1 = Refl<C>::of_slot(1, gq);
        o1 = j * LDV + Frag<C>::roff(0, gq);
        t0 = s0 * 8 + j;
        t1 = s1 * 8 + j;
        v0 = s0 * LDV + i;
        v1 = s1 * LDV + i;
        asm volatile("" : "+v"(o1), "+v"(t0), "+v"(t1), "+v"(v0), "+v"(v1));
    }
    // p = V^T y.  In f32 four partial sums: with one, the error of the whole reduction was larger by 3, 7 and 7 % (nb =
    // 32, 64, 128; n = 600, mean of 48 bands), for the same time; in f64 they cost 0.4 (two) to 4 % for an error within
    // the means' spread of 3 %.
    __device__ __forceinline__ acc_t inner(const C* V, const acc_t (&y)[NTL]) const
    {
        constexpr int NP = sizeof(C) == 4 ? 4 : 1;
        acc_t p[NP];
#pragma unroll
        for (int q = 0; q < NP; ++q)
#pragma unroll
            for (int r = 0; r < 4; ++r) p[q][r] = 0;
#pragma unroll
        for (int a = 0; a < NTL; ++a) {
            C v[4];
            Frag<C>::ld4(V + o1 + 16 * a, 0, v);
#pragma unroll
            for (int r = 0; r < 4; ++r) p[r % NP] = Frag<C>::mma(v[r], y[a][r], p[r % NP]);
        }
#pragma unroll
        for (int w = NP; w > 1; w /= 2)
#pragma unroll
            for (int q = 0; q < w / 2; ++q)
#pragma unroll
                for (int r = 0; r < 4; ++r) p[q][r] += p[q + w / 2][r];
        return p[0];
    }
    // z = -T^T p in registers 0 and 1; lines that are not `on` get zero
    __device__ __forceinline__ acc_t middle(const C* T, const acc_t& p, bool on) const
    {
        acc_t z;
#pragma unroll
        for (int r = 0; r < 4; ++r) z[r] = 0;
        z = Frag<C>::mma(-T[t0], on ? p[0] : (C)0, z);
        return Frag<C>::mma(-T[t1], on ? p[1] : (C)0, z);
    }
    // y_a += V_a z, a = A0 .. A1-1
    template <int A0, int A1> __device__ __forceinline__ void outer(const C* V, acc_t (&y)[NTL], const acc_t& z) const
    {
#pragma unroll
        for (int a = A0; a < A1; ++a) y[a] = Frag<C>::mma(V[v0 + 16 * a], z[0], y[a]);
#pragma unroll
        for (int a = A0; a < A1; ++a) y[a] = Frag<C>::mma(V[v1 + 16 * a], z[1], y[a]);
    }
};

// Shape of the band reduction kernel.  Apply waves, and one more for the panels.  A wave has a `look` tile
// (sixteen rows of Z / columns of A3, of which the next panel waits for a corner) or a `rest` tile
// (rows of U / columns of Z, wanted a phase later), or one of each (B = 128).
template <typename C, int B> struct ReduceShape {
    static constexpr int NTL = B / 16;
    static constexpr int NA = B == 128 ? NTL : 2 * NTL;
    static constexpr bool BOTH = NA == NTL;
    static constexpr int NT = (NA + 1) * kWave;
    // rows of consecutive columns of S and consecutive lines of V are LD and LDV apart: both directions of a
    // tile, and its operands, then fall on different LDS banks
    static constexpr int LD = (BOTH ? 2 : 3) * B + (sizeof(C) == 4 ? 4 : 18);
    static constexpr int LDV = B + (sizeof(C) == 4 ? 8 : 12);
    static constexpr int oV = B * LD, oT = oV + 2 * 8 * LDV, oF = oT + 2 * 64, kElems = oF + 64;   // LDS carve: S, two V, two T, F
    static constexpr size_t kSmemBytes = sizeof(C) * (size_t)kElems;
    // a wave moves sixteen block columns: 64 rows (or 64 / B columns of B rows) at a time
    static constexpr int RG = B >= kWave ? B / kWave : 1;      // row groups of a column
    static constexpr int CG = B >= kWave ? 1 : kWave / B;      // columns per access
    static constexpr int PER = RG * 16 / CG;                   // accesses
};

// WIDE: lane offsets into a block of up to 15 columns do not fit 32 bits.
template <typename C, int B, bool WIDE>
__global__ __launch_bounds__((ReduceShape<C, B>::NT)) void band_reduce_kernel(C* __restrict__ band, int64_t ldab, int64_t n,
                                                                             int* __restrict__ ctrl,
                                                                             int* __restrict__ progress, int spin_limit)
{
    // A step has four phases with a barrier behind each:
    //   P1  panel wave: right panel                | rest of the left reflectors of the step before (A3 below its
    //                                              | first sixteen rows; Z, which then goes back), this step's Z in
    //   P2  (first sixteen columns of Z transformed; the rows of U fetched from LDS)
    //   P3  panel wave: left panel                 | rest of the right reflectors (Z; U, which goes back from the
    //                                              | registers), the block right of Z (A3) in, over U
    //   P4  (first sixteen rows of A3 transformed; the columns of Z fetched from LDS)
    // so that of the two block reflectors only what the next panel needs (P2, P4) stands on the chain.
    using SH = ReduceShape<C, B>;
    using F = Frag<C>;
    typedef typename F::acc_t acc_t;
    constexpr int D = 8, LD = SH::LD, LDV = SH::LDV, NTL = SH::NTL, NA = SH::NA, PER = SH::PER, RG = SH::RG, CG = SH::CG;
    constexpr bool BOTH = SH::BOTH;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    // S[row + col * LD]: U / A3 in rows 0 .. B-1, Z behind them, where LDS has room in two places in turn, so that
    // the next Z need not wait until the last one is out
    C* S = reinterpret_cast<C*>(smem_raw);
    C* const Vr = S + SH::oV;                     // reflectors of the right panel, of the left one
    C* const Vl = Vr + 8 * LDV;
    C* const Tr = S + SH::oT;
    C* const Tl = Tr + 64;
    C* const Fs = S + SH::oF;                     // triangular factor of a panel
    __shared__ int sh_s;
    __shared__ volatile int sh_fail, sh_seen;     // sh_seen: progress of the predecessor as last polled
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool pw = wv == NA;
    const bool lead = tid == NA * kWave;
    const bool look = !pw && wv < NTL, rest = !pw && (BOTH || wv >= NTL);
    const int tile = BOTH ? wv : wv % NTL;
    // The rest tiles begin behind the panel's eight lines, which the last tile takes along unchanged.  A wave
    // moves the columns of its tile in two runs of eight (which do not wrap).
    const int lk0 = 16 * tile, lk1 = lk0 + 8, rk0 = 16 * tile + D, rk1 = (rk0 + 8) & (B - 1);
    struct Me {
        int i, gq;         // fragment coordinates
        int mrow, mcol;    // moving blocks: row and first column
        int lline, rline;  // lines of the two tiles
        bool ron;          // whether the reflectors apply to rline
        int lrow, rrow, lcol, rcol;   // offsets of the tiles' first elements as rows, as columns
    };
    Me me;
    BlockRefl<C, B, LDV> refl;
    auto place = [&](int l) {
        me.i = l & 15;
        me.gq = l >> 4;
        me.mrow = B >= kWave ? l : l % B;
        me.mcol = B >= kWave ? 0 : l / B;
        me.lline = 16 * tile + me.i;
        me.rline = (D + 16 * tile + me.i) & (B - 1);
        me.ron = me.rline >= D;
        me.lrow = me.lline + F::roff(0, me.gq) * LD;
        me.rrow = me.rline + F::roff(0, me.gq) * LD;
        me.lcol = me.lline * LD + F::roff(0, me.gq);
        me.rcol = me.rline * LD + F::roff(0, me.gq);
        asm volatile("" : "+v"(me.lrow), "+v"(me.rrow), "+v"(me.lcol), "+v"(me.rcol));
        refl.init(me.i, me.gq);
    };
    place(lane);
    using Ld = std::conditional_t<WIDE, int64_t, int>;
    using Off = std::conditional_t<WIDE, int64_t, unsigned>;
    const Ld ldm1 = (Ld)(ldab - 1);
    const int64_t ku = 2 * (int64_t)B - 1;
    const int64_t nsweeps = (n - 1) / D;
#ifdef SVB_CHASE_TIMING
    unsigned long long tacc[8] = {0, 0, 0, 0, 0, 0, 0, 0}, tlast = 0, nstep_acc = 0;
#define RMARK(slot_) do { if (lead) { unsigned long long now_ = wall_clock64(); tacc[slot_] += now_ - tlast; tlast = now_; } } while (0)
#else
#define RMARK(slot_) do { } while (0)
#endif

    // Progress of a sweep: 2k+1 once the upper block U of its step k and the corner that the step's left panel
    // leaves in Z are final in the band, 2k+2 once all of Z is and the corner that the next step's right panel
    // leaves in that step's U.  The corners (D x D) go to the band by themselves, ahead of their blocks: a
    // successor's Z needs no more of this sweep's step t+1 than U and the corner of Z, its A3 no more than Z
    // and the corner of the U after it.  (The block stores that repeat them are acknowledged before the progress
    // that lets the successor write there.)
    // Waits (one lane) until sweep s-1 has reached `need`.  One wave at a time polls (`polls`), the others watch
    // what it saw; an expired wait sets sh_fail.  A poll takes about a microsecond there and back, so the first is
    // asked for a phase ahead (`early`).
    auto poll = [&](int64_t s) -> int {
        return s > 0 ? __hip_atomic_load(&progress[(s - 1) * kProgressStride], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
    };
    auto wait_for = [&](int64_t s, int need, bool polls, int early) {
        if (lane == 0 && s > 0) {
            int spins = 0;
            if (polls) {
                int seen = early;
                while (seen < need) {
                    seen = poll(s);
                    if (seen >= need) break;
                    if (++spins > spin_limit) {
                        atomicExch(&ctrl[1], 1);
                        sh_fail = 1;
                        break;
                    }
                    __builtin_amdgcn_s_sleep(1);
                }
                sh_seen = seen;
            } else {
                while (sh_seen < need && !sh_fail) __builtin_amdgcn_s_sleep(1);
            }
        }
        asm volatile("" ::: "memory");   // (the loads that follow stay behind it)
    };
    auto publish = [&](int64_t s, int value) {
        if (lane == 0) __hip_atomic_store(&progress[s * kProgressStride], value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    // Moving the sixteen columns of a block that belong to this wave: two runs of eight, the first from
    // column k0, the second from k1; this lane moves row mrow (and those 64 below) of every CG-th column.
    // (Scalar column addresses and a 32-bit lane offset.)
    auto entry = [&](int64_t r0, int64_t cb, int col) -> char* {
        return reinterpret_cast<char*>(band + ((r0 - cb + ku) + cb * ldab) + (int64_t)col * ldm1);
    };
    auto at = [](char* p, Off off) -> C* { return reinterpret_cast<C*>(p + off); };
    // (entries outside the matrix, or above row `from`, are not touched and read as zero)
    auto load_cols = [&](C (&pre)[PER], int64_t r0, int64_t cb, int k0, int k1, int from) {
        const bool full = r0 + B <= n && cb + B <= n && from == 0;
        const int nrow = (int)min((int64_t)B, n - r0), ncol = (int)max((int64_t)0, min((int64_t)B, n - cb));
        const Off off = (Off)(me.mrow + me.mcol * ldm1) * (Off)sizeof(C);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int kc = h ? k1 : k0;
            char* p = entry(r0, cb, kc);
            if (full) {
#pragma unroll
                for (int q = 0; q < PER / 2; ++q) {
                    pre[h * (PER / 2) + q] = rgld(at(p, off) + (q % RG) * kWave);
                    if (q % RG == RG - 1) p += CG * ldm1 * (int64_t)sizeof(C);
                }
            } else {
#pragma unroll
                for (int q = 0; q < PER / 2; ++q) {
                    const int row = me.mrow + (q % RG) * kWave, col = kc + (q / RG) * CG + me.mcol;
                    C v = 0;
                    if (row < nrow && row >= from && col < ncol) v = rgld(at(p, off) + (q % RG) * kWave);
                    pre[h * (PER / 2) + q] = v;
                    if (q % RG == RG - 1) p += CG * ldm1 * (int64_t)sizeof(C);
                }
            }
        }
    };
    auto put_cols = [&](C* dst, const C (&pre)[PER], int k0, int k1) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            int o = me.mrow + ((h ? k1 : k0) + me.mcol) * LD;
            asm volatile("" : "+v"(o));
#pragma unroll
            for (int q = 0; q < PER / 2; ++q) dst[o + (q % RG) * kWave + (q / RG) * CG * LD] = pre[h * (PER / 2) + q];
        }
    };
    auto store_cols = [&](const C* src, int64_t r0, int64_t cb, int k0, int k1) {
        const bool full = r0 + B <= n && cb + B <= n;
        const int nrow = (int)min((int64_t)B, n - r0), ncol = (int)min((int64_t)B, n - cb);
        const Off off = (Off)(me.mrow + me.mcol * ldm1) * (Off)sizeof(C);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int kc = h ? k1 : k0;
            int o = me.mrow + (kc + me.mcol) * LD;
            asm volatile("" : "+v"(o));
            C v[PER / 2];
#pragma unroll
            for (int q = 0; q < PER / 2; ++q) v[q] = src[o + (q % RG) * kWave + (q / RG) * CG * LD];
            char* p = entry(r0, cb, kc);
            if (full) {
#pragma unroll
                for (int q = 0; q < PER / 2; ++q) {
                    rgst(at(p, off) + (q % RG) * kWave, v[q]);
                    if (q % RG == RG - 1) p += CG * ldm1 * (int64_t)sizeof(C);
                }
            } else {
#pragma unroll
                for (int q = 0; q < PER / 2; ++q) {
                    const int row = me.mrow + (q % RG) * kWave, col = kc + (q / RG) * CG + me.mcol;
                    if (row < nrow && col < ncol) rgst(at(p, off) + (q % RG) * kWave, v[q]);
                    if (q % RG == RG - 1) p += CG * ldm1 * (int64_t)sizeof(C);
                }
            }
        }
    };
    // tiles between LDS and registers: rows of a block (element e of line l at p[l + e * LD]) and columns
    // (p[e + l * LD])
    auto get_rows = [&](acc_t (&y)[NTL], const C* p, int o) {
#pragma unroll
        for (int a = 0; a < NTL; ++a)
#pragma unroll
            for (int r = 0; r < 4; ++r) y[a][r] = p[o + (16 * a + F::roff(r, 0)) * LD];
    };
    auto put_row_tile = [&](const acc_t& y, int a, C* p, int o) {
#pragma unroll
        for (int r = 0; r < 4; ++r) p[o + (16 * a + F::roff(r, 0)) * LD] = y[r];
    };
    auto get_cols = [&](acc_t (&y)[NTL], const C* p, int o) {
#pragma unroll
        for (int a = 0; a < NTL; ++a) {
            C v[4];
            F::ld4(p + o + 16 * a, 0, v);
#pragma unroll
            for (int r = 0; r < 4; ++r) y[a][r] = v[r];
        }
    };
    // the panel's own lines in a rest tile (line j of the panel in this lane if 0 <= j < 8): the triangular factor,
    // zero beyond
    auto put_factor = [&](acc_t (&y)[NTL], int j) {
        C f[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) f[r] = Fs[(j & 7) * 8 + (F::roff(r, me.gq) & 7)];
        const bool own = j >= 0 && j < D;
#pragma unroll
        for (int a = 0; a < NTL; ++a)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const C v = a == 0 && F::roff(r, me.gq) <= j ? f[r] : (C)0;
                y[a][r] = own ? v : y[a][r];
            }
    };
    auto put_col_tile = [&](const acc_t& y, int a, C* p, int o) {
        const C v[4] = {y[0], y[1], y[2], y[3]};
        F::st4(p + o + 16 * a, 0, v);
    };

    // Every single-lane section is followed by a barrier before the next one (no divergent
    // region spans a loop back-edge).
    for (;;) {
        if (lead) {
            sh_s = atomicAdd(&ctrl[0], 1);
            sh_fail = __hip_atomic_load(&ctrl[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            sh_seen = 0;
        }
        __syncthreads();
        const int64_t s = __builtin_amdgcn_readfirstlane(sh_s);
        __syncthreads();
        if (s >= nsweeps) break;
        const int64_t c00 = (s + 1) * D;
        const int nsteps = (int)((n - 1 - c00) / B) + 1;
        // ---- prologue: the sweep's own D rows (rows of the predecessor's first Z, and the corner of its next
        // step's U); the first Z follows in P1 like every other
        if (wv == 0) wait_for(s, 2, true, 0);
        __syncthreads();
        const bool failed = sh_fail != 0;
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        if (!failed && look) {
            C pre[PER];
            load_cols(pre, c00 - B, c00, lk0, lk1, B - D);
            put_cols(S, pre, lk0, lk1);
        }
        __syncthreads();
        // The panel wave and the apply waves run loops of their own (same barriers): nothing one of them keeps
        // takes registers of the other.
        auto z_at = [&](int t) -> C* { return S + (BOTH || !(t & 1) ? B : 2 * B); };
        auto panels = [&] {
#ifdef SVB_CHASE_TIMING
            if (lead) { tlast = wall_clock64(); nstep_acc += nsteps; }
#endif
            __builtin_amdgcn_s_setprio(3);
            for (int t = 0; t < nsteps; ++t) {
                PanelTail<C> tail;
                panel_wave<C, B, D, LD, LDV, true>(S + (t == 0 ? B - D : 0), Vr, tail);
                RMARK(0);
                lds_barrier();   // end of P1
                RMARK(1);
                if (sh_fail) break;
                panel_rest<C>(tail, Tr, Fs);
                lds_barrier();
                lds_barrier();   // end of P2
                RMARK(2);
                panel_wave<C, B, D, LD, LDV, false>(z_at(t), Vl, tail);
                RMARK(3);
                lds_barrier();   // end of P3
                RMARK(4);
                panel_rest<C>(tail, Tl, Fs);
                lds_barrier();
                lds_barrier();   // end of P4
                RMARK(5);
            }
            __builtin_amdgcn_s_setprio(0);
        };
        auto apply = [&](auto role) {
            constexpr bool look = decltype(role)::value != 1, rest = decltype(role)::value != 0;
            const bool corner = rest && tile == NTL - 1;   // the wave whose tile takes the panel's lines along
            // Places are formed here, once a sweep, and not held across the ticket loop for both roles: held, 27 to 35
            // registers were spilled at nb = 64 (reloaded at each sweep's start; f32, n = 8192: 14.2 -> 12.8 ms inside
            // svb_svdvals, 13.8 -> 12.8 by itself).  (One role at nb = 128: nothing to separate, and it would spill two.)
            if constexpr (!BOTH) {
                int l = lane;
                asm volatile("" : "+v"(l));
                place(l);
            }
            if (look) __builtin_amdgcn_s_setprio(2);
            int early_z = 0, early_a = 0;
            acc_t cl[NTL], cr[NTL], clz, crz;   // tiles of the left reflectors, P4 to the next step's P1
            for (int t = 0;; ++t) {
                const int64_t c0 = c00 + (int64_t)t * B;
                C* const Z = z_at(t);
                // ---- P1
                if (look) {
                    if (t > 0) {
                        refl.template outer<1, NTL>(Vl, cl, clz);
#pragma unroll
                        for (int a = 1; a < NTL; ++a) put_col_tile(cl[a], a, S, me.lcol);
                    }
                    if (!rest && t < nsteps) {
                        // this step's Z shares a corner with the predecessor's Z of step t+1
                        C pre[PER];
                        wait_for(s, 2 * t + 3, tile == 0, early_z);
                        load_cols(pre, c0, c0, lk0, lk1, 0);
                        put_cols(Z, pre, lk0, lk1);
                    }
                }
                if (rest) {
                    C* const Zp = z_at(t - 1);
                    if (t > 0) {
                        crz = refl.inner(Vl, cr);
                        crz = refl.middle(Tl, crz, me.ron);
                        refl.template outer<0, NTL>(Vl, cr, crz);
#pragma unroll
                        for (int a = 0; a < NTL; ++a) put_col_tile(cr[a], a, Zp, me.rcol);
                        if (corner && t < nsteps) {
                            stores_done();
                            publish(s, 2 * t - 1);
                        }
                    }
                    if (look && t < nsteps) {
                        C pre[PER];
                        wait_for(s, 2 * t + 3, tile == 0, early_z);
                        load_cols(pre, c0, c0, rk0, rk1, 0);
                        if (t > 0) store_cols(Zp, c0 - B, c0 - B, rk0, rk1);
                        put_cols(Z, pre, rk0, rk1);
                    } else if (t > 0) {
                        store_cols(Zp, c0 - B, c0 - B, rk0, rk1);
                    }
                    stores_done();   // every block of step t-1 is in the band before the barrier
                }
                if (t == nsteps) break;
                lds_barrier();
                if (sh_fail) break;
                // ---- P2
                acc_t rl[NTL], rr[NTL], rlz, rrz;   // tiles of the right reflectors, P2 to P3
                if (look && tile == 0) early_a = poll(s);
                if (look) {
                    get_rows(rl, Z, me.lrow);
                    rlz = refl.inner(Vr, rl);
                }
                if (rest) get_rows(rr, S, me.rrow);
                lds_barrier();
                if (look) {
                    rlz = refl.middle(Tr, rlz, true);
                    refl.template outer<0, 1>(Vr, rl, rlz);
                    put_row_tile(rl[0], 0, Z, me.lrow);
                }
                if (corner) {
                    // (the panel's lines are rows 0 .. 7, in the first step the last eight)
                    const int j = t == 0 ? me.rline - (B - D) : me.rline;
                    put_factor(rr, j);
                    char* p = entry(c0 - B, c0, 0);
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int col = F::roff(r, me.gq);
                        if (j >= 0 && j < D && col < D && c0 + col < n)
                            rgst(at(p, (Off)(me.rline + col * ldm1) * (Off)sizeof(C)), rr[0][r]);
                    }
                }
                lds_barrier();
                // ---- P3
                {
                    auto look_rest = [&] {
                        refl.template outer<1, NTL>(Vr, rl, rlz);
#pragma unroll
                        for (int a = 1; a < NTL; ++a) put_row_tile(rl[a], a, Z, me.lrow);
                    };
                    auto upper = [&] {
                        if (t > 0) {
                            rrz = refl.inner(Vr, rr);
                            rrz = refl.middle(Tr, rrz, me.ron);
                            refl.template outer<0, NTL>(Vr, rr, rrz);
                        }
                        if (corner && t > 0) {
                            stores_done();
                            publish(s, 2 * t);
                        }
                        // (straight from the registers: sixteen consecutive rows a column)
                        char* p = entry(c0 - B, c0, 0);
                        const Off off = (Off)(me.rline + F::roff(0, me.gq) * ldm1) * (Off)sizeof(C);
                        const bool full = t > 0 && c0 + B <= n;
                        const int ncol = (int)min((int64_t)B, n - c0) - F::roff(0, me.gq);
                        if (full) {
#pragma unroll
                            for (int a = 0; a < NTL; ++a)
#pragma unroll
                                for (int r = 0; r < 4; ++r) {
                                    rgst(at(p, off), rr[a][r]);
                                    p += (r < 3 ? F::roff(1, 0) : 16 - 3 * F::roff(1, 0)) * ldm1 * (int64_t)sizeof(C);
                                }
                        } else if (t > 0 || me.rline >= B - D) {
#pragma unroll
                            for (int a = 0; a < NTL; ++a)
#pragma unroll
                                for (int r = 0; r < 4; ++r) {
                                    if (16 * a + F::roff(r, 0) < ncol) rgst(at(p, off), rr[a][r]);
                                    p += (r < 3 ? F::roff(1, 0) : 16 - 3 * F::roff(1, 0)) * ldm1 * (int64_t)sizeof(C);
                                }
                        }
                    };
                    // the block right of Z lies in the predecessor's Z of step t+1, its U of that step and the
                    // corner of the U after it
                    if (look) {
                        C pre[PER];
                        if (rest) look_rest();
                        wait_for(s, 2 * t + 4, tile == 0, early_a);
                        load_cols(pre, c0, c0 + B, lk0, lk1, 0);
                        if (rest) upper();
                        else look_rest();
                        put_cols(S, pre, lk0, lk1);
                    } else {
                        upper();
                    }
                    if (rest) stores_done();   // U is in the band before the barrier
                }
                lds_barrier();
                // ---- P4
                if (look && tile == 0) early_z = poll(s);
                if (look) {
                    get_cols(cl, S, me.lcol);
                    clz = refl.inner(Vl, cl);
                }
                if (rest) get_cols(cr, Z, me.rcol);
                lds_barrier();
                if (look) {
                    clz = refl.middle(Tl, clz, true);
                    refl.template outer<0, 1>(Vl, cl, clz);
                    put_col_tile(cl[0], 0, S, me.lcol);
                }
                if (corner) {
                    put_factor(cr, me.rline);
                    char* p = entry(c0, c0, 0);
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int row = F::roff(r, me.gq);
                        if (me.rline < D && row < D && c0 + row < n && c0 + me.rline < n)
                            rgst(at(p, (Off)(row + me.rline * ldm1) * (Off)sizeof(C)), cr[0][r]);
                    }
                }
                lds_barrier();
            }
            if (look) __builtin_amdgcn_s_setprio(0);
        };
        if (!failed) {
            if (pw) panels();
            else if constexpr (BOTH) apply(std::integral_constant<int, 2>{});
            else if (look) apply(std::integral_constant<int, 0>{});
            else apply(std::integral_constant<int, 1>{});
        }
        __syncthreads();
        if (lead) __hip_atomic_store(&progress[s * kProgressStride], kSweepDone, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
    }
#ifdef SVB_CHASE_TIMING
    if (lead) {
        unsigned long long* acc = reinterpret_cast<unsigned long long*>(ctrl + 8);
        for (int q = 0; q < 8; ++q) atomicAdd(&acc[q], tacc[q]);
        atomicAdd(&acc[8], nstep_acc);
    }
#endif
#undef RMARK
}

// The in-band form, where two blocks do not fit in LDS (f64 at B = 128): only the diagonal block Z lives in
// LDS, the upper block U and the block right of Z are transformed where they lie, in the packed band in
// device memory.  8*B apply threads, wave 0 of which factors the panels.  Z is moved
// by "traffic" waves, each lane keeping one block row: a wave covers 64 consecutive rows of
// a column at a time and steps through the columns with a fixed stride, so that its
// addresses are a scalar base, advanced by a scalar per step, plus a fixed lane offset.
template <int B> struct InbandShape {
    static_assert(B >= kWave, "whole groups of 64 rows a column");
    static constexpr int NT = 8 * B;
    static constexpr int NWV = NT / kWave;
    static constexpr int PWV = 0;                                 // the panel wave
    static constexpr int GPC = B / kWave;                         // 64-row groups per block column
    static constexpr int NTW = (NWV - 1) / GPC * GPC;             // waves that move Z
    static constexpr int JS = NTW / GPC;                          // column step of a traffic wave
    static constexpr int PER = (B + JS - 1) / JS;                 // accesses per traffic wave and block
};

template <typename C, int B, int D>
__global__ __launch_bounds__(InbandShape<B>::NT) void band_reduce_inband_kernel(C* __restrict__ band, int64_t ldab, int64_t n,
                                                                        int* __restrict__ ctrl,
                                                                        int* __restrict__ progress, int spin_limit)
{
    // The panel wave draws the sweep, waits for the predecessor, factors the two panels of a
    // step and publishes progress.  The traffic waves move Z between device memory
    // and LDS; the right panel of step t runs beside the exchange of step t-1's Z for this step's.
    using SH = InbandShape<B>;
    static_assert(SH::NT == 1024 && sizeof(C) == 8, "waves 0-7 on LDS lines, waves 8-15 on band lines, sixteen each; Frag of f64");
    constexpr int LD = B + 1, PER = SH::PER, JS = SH::JS;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    C* S = reinterpret_cast<C*>(smem_raw);        // rows and columns c0 .. c0+B-1: S[row + col*LD]
    C* Vs = S + ((B * LD + 3) & ~3);              // (B + 4) * D
    C* Ts = Vs + (B + 4) * D;                     // D * D
    __shared__ int sh_s, sh_fail, sh_back;   // sh_back: traffic waves whose stores of a block have been acknowledged
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);       // wave-uniform: scalar branches below
    const bool pw = wv == SH::PWV;
    const bool lead = tid == SH::PWV * kWave;                      // first lane of the panel wave
    const int tw = wv - 1;                       // index among the traffic waves
    const bool traffic = !pw && tw < SH::NTW;
    // this lane's block row and first block column
    const int ii = (tw % SH::GPC) * kWave + lane;
    const int jj0 = tw / SH::GPC;
    const int ldm1 = (int)(ldab - 1);
    const int64_t ku = 2 * (int64_t)B - 1;
#ifdef SVB_CHASE_TIMING
    unsigned long long tacc[8] = {0, 0, 0, 0, 0, 0, 0, 0}, tlast = 0, nstep_acc = 0;
#define RMARK(slot_) do { if (lead) { unsigned long long now_ = wall_clock64(); tacc[slot_] += now_ - tlast; tlast = now_; } } while (0)
#else
#define RMARK(slot_) do { } while (0)
#endif
    const int64_t nsweeps = (n - 1) / D;

    // A B x B block of the band whose first element is entry (r0, cb): this lane's first
    // element of it, and the numbers of its rows and columns that lie inside the matrix.
    struct Blk { C* p; int nrow, ncol; };
    auto block_at = [&](int64_t r0, int64_t cb) -> Blk {
        Blk k;
        k.p = band + ((r0 - cb + ku) + cb * ldab) + (ii + (int64_t)jj0 * ldm1);
        k.nrow = (int)max((int64_t)0, min((int64_t)B, n - r0));
        k.ncol = (int)max((int64_t)0, min((int64_t)B, n - cb));
        return k;
    };
    // access q of a block: element (ii, jj0 + q*JS), at k.p + q*JS*ldm1 in the band and at
    // lds0 + q*JS*LD in LDS; loads of elements outside the matrix read the band's first entry
    // and are masked where the value is consumed (masking at once would wait for the load)
    auto inside = [&](const Blk& k, int q) -> bool { return ii < k.nrow && jj0 + q * JS < k.ncol; };
    auto gload = [&](const Blk& k, int q) -> C {
        const C* p = inside(k, q) ? k.p + (int64_t)(q * JS) * ldm1 : band;
        return rgld(p);
    };
    auto gstore = [&](const Blk& k, int q, C v) { rgst(k.p + (int64_t)(q * JS) * ldm1, v); };
    // Progress of a sweep: 2k+1 once the upper block U of its step k is final in the band (and
    // every block of the steps before), 2k+2 once all blocks of step k are.
    // poll: the predecessor's progress, requested ahead of the work it is checked after;
    // wait_for: waits (one lane) until sweep s-1 has reached `need`, `seen` being an earlier
    // poll; an expired wait sets sh_fail
    auto poll = [&](int64_t s) -> int {
        return (lead && s > 0) ? __hip_atomic_load(&progress[(s - 1) * kProgressStride], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
    };
    auto publish = [&](int64_t s, int value) {
        if (lead) __hip_atomic_store(&progress[s * kProgressStride], value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    auto wait_for = [&](int64_t s, int need, int seen) {
        if (lead && s > 0 && seen < need) {
            int spins = 0;
            while (__hip_atomic_load(&progress[(s - 1) * kProgressStride], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < need) {
                if (++spins > spin_limit) {
                    atomicExch(&ctrl[1], 1);
                    sh_fail = 1;
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
            }
        }
    };

    // A block written back by the traffic waves is published by the last of them to have its
    // stores acknowledged, not by the panel wave at the next barrier, which comes up to a
    // panel factorisation later: the successor sweep is waiting for exactly this.
    auto block_back = [&](int64_t s, int value) {
        stores_done();
        if (lane == 0) {
            const int arrived = atomicAdd(&sh_back, 1);
            if (arrived == SH::NTW - 1) {
                sh_back = 0;
                __hip_atomic_store(&progress[s * kProgressStride], value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    };

    // Every single-lane section is followed by a barrier before the next one (no divergent
    // region spans a loop back-edge).
    for (;;) {
        if (lead) {
            sh_s = atomicAdd(&ctrl[0], 1);
            sh_fail = __hip_atomic_load(&ctrl[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            sh_back = 0;
        }
        __syncthreads();
        const int64_t s = __builtin_amdgcn_readfirstlane(sh_s);
        __syncthreads();
        if (s >= nsweeps) break;
        const int64_t c00 = (s + 1) * D;
        const int nsteps = (int)((n - 1 - c00) / B) + 1;
#ifdef SVB_CHASE_TIMING
        if (lead) tlast = wall_clock64();
#endif
        // ---- prologue: the sweep's own D rows and the first diagonal block, straight into LDS
        // (the first diagonal block was last touched by the predecessor's step 1)
        wait_for(s, 4, 0);
        __syncthreads();
        bool failed = sh_fail != 0;
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        C pre[PER];   // traffic waves: the next Z
        if (!failed && traffic) {
            const Blk zb = block_at(c00, c00);
            const int lds0 = ii + jj0 * LD;
#pragma unroll
            for (int q = 0; q < PER; ++q) pre[q] = gload(zb, q);
#pragma unroll
            for (int q = 0; q < PER; ++q) {
                if (jj0 + q * JS < B) S[lds0 + q * JS * LD] = inside(zb, q) ? pre[q] : (C)0;
            }
        }
        __syncthreads();
        RMARK(7);
        int seen_next = 0;   // the predecessor's progress as polled during the previous step's last phase
        for (int t = 0; t < nsteps && !failed; ++t) {
            const int64_t c0 = c00 + (int64_t)t * B;
            // opaque per-step copy: without it every LDS index below is hoisted out of the step
            // loop and held in (spilled) registers
            int lds0 = ii + jj0 * LD;
            asm volatile("" : "+v"(lds0));
#ifdef SVB_CHASE_TIMING
            if (lead) { tlast = wall_clock64(); ++nstep_acc; }
#endif
            if (t > 0) {
                // this step's Z (requested in S1) has a corner that the left half of the predecessor's
                // step t+1 wrote
                wait_for(s, 2 * t + 4, seen_next);
                lds_barrier();
                failed = sh_fail != 0;
                if (failed) break;
            }
            // ---- S1: right panel (LQ of X)  ||  Z of the previous step back, this step's Z in
            const int ncol = (int)min((int64_t)B, n - c0);                            // columns c0 .. inside the matrix
            const int64_t rho = (t == 0) ? c00 - D : c0 - B;                          // first row of X
            if (pw) {
                panel_wave_spread<C, B, D, true>(band + (rho - c0 + ku) + c0 * ldab, 1, ldm1, Vs, Ts, ncol);
            } else if (traffic && t > 0) {
                // this step's Z is requested here (its registers would otherwise be live across the
                // in-band applies, which need theirs), the previous Z goes back meanwhile
                const Blk zp = block_at(c0 - B, c0 - B), zc = block_at(c0, c0);
#pragma unroll
                for (int q = 0; q < PER; ++q) pre[q] = gload(zc, q);
#pragma unroll
                for (int q = 0; q < PER; ++q)
                    if (inside(zp, q)) gstore(zp, q, S[lds0 + q * JS * LD]);
                // every block of step t-1 is final (the in-band stores of its last phase were
                // acknowledged before that phase's barrier)
                block_back(s, 2 * t);
#pragma unroll
                for (int q = 0; q < PER; ++q)
                    if (jj0 + q * JS < B) S[lds0 + q * JS * LD] = inside(zc, q) ? pre[q] : (C)0;
            }
            RMARK(0);
            // every wave's band stores of the previous step (and the panel's) are acknowledged
            // before the barrier that precedes the progress store
            stores_done();
            lds_barrier();
            RMARK(1);
            // ---- S3: block reflector onto the rows below X
            {
                // (waves 0 .. 7: the rows of Z, in LDS; waves 8 .. 15: rows D .. B-1 of U, in the band; none in the
                // first step, whose X is the sweep's own rows)
                if (wv < 8) {
                    apply_tile<C, B, D>(S + 16 * wv, LD, 1, 16, Vs, Ts);
                } else if (t > 0) {
                    const int row = D + 16 * (wv - 8);
                    apply_tile_g<C, B, D>(band + ((c0 - B + row) - c0 + ku) + c0 * ldab, ldm1, 1, B - row, ncol, Vs, Ts);
                    stores_done();
                }
            }
            lds_barrier();
            RMARK(2);
            publish(s, 2 * t + 1);   // U was transformed where it lies; the stores are acknowledged
            // ---- S4: left panel (QR of Z's first D columns)
            const int seen2 = poll(s);
            if (pw) panel_wave_spread<C, B, D, false>(S, LD, 1, Vs, Ts, B);
            RMARK(3);
            lds_barrier();
            // the block right of Z (transformed where it lies in S5) was last touched by the right
            // half of the predecessor's step t+2, whose result is that step's upper block
            wait_for(s, 2 * t + 5, seen2);
            lds_barrier();
            failed = sh_fail != 0;
            if (failed) break;
            RMARK(4);
            seen_next = poll(s);
            // ---- S5: block reflector onto the other columns of Z and onto A3
            {
                // waves 0 .. 7: columns D .. B-1 of Z, in LDS; waves 8 .. 15: the columns of the block right of Z, in
                // the band
                if (wv < 8) {
                    apply_tile<C, B, D>(S + (D + 16 * wv) * LD, 1, LD, B - D - 16 * wv, Vs, Ts);
                } else {
                    const int nrow = (int)min((int64_t)B, n - c0);
                    const int64_t cg = c0 + B + 16 * (wv - 8);
                    if (cg < n) {   // (none of the sixteen inside, as in all of a sweep's last step: most of the work at n <= 136)
                        apply_tile_g<C, B, D>(band + (c0 - cg + ku) + cg * ldab, 1, ldm1, (int)min((int64_t)16, n - cg), nrow, Vs, Ts);
                        stores_done();
                    }
                }
            }
            lds_barrier();
            RMARK(5);
        }
        // ---- epilogue: the last step's Z back (nothing is right of it)
        if (!failed && traffic) {
            const int64_t c0 = c00 + (int64_t)(nsteps - 1) * B;
            const Blk zl = block_at(c0, c0);
            const int lds0 = ii + jj0 * LD;
#pragma unroll
            for (int q = 0; q < PER; ++q)
                if (inside(zl, q)) gstore(zl, q, S[lds0 + q * JS * LD]);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        }
        __syncthreads();
        if (lead) __hip_atomic_store(&progress[s * kProgressStride], kSweepDone, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
    }
#ifdef SVB_CHASE_TIMING
    if (lead) {
        unsigned long long* acc = reinterpret_cast<unsigned long long*>(ctrl + 8);
        for (int q = 0; q < 8; ++q) atomicAdd(&acc[q], tacc[q]);
        atomicAdd(&acc[8], nstep_acc);
    }
#endif
#undef RMARK
}

__global__ __launch_bounds__(256) void reduce_clear_kernel(int* __restrict__ p, int64_t count)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0;
}

template <typename C, int B>
int launch_band_reduce(int64_t n, C* band, int64_t ldab, int* ctrl, hipStream_t s)
{
    constexpr int D = 8;
    // two blocks in LDS where they fit, otherwise only the diagonal block
    constexpr bool inband = ReduceShape<C, B>::kSmemBytes > 160 * 1024 - 256;
    void (*kern)(C*, int64_t, int64_t, int*, int*, int);
    size_t smem;
    int nt;
    const bool wide = !inband && ldab > ((int64_t)1 << 26);
    if constexpr (inband) {
        kern = band_reduce_inband_kernel<C, B, D>;
        smem = sizeof(C) * (size_t)(((B * (B + 1) + 3) & ~3) + (B + 4) * D + D * D);
        nt = InbandShape<B>::NT;
    } else {
        // (offsets of 32 bits: 7 columns of f64, 12 of f32 from the first of a block are less than 2^32 bytes away)
        kern = wide ? band_reduce_kernel<C, B, true> : band_reduce_kernel<C, B, false>;
        smem = ReduceShape<C, B>::kSmemBytes;
        nt = ReduceShape<C, B>::NT;
    }
    static bool attr_set[2] = {false, false};
    if (!attr_set[wide]) {
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        attr_set[wide] = true;
    }
    const int64_t nsweeps = (n - 1) / D;
    const int64_t count = 64 + nsweeps * kProgressStride;
    const int cb = (int)((count + 255) / 256);
    hipLaunchKernelGGL(reduce_clear_kernel, dim3(cb > 256 ? 256 : cb), dim3(256), 0, s, ctrl, count);
    if (nsweeps <= 0) return SVB_OK;
    const int grid = (int)min((int64_t)env_int("SVB_REDUCE_GRID", 256), nsweeps);
    const int spin_limit = env_int("SVB_CHASE_SPIN", 1 << 20);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(nt), smem, s, band, ldab, n, ctrl, ctrl + 64, spin_limit);
    return hipGetLastError() == hipSuccess ? SVB_OK : SVB_ERR_DEVICE;
}

}  // namespace

// ctrl: 64 ints (ticket, error flag, timing slots) followed by the progress counters of the (n - 1) / 8 block sweeps
size_t band_reduce_workspace_bytes(int64_t n) { return (size_t)((64 + n / 8 * kProgressStride) * 4 + 255) / 256 * 256; }

bool band_reduce_supported(int nb, size_t elem_size)
{
    (void)elem_size;
    return nb == 32 || nb == 64 || nb == 128;
}

template <typename C>
int run_band_reduce(int64_t n, int nb, C* band, int64_t ldab, int* ctrl, hipStream_t s)
{
    if (nb == 32) return launch_band_reduce<C, 32>(n, band, ldab, ctrl, s);
    if (nb == 64) return launch_band_reduce<C, 64>(n, band, ldab, ctrl, s);
    if (nb == 128) return launch_band_reduce<C, 128>(n, band, ldab, ctrl, s);
    return SVB_ERR_UNSUPPORTED;
}

template int run_band_reduce<double>(int64_t, int, double*, int64_t, int*, hipStream_t);
template int run_band_reduce<float>(int64_t, int, float*, int64_t, int*, hipStream_t);

}  // namespace svb
