// Stage 3 on the device: singular values of the upper bidiagonal (d, e) by
// bisection (paper Section 3, final stage; the paper solves the bidiagonal on
// the CPU with LAPACK and names it the cheapest stage.  Once stages 1-2 run
// in tens of milliseconds a host solve dominates time-to-singular-values, so
// the same bisection that the host entry point svb_bdsvals performs is also
// available on the GPU).
//
// Count of singular values below x, by the Sturm sequence of the Golub-Kahan tridiagonal (zero
// diagonal, off-diagonals d_1, e_1, d_2, ..): with r_k = (-1)^k det(T_k - x I),
//   r_{2j+1} = x r_{2j} - e_{j-1}^2 r_{2j-1},   r_{2j+2} = x r_{2j+1} - d_j^2 r_{2j},
// the number of sign changes is the number of singular values >= x.  Two fused multiply-adds per row
// are all that depends on the row before, no division; computed r are those of a matrix whose
// entries differ by a few units in the last place, so small values keep their relative accuracy.
// The pair is scaled back to [1/2, 1) every eight rows (a row shrinks it by no more than x^2 and the
// rounding of a cancellation: every two rows for x below 2^-50); a count in which it fell below
// 2^-800 in between (exact zeros) is done again with the differential stationary qd recurrence, which
// forms ratios and needs a reciprocal per row.  Squares are taken after scaling by
// the largest entry, always in fp64.  A first kernel counts at 4096 shared points of
// [0, bound]; every singular value then starts from the cell it falls in and is refined by
// multisection (several points per round, one lane each).
#include "svb_internal.h"

namespace svb {

namespace {

constexpr int kPrepThreads = 1024;

// ws[0] = scale, ws[1] = upper bound for sigma_max / scale; from ws + 8 on the squares of the scaled
// entries, row by row: e_{j-1}^2, d_j^2 (e_{-1} = 0).
template <typename C>
__global__ __launch_bounds__(kPrepThreads) void bd_prep_kernel(const C* __restrict__ d, const C* __restrict__ e,
                                                               int64_t n, double* __restrict__ ws)
{
    __shared__ double red[2][kPrepThreads / kWave];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    double zmax = 0.0, bound = 0.0;
    bool bad = false;
    for (int64_t j = tid; j < n; j += kPrepThreads) {
        const double a = fabs((double)d[j]);
        const double b = j + 1 < n ? fabs((double)e[j]) : 0.0;
        const double bp = j > 0 ? fabs((double)e[j - 1]) : 0.0;
        bad = bad || !(a <= 1.79e308) || !(b <= 1.79e308);
        zmax = fmax(zmax, fmax(a, b));
        bound = fmax(bound, a + fmax(b, bp));
    }
    if (bad) { zmax = NAN; bound = NAN; }
    for (int off = 32; off > 0; off >>= 1) {
        const double z2 = __shfl_xor(zmax, off, kWave), b2 = __shfl_xor(bound, off, kWave);
        zmax = (zmax != zmax || z2 != z2) ? NAN : fmax(zmax, z2);
        bound = (bound != bound || b2 != b2) ? NAN : fmax(bound, b2);
    }
    if (lane == 0) { red[0][wave] = zmax; red[1][wave] = bound; }
    __syncthreads();
    zmax = 0.0; bound = 0.0;
    for (int w = 0; w < kPrepThreads / kWave; ++w) {
        const double z2 = red[0][w], b2 = red[1][w];
        zmax = (zmax != zmax || z2 != z2) ? NAN : fmax(zmax, z2);
        bound = (bound != bound || b2 != b2) ? NAN : fmax(bound, b2);
    }
    const double scale = zmax > 0.0 ? zmax : 1.0;  // NaN stays NaN through the comparisons below
    if (tid == 0) {
        ws[0] = (zmax != zmax) ? NAN : scale;
        ws[1] = bound / scale * (1.0 + 1e-14) + 1e-300;
    }
    double* z = ws + 8;
    for (int64_t j = tid; j < n; j += kPrepThreads) {
        const double a = (double)d[j] / scale;
        const double b = j > 0 ? (double)e[j - 1] / scale : 0.0;
        z[2 * j] = b * b;
        z[2 * j + 1] = a * a;
    }
}

constexpr int64_t kMinGuess = 300;        // rows from which a round costs more than the interpolation
constexpr double kSmallPoint = 0x1p-50;   // below: two rows between rescalings, else eight
constexpr int kGrid = 4096;   // points of the shared first partition of [0, bound]

__device__ __forceinline__ double lane_value(double v, int lane)
{
    const long long b = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), lane);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __builtin_bit_cast(double, ((long long)hi << 32) | (long long)(unsigned)lo);
}

// Number of singular values below x by the qd recurrence
//   t_1 = -x^2,  D_j = d_j^2 + t_j,  t_{j+1} = -x^2 + e_j^2 * t_j / D_j   (the number of negative D_j).
// All 64 lanes of the wave walk the same rows, so the rows are fetched 64 at a time, one per lane,
// and handed round as wave-uniform scalars.  Rows past n are padded so that they never count.
__device__ __attribute__((noinline)) int64_t qd_count(const double* __restrict__ z, int64_t n, double x)
{
    const int lane = threadIdx.x & (kWave - 1);
    const double pivmin = 1e-300, x2 = x * x;
    double s = 0.0;      // t_j / D_j of the row before
    int64_t cnt = 0;
    for (int64_t j0 = 0; j0 < n; j0 += kWave) {
        const bool in = j0 + lane < n;
        const double ej = in ? z[2 * (j0 + lane)] : 0.0, dj = in ? z[2 * (j0 + lane) + 1] : 1e300;
#pragma unroll 8
        for (int jj = 0; jj < kWave; ++jj) {
            const double dd = lane_value(dj, jj), ee = lane_value(ej, jj);
            const double t = ee * s - x2;
            double D = dd + t;
            if (fabs(D) < pivmin) D = -pivmin;
            cnt += D < 0.0 ? 1 : 0;
            double r = __builtin_amdgcn_rcp(D);      // reciprocal + one Newton step instead of a full division
            r = fma(r, fma(-D, r, 1.0), r);
            s = t * r;
        }
    }
    return cnt;
}

// Number of singular values below x (one x > 0 per lane, every lane of the wave active) by the
// recurrence in the header.  The rows are the same for every lane: they come in as scalars, a
// block of eight ahead.  What bounds it is the issue of its instructions (per row two products,
// two fused multiply-adds, two shifts that collect the signs, and the rescaling: about 7, of 5
// cycles each from a lone wave; the dependent chain is 16 cycles a row): 50 cycles a row measured
// against 92 for the qd form above; the whole stage at n = 8192: 7.02 -> 3.37 ms (f64), 4.04 -> 1.81
// (f32), at n = 32768: 50 -> 23 and 27 -> 12.
// f 2^fe: the last member of the sequence, det up to its sign, a polynomial in x whose zeros are the values
// (f = 0 where the count was done again in the other form); formed if POLY, for some 5 % of the time.
template <int EVERY, bool POLY>
__device__ __forceinline__ int64_t sequence_count(const double* __restrict__ z, int64_t n, double x, double& f, int& fe)
{
    constexpr int R = 8;
    double h = 0.0, b = 1.0;          // r_{2j-1}, r_{2j}
    unsigned signs = 0;               // of the last 32 members of the sequence, the latest in bit 0
    int changes = 0;
    // smallest size the pair had before a rescaling: over all of them, and over those at the end of a block
    // without the ones in between (`moved`: powers of two these took out), which is what EVERY = R sees.
    // Points of either kind are judged by the same number in both forms: the outcome depends on x alone,
    // not on the other lanes of the wave.
    double low = 1.0, low_block = 1.0;
    int moved = 0, shift = 0;
    auto row = [&](double ee, double dd) {
        const double nh = fma(x, b, -(ee * h));
        const double nb = fma(x, nh, -(dd * b));
        signs = __builtin_amdgcn_alignbit(signs, (unsigned)(__builtin_bit_cast(unsigned long long, nh) >> 32), 31);
        signs = __builtin_amdgcn_alignbit(signs, (unsigned)(__builtin_bit_cast(unsigned long long, nb) >> 32), 31);
        h = nh;
        b = nb;
    };
    auto rescale = [&](bool last) {
        const double m = fmax(fabs(h), fabs(b));
        const int e = -__builtin_amdgcn_frexp_exp(m);
        low = fmin(low, m);
        if (POLY) shift += e;
        if (EVERY < R) {
            if (last) low_block = fmin(low_block, __builtin_amdgcn_ldexp(m, moved));
            moved = last ? 0 : moved - e;
        }
        h = __builtin_amdgcn_ldexp(h, e);
        b = __builtin_amdgcn_ldexp(b, e);
    };
    // Two blocks of rows in scalar registers: one is on its way while the other is worked on.  Left to
    // itself the compiler moves the loads to where their values are used, and every block waits for
    // them: the fence keeps them in front of the rows, the empty statement takes delivery behind them.
    const int nblk = (int)(n / R);
    double za[2 * R], zb[2 * R];
    auto fetch = [&](double (&q)[2 * R], int k) {
        const double* __restrict__ p = z + (int64_t)(k < nblk ? k : 0) * (2 * R);
#pragma unroll
        for (int i = 0; i < 2 * R; ++i) q[i] = p[i];
        __builtin_amdgcn_sched_barrier(0);
    };
    auto block = [&](const double (&q)[2 * R]) {
#pragma unroll
        for (int i = 0; i < R; ++i) {
            row(q[2 * i], q[2 * i + 1]);
            if ((i + 1) % EVERY == 0) rescale(i + 1 == R);
        }
        changes += __builtin_popcount((signs ^ (signs >> 1)) & 0xffffu);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto arrived = [&](double (&q)[2 * R]) {
#pragma unroll
        for (int i = 0; i < 2 * R; ++i) asm volatile("" : "+s"(q[i]));
    };
    if (nblk > 0) fetch(za, 0);
    for (int k = 0; k < nblk; k += 2) {
        arrived(za);
        fetch(zb, k + 1);
        block(za);
        if (k + 1 == nblk) break;
        arrived(zb);
        fetch(za, k + 2);
        block(zb);
    }
    for (int64_t j = (int64_t)nblk * R; j < n; ++j) {
        row(z[2 * j], z[2 * j + 1]);
        changes += __builtin_popcount((signs ^ (signs >> 1)) & 3u);
        rescale(true);
    }
    // (every lane walks along, each keeps its own: two values next to each other have to see the same count
    // at the same point, whatever the rest of their waves does, or they could come out in the wrong order)
    const bool redo = (EVERY < R && x >= kSmallPoint ? low_block : low) < 0x1p-800;
    int64_t count = n - changes;
    if (POLY) {
        f = redo ? 0.0 : b;
        fe = -shift;
    }
    if (__any(redo)) {
        const int64_t c = qd_count(z, n, x);
        count = redo ? c : count;
    }
    return count;
}
template <bool POLY> __device__ __forceinline__ int64_t sturm_count(const double* __restrict__ z, int64_t n, double x, double& f, int& fe)
{
    return __any(x < kSmallPoint) ? sequence_count<2, POLY>(z, n, x, f, fe) : sequence_count<8, POLY>(z, n, x, f, fe);
}

// counts at the points x_i = bound * i / kGrid, i = 1 .. kGrid - 1 (x_0 counts 0, x_kGrid counts n)
__global__ __launch_bounds__(64) void bd_grid_kernel(const double* __restrict__ ws, int64_t n, int* __restrict__ gcnt)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;   // 0 .. kGrid-1, all lanes stay active
    const double scale = ws[0], hi0 = ws[1];
    const double* __restrict__ z = ws + 8;
    int64_t c = 0;
    if (scale == scale) {
        const double x = hi0 * ((double)max(i, 1) / kGrid);   // (x = 0 would send its wave the slow ways)
        double f;
        int fe;
        c = sturm_count<false>(z, n, x, f, fe);
    }
    gcnt[i] = i == 0 ? 0 : (int)min(c, n);
    if (i == 0) gcnt[kGrid] = (int)n;
}

// 1 / x for guesses
__device__ __forceinline__ double quick_rcp(double x)
{
    const double r = __builtin_amdgcn_rcp(x);
    return fma(r, fma(-x, r, 1.0), r);
}

// Where the polynomial through the nodes of a bracket vanishes inside it: t in (0, 1), 0 and 1 being the bracket's
// ends, nodes 0 and 1.  M nodes; Newton's form, Newton's method from x on, kept inside a shrinking bracket.
template <int M>
__device__ __forceinline__ double interpolated_zero(const double (&t)[6], const double (&c)[6], bool negative, double x)
{
    double a = 0.0, b = 1.0;
#pragma unroll 1
    for (int it = 0; it < 7; ++it) {
        double p = c[M - 1], dp = 0.0;
#pragma unroll
        for (int i = M - 2; i >= 0; --i) {
            dp = fma(dp, x - t[i], p);
            p = fma(p, x - t[i], c[i]);
        }
        if ((p < 0.0) == negative) a = x;
        else b = x;
        const double nx = fma(-p, quick_rcp(dp), x);
        x = nx > a && nx < b ? nx : 0.5 * (a + b);
    }
    return x;
}

// Multisection: P lanes per singular value, each counting at one of P interior points of the value's current
// interval.  The Sturm recurrence is one long dependent chain per point and a wave costs the
// same whether it refines 64 values by 2 or 4 values by 17 per round, so while the compute
// units have waves to spare the extra points are free and the number of rounds drops.
// The points are equally spaced (the interval shrinks by P + 1) until the value is alone in its interval.  From
// then on the counts' recurrence has more to say: its last member is a polynomial that changes sign at the value,
// known at the P points and the ends.  The next points are laid around the zero of the interpolating polynomial
// through the nodes next to the value (up to six, none beyond another value), at distances delta,
// delta 4, delta 16, .. (P = 16) on both sides, delta being half of what two more nodes can be expected to change, or
// what the tolerance still asks for.  The counts alone decide which interval is taken, so a bad guess costs a round
// and nothing else; the points are equally spaced after a round that gained less than that, where the interpolation has
// not settled, and where equal spacing is enough to end.
// The polynomial is formed, and known ends asked for, only for values that are alone (and in the first round), the
// ends only once: a point where it is not to be had (the count was done again: singular matrices) counts as known, and
// at zero it is a product of the diagonal.  A form that asked for both ends in every round of every value until it
// had them took 3.3 times as long as equal spacing on singular matrices (0.44 -> 1.59 ms at n = 700) and up to 1.4 times on
// tight clusters.
// Values that share an interval see the same points, those that do not are in order already: they come out in order.
// Bidiagonal of a Gaussian matrix, ms with equal spacing only -> with guesses (whole stage): f64 n = 500 0.145 -> 0.107,
// n = 6000 (10 -> 5 rounds) 2.35 -> 1.53, n = 20000 13.5 -> 8.4; f32 n = 6000 (5 -> 3) 1.32 -> 1.03.  What is left at n = 6000 is a
// wave and a half per SIMD, the last of which take seven rounds.
template <typename C, int P, bool GUESS>
__global__ __launch_bounds__(64) void bd_multisect_kernel(const double* __restrict__ ws, int64_t n,
                                                           C* __restrict__ sigma, double rel_tol,
                                                           double floor_frac, const int* __restrict__ gcnt)
{
    constexpr int VPW = kWave / P;   // values per wave
    const int lane = threadIdx.x, grp = lane / P, q = lane % P;
    const int64_t kraw = (int64_t)blockIdx.x * VPW + grp;  // ascending index
    const int64_t k = min(kraw, n - 1);   // surplus lanes repeat the last value: the wave stays whole
    const double scale = ws[0], hi0 = ws[1];
    const double* __restrict__ z = ws + 8;
    if (scale != scale) {  // non-finite input: poison the output, the caller maps it to a status
        if (kraw < n && q == 0) sigma[n - 1 - k] = (C)NAN;
        return;
    }
    if (hi0 <= 2e-300) {   // all entries are zero (the bound is its own guard term): so are the values
        if (kraw < n && q == 0) sigma[n - 1 - k] = (C)0;
        return;
    }
    // first interval from the shared partition: gcnt[a] < k+1 <= gcnt[b] with b = a+1
    int a = 0, b = kGrid;
    while (b - a > 1) {
        const int m = (a + b) >> 1;
        if (gcnt[m] >= k + 1) b = m;
        else a = m;
    }
    double lo = hi0 * ((double)a / kGrid), hi = b == kGrid ? hi0 : hi0 * ((double)b / kGrid);
    // width relative to the value, or to floor_frac times the bound on the largest value if that is more
    auto wanted = [&]() -> double { return rel_tol * fmax(hi, floor_frac * hi0) + 1e-38 * hi0; };
    // whether to go on, and the first of the round's points that is above the value (P: none); the points of a value
    // are ascending, so its lanes read: below .. below, above .. above.  Rounding may have put a point on an end of
    // the interval, where the count is known.
    auto is_open = [&]() -> bool {
        const double mid = 0.5 * (lo + hi);
        return (hi - lo > wanted()) && (mid > lo && mid < hi);
    };
    auto first_above = [&](double x, int64_t cnt) -> int {
        const unsigned long long m = __ballot(x >= hi || (x > lo && cnt >= k + 1)) >> (grp * P);
        const unsigned long long mine = P == 64 ? m : (m & ((1ull << P) - 1ull));
        return mine ? __builtin_ctzll(mine) : P;
    };
    const double frac = (double)(q + 1) / (P + 1);
    if constexpr (!GUESS) {
        for (int it = 0; it < 200; ++it) {
            const bool open = is_open();
            if (!__any(open)) break;            // wave-uniform exit: the row hand-over needs every lane
            const double w = hi - lo, x = fmin(fmax(fma(w, frac, lo), lo), hi);
            double f;
            int fe;
            const int first = first_above(x, sturm_count<false>(z, n, x, f, fe));
            if (open) {
                // (the same expressions the lanes first - 1 and first evaluated their points with)
                const double nlo = first == 0 ? lo : fmin(fmax(fma(w, (double)first / (P + 1), lo), lo), hi);
                const double nhi = first == P ? hi : fmin(fmax(fma(w, (double)(first + 1) / (P + 1), lo), lo), hi);
                lo = nlo;
                hi = nhi;
            }
        }
    } else {
        // the round's nodes of every value: 0 the interval's lower end, P + 1 its upper end
        __shared__ double sx[VPW][P + 2], sf[VPW][P + 2];
        __shared__ int se[VPW][P + 2], sc[VPW][P + 2];
        double* const X = sx[grp];
        double* const Fv = sf[grp];
        int* const E = se[grp];
        int* const N = sc[grp];
        // the polynomial at the ends: NaN where not formed, 0 where not to be had
        double flo = NAN, fhi = NAN;
        int elo = 0, ehi = 0, nlo = gcnt[a], nhi = gcnt[b];
        bool guess = false;
        double centre = 0.0, delta = 0.0;
        // this lane's offset from a guess, in units of delta: -G^(P/2-1) .. -1, 1 .. G^(P/2-1), G = 4, 16, 256
        const int step = 32 / P * (q < P / 2 ? P / 2 - 1 - q : q - P / 2);
        const double offset = __builtin_amdgcn_ldexp(q < P / 2 ? -1.0 : 1.0, step), frac_ends = (double)q / (P - 1);
        // the polynomial at zero, (-1)^n d_1^2 d_2^2 .., by all lanes together
        auto at_zero = [&](int& fe) -> double {
            double p = 1.0;
            int e = 0;
            auto scaled = [&](double v) {
                const int d = __builtin_amdgcn_frexp_exp(v);
                p = __builtin_amdgcn_ldexp(v, -d);
                e += d;
            };
            for (int64_t j = lane; j < n; j += kWave) scaled(p * z[2 * j + 1]);
            for (int off = 32; off > 0; off >>= 1) {
                const double p2 = __shfl_xor(p, off, kWave);
                const int e2 = __shfl_xor(e, off, kWave);
                scaled(p * p2);
                e += e2;
            }
            fe = e;
            return (n & 1) ? -p : p;
        };
        // intervals up to this many times the wanted width (one round, P = 4: two) are left to equal spacing
        constexpr double kNear = P >= 8 ? P + 1.0 : (P + 1.0) * (P + 1.0);
        for (int it = 0; it < 200; ++it) {
            const bool open = is_open();
            if (!__any(open)) break;
            const double w = hi - lo, far = w * quick_rcp(kNear * wanted());
            const bool alone = nlo == k && nhi == k + 1, at0 = open && alone && lo == 0.0 && flo != flo && far > P + 1;
            if (__any(at0)) {
                int e;
                const double p = at_zero(e);
                if (at0) { flo = p; elo = e; }
            }
            // equally spaced points inside the interval, or, where the polynomial at an end is still to be formed, with
            // the ends
            const bool known = flo + fhi == flo + fhi, useless = flo == 0.0 || fhi == 0.0;
            const bool ends = alone && lo > 0.0 && !known && !useless && far > P - 1;
            const double x = fmin(fmax(guess ? fma(delta, offset, centre) : fma(w, ends ? frac_ends : frac, lo), lo), hi);
            const bool poly = guess || ends || ((alone ? !useless : it == 0 && nhi - nlo <= P) && far > P + 1);
            double f = NAN;
            int fe = 0;
            const int64_t cnt = __any(open && poly) ? sturm_count<true>(z, n, x, f, fe) : sturm_count<false>(z, n, x, f, fe);
            const int first = first_above(x, cnt);
            X[q + 1] = x; Fv[q + 1] = f; E[q + 1] = fe; N[q + 1] = (int)min(cnt, n);
            if (q == 0) {
                X[0] = lo; Fv[0] = flo; E[0] = elo; N[0] = nlo;
                X[P + 1] = hi; Fv[P + 1] = fhi; E[P + 1] = ehi; N[P + 1] = nhi;
            }
            __syncthreads();
            if (open) {
                lo = X[first]; flo = Fv[first]; elo = E[first]; nlo = N[first];
                hi = X[first + 1]; fhi = Fv[first + 1]; ehi = E[first + 1]; nhi = N[first + 1];
                const bool gained = (hi - lo) * (P - 1) <= w * 1.0001;
                guess = false;
                const double wn = hi - lo, want = wanted();
                if (gained && nlo == k && nhi == k + 1 && flo * fhi < 0.0 && wn > kNear * want) {
                    // nodes outwards from the bracket, those between the neighbouring values only
                    double t[6], y[6], c[6];
                    const double wi = quick_rcp(wn);
                    const int e0 = max(elo, ehi);
                    t[0] = 0.0; t[1] = 1.0;
                    y[0] = __builtin_amdgcn_ldexp(flo, elo - e0);
                    y[1] = __builtin_amdgcn_ldexp(fhi, ehi - e0);
                    int l = first, r = first + 1, nodes = 2;
#pragma unroll
                    for (int j = 2; j < 6; ++j) {
                        const int i = (j & 1) ? r + 1 : l - 1;
                        const int ic = min(max(i, 0), P + 1);
                        const double xi = X[ic], fi = Fv[ic];
                        const bool use = nodes == j && i >= 0 && i <= P + 1 && fi == fi && fi != 0.0 &&
                                         ((j & 1) ? (xi > X[r] && N[ic] == k + 1) : (xi < X[l] && N[ic] == k));
                        t[j] = (xi - lo) * wi;
                        y[j] = __builtin_amdgcn_ldexp(fi, min(max(E[ic] - e0, -1000), 500));
                        if (use) {
                            ++nodes;
                            if (j & 1) r = i;
                            else l = i;
                        }
                    }
                    // divided differences
#pragma unroll
                    for (int j = 0; j < 6; ++j) c[j] = y[j];
#pragma unroll
                    for (int d = 1; d < 6; ++d)
#pragma unroll
                        for (int j = 5; j >= d; --j)
                            if (j < nodes) c[j] = (c[j] - c[j - 1]) * quick_rcp(t[j] - t[j - d]);
                    const double zs = y[0] * quick_rcp(y[0] - y[1]);
                    double z0, z1;
                    if (nodes == 6) {
                        z0 = interpolated_zero<6>(t, c, y[0] < 0.0, zs);
                        z1 = interpolated_zero<4>(t, c, y[0] < 0.0, zs);
                    } else if (nodes >= 4) {
                        z0 = interpolated_zero<4>(t, c, y[0] < 0.0, zs);
                        z1 = interpolated_zero<3>(t, c, y[0] < 0.0, zs);
                    } else {
                        z0 = zs;
                        z1 = z0 + z0 * (1.0 - z0);
                    }
                    centre = fma(wn, z0, lo);
                    // (the next two nodes would change about d1 d1 / d2 more, d1 and d2 being what the last and the ones
                    // before them changed)
                    const double d1 = fabs(z0 - z1), d2 = fabs(z1 - zs);
                    const double d = nodes >= 4 ? 0.5 * fmin(fmax(d1 * d1 * quick_rcp(fmax(d2, 1e-300)), d1 * (1.0 / 4096)), d1) : 0.25 * d1;
                    delta = fmax(wn * d, 0.45 * want);
                    guess = centre >= lo && centre <= hi && d1 < 0.05;
                }
            }
            __syncthreads();
        }
    }
    if (kraw < n && q == 0) sigma[n - 1 - k] = (C)(0.5 * (lo + hi) * scale);
}

}  // namespace

// doubles: scale, bound, 6 spare, the squares (two a row); then the counts at the partition points
size_t bdsvals_dev_workspace_bytes(int64_t n) { return (size_t)(8 + 2 * n) * sizeof(double) + (size_t)(kGrid + 8) * sizeof(int); }

template <typename C>
int run_bdsvals_dev(int64_t n, const C* d, const C* e, C* sigma, void* work, double rel_tol, double floor_frac,
                    hipStream_t s)
{
    double* ws = static_cast<double*>(work);
    hipLaunchKernelGGL((bd_prep_kernel<C>), dim3(1), dim3(kPrepThreads), 0, s, d, e, n, ws);
    int* gcnt = reinterpret_cast<int*>(ws + 8 + 2 * n);
    hipLaunchKernelGGL(bd_grid_kernel, dim3(kGrid / 64), dim3(64), 0, s, ws, n, gcnt);
    // points per value: as many as keep the launch at about two waves per SIMD
    int p = env_int("SVB_STAGE3_POINTS", 0);
    if (p <= 0) p = n <= 8192 ? 16 : (n <= 16384 ? 8 : (n <= 32768 ? 4 : (n <= 65536 ? 2 : 1)));
    auto launch = [&](auto kern, int pp) {
        const int vpw = kWave / pp;
        hipLaunchKernelGGL(kern, dim3((unsigned)((n + vpw - 1) / vpw)), dim3(64), 0, s, ws, n, sigma, rel_tol, floor_frac,
                           gcnt);
    };
    // Guessed rounds need four points at least to interpolate, rows enough that a round costs more than the
    // interpolation, and rounds enough to save some: a wave goes on until the last of its values is done, so where equal
    // spacing takes five rounds a single guess that misses costs what the others gained.  Time with guesses over time
    // without, Gaussian / log-uniform / graded bidiagonals, n = 500 .. 32768, by the width asked for, relative to every value:
    // 2^-20 .75 - .98 / 1.0 - 1.2 / .96 - 1.1; 2^-29 .72 - .82 / .89 - .99 / .87 - .93 (n > 16384, four points: .96 / 1.05
    // / .99); 2^-37 .62 - .80 / .80 - .93 / .79 - .93; 2^-52 .65 - .85 / .70 - .87 / .75 - .90; relative to an eighth of the
    // bound at least: 2^-29 .86 - 1.07 / 1.0 - 1.14 / 1.1 - 1.2; 2^-37 .77 - .89 / .86 - .98 / 1.06 - 1.11; 2^-52 .66 - .92 /
    // .70 - .98 / .87 - 1.1.  Tight clusters gain nothing and lose up to 1.19 (2^-29, 2^-37), 1.06 (2^-52).
    const bool guess = n >= kMinGuess && (rel_tol <= 0x1p-36 || (rel_tol <= 0x1p-28 && floor_frac == 0.0 && p >= 8));
    if (p >= 16) guess ? launch(bd_multisect_kernel<C, 16, true>, 16) : launch(bd_multisect_kernel<C, 16, false>, 16);
    else if (p >= 8) guess ? launch(bd_multisect_kernel<C, 8, true>, 8) : launch(bd_multisect_kernel<C, 8, false>, 8);
    else if (p >= 4) guess ? launch(bd_multisect_kernel<C, 4, true>, 4) : launch(bd_multisect_kernel<C, 4, false>, 4);
    else if (p >= 2) launch(bd_multisect_kernel<C, 2, false>, 2);
    else launch(bd_multisect_kernel<C, 1, false>, 1);
    return hipGetLastError() == hipSuccess ? SVB_OK : SVB_ERR_DEVICE;
}

template int run_bdsvals_dev<double>(int64_t, const double*, const double*, double*, void*, double, double, hipStream_t);
template int run_bdsvals_dev<float>(int64_t, const float*, const float*, float*, void*, double, double, hipStream_t);

}  // namespace svb
