// Stage 2, narrow bands: band -> bidiagonal for a band of D = 8 super-diagonals
// (paper Section 3, second stage; the paper points to cache-efficient tile kernels and a
// communication-avoiding strategy without giving the algorithm).
//
// The chase itself is the one described in stage2_chase.hip (sweep i, step t at
// c0 = i + 1 + t*D: right reflector from row r on columns c0.., left reflector from column
// c0 on rows c0..; half step h of sweep i+1, h = 2t for the right and 2t + 1 for the left
// reflector of step t, after half step h + 3 of sweep i).  That is one chain of 4n half steps
// for the whole matrix, so what counts is the latency of a half step and what a hand-over adds.
//
// A workgroup owns a BUNDLE of NW consecutive sweeps inside a ring of the band's columns in LDS:
// four sweeps per compute wave, four half steps apart, sixteen lanes each, one row (right) or
// column (left) of the step per lane.  A half step is 8 LDS reads, the reflector, 8 LDS writes.  Its
// pivot does not come through LDS: it is the first element of the lines that lanes 8 .. 15 have
// just transformed, handed round by row broadcasts, so the reflector's scalars are formed while
// the lines are on their way (LDS operations of a wave complete in order: no wait between its
// writes and its next reads).  Waves follow each
// other through progress counters in LDS, a half step of slack apart, so no workgroup barrier
// stands in the chain.  Two more waves do the traffic: one brings columns in as soon as the
// previous bundle has published them, one writes finished columns back and publishes them.
// Bundles are pipelined over workgroups through a ticket counter and a per-bundle count of
// written-back columns (bounded waits, as in stage2_chase.hip).
//
// Packed band: entry (i,j) at band[(i - j + ku) + j*ldab]; ku >= 2D-1 and ldab >= ku + D.
#include <type_traits>

#include "svb_internal.h"
#include "lane_ops.h"

namespace svb {

namespace {

constexpr int kAllFlushed = 0x7fffffff;
constexpr int kAllDone = 0x3fffffff;    // progress of a wave (or the loader) that has finished its bundle

template <typename C> __device__ __forceinline__ C ngld(const C* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename C> __device__ __forceinline__ void ngst(C* p, C v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// progress counters in LDS
__device__ __forceinline__ int lds_get(const int* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void lds_set(int* p, int v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Keeps the compiler from moving memory accesses across; the LDS unit itself takes the
// operations of one wave in order, so a counter written after the data is seen after the data.
__device__ __forceinline__ void order_lds() { asm volatile("" ::: "memory"); }

// the pivot (p_0 .. p_7) from lanes 8 .. 15 of the row
template <typename C> __device__ __forceinline__ void row_pivot(C x, C (&p)[8])
{
    p[0] = row_lane<8>(x); p[1] = row_lane<9>(x); p[2] = row_lane<10>(x); p[3] = row_lane<11>(x);
    p[4] = row_lane<12>(x); p[5] = row_lane<13>(x); p[6] = row_lane<14>(x); p[7] = row_lane<15>(x);
}

// is x (a sum of squares, >= 0) so small or so large that the reflector's scalars may leave the
// type's range (also true for a NaN)?  One unsigned comparison of the upper bits.
__device__ __forceinline__ bool extreme(float x)     // outside [2^-100, 2^120]
{
    constexpr unsigned lo = (127u - 100u) << 23, hi = (127u + 120u) << 23;
    return __builtin_bit_cast(unsigned, x) - lo > hi - lo;
}
__device__ __forceinline__ bool extreme(double x)    // outside [2^-960, 2^1016]
{
    constexpr unsigned lo = (1023u - 960u) << 20, hi = (1023u + 1016u) << 20;
    return (unsigned)(__builtin_bit_cast(unsigned long long, x) >> 32) - lo > hi - lo;
}

__device__ __forceinline__ int exponent_of(float x) { return __builtin_amdgcn_frexp_expf(x); }
__device__ __forceinline__ int exponent_of(double x) { return __builtin_amdgcn_frexp_exp(x); }

// reflect_line (below) for a pivot whose sum of squares leaves the type's range: the pivot scaled
// by a power of two (H depends on its direction only), the lines themselves as they are.
template <typename C, int D>
__device__ __forceinline__ void extreme_line(C (&a)[D], C (&p)[D], bool pivot)
{
    C big = 0;
#pragma unroll
    for (int k = 0; k < D; ++k) big = fmax(big, fabs(p[k]));
    const int ex = big == (C)0 ? 0 : exponent_of(big);
    C ss = 0, q = 0;
#pragma unroll
    for (int k = 1; k < D; ++k) {
        p[k] = ldexp(p[k], -ex);         // below 1
        ss = fma(p[k], p[k], ss);
        q = fma(p[k], a[k], q);
    }
    const C al = ldexp(p[0], -ex);
    const C beta = copysign(sqrt(fma(al, al, ss)), -al), den = al - beta;
    const bool ident = ss == (C)0;
    const C w = ident ? (C)0 : fma(den, a[0], q) / ((C)0.5 * fma(den, den, ss));
    const C first = ident ? a[0] : ldexp(beta, ex);
    a[0] = pivot ? first : fma(-den, w, a[0]);
#pragma unroll
    for (int k = 1; k < D; ++k) a[k] = pivot ? (C)0 : fma(-w, p[k], a[k]);
}

// The reflector of the pivot line p applied to this lane's line a; on the lane that holds the
// pivot itself (pivot: a = p) the line becomes (beta, 0, ..).  H = I - g u u^T with u = (den, tail),
// den = alpha - beta, g = 2 / u^T u: orthogonal to working precision whatever the rounding of
// beta, and with no division but g's reciprocal.  A zero tail gives H = I, exactly.  Returns the
// mask of lanes whose pivot's sum of squares was of extreme size (their lines are then undefined:
// extreme_line on a fresh copy).
template <typename C, int D>
__device__ __forceinline__ unsigned long long reflect_line(C (&a)[D], const C (&p)[D], bool pivot)
{
    C sa = p[1] * p[1], sb = p[2] * p[2];
#pragma unroll
    for (int k = 3; k < D; ++k) {
        if (k & 1) sa = fma(p[k], p[k], sa);
        else sb = fma(p[k], p[k], sb);
    }
    const C alpha = p[0], ss = sa + sb, x2 = fma(alpha, alpha, ss);
    // (formed here, long before the branch that reads it: a branch right behind the comparison
    // it depends on costs some 50 cycles)
    unsigned long long ext = __builtin_amdgcn_ballot_w64(extreme(x2));
    const bool ident = ss == (C)0;
    ext &= ~__builtin_amdgcn_ballot_w64(ident);
    const bool keep = ident || pivot;
    asm volatile("" : "+s"(ext));
    const C beta = copysign(newton_sqrt(x2), -alpha);
    const C den = alpha - beta;
    const C g = newton_rcp(fma(den, den, ss));       // half of g
    const C kept = pivot ? (ident ? alpha : beta) : a[0];
    C da = p[1] * a[1], db = p[2] * a[2];
#pragma unroll
    for (int k = 3; k < D; ++k) {
        if (k & 1) da = fma(p[k], a[k], da);
        else db = fma(p[k], a[k], db);
    }
    const C q = fma(den, a[0], da) + db;
    // the multiple of u taken off this line: none for H = I; on the pivot's lane a = p, and
    // a - 1 * a = 0 exactly
    const C w = keep ? (pivot ? (C)1 : (C)0) : (q + q) * g;
    a[0] = keep ? kept : fma(-den, w, a[0]);     // (H = I also where everything is zero and den a NaN)
#pragma unroll
    for (int k = 1; k < D; ++k) a[k] = fma(-w, p[k], a[k]);
    return ext;
}

// Shape of a bundle: NW sweeps, four per compute wave, two traffic waves behind them; ring of WC
// columns, column c of the bundle (counted from its first) at ring index (c + RING0) mod WC.  The ring has
// 8 columns in front and 16 behind: the first 8 columns are mirrored behind the end, so that the
// 8 columns of a right reflector lie side by side wherever they start; what its mirrored write
// adds around them is never read.  Behind that: zeros, on which sweeps work that have not begun.
// (A bundle's first column sits at ring index RING0: its begin is clear of the ring's ends.)
template <int NW_, int WC_> struct NarrowShape {
    static constexpr int NW = NW_, WC = WC_, D = 8, RS = 3 * D;
    static constexpr int WAVES = NW / 4, NT = (WAVES + 2) * kWave;
    static constexpr int RING0 = 64;
    static constexpr int IDLE = (WC + 16) * RS, NIDLE = 16 * RS + 2 * D;   // the zeros
    static constexpr int ELEMS = 8 * RS + IDLE + NIDLE;
    // columns past the matrix that the last steps of a wave touch: sweeps of a wave that have ended go
    // on (on zero columns, with H = I) until its last one has
    static constexpr int PAST = 6 * D + 3 * D;
    // a wave follows its predecessor at 18 half steps at best, so the columns between the first wave's
    // front (17 ahead of its step) and the last sweep's back span at least 9 - NW + 64 WAVES; two units
    // of 8 for the traffic waves' granularity on top have to fit (more lets the waves drift apart)
    static_assert(9 - NW + 64 * WAVES + 16 <= WC && WC % 8 == 0 && NW % 8 == 0, "ring too small");
};

template <typename C, typename SH>
__global__ __launch_bounds__(SH::NT) void chase_narrow_kernel(C* __restrict__ band, int64_t ldab, int64_t ku,
                                                              int64_t n, int* __restrict__ ctrl,
                                                              int* __restrict__ flushed, int stride, int spin_limit)
{
    constexpr int D = SH::D, RS = SH::RS, NW = SH::NW, WC = SH::WC, WAVES = SH::WAVES;
    constexpr int UNITS = sizeof(C) == 8 ? 4 : 8;   // units of 8 columns a traffic wave moves at a time, at most
    constexpr int PER = D * RS / kWave;      // elements of a unit per lane
    extern __shared__ __align__(16) unsigned char smem_raw[];
    C* win = reinterpret_cast<C*>(smem_raw) + 8 * RS;
    __shared__ int sh_b, sh_fail;
    // progress in half steps: [0] columns brought in, counted as the half steps of the first wave they
    // allow; [1 + j] half steps wave j has completed.  Wave j may run its half step S once [j] >= S + 16
    // (a wave's 64 lanes write 64 copies: no lane mask, no bank conflict)
    __shared__ int sh_prog[WAVES + 1][kWave];
    __shared__ int sh_freed;                 // columns written back (the ring's space behind them is free)
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t nsweeps = n - 2;                         // sweeps 0 .. n-3
    const int64_t nbundles = (nsweeps + NW - 1) / NW;
    for (int e = tid; e < SH::NIDLE; e += SH::NT) win[SH::IDLE + e] = (C)0;

    for (;;) {
        if (tid == 0) {
            sh_b = atomicAdd(&ctrl[0], 1);
            sh_fail = __hip_atomic_load(&ctrl[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            sh_freed = 0;
        }
        if (wv <= WAVES) sh_prog[wv][lane] = 0;
        __syncthreads();
        const int64_t b = __builtin_amdgcn_readfirstlane(sh_b);   // (a scalar, and all that follows from it)
        if (b >= nbundles) break;
        const int64_t i0 = b * NW;
        const int ncols = (int)(n - i0);                   // columns of the bundle inside the matrix
        const int nunits = (ncols + SH::PAST + D - 1) / D; // units brought in (zeros past the matrix)

        if (wv < WAVES) {
            // ---- compute wave: sweeps 4 wv + g, g = lane / 16, group g running 4g half steps behind group 0
            const int sub = lane & 15, grp = lane >> 4;
            const int left = ncols - 3 - 4 * wv;           // sweeps from this wave's first to the matrix's last
            int smax = 0;                                  // half steps of this wave
            for (int g = 0; g < 4; ++g) smax = max(smax, left >= g ? 4 * g + 2 * ((left - g) / D + 1) : 0);
            // ring offset of column c0 of the group's current step, once it has begun
            constexpr int RING = WC * RS;
            int off = SH::IDLE, inc = 0;
            // waits until the predecessor's progress is `need`; false if the bundle has failed
            auto follow = [&](int need) -> bool {
                for (;;) {
                    // (both are waited for in here: nothing is outstanding where the fast path goes on)
                    const int now = __builtin_amdgcn_readfirstlane(lds_get(&sh_prog[wv][0]));
                    const int bad = __builtin_amdgcn_readfirstlane(lds_get(&sh_fail));
                    if (now >= need) return true;
                    if (bad) return false;
                }
            };
            int seen = 0;   // the predecessor's progress, read ahead with the lines of the half step before
            C x = 0;        // lanes 8 .. 15 of a row: the next half step's pivot
            const unsigned long long lanes0 = 0x0001000100010001ull;
            // One step (both half steps) of the four sweeps.  piv: the lanes that hold the right
            // reflector's pivot.  WRAP: some sweep is near the ends of the ring.  A sweep that has not begun
            // works on zeros, one that has ended on the zero columns behind the matrix (H = I).
            auto step = [&](int S, unsigned long long piv, auto wrap_c) {
                constexpr bool WRAP = decltype(wrap_c)::value;
                C a[D], p[D];
                auto redo = [&](C* base, int es, bool pivot) {   // (rare) from the lines as they still are in LDS
#pragma unroll
                    for (int k = 0; k < D; ++k) a[k] = base[k * es];
                    extreme_line<C, D>(a, p, pivot);
                };
                // -- right reflector: lane = row c0 - 8 + sub
                C* base = win + off + sub + (D - 1);
#pragma unroll
                for (int k = 0; k < D; ++k) a[k] = base[k * (RS - 1)];
                row_pivot(x, p);
                bool pivot = __builtin_amdgcn_inverse_ballot_w64(piv);
                unsigned long long ext = reflect_line<C, D>(a, p, pivot);
                if (__builtin_expect(ext != 0, 0)) {
                    if (ext >> lane & 1) redo(base, RS - 1, pivot);
                }
                if (WRAP) {
                    // columns among the ring's first 8, or past its end: the other copy as well
                    C* other = base + (off < D * RS ? RING : off > RING - D * RS && off < RING ? -RING : 0);
#pragma unroll
                    for (int k = 0; k < D; ++k) other[k * (RS - 1)] = a[k];
                }
#pragma unroll
                for (int k = 0; k < D; ++k) base[k * (RS - 1)] = a[k];
                x = a[0];   // rows c0 .. c0 + 7 of column c0: the left reflector's pivot
                order_lds();
                // -- left reflector: lane = column c0 + sub, pivot on lane 0
                const int ahead = lds_get(&sh_prog[wv][0]);
                int oc = off + sub * RS;
                if (WRAP) oc = oc >= RING && off < RING ? oc - RING : oc;
                base = win + oc + 2 * D - 1 - sub;
#pragma unroll
                for (int k = 0; k < D; ++k) a[k] = base[k];
                row_pivot(x, p);
                pivot = sub == 0;
                ext = reflect_line<C, D>(a, p, pivot);
                seen = __builtin_amdgcn_readfirstlane(ahead);            // (here: waits for no write)
                if (__builtin_expect(ext != 0, 0)) {
                    if (ext >> lane & 1) redo(base, 1, pivot);
                }
                if (WRAP) {
                    C* other = base + (oc < D * RS ? RING : 0);
#pragma unroll
                    for (int k = 0; k < D; ++k) other[k] = a[k];
                }
#pragma unroll
                for (int k = 0; k < D; ++k) base[k] = a[k];
                x = a[0];   // row c0 of columns c0 + 8 .. c0 + 15: the next step's pivot
                order_lds();
                lds_set(&sh_prog[wv + 1][lane], S + 2);
                off += inc;
                if (WRAP) off = off >= RING && inc != 0 ? off - RING : off;
            };
            // Steps S .. end - 2, the first with the pivot lanes piv; false if the bundle has failed.
            auto run = [&](int S, int end, unsigned long long piv, auto wrap_c) -> bool {
                for (; S < end; S += 2) {
                    if (__builtin_expect(seen < S + 17, 0)) {
                        if (!follow(S + 17)) return false;
                    }
                    order_lds();
                    step(S, piv, wrap_c);
                    piv = lanes0;
                }
                return true;
            };
            // Every step of every wave has to keep the same pace: the next wave follows ten steps behind, so
            // ten slow steps in a row anywhere (the begin, the ring's ends) set the rate at which bundles
            // follow each other.  So the steps run in a few long loops, with what is special between them.
            bool good = true;
            int ring = SH::RING0 + 4 * wv + 1;   // ring index of the first sweep's column (the others: 15, 30, 45 behind)
            for (int S = 0; S < smax && good;) {
                unsigned long long piv = lanes0;
                int end = smax;
                if (S < 16) {
                    // a sweep begins: its first pivot is row c0 - 1 (lane 7; the rows above it are zero in these
                    // columns) and comes from LDS
                    if (__builtin_expect(seen < S + 17, 0)) {
                        if (!follow(S + 17)) break;
                    }
                    order_lds();
                    piv += 0x7full << (4 * S);
                    const bool begins = grp == S >> 2;
                    off = begins ? (SH::RING0 + 4 * wv + grp + 1) * RS : off;
                    inc = begins ? D * RS : inc;
                    const C y = win[off + (sub & 7) * (RS - 1) + 2 * D - 2];
                    x = begins ? y : x;
                    end = min(end, S + 4);
                }
                const bool plain = ring >= 45 + D && ring <= WC - 2 * D;
                const int room = plain ? (WC - 2 * D - ring) / D + 1
                                       : (45 + 2 * D - 1 - (ring >= 45 + D ? ring - WC : ring)) / D;
                end = min(end, S + 2 * room);
                if (plain) good = run(S, end, piv, std::false_type{});
                else good = run(S, end, piv, std::true_type{});
                ring += (end - S) / 2 * D;
                ring = ring >= WC ? ring - WC : ring;
                S = end;
            }
            // finished once the predecessor is (a wave without sweeps only passes that on)
            if (good && follow(kAllDone)) lds_set(&sh_prog[wv + 1][lane], kAllDone);
        } else {
            // ---- traffic waves (ahead of the compute waves on their SIMD: short work that others wait for)
            __builtin_amdgcn_s_setprio(3);
            // element q of a unit held by this lane: column ucol[q], storage row urow[q] (row 23 is padding)
            int ucol[PER], urow[PER];
            C* first[PER];                       // band entry of element q of unit 0
#pragma unroll
            for (int q = 0; q < PER; ++q) {
                const int e = lane + q * kWave;
                ucol[q] = e / RS;
                urow[q] = e % RS;
                first[q] = band + (urow[q] - (2 * D - 1) + ku) + (i0 + ucol[q]) * ldab;
            }
            // are all entries of units u .. u + nu - 1 inside the matrix; is element q of unit u
            auto interior = [&](int u, int nu) -> bool { return i0 + (int64_t)u * D >= 2 * D - 1 && (u + nu + 1) * D <= ncols; };
            auto inside = [&](int u, int q) -> bool {
                const int j = u * D + ucol[q];
                const int64_t i = i0 + j + urow[q] - (2 * D - 1);
                return urow[q] < RS - 1 && j < ncols && i >= 0 && i < n;
            };
            const int64_t ustep = D * ldab;
            if (wv == WAVES) {
                // ---- loader
                int u = 0, seen = b > 0 ? 0 : kAllFlushed, spins = 0;
                while (u < nunits) {
                    // room in the ring, and columns the previous bundle has finished
                    const int room = (__builtin_amdgcn_readfirstlane(lds_get(&sh_freed)) + WC) / D - u;
                    const int have = seen >= n ? nunits : (int)((seen - i0) / D);
                    const int nu = min(min(have, nunits) - u, min(room, UNITS));
                    if (nu <= 0) {
                        if (__builtin_amdgcn_readfirstlane(lds_get(&sh_fail))) break;
                        if (room > 0) {
                            seen = __builtin_amdgcn_readfirstlane(
                                __hip_atomic_load(&flushed[(b - 1) * stride], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
                            if (seen < n && (seen - i0) / D <= u) {
                                // the wait for the previous bundle is bounded
                                if (++spins > spin_limit) {
                                    if (lane == 0) { atomicExch(&ctrl[1], 1); lds_set(&sh_fail, 1); }
                                    break;
                                }
                                __builtin_amdgcn_s_sleep(1);
                            }
                        } else {
                            __builtin_amdgcn_s_sleep(4);
                        }
                        continue;
                    }
                    spins = 0;
                    C v[UNITS][PER];
                    if (interior(u, nu)) {
#pragma unroll
                        for (int x = 0; x < UNITS; ++x)
                            if (x < nu) {
#pragma unroll
                                for (int q = 0; q < PER; ++q) v[x][q] = ngld(first[q] + (u + x) * ustep);
                            }
                    } else {
#pragma unroll
                        for (int x = 0; x < UNITS; ++x)
                            if (x < nu) {
#pragma unroll
                                for (int q = 0; q < PER; ++q) v[x][q] = inside(u + x, q) ? ngld(first[q] + (u + x) * ustep) : (C)0;
                            }
                    }
                    // (the next answer of the previous bundle travels with the columns)
                    if (seen < n)
                        seen = __hip_atomic_load(&flushed[(b - 1) * stride], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                    for (int x = 0; x < UNITS; ++x)
                        if (x < nu) {
                            const int ring = (SH::RING0 + (u + x) * D) % WC;
#pragma unroll
                            for (int q = 0; q < PER; ++q) {
                                win[ring * RS + lane + q * kWave] = v[x][q];
                                if (ring == 0) win[WC * RS + lane + q * kWave] = v[x][q];
                            }
                        }
                    seen = __builtin_amdgcn_readfirstlane(seen);
                    u += nu;
                    order_lds();
                    // half step S of the first wave touches the columns below 8 (S / 2) + 17
                    const int cols = u * D;
                    lds_set(&sh_prog[0][lane], u == nunits ? kAllDone : (cols >= 17 ? 2 * ((cols - 17) / D) + 17 : 0));
                }
            } else {
                // ---- writer: columns below the last sweep's current step are final
                int u = 0;
                const int last = (ncols + D - 1) / D;
                while (u < last) {
                    const int done = __builtin_amdgcn_readfirstlane(lds_get(&sh_prog[WAVES][0]));
                    order_lds();
                    const int fin = done >= kAllDone ? last : (done < 12 ? 0 : NW / D + ((done - 12) >> 1));
                    const int nu = min(min(fin, last) - u, UNITS);
                    if (nu <= 0) {
                        if (__builtin_amdgcn_readfirstlane(lds_get(&sh_fail))) break;
                        __builtin_amdgcn_s_sleep(1);
                        continue;
                    }
                    C v[UNITS][PER];
#pragma unroll
                    for (int x = 0; x < UNITS; ++x)
                        if (x < nu) {
                            const int ring = (SH::RING0 + (u + x) * D) % WC;
#pragma unroll
                            for (int q = 0; q < PER; ++q) v[x][q] = win[ring * RS + lane + q * kWave];
                        }
                    if (interior(u, nu)) {
#pragma unroll
                        for (int x = 0; x < UNITS; ++x)
                            if (x < nu) {
#pragma unroll
                                for (int q = 0; q < PER; ++q)
                                    if (urow[q] < RS - 1) ngst(first[q] + (u + x) * ustep, v[x][q]);
                            }
                    } else {
#pragma unroll
                        for (int x = 0; x < UNITS; ++x)
                            if (x < nu) {
#pragma unroll
                                for (int q = 0; q < PER; ++q)
                                    if (inside(u + x, q)) ngst(first[q] + (u + x) * ustep, v[x][q]);
                            }
                    }
                    u += nu;
                    order_lds();
                    if (lane == 0) lds_set(&sh_freed, u * D);
                    // the stores are device-scope atomics: once acknowledged (vmcnt = 0) they are visible
                    // to every workgroup, no cache write-back is needed
                    __builtin_amdgcn_s_waitcnt(0x0f70);
                    order_lds();
                    if (lane == 0)
                        __hip_atomic_store(&flushed[b * stride], u == last ? kAllFlushed : (int)(i0 + u * D), __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
                }
                // (also when a wait has expired: the next bundle must not wait for this one)
                if (lane == 0)
                    __hip_atomic_store(&flushed[b * stride], kAllFlushed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            __builtin_amdgcn_s_setprio(0);
        }
        __syncthreads();
    }
}

__global__ __launch_bounds__(256) void narrow_clear_kernel(int* __restrict__ p, int64_t np, int* __restrict__ q, int64_t nq)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < np + nq; i += (int64_t)gridDim.x * blockDim.x)
        (i < np ? p[i] : q[i - np]) = 0;
}

}  // namespace

// ctrl: 64 ints (ticket, error flag) followed by one flushed counter per bundle, unless the caller has room to keep
// these apart (`spread`, 8 ints a bundle): one bundle polls while another writes beside it
size_t chase_narrow_workspace_bytes(int64_t n) { return (size_t)(64 + n / 8 + 8) * sizeof(int); }

// Sweeps per bundle.  Latencies set the pace (measured: a plain vector instruction 5 cycles from the
// same wave, 8 if it needs the previous one's result, a branch on a vector comparison over 50), so one
// wave per SIMD runs a half step in about 470 cycles (f32), two in 600: small bundles keep a half
// step short, large ones spread the 6 us of a hand-over through device memory.  us per sweep with
// 16 / 24 / 32 sweeps, n = 256: f32 1.51 / 1.39 / 1.38, f64 1.73 / 1.65 / 1.66; n = 8192: f32
// 1.52 / 1.53 / 1.60, f64 1.95 / 2.32 / 2.42 (twice the issue slots per half step, so sharing a SIMD
// costs more).  The form before this one (48 sweeps in lock step behind workgroup barriers, pivots
// read from LDS, chunks of columns moved by the same waves) took 4.13 (f32) and 4.6 (f64).  The ring
// is what the waves of a bundle may drift apart: in f64 nearly all of LDS (704 columns, 143 KB), in f32 1024
// columns (102 KB), beyond which nothing is gained (1536 columns: 1.42 instead of 1.38 us at n = 256, 1.52
// instead of 1.53 at 8192).
template <typename C>
int run_chase_narrow(int64_t n, C* band, int64_t ldab, int64_t ku, int* ctrl, int* spread, hipStream_t s)
{
    using SH = std::conditional_t<sizeof(C) == 8, NarrowShape<16, 704>, NarrowShape<24, 1024>>;
    if (n < 3) return SVB_OK;
    const size_t smem = sizeof(C) * (size_t)SH::ELEMS;
    auto kern = chase_narrow_kernel<C, SH>;
    static bool attr_set = false;
    if (!attr_set) {
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        attr_set = true;
    }
    const int64_t nbundles = (n - 2 + SH::NW - 1) / SH::NW;
    int* const flushed = spread ? spread : ctrl + 64;
    const int stride = spread ? 8 : 1;
    const int64_t count = nbundles * stride;
    int cb = (int)((64 + count + 255) / 256);
    hipLaunchKernelGGL(narrow_clear_kernel, dim3(cb > 256 ? 256 : cb), dim3(256), 0, s, ctrl, (int64_t)64, flushed, count);
    const int grid = (int)min((int64_t)env_int("SVB_NARROW_GRID", 128), nbundles);
    const int spin_limit = env_int("SVB_CHASE_SPIN", 1 << 20);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(SH::NT), smem, s, band, ldab, ku, n, ctrl, flushed, stride, spin_limit);
    return hipGetLastError() == hipSuccess ? SVB_OK : SVB_ERR_DEVICE;
}

template int run_chase_narrow<double>(int64_t, double*, int64_t, int64_t, int*, int*, hipStream_t);
template int run_chase_narrow<float>(int64_t, float*, int64_t, int64_t, int*, int*, hipStream_t);

}  // namespace svb
