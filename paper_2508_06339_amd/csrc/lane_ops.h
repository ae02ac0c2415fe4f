// Lane-to-lane operations that stay in the vector registers (gfx950): broadcasts inside rows of 16
// lanes (data-parallel primitives) and swaps of lane groups.  A value fetched this way costs an
// instruction or two (5 cycles each) against 50 for a trip through LDS and 70 for a shuffle.
#pragma once

#include <hip/hip_runtime.h>
#include <utility>

namespace svb {

// value of lane K of this lane's row of 16
template <int K> __device__ __forceinline__ int row_lane(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, 0x150 + K, 0xF, 0xF, true);
}
// sum of the two rows of 16 of each half of the wave / of the two halves, in all of them (the two
// operands of a swap are the same register: it leaves the value and its partner's)
__device__ __forceinline__ float rows_sum(float v)
{
    const unsigned u = __builtin_bit_cast(unsigned, v);
    const auto t = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    const unsigned t0 = t[0], t1 = t[1];   // (a bit cast of t[1] itself would read t[0])
    const unsigned q = __builtin_bit_cast(unsigned, __builtin_bit_cast(float, t0) + __builtin_bit_cast(float, t1));
    const auto h = __builtin_amdgcn_permlane32_swap(q, q, false, false);
    const unsigned h0 = h[0], h1 = h[1];
    return __builtin_bit_cast(float, h0) + __builtin_bit_cast(float, h1);
}
struct Words { unsigned lo, hi; };
__device__ __forceinline__ double rows_sum(double v)
{
    const Words u = __builtin_bit_cast(Words, v);
    const auto a = __builtin_amdgcn_permlane16_swap(u.lo, u.lo, false, false);
    const auto b = __builtin_amdgcn_permlane16_swap(u.hi, u.hi, false, false);
    const double w = __builtin_bit_cast(double, Words{a[0], b[0]}) + __builtin_bit_cast(double, Words{a[1], b[1]});
    const Words q = __builtin_bit_cast(Words, w);
    const auto c = __builtin_amdgcn_permlane32_swap(q.lo, q.lo, false, false);
    const auto d = __builtin_amdgcn_permlane32_swap(q.hi, q.hi, false, false);
    return __builtin_bit_cast(double, Words{c[0], d[0]}) + __builtin_bit_cast(double, Words{c[1], d[1]});
}
// sums of a and of b over the four rows of 16 (for every position in a row), in all of them, and those of position
// K as scalars ak and bk, which are there first; the two travel through the swaps of row groups together
__device__ __forceinline__ float lane_value(float v, int lane)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}
template <int K> __device__ __forceinline__ void rows_sum2(float& a, float& b, float& ak, float& bk)
{
    const auto t = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, b), false, false);
    const unsigned t0 = t[0], t1 = t[1];   // rows a0 b0 a2 b2 and a1 b1 a3 b3
    const unsigned q = __builtin_bit_cast(unsigned, __builtin_bit_cast(float, t0) + __builtin_bit_cast(float, t1));
    const auto h = __builtin_amdgcn_permlane32_swap(q, q, false, false);
    const unsigned h0 = h[0], h1 = h[1];
    const float s = __builtin_bit_cast(float, h0) + __builtin_bit_cast(float, h1);   // rows a b a b
    ak = lane_value(s, K);
    bk = lane_value(s, 16 + K);
    const unsigned w = __builtin_bit_cast(unsigned, s);
    const auto f = __builtin_amdgcn_permlane16_swap(w, w, false, false);
    const unsigned f0 = f[0], f1 = f[1];
    a = __builtin_bit_cast(float, f0);
    b = __builtin_bit_cast(float, f1);
}
__device__ __forceinline__ double lane_value(double v, int lane)
{
    const Words u = __builtin_bit_cast(Words, v);
    return __builtin_bit_cast(double, Words{(unsigned)__builtin_amdgcn_readlane((int)u.lo, lane),
                                            (unsigned)__builtin_amdgcn_readlane((int)u.hi, lane)});
}
template <int K> __device__ __forceinline__ void rows_sum2(double& a, double& b, double& ak, double& bk)
{
    const Words u = __builtin_bit_cast(Words, a), v = __builtin_bit_cast(Words, b);
    const auto tl = __builtin_amdgcn_permlane16_swap(u.lo, v.lo, false, false);
    const auto th = __builtin_amdgcn_permlane16_swap(u.hi, v.hi, false, false);
    const Words q = __builtin_bit_cast(Words, __builtin_bit_cast(double, Words{tl[0], th[0]}) +
                                                  __builtin_bit_cast(double, Words{tl[1], th[1]}));
    const auto hl = __builtin_amdgcn_permlane32_swap(q.lo, q.lo, false, false);
    const auto hh = __builtin_amdgcn_permlane32_swap(q.hi, q.hi, false, false);
    const double s = __builtin_bit_cast(double, Words{hl[0], hh[0]}) + __builtin_bit_cast(double, Words{hl[1], hh[1]});
    ak = lane_value(s, K);
    bk = lane_value(s, 16 + K);
    const Words w = __builtin_bit_cast(Words, s);
    const auto fl = __builtin_amdgcn_permlane16_swap(w.lo, w.lo, false, false);
    const auto fh = __builtin_amdgcn_permlane16_swap(w.hi, w.hi, false, false);
    a = __builtin_bit_cast(double, Words{fl[0], fh[0]});
    b = __builtin_bit_cast(double, Words{fl[1], fh[1]});
}
// a number that orders as |x| does: for a double its upper word, read as a float (two of them a maximum
// instruction takes, and it needs no quieting; above 2^1017 it is a NaN, which a maximum passes over)
__device__ __forceinline__ float magnitude(float x) { return fabsf(x); }
__device__ __forceinline__ float magnitude(double x)
{
    return fabsf(__builtin_bit_cast(float, (unsigned)(__builtin_bit_cast(unsigned long long, x) >> 32)));
}
// maximum over the lanes that agree in the lower four bits of their number (four of them), in all of them
__device__ __forceinline__ float rows_max(float v)
{
    const unsigned u = __builtin_bit_cast(unsigned, v);
    const auto t = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    const unsigned t0 = t[0], t1 = t[1];
    const unsigned q = __builtin_bit_cast(unsigned, fmaxf(__builtin_bit_cast(float, t0), __builtin_bit_cast(float, t1)));
    const auto h = __builtin_amdgcn_permlane32_swap(q, q, false, false);
    const unsigned h0 = h[0], h1 = h[1];
    return fmaxf(__builtin_bit_cast(float, h0), __builtin_bit_cast(float, h1));
}
// bitwise or over the lanes that agree in the lower four bits of their number (four of them), in all of them
__device__ __forceinline__ unsigned rows_or(unsigned v)
{
    const auto t = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    const unsigned q = t[0] | t[1];
    const auto h = __builtin_amdgcn_permlane32_swap(q, q, false, false);
    return h[0] | h[1];
}
template <int K> __device__ __forceinline__ float row_lane(float v)
{
    return __builtin_bit_cast(float, row_lane<K>(__builtin_bit_cast(int, v)));
}
template <int K> __device__ __forceinline__ double row_lane(double v)
{
    const Words u = __builtin_bit_cast(Words, v);
    return __builtin_bit_cast(double, Words{(unsigned)row_lane<K>((int)u.lo), (unsigned)row_lane<K>((int)u.hi)});
}


// Multiply-adds whose first factor is the value of lane K of the lane's row of sixteen, taken as the operand is
// read: p[i mod 4] = sum of row_lane<K>(x[i]) x[i], and x[i] += row_lane<K>(x[i]) w.  (The compiler makes a move
// and a multiply-add of these.  An operand that is read across lanes may not have been written by the last two
// vector instructions: two wait states in front; inside a group of eight nothing that was written is read so.  The
// compiler does not see what a group writes, so behind it the caller has to keep the same distance: the results go
// through an ordinary vector instruction or another of these groups before a lane operation (permlane, readlane, a
// data-parallel move) reads them.)
#define SVB_BCAST " row_mask:0xf bank_mask:0xf\n\t"
#define SVB_DOT8(T, FIRST, C0)                                                                             \
    asm("s_nop 1\n\t"                                                                                      \
        FIRST T "_dpp %0, %4, %4 row_newbcast:%12" SVB_BCAST                                               \
        FIRST T "_dpp %1, %5, %5 row_newbcast:%12" SVB_BCAST                                               \
        FIRST T "_dpp %2, %6, %6 row_newbcast:%12" SVB_BCAST                                               \
        FIRST T "_dpp %3, %7, %7 row_newbcast:%12" SVB_BCAST                                               \
        "v_fmac_" T "_dpp %0, %8, %8 row_newbcast:%12" SVB_BCAST                                           \
        "v_fmac_" T "_dpp %1, %9, %9 row_newbcast:%12" SVB_BCAST                                           \
        "v_fmac_" T "_dpp %2, %10, %10 row_newbcast:%12" SVB_BCAST                                         \
        "v_fmac_" T "_dpp %3, %11, %11 row_newbcast:%12 row_mask:0xf bank_mask:0xf"                        \
        : C0(p[0]), C0(p[1]), C0(p[2]), C0(p[3])                                                           \
        : "v"(x[i]), "v"(x[i + 1]), "v"(x[i + 2]), "v"(x[i + 3]), "v"(x[i + 4]), "v"(x[i + 5]),            \
          "v"(x[i + 6]), "v"(x[i + 7]), "n"(K))
#define SVB_AXPY8(T)                                                                                       \
    asm("s_nop 1\n\t"                                                                                      \
        "v_fmac_" T "_dpp %0, %0, %8 row_newbcast:%9" SVB_BCAST                                            \
        "v_fmac_" T "_dpp %1, %1, %8 row_newbcast:%9" SVB_BCAST                                            \
        "v_fmac_" T "_dpp %2, %2, %8 row_newbcast:%9" SVB_BCAST                                            \
        "v_fmac_" T "_dpp %3, %3, %8 row_newbcast:%9" SVB_BCAST                                            \
        "v_fmac_" T "_dpp %4, %4, %8 row_newbcast:%9" SVB_BCAST                                            \
        "v_fmac_" T "_dpp %5, %5, %8 row_newbcast:%9" SVB_BCAST                                            \
        "v_fmac_" T "_dpp %6, %6, %8 row_newbcast:%9" SVB_BCAST                                            \
        "v_fmac_" T "_dpp %7, %7, %8 row_newbcast:%9 row_mask:0xf bank_mask:0xf"                           \
        : "+v"(x[i]), "+v"(x[i + 1]), "+v"(x[i + 2]), "+v"(x[i + 3]), "+v"(x[i + 4]), "+v"(x[i + 5]),      \
          "+v"(x[i + 6]), "+v"(x[i + 7])                                                                   \
        : "v"(w), "n"(K))
// acc[j] += row_lane<K>(c[j]) t, j = K + 1 .. 7
#define SVB_COL1(T, A, B) "v_fmac_" T "_dpp %" #A ", %" #B ", %14 row_newbcast:%15" SVB_BCAST
#define SVB_COL7(T)                                                                                        \
    if constexpr (K == 0)                                                                                  \
        asm("s_nop 1\n\t" SVB_COL1(T, 0, 7) SVB_COL1(T, 1, 8) SVB_COL1(T, 2, 9) SVB_COL1(T, 3, 10) SVB_COL1(T, 4, 11) SVB_COL1(T, 5, 12) SVB_COL1(T, 6, 13) SVB_COL_ARGS); \
    if constexpr (K == 1)                                                                                  \
        asm("s_nop 1\n\t" SVB_COL1(T, 1, 8) SVB_COL1(T, 2, 9) SVB_COL1(T, 3, 10) SVB_COL1(T, 4, 11) SVB_COL1(T, 5, 12) SVB_COL1(T, 6, 13) SVB_COL_ARGS); \
    if constexpr (K == 2)                                                                                  \
        asm("s_nop 1\n\t" SVB_COL1(T, 2, 9) SVB_COL1(T, 3, 10) SVB_COL1(T, 4, 11) SVB_COL1(T, 5, 12) SVB_COL1(T, 6, 13) SVB_COL_ARGS); \
    if constexpr (K == 3)                                                                                  \
        asm("s_nop 1\n\t" SVB_COL1(T, 3, 10) SVB_COL1(T, 4, 11) SVB_COL1(T, 5, 12) SVB_COL1(T, 6, 13) SVB_COL_ARGS); \
    if constexpr (K == 4)                                                                                  \
        asm("s_nop 1\n\t" SVB_COL1(T, 4, 11) SVB_COL1(T, 5, 12) SVB_COL1(T, 6, 13) SVB_COL_ARGS);          \
    if constexpr (K == 5) asm("s_nop 1\n\t" SVB_COL1(T, 5, 12) SVB_COL1(T, 6, 13) SVB_COL_ARGS);           \
    if constexpr (K == 6) asm("s_nop 1\n\t" SVB_COL1(T, 6, 13) SVB_COL_ARGS)
#define SVB_COL_ARGS                                                                                       \
    : "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3]), "+v"(acc[4]), "+v"(acc[5]), "+v"(acc[6]), "+v"(acc[7])     \
    : "v"(c[1]), "v"(c[2]), "v"(c[3]), "v"(c[4]), "v"(c[5]), "v"(c[6]), "v"(c[7]), "v"(t), "n"(K)
template <int K> __device__ __forceinline__ void row_lane_columns(float (&acc)[8], const float (&c)[8], float t)
{
    SVB_COL7("f32");
}
template <int K> __device__ __forceinline__ void row_lane_columns(double (&acc)[8], const double (&c)[8], double t)
{
    SVB_COL7("f64");
}
template <int K, int N> __device__ __forceinline__ void row_lane_dot(const float (&x)[N], float (&p)[4])
{
    static_assert(N % 8 == 0, "groups of eight");
#pragma unroll
    for (int i = 0; i < N; i += 8) {
        if (i == 0) SVB_DOT8("f32", "v_mul_", "=&v");
        else SVB_DOT8("f32", "v_fmac_", "+v");
    }
}
template <int K, int N> __device__ __forceinline__ void row_lane_dot(const double (&x)[N], double (&p)[4])
{
    static_assert(N % 8 == 0, "groups of eight");
#pragma unroll
    for (int i = 0; i < 4; ++i) p[i] = 0;
#pragma unroll
    for (int i = 0; i < N; i += 8) SVB_DOT8("f64", "v_fmac_", "+v");
}
template <int K, int N> __device__ __forceinline__ void row_lane_axpy(float (&x)[N], float w)
{
    static_assert(N % 8 == 0, "groups of eight");
#pragma unroll
    for (int i = 0; i < N; i += 8) SVB_AXPY8("f32");
}
template <int K, int N> __device__ __forceinline__ void row_lane_axpy(double (&x)[N], double w)
{
    static_assert(N % 8 == 0, "groups of eight");
#pragma unroll
    for (int i = 0; i < N; i += 8) SVB_AXPY8("f64");
}
#undef SVB_DOT8
#undef SVB_AXPY8
#undef SVB_COL1
#undef SVB_COL7
#undef SVB_COL_ARGS
#undef SVB_BCAST

// swap of a's upper half with b's lower half / of the odd rows of sixteen lanes of a with the even rows of b
__device__ __forceinline__ void swap_halves(float& a, float& b)
{
    const auto t = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, b), false, false);
    const unsigned t0 = t[0], t1 = t[1];
    a = __builtin_bit_cast(float, t0);
    b = __builtin_bit_cast(float, t1);
}
__device__ __forceinline__ void swap_rows(float& a, float& b)
{
    const auto t = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, b), false, false);
    const unsigned t0 = t[0], t1 = t[1];
    a = __builtin_bit_cast(float, t0);
    b = __builtin_bit_cast(float, t1);
}
__device__ __forceinline__ void swap_halves(double& a, double& b)
{
    const Words u = __builtin_bit_cast(Words, a), v = __builtin_bit_cast(Words, b);
    const auto l = __builtin_amdgcn_permlane32_swap(u.lo, v.lo, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(u.hi, v.hi, false, false);
    a = __builtin_bit_cast(double, Words{l[0], h[0]});
    b = __builtin_bit_cast(double, Words{l[1], h[1]});
}
__device__ __forceinline__ void swap_rows(double& a, double& b)
{
    const Words u = __builtin_bit_cast(Words, a), v = __builtin_bit_cast(Words, b);
    const auto l = __builtin_amdgcn_permlane16_swap(u.lo, v.lo, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(u.hi, v.hi, false, false);
    a = __builtin_bit_cast(double, Words{l[0], h[0]});
    b = __builtin_bit_cast(double, Words{l[1], h[1]});
}
template <int CTRL> __device__ __forceinline__ float dpp(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
template <int CTRL> __device__ __forceinline__ double dpp(double v)
{
    const Words u = __builtin_bit_cast(Words, v);
    return __builtin_bit_cast(double, Words{(unsigned)__builtin_amdgcn_update_dpp(0, (int)u.lo, CTRL, 0xF, 0xF, true),
                                            (unsigned)__builtin_amdgcn_update_dpp(0, (int)u.hi, CTRL, 0xF, 0xF, true)});
}
constexpr int kRor8 = 0x128, kHalfMirror = 0x141, kSwap2 = 0x4E, kSwap1 = 0xB1;   // row_ror:8, row_half_mirror, quad_perm
// sum over the wave in every lane
template <typename C> __device__ __forceinline__ C wave_sum(C v)
{
    v = rows_sum(v);
    v += dpp<kRor8>(v);
    v += dpp<kHalfMirror>(v);
    v += dpp<kSwap2>(v);
    return v + dpp<kSwap1>(v);
}

// f(integral constant 0), f(integral constant 1), .., f(integral constant N - 1)
template <typename Fn, int... K> __device__ __forceinline__ void unrolled(Fn&& f, std::integer_sequence<int, K...>)
{
    (f(std::integral_constant<int, K>{}), ...);
}
template <int N, typename Fn> __device__ __forceinline__ void unroll(Fn&& f)
{
    unrolled(f, std::make_integer_sequence<int, N>{});
}

// workgroup barrier that orders LDS traffic only (s_waitcnt lgkmcnt(0); gfx9 encoding: vmcnt = 63, expcnt = 7,
// lgkmcnt = 0): global accesses stay in flight
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_s_waitcnt(0xc07f);
    __builtin_amdgcn_s_barrier();
}

}  // namespace svb
