// Line diffusion on the matrix cores.
//
// The one-dimensional diffusion exp(h d^2/dx^2) of Eq. (5) on a line of N
// points is a real symmetric matrix, the same for the real and the imaginary
// parts, so many lines at once are a matrix product: a wavefront holds N rows
// (the points of the line) by 16 columns and multiplies them by the matrix
// with v_mfma_{f32,f64}_16x16x4.  Against the register transforms of fft.h
// this has no twiddles, no LDS exchange and no barrier inside a line, at the
// price of more arithmetic, on units that those transforms leave idle.
//
// Symmetry cuts the arithmetic.  The matrix of a periodic line depends on
// i - j only and is even, so it commutes with the shift by N/2 and with the
// reflection n -> N - 1 - n.  With x_n +- x_{n+N/2} it splits into two
// matrices of N/2 points (2 ways), and with the reflection of each into four
// of N/4 (4 ways): N multiplications per point instead of 4 N.  Between walls
// (reflecting or absorbing) the matrix depends on i - j and i + j and keeps the
// reflection only: halves.
//
// Layout.  A group is 16 lanes; the wavefront's four groups g hold the rows,
// lane % 16 is the column.  The product's result sits in the lanes and
// registers in which its operand did (the table of matrix entries is permuted
// to make it so), so diffusions chain without moving data.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "fft.h"

namespace pft {

// How a line of N points is split: `ways` independent matrices of S points
// each, R = S / 4 rows of each per group, in RB blocks of the 16-row product.
// The split with the fewest products: lengths whose quarter is a multiple of
// four rows go 4 ways, else halves, and up to 20 points one dense product of
// padded rows costs no more than two halves.
template <int N, bool WALL = false>
struct MSplit {
    static constexpr int ways = N <= 20 ? 1 : (!WALL && N % 16 == 0 && N >= 48) ? 4 : 2;
    static constexpr int S = N / ways;
    static_assert(S % 4 == 0, "rows must spread over the four groups");
    static constexpr int R = S / 4;
    static constexpr int RB = (R + 3) / 4;
    static constexpr int NR = N / 4;                       // rows a lane holds
    static constexpr int kSums = ways * RB * R * 64;       // walls: row sums follow the matrices
    static constexpr int kFrag = kSums + (WALL ? (S + 63) / 64 * 64 : 0);  // table entries
};

// Row of a sub-matrix that group g holds in its register rr, chosen by the
// accesses along a contiguous line.  Complex float: R consecutive points per
// lane (64 points in complex float: z pass 9.4 us; eight consecutive points over
// the groups per instruction, as below, 16.8 us).  Complex double: register
// pairs of consecutive points, the groups side by side, eight points (128
// bytes) per instruction; an odd last register takes the four rows left (z pass
// of 64 points 13.7 us with four points per instruction, 11.2 us with eight).
template <typename T>
__host__ __device__ constexpr int mrow(int g, int rr, int R)
{
    return sizeof(T) == 4 ? g * R + rr : rr < R / 2 * 2 ? 8 * (rr / 2) + 2 * g + rr % 2 : 4 * rr + g;
}
// The point of the line that sub-vector t holds in row m.
template <int N, bool WALL = false>
__host__ __device__ constexpr int mpoint(int t, int m)
{
    constexpr int W = MSplit<N, WALL>::ways;
    if (WALL && W == 2) return t == 0 ? m : N - 1 - m;
    if (W == 4) return t == 0 ? m : t == 1 ? N / 2 - 1 - m : t == 2 ? N / 2 + m : N - 1 - m;
    if (W == 2) return t == 0 ? m : N / 2 + m;
    return m;
}

// Whether sub-vector t runs against the line's direction.
template <int N, bool WALL = false>
constexpr bool mreversed(int t)
{
    return MSplit<N, WALL>::ways == 4 ? t % 2 == 1 : WALL && t == 1;
}

using mf4 = float __attribute__((ext_vector_type(4)));
using md4 = double __attribute__((ext_vector_type(4)));

template <typename T>
using macc = std::conditional_t<sizeof(T) == 4, mf4, md4>;

__device__ __forceinline__ mf4 mprod(float a, float b, mf4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
__device__ __forceinline__ md4 mprod(double a, double b, md4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }

// Sums and differences that split the line, and their inverse (scale in the table).
template <int N, bool WALL, typename T>
__device__ __forceinline__ void msplit(T (&x)[N / 4])
{
    using M = MSplit<N, WALL>;
    constexpr int R = M::R;
    sfor<0, R>([&](auto I) {
        constexpr int i = decltype(I)::value;
        if constexpr (M::ways == 4) {
            const T s0 = x[i] + x[2 * R + i], d0 = x[i] - x[2 * R + i];
            const T s1 = x[R + i] + x[3 * R + i], d1 = x[R + i] - x[3 * R + i];
            x[i] = s0 + s1;
            x[R + i] = s0 - s1;
            x[2 * R + i] = d0 + d1;
            x[3 * R + i] = d0 - d1;
        } else if constexpr (M::ways == 2) {
            const T a = x[i], b = x[R + i];
            x[i] = a + b;
            x[R + i] = a - b;
        }
    });
}
template <int N, bool WALL, typename T>
__device__ __forceinline__ void mjoin(T (&x)[N / 4])
{
    using M = MSplit<N, WALL>;
    constexpr int R = M::R;
    sfor<0, R>([&](auto I) {
        constexpr int i = decltype(I)::value;
        if constexpr (M::ways == 4) {
            const T s0 = x[i] + x[R + i], s1 = x[i] - x[R + i];
            const T d0 = x[2 * R + i] + x[3 * R + i], d1 = x[2 * R + i] - x[3 * R + i];
            x[i] = s0 + d0;
            x[R + i] = s1 + d1;
            x[2 * R + i] = s0 - d0;
            x[3 * R + i] = s1 - d1;
        } else if constexpr (M::ways == 2) {
            const T a = x[i], b = x[R + i];
            x[i] = a + b;
            x[R + i] = a - b;
        }
    });
}

// The value of lane `l`, the same in every lane.
__device__ __forceinline__ float mlane(float x, int l)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), l));
}
__device__ __forceinline__ double mlane(double x, int l)
{
    const long long b = __builtin_bit_cast(long long, x);
    const int lo = __builtin_amdgcn_readlane((int)b, l), hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
    return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}

// x <- D x for NC columns sets (complex float: real and imaginary parts).
//
// A constant passes through D unchanged, so one value c of the strip is taken
// out before the product and put back after it: D x = D (x - c) + c.  The
// products then add up to the line's variation, not to its mean.  Added to the
// mean, the matrix's smallest entries would round away, all in the same
// direction, which shows as a drift of Q over the contour (4e-6 against 2e-7
// in complex float over 100 steps at 64^3).
// f: the matrix's table, [ways][RB][R][64 lanes], in LDS or global memory.
// Between walls the constant comes back times the row sums of the table
// (absorbing walls do not keep it).
template <int N, int NC, bool WALL = false, typename T>
__device__ __forceinline__ void mdiffuse(T (&x)[NC][N / 4], const T* f)
{
    using M = MSplit<N, WALL>;
    constexpr int R = M::R, RB = M::RB;
    const int lane = threadIdx.x & 63;
    T mean[NC];  // `ways` times the constant: its share of the first sub-vector
    sfor<0, NC>([&](auto C) {
        constexpr int c = decltype(C)::value;
        msplit<N, WALL>(x[c]);
        if constexpr (NC == 2)
            mean[c] = mlane(x[c][0], 0);
        else
            mean[c] = (lane & 1) ? mlane(x[c][0], 1) : mlane(x[c][0], 0);
        sfor<0, R>([&](auto I) { x[c][decltype(I)::value] -= mean[c]; });
    });
    sfor<0, M::ways>([&](auto TI) {
        constexpr int t = decltype(TI)::value;
        macc<T> acc[NC][RB];
        sfor<0, NC>([&](auto C) { sfor<0, RB>([&](auto B) { acc[decltype(C)::value][decltype(B)::value] = macc<T>{0, 0, 0, 0}; }); });
        sfor<0, R>([&](auto SI) {
            constexpr int s = decltype(SI)::value;
            sfor<0, RB>([&](auto B) {
                constexpr int rb = decltype(B)::value;
                const T a = f[((t * RB + rb) * R + s) * 64 + lane];
                sfor<0, NC>([&](auto C) {
                    constexpr int c = decltype(C)::value;
                    acc[c][rb] = mprod(a, x[c][t * R + s], acc[c][rb]);
                });
            });
        });
        sfor<0, NC>([&](auto C) {
            sfor<0, R>([&](auto I) {
                constexpr int i = decltype(I)::value;
                x[decltype(C)::value][t * R + i] = acc[decltype(C)::value][i / 4][i % 4];
            });
        });
    });
    sfor<0, R>([&](auto I) {
        constexpr int i = decltype(I)::value;
        T r;
        if constexpr (WALL)
            r = f[M::kSums + mrow<T>(lane >> 4, i, R)];
        else
            r = T(1.0 / M::ways);
        sfor<0, NC>([&](auto C) { x[decltype(C)::value][i] += mean[decltype(C)::value] * r; });
    });
    sfor<0, NC>([&](auto C) { mjoin<N, WALL>(x[decltype(C)::value]); });
}

// ------------------------------------------------- pairs of lanes (double) --
// Complex double holds the real part of a column in an even lane and the
// imaginary part in the odd lane beside it.
template <int CTRL>
__device__ __forceinline__ double mdpp(double x)
{
    const long long b = __builtin_bit_cast(long long, x);
    const int lo = __builtin_amdgcn_mov_dpp((int)b, CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xf, 0xf, true);
    return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double mswap(double x) { return mdpp<0xB1>(x); }   // the partner's value
__device__ __forceinline__ double meven(double x) { return mdpp<0xA0>(x); }   // the even lane's
__device__ __forceinline__ double modd(double x) { return mdpp<0xF5>(x); }    // the odd lane's

}  // namespace pft
