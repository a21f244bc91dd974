// Host side of the matrix-core line diffusion (mfma.h): the table of one
// axis's diffusion matrix, in the order in which the lanes read it.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstddef>
#include <numeric>
#include <vector>

#include "mfma.h"

namespace pft {

// Split of a line (MSplit for a length known at run time).
struct MSplitRt {
    int N, ways, S, R, RB;
    explicit MSplitRt(int n)
        : N(n), ways(n <= 20 ? 1 : (n % 16 == 0 && n >= 48) ? 4 : 2), S(n / ways), R(S / 4), RB((R + 3) / 4)
    {
    }
    size_t size() const { return (size_t)ways * RB * R * 64; }
};

// Table of the matrix whose eigenvalue at mode k (natural DFT order, even in
// k) is g[k], with g[0] = 1.  The entry (i, j) is c[i - j], c the inverse DFT of g.  Each
// sub-matrix follows from c: with cs[m] = c[m] + c[m + N/2] (period N/2) and
// cd[m] = c[m] - c[m + N/2] (changing sign after N/2), the halves are cs[i - j]
// and cd[i - j], and their even and odd parts under n -> N/2 - 1 - n add or
// subtract cs[i + j + 1], and subtract or add cd[i + j + 1].  The 1/ways of the
// recombination is folded in.
//
// The k = 0 mode (factor 1) passes through the row sums of the first
// sub-matrix, and a row sum that is off by a rounding would scale the mean of q
// by the same factor at every step of the sweep.  The rounded entries of each
// row are therefore adjusted, from the largest to the smallest, until they add
// up to 1 / ways.
template <typename T>
void mtable(int N, const std::vector<double>& g, T* out)
{
    const MSplitRt M(N);
    std::vector<double> cosn(N), c(N, 0.0);
    for (int j = 0; j < N; ++j) cosn[j] = std::cos(6.283185307179586476925286766559 * std::min(j, N - j) / N);
    for (int m = 0; m <= N / 2; ++m) {
        double s = 0.0;
        for (int k = N - 1; k >= 0; --k) s += g[k] * cosn[(int)(((long)k * m) % N)];
        c[m] = s / N;
        c[(N - m) % N] = c[m];
    }
    auto C = [&](int m) { return c[((m % N) + N) % N]; };
    auto cs = [&](int m) { return C(m) + C(m + N / 2); };
    auto cd = [&](int m) { return C(m) - C(m + N / 2); };
    auto entry = [&](int t, int i, int j) {
        if (M.ways == 1) return C(i - j);
        if (M.ways == 2) return 0.5 * (t == 0 ? cs(i - j) : cd(i - j));
        const double a = t < 2 ? cs(i - j) : cd(i - j), b = t < 2 ? cs(i + j + 1) : -cd(i + j + 1);
        return 0.25 * (t % 2 == 0 ? a + b : a - b);
    };
    std::vector<T> K((size_t)M.S * M.S);
    std::vector<int> order(M.S);
    for (int t = 0; t < M.ways; ++t) {
        for (int i = 0; i < M.S; ++i) {
            T* row = &K[(size_t)i * M.S];
            for (int j = 0; j < M.S; ++j) row[j] = T(entry(t, i, j));
            if (t == 0) {
                long double s = 1.0L / M.ways;
                for (int j = 0; j < M.S; ++j) s -= (long double)row[j];
                std::iota(order.begin(), order.end(), 0);
                std::sort(order.begin(), order.end(), [&](int a, int b) {
                    return std::fabs(row[a]) != std::fabs(row[b]) ? std::fabs(row[a]) > std::fabs(row[b]) : a < b;
                });
                for (int j : order) {
                    const T v = T((long double)row[j] + s);
                    s -= (long double)v - (long double)row[j];
                    row[j] = v;
                }
            }
        }
        for (int rb = 0; rb < M.RB; ++rb)
            for (int s = 0; s < M.R; ++s)
                for (int lane = 0; lane < 64; ++lane) {
                    // operand row i of the 16-row product, and its k index (the lane's group)
                    const int i = lane % 16, gk = lane / 16;
                    const int go = sizeof(T) == 4 ? i / 4 : i % 4, ro = 4 * rb + (sizeof(T) == 4 ? i % 4 : i / 4);
                    out[(((size_t)t * M.RB + rb) * M.R + s) * 64 + lane] =
                        ro < M.R ? K[(size_t)mrow<T>(go, ro, M.R) * M.S + mrow<T>(gk, s, M.R)] : T(0);
                }
    }
}

}  // namespace pft
