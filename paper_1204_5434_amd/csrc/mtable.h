// Host side of the matrix-core line diffusion (mfma.h): the table of one
// axis's diffusion matrix, in the order in which the lanes read it.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstddef>
#include <vector>

#include "mfma.h"

namespace pft {

// Split of a line (MSplit for a length known at run time).
struct MSplitRt {
    int N, ways, S, R, RB;
    bool wall;
    explicit MSplitRt(int n, bool w = false)
        : N(n), ways(n <= 20 ? 1 : (!w && n % 16 == 0 && n >= 48) ? 4 : 2), S(n / ways), R(S / 4), RB((R + 3) / 4), wall(w)
    {
    }
    size_t sums() const { return (size_t)ways * RB * R * 64; }
    size_t size() const { return sums() + (wall ? (size_t)(S + 63) / 64 * 64 : 0); }
};

// Table of the matrix whose eigenvalue at mode k is g[k], g[0] = 1.
//
// Periodic (wall 0; natural DFT order, even in k): the entry (i, j) is
// c[i - j], c the inverse DFT of g.  Each sub-matrix follows from c: with
// cs[m] = c[m] + c[m + N/2] (period N/2) and cd[m] = c[m] - c[m + N/2] (changing
// sign after N/2), the halves are cs[i - j] and cd[i - j], and their even and
// odd parts under n -> N/2 - 1 - n add or subtract cs[i + j + 1], and subtract
// or add cd[i + j + 1].
//
// Walls (1 reflecting, cosine modes k = 0..N-1; 2 absorbing, sine modes
// k = 1..N, g[N] the last): the orthonormal modes give c[i - j] + c[i + j + 1]
// or c[i - j] - c[i + j + 1] with c[m] the sum of g[k] cos(pi k m / N) / N, the
// modes of constant magnitude (k = 0, k = N) at half weight.  The sub-matrices
// are the even and odd parts under n -> N - 1 - n.
//
// The 1/ways of the recombination is folded in.
//
// The k = 0 mode (factor 1) passes through the row sums of the first
// sub-matrix, and a row sum that is off by a rounding would scale the mean of q
// by the same factor at every step of the sweep.  Rounded entries of each row
// are therefore adjusted until the row adds up to the exact sum, 1 / ways
// without absorbing walls.
template <typename T>
void mtable(int N, int wall, const std::vector<double>& g, T* out)
{
    const MSplitRt M(N, wall != 0);
    const int P = wall ? 2 * N : N;  // c has period P, and is even
    std::vector<double> cosn(P), c(P, 0.0);
    for (int j = 0; j < P; ++j) cosn[j] = std::cos(6.283185307179586476925286766559 * std::min(j, P - j) / P);
    const int K = wall == 2 ? N + 1 : N;
    for (int m = 0; m <= P / 2; ++m) {
        double s = 0.0;
        for (int k = K - 1; k >= 0; --k) {
            const double w = !wall ? 1.0 : (k == 0 || k == N) ? 0.5 : 1.0;
            if (wall == 2 && k == 0) continue;
            s += w * g[k] * cosn[(int)(((long)k * m) % P)];
        }
        c[m] = s / N;
        c[(P - m) % P] = c[m];
    }
    // The entries as a difference part f[i - j] and a sum part h[i + j + 1] per
    // sub-matrix: f and h of it, indices shifted by N.
    const int H = N / 2;
    std::vector<double> f(3 * N + 1), h(3 * N + 1);
    auto parts = [&](int t) {
        for (int m = -N; m <= 2 * N; ++m) {
            const int p = (m + 2 * P) % P;
            double df = c[p], sm = 0.0;
            if (wall) {
                const double sg = wall == 1 ? 1.0 : -1.0;
                sm = sg * c[p];
                if (M.ways == 2) {  // even and odd parts under n -> N - 1 - n
                    const double q = c[(m + N + P) % P], od = t == 0 ? 1.0 : -1.0;
                    df = 0.5 * (c[p] + od * sg * q);
                    sm = 0.5 * (sg * c[p] + od * q);
                }
            } else if (M.ways > 1) {
                const double q = c[(m + H + 2 * P) % P];
                const bool sum = M.ways == 2 ? t == 0 : t < 2;
                df = (sum ? c[p] + q : c[p] - q) / M.ways;
                if (M.ways == 4) sm = (sum == (t % 2 == 0)) ? df : -df;
            }
            f[m + N] = df;
            h[m + N] = sm;
        }
    };
    std::vector<T> rows((size_t)M.S * M.S);
    for (int t = 0; t < M.ways; ++t) {
        parts(t);
        for (int i = 0; i < M.S; ++i) {
            T* row = &rows[(size_t)i * M.S];
            long double sum = 0.0L;
            for (int j = 0; j < M.S; ++j) {
                const double v = f[i - j + N] + h[i + j + 1 + N];
                row[j] = T(v);
                sum += v;
            }
            if (t > 0) continue;
            if (wall != 2) sum = 1.0L / M.ways;
            if (wall) out[M.sums() + i] = T(sum);
            for (int j = 0; j < M.S; ++j) sum -= (long double)row[j];
            // what is left goes to the smallest entry well above it, again for
            // that entry's own rounding
            for (int k = 0; k < 3 && sum != 0.0L; ++k) {
                int at = -1;
                for (int j = 0; j < M.S; ++j)
                    if (std::fabs(row[j]) >= 64 * std::fabs((double)sum) && (at < 0 || std::fabs(row[j]) < std::fabs(row[at])))
                        at = j;
                if (at < 0) break;
                const T v = T((long double)row[at] + sum);
                sum -= (long double)v - (long double)row[at];
                row[at] = v;
            }
        }
        for (int rb = 0; rb < M.RB; ++rb)
            for (int s = 0; s < M.R; ++s)
                for (int lane = 0; lane < 64; ++lane) {
                    // operand row i of the 16-row product, and its k index (the lane's group)
                    const int i = lane % 16, gk = lane / 16;
                    const int go = sizeof(T) == 4 ? i / 4 : i % 4, ro = 4 * rb + (sizeof(T) == 4 ? i % 4 : i / 4);
                    out[(((size_t)t * M.RB + rb) * M.R + s) * 64 + lane] =
                        ro < M.R ? rows[(size_t)mrow<T>(go, ro, M.R) * M.S + mrow<T>(gk, s, M.R)] : T(0);
                }
    }
}

}  // namespace pft
