// Arguments and lane-level building blocks of the passes on the matrix cores:
// strips of columns held by a wavefront (see mfma.h), their memory accesses and
// pointwise products.
#pragma once

#include "kernels.h"
#include "mfma.h"

namespace pft {

// Arguments of the yz pass (and of the z pass alone, which reads the z tables
// only).  The f.. are matrix tables (mfma.h).
template <typename T>
struct MArgs {
    int skip;        // batched launches: this replica has no work at this position
    int nplanes;     // yz pass: nx
    int nlines;      // z pass: nx ny lines of nz contiguous points
    int has_prev, has_next, scheme;
    cx<T>* U;
    cx<T>* V;
    const cx<T>* qin;  // start value when there is no previous step (NULL: q = 1)
    cx<T>* qout;       // where the completed q is stored (NULL: not stored)
    const cx<T>* Ep;   // E4 table of the step being completed
    const T* fyh_p;    // its y and z matrices for h/2
    const T* fzh_p;
    const cx<T>* En;   // E4 table of the step being started
    const T* fzh_n;    // its matrices for h/2 and h
    const T* fzf_n;
    const T* fyh_n;
    const T* fyf_n;
    cx<T>* hcap;       // reverse mode: the completed step's last diffused value
};

// What a wavefront holds of a strip: 16 columns of N rows.  Complex float: 16
// complex columns, a lane holds both parts (NC = 2); complex double: 8 complex
// columns, real and imaginary parts in neighbouring lanes.
template <typename T, int N>
struct MStrip {
    static constexpr int NC = sizeof(T) == 4 ? 2 : 1;
    static constexpr int CPS = sizeof(T) == 4 ? 16 : 8;  // complex columns
    T v[NC][N / 4];
};

// What a lane does with its strip: its rows' addresses, and the pointwise
// complex products.
template <typename T, int N, bool WALL = false>
struct MLane {
    using S = MStrip<T, N>;
    using M = MSplit<N, WALL>;
    static constexpr int R = M::R, NR = N / 4;
    int g, comp;  // row group, component (complex double)

    __device__ __forceinline__ MLane()
    {
        g = (threadIdx.x >> 4) & 3;
        comp = threadIdx.x & 1;
    }
    // q = 1
    __device__ __forceinline__ void one(MStrip<T, N>& x) const
    {
        sfor<0, NR>([&](auto K) {
            constexpr int k = decltype(K)::value;
            if constexpr (S::NC == 2) {
                x.v[0][k] = T(1);
                x.v[1][k] = T(0);
            } else {
                x.v[0][k] = comp ? T(0) : T(1);
            }
        });
    }
    // Contiguous lines in complex double: a register pair is two consecutive
    // points of the line; each lane of a column's pair accesses one of them whole
    // (16 bytes), and they swap: the even lane keeps the real parts.
    // f(lo, hi, a) per register pair with the point a of register lo (a + 1 of
    // hi), s(k, a) for an odd last register.
    template <class F, class G>
    __device__ __forceinline__ void along(F&& f, G&& s) const
    {
        sfor<0, M::ways>([&](auto TI) {
            constexpr int t = decltype(TI)::value;
            sfor<0, R / 2>([&](auto I) {
                constexpr int i = 2 * decltype(I)::value;
                constexpr int lo = mreversed<N, WALL>(t) ? i + 1 : i, hi = 2 * i + 1 - lo;
                f(std::integral_constant<int, t * R + lo>{}, std::integral_constant<int, t * R + hi>{},
                  mpoint<N, WALL>(t, mrow<T>(g, lo, R)));
            });
            if constexpr (R % 2) s(std::integral_constant<int, t * R + R - 1>{}, mpoint<N, WALL>(t, mrow<T>(g, R - 1, R)));
        });
    }
    __device__ __forceinline__ void load_line(MStrip<T, N>& x, const cx<T>* p, bool act) const
    {
        if constexpr (S::NC == 2) {
            load(x, p, 1, act);
        } else if (act) {
            along(
                [&](auto LO, auto HI, int a) {
                    const cx<T> w = p[a + comp];
                    const T other = mswap(comp ? w.re : w.im);
                    x.v[0][decltype(LO)::value] = comp ? other : w.re;
                    x.v[0][decltype(HI)::value] = comp ? w.im : other;
                },
                [&](auto K, int a) { x.v[0][decltype(K)::value] = reinterpret_cast<const T*>(p)[2 * a + comp]; });
        } else {
            sfor<0, NR>([&](auto K) { x.v[0][decltype(K)::value] = T(0); });
        }
    }
    __device__ __forceinline__ void store_line(const MStrip<T, N>& x, cx<T>* p, bool act) const
    {
        if constexpr (S::NC == 2) {
            store(x, p, 1, act);
        } else if (act) {  // both lanes of a pair share their column
            along(
                [&](auto LO, auto HI, int a) {
                    const T u = x.v[0][decltype(LO)::value], w = x.v[0][decltype(HI)::value];
                    const T other = mswap(comp ? u : w);
                    p[a + comp] = cx<T>{comp ? other : u, comp ? w : other};
                },
                [&](auto K, int a) { reinterpret_cast<T*>(p)[2 * a + comp] = x.v[0][decltype(K)::value]; });
        }
    }
    // row n of the line is p[n * stride]
    __device__ __forceinline__ void load(MStrip<T, N>& x, const cx<T>* p, int stride, bool act) const
    {
        each([&](auto TI, auto I, int pt) {
            constexpr int k = decltype(TI)::value * R + decltype(I)::value;
            if constexpr (S::NC == 2) {
                const cx<T> a = act ? p[(int64_t)pt * stride] : cx<T>{T(0), T(0)};
                x.v[0][k] = a.re;
                x.v[1][k] = a.im;
            } else {
                x.v[0][k] = act ? reinterpret_cast<const T*>(p)[2 * ((int64_t)pt * stride) + comp] : T(0);
            }
        });
    }
    __device__ __forceinline__ void store(const MStrip<T, N>& x, cx<T>* p, int stride, bool act) const
    {
        if (!act) return;
        each([&](auto TI, auto I, int pt) {
            constexpr int k = decltype(TI)::value * R + decltype(I)::value;
            if constexpr (S::NC == 2)
                p[(int64_t)pt * stride] = cx<T>{x.v[0][k], x.v[1][k]};
            else
                reinterpret_cast<T*>(p)[2 * ((int64_t)pt * stride) + comp] = x.v[0][k];
        });
    }
    // every (sub-vector, row) of this lane with its point of the line
    template <class F>
    __device__ __forceinline__ void each(F&& f) const
    {
        sfor<0, M::ways>([&](auto TI) {
            sfor<0, R>([&](auto I) { f(TI, I, mpoint<N, WALL>(decltype(TI)::value, mrow<T>(g, decltype(I)::value, R))); });
        });
    }
    // x *= e
    __device__ __forceinline__ void mul(MStrip<T, N>& x, const MStrip<T, N>& e) const
    {
        sfor<0, NR>([&](auto K) {
            constexpr int k = decltype(K)::value;
            if constexpr (S::NC == 2) {
                const T re = x.v[0][k] * e.v[0][k] - x.v[1][k] * e.v[1][k];
                x.v[1][k] = x.v[0][k] * e.v[1][k] + x.v[1][k] * e.v[0][k];
                x.v[0][k] = re;
            } else {
                const T er = meven(e.v[0][k]), ei = modd(e.v[0][k]);
                x.v[0][k] = x.v[0][k] * er + mswap(x.v[0][k]) * (comp ? ei : -ei);
            }
        });
    }
    __device__ __forceinline__ void square(MStrip<T, N>& e) const
    {
        sfor<0, NR>([&](auto K) {
            constexpr int k = decltype(K)::value;
            if constexpr (S::NC == 2) {
                const T re = e.v[0][k] * e.v[0][k] - e.v[1][k] * e.v[1][k];
                e.v[1][k] = T(2) * e.v[0][k] * e.v[1][k];
                e.v[0][k] = re;
            } else {
                const T er = meven(e.v[0][k]), ei = modd(e.v[0][k]);
                e.v[0][k] = comp ? T(2) * er * ei : er * er - ei * ei;
            }
        });
    }
    // (4 x - v) / 3; complex float in double with one rounding
    __device__ __forceinline__ void combine(MStrip<T, N>& x, const MStrip<T, N>& v) const
    {
        constexpr double third = 1.0 / 3.0;
        sfor<0, S::NC>([&](auto C) {
            sfor<0, NR>([&](auto K) {
                constexpr int c = decltype(C)::value, k = decltype(K)::value;
                if constexpr (S::NC == 2)
                    x.v[c][k] = float((4.0 * double(x.v[c][k]) - double(v.v[c][k])) * third);
                else
                    x.v[c][k] = third * (4.0 * x.v[c][k] - v.v[c][k]);
            });
        });
    }
};

}  // namespace pft
