// Fused yz-plane pass and x pass of the Richardson split step, Eq. (12), on
// the matrix cores (mfma.h).  The passes are those of planes.h and kernels.h:
//
//   yz: U = Dz_{h/2} Dy_{h/2} U,  q' = (4 E4 U - V) / 3 (stored),
//       U = Dy_{h/2} Dz_{h/2} (E4 q'),  V = Dy_h Dz_h (E2 q')
//   x:  U = Dx_{h/2} (E2 Dx_{h/2} U),   V = E2 Dx_h V
//
// and the plain split step uses V alone.
//
// A wavefront of the yz pass holds a strip of 16 columns of one plane (16
// complex float columns, or 8 complex double ones with real and imaginary
// parts in neighbouring lanes) with all their rows in registers; the plane goes
// through LDS three times, where the strips turn from columns (y in the rows)
// to rows (z in the rows) and back.
#pragma once

#include <hip/hip_runtime.h>

#include "kernels.h"
#include "mfma.h"

namespace pft {

// Arguments of the yz pass.  The f.. are matrix tables (mfma.h).
template <typename T>
struct MArgs {
    int skip;        // batched launches: this replica has no work at this position
    int nplanes;     // nx
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

// Arguments of the x pass.
template <typename T>
struct MXArgs {
    int skip;
    int ncols;       // ny nz contiguous columns
    cx<T>* U;        // NULL: V only (plain split step)
    cx<T>* V;
    const cx<T>* E;  // E4 table (NULL: no multiply)
    const T* fh;     // x matrices for h/2 and h
    const T* ff;
    cx<T>* capU;     // reverse mode: U and V after their first diffusion
    cx<T>* capV;
};

template <typename T, int N>
struct MShape {
    static constexpr int NC = sizeof(T) == 4 ? 2 : 1;   // components a lane holds
    static constexpr int CPS = sizeof(T) == 4 ? 16 : 8; // complex columns per strip
    // planes per workgroup: whole strips
    static constexpr int PW = (N % CPS == 0) ? 1 : (2 * N % CPS == 0) ? 2 : 4;
    static constexpr int kStrips = PW * N / CPS;
    static constexpr int kThreads = 64 * kStrips;
    static constexpr int RP = N + 1;  // odd pitch: strips of rows and of columns both spread over the banks
    // complex double at 128: the plane exceeds LDS, real and imaginary parts go through it one after the other
    static constexpr bool kHalves = (int64_t)PW * N * RP * (int64_t)sizeof(cx<T>) > 160 * 1024;
    static constexpr int kPlaneBytes = PW * N * RP * (int)sizeof(T) * (kHalves ? 1 : 2);
    // Matrix tables in LDS: all four of a pass where they fit beside the plane,
    // one at a time where that fits, else read from global memory.
    static constexpr int kFragBytes = MSplit<N>::kFrag * (int)sizeof(T);
    static constexpr int kPlanePad = (kPlaneBytes + 15) / 16 * 16;
    static constexpr int kSlots = kPlanePad + 4 * kFragBytes <= 160 * 1024 ? 4 : kPlanePad + kFragBytes <= 160 * 1024 ? 1 : 0;
    static constexpr int kLdsBytes = kPlanePad + kSlots * kFragBytes;
    // registers of a strip, and what a lane may use at this workgroup size
    static constexpr int kStripRegs = NC * (N / 4) * (int)sizeof(T) / 4;
    static constexpr int kRegs = 512 / ((kStrips + 3) / 4);
    // V and E are loaded before U's transforms where three strips fit the registers
    static constexpr bool kEarly = 4 * kStripRegs + 64 <= kRegs;
};

// One strip's values: NC components by NR rows.
template <typename T, int N>
struct MStrip {
    T v[MShape<T, N>::NC][N / 4];
};

// What a lane does with its strip: addresses along both layouts, and the
// pointwise complex products.
template <typename T, int N>
struct MLane {
    using S = MShape<T, N>;
    using M = MSplit<N>;
    static constexpr int R = M::R, NR = N / 4;
    int g, comp;  // row group, component (complex double)

    __device__ __forceinline__ MLane()
    {
        g = (threadIdx.x >> 4) & 3;
        comp = threadIdx.x & 1;
    }
    // rows along a strided direction: element (row) at p + row * stride
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
            sfor<0, R>([&](auto I) { f(TI, I, mpoint<N>(decltype(TI)::value, mrow<T>(g, decltype(I)::value, R))); });
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

template <typename T, int N>
__device__ __forceinline__ void myz_body(const MArgs<T>& A, unsigned bid, unsigned char* smem)
{
    using S = MShape<T, N>;
    constexpr int NC = S::NC, RP = S::RP;
    using Strip = MStrip<T, N>;
    const MLane<T, N> L;
    const int cc = (int)(threadIdx.x >> 6) * S::CPS + ((int)threadIdx.x & 15) / (16 / S::CPS);
    const int pw = S::PW == 1 ? 0 : cc / N, col = S::PW == 1 ? cc : cc % N;
    const int plane = (int)bid * S::PW + pw;
    const bool act = S::PW == 1 || plane < A.nplanes;
    const int64_t pbase = (int64_t)plane * N * N;
    const int64_t oc = pbase + col, orow = pbase + (int64_t)col * N;
    T* sh = reinterpret_cast<T*>(smem);

    // Matrix tables: slot 0 (1, 2, 3) of LDS holds the y and z tables for h/2
    // and the z and y tables for h; with one slot each is brought in when the
    // plane turns, or by itself.
    T* const fs = reinterpret_cast<T*>(smem + S::kPlanePad);
    constexpr int kFrag = MSplit<N>::kFrag;
    using Quad = float __attribute__((ext_vector_type(4)));
    constexpr int kQuads = S::kFragBytes / 16;
    constexpr int kCopy = (kQuads + S::kThreads - 1) / S::kThreads;
    struct Copy {
        Quad r[kCopy];
    };
    auto fetch = [&](Copy& c, const T* f) {
        sfor<0, kCopy>([&](auto I) {
            const int i = decltype(I)::value * S::kThreads + (int)threadIdx.x;
            if (i < kQuads) c.r[decltype(I)::value] = reinterpret_cast<const Quad*>(f)[i];
        });
    };
    auto commit = [&](const Copy& c, int slot) {
        sfor<0, kCopy>([&](auto I) {
            const int i = decltype(I)::value * S::kThreads + (int)threadIdx.x;
            if (i < kQuads) reinterpret_cast<Quad*>(fs + slot * kFrag)[i] = c.r[decltype(I)::value];
        });
    };
    auto bring = [&](const T* f, int slot) {
        Copy c;
        fetch(c, f);
        __syncthreads();
        commit(c, slot);
        __syncthreads();
    };
    auto diff = [&](Strip& x, const T* f, int slot) {
        if constexpr (S::kSlots == 0)
            mdiffuse<N, NC>(x.v, f);
        else
            mdiffuse<N, NC>(x.v, static_cast<const T*>(fs + (S::kSlots == 4 ? slot : 0) * kFrag));
    };
    // turn a strip of columns into a strip of rows, and back; f: the table that
    // the next diffusion reads (one slot)
    auto turn = [&](Strip& x, bool to_rows, const T* f) {
        Copy c;
        if constexpr (S::kSlots == 1) {
            if (f) fetch(c, f);
        }
        const int wbase = pw * N * RP + (to_rows ? col : col * RP), ws = to_rows ? RP : 1;
        const int rbase = pw * N * RP + (to_rows ? col * RP : col), rs = to_rows ? 1 : RP;
        constexpr int R = MSplit<N>::R;
        if constexpr (NC == 2) {
            cx<T>* s2 = reinterpret_cast<cx<T>*>(sh);
            __syncthreads();
            if constexpr (S::kSlots == 1) {
                if (f) commit(c, 0);
            }
            L.each([&](auto TI, auto I, int pt) {
                constexpr int k = decltype(TI)::value * R + decltype(I)::value;
                s2[wbase + pt * ws] = cx<T>{x.v[0][k], x.v[1][k]};
            });
            __syncthreads();
            L.each([&](auto TI, auto I, int pt) {
                constexpr int k = decltype(TI)::value * R + decltype(I)::value;
                const cx<T> a = s2[rbase + pt * rs];
                x.v[0][k] = a.re;
                x.v[1][k] = a.im;
            });
        } else if constexpr (!S::kHalves) {
            __syncthreads();
            if constexpr (S::kSlots == 1) {
                if (f) commit(c, 0);
            }
            L.each([&](auto TI, auto I, int pt) {
                sh[2 * (wbase + pt * ws) + L.comp] = x.v[0][decltype(TI)::value * R + decltype(I)::value];
            });
            __syncthreads();
            L.each([&](auto TI, auto I, int pt) {
                x.v[0][decltype(TI)::value * R + decltype(I)::value] = sh[2 * (rbase + pt * rs) + L.comp];
            });
        } else {
            for (int half = 0; half < 2; ++half) {
                __syncthreads();
                if constexpr (S::kSlots == 1) {
                    if (f && half == 0) commit(c, 0);
                }
                if (L.comp == half)
                    L.each([&](auto TI, auto I, int pt) {
                        sh[wbase + pt * ws] = x.v[0][decltype(TI)::value * R + decltype(I)::value];
                    });
                __syncthreads();
                if (L.comp == half)
                    L.each([&](auto TI, auto I, int pt) {
                        x.v[0][decltype(TI)::value * R + decltype(I)::value] = sh[rbase + pt * rs];
                    });
            }
        }
    };

    Strip q, e;
    bool have_e = false;
    const bool rqm4 = A.scheme == kSchemeRQM4;
    if (A.has_prev && rqm4) {
        L.load(q, A.U + oc, N, act);
        Strip v;
        if constexpr (S::kEarly) {
            L.load(v, A.V + orow, 1, act);
            L.load(e, A.Ep + orow, 1, act);
        }
        if constexpr (S::kSlots == 4) {
            Copy c0, c1;
            fetch(c0, A.fyh_p);
            fetch(c1, A.fzh_p);
            commit(c0, 0);
            commit(c1, 1);
            if (A.has_next) {
                fetch(c0, A.fzf_n);
                fetch(c1, A.fyf_n);
                commit(c0, 2);
                commit(c1, 3);
            }
            __syncthreads();
        } else if constexpr (S::kSlots == 1) {
            bring(A.fyh_p, 0);
        }
        diff(q, A.fyh_p, 0);
        turn(q, true, A.fzh_p);
        diff(q, A.fzh_p, 1);
        if (A.hcap) L.store(q, A.hcap + orow, 1, act);
        if constexpr (!S::kEarly) L.load(e, A.Ep + orow, 1, act);
        have_e = true;
        L.mul(q, e);
        if constexpr (!S::kEarly) L.load(v, A.V + orow, 1, act);
        L.combine(q, v);
    } else if (A.has_prev) {
        L.load(q, A.V + orow, 1, act);
        if (A.hcap) L.store(q, A.hcap + orow, 1, act);
        L.load(e, A.Ep + orow, 1, act);
        have_e = true;
        L.mul(q, e);
        L.mul(q, e);
    } else if (A.qin) {
        L.load(q, A.qin + orow, 1, act);
    } else {
        sfor<0, N / 4>([&](auto K) {
            constexpr int k = decltype(K)::value;
            if constexpr (NC == 2) {
                q.v[0][k] = T(1);
                q.v[1][k] = T(0);
            } else {
                q.v[0][k] = L.comp ? T(0) : T(1);
            }
        });
    }
    if (A.qout) L.store(q, A.qout + orow, 1, act);

    if (A.has_next) {
        if constexpr (S::kSlots == 4) {
            // tables of this step that are not in LDS yet
            if (!(A.has_prev && rqm4)) {
                Copy c0, c1;
                fetch(c0, A.fzf_n);
                fetch(c1, A.fyf_n);
                commit(c0, 2);
                commit(c1, 3);
                __syncthreads();
            }
            if (rqm4 && !(A.has_prev && A.fyh_n == A.fyh_p && A.fzh_n == A.fzh_p)) {
                Copy c0, c1;
                fetch(c0, A.fyh_n);
                fetch(c1, A.fzh_n);
                __syncthreads();
                commit(c0, 0);
                commit(c1, 1);
                __syncthreads();
            }
        }
        if (!(have_e && A.En == A.Ep)) L.load(e, A.En + orow, 1, act);
        L.mul(q, e);
        Strip w = q;
        L.mul(w, e);
        if (rqm4) {
            if constexpr (S::kSlots == 1) {
                if (!(A.has_prev && A.fzh_n == A.fzh_p)) bring(A.fzh_n, 0);
            }
            diff(q, A.fzh_n, 1);
            turn(q, false, A.fyh_n);
            diff(q, A.fyh_n, 0);
            L.store(q, A.U + oc, N, act);
        }
        if constexpr (S::kSlots == 1) bring(A.fzf_n, 0);
        diff(w, A.fzf_n, 2);
        turn(w, false, A.fyf_n);
        diff(w, A.fyf_n, 3);
        L.store(w, A.V + oc, N, act);
    }
}

// One or two sweeps (blockIdx.y) per launch.
template <typename T, int N>
__global__ __launch_bounds__((MShape<T, N>::kThreads)) void k_myz(MArgs<T> A0, MArgs<T> A1)
{
    __shared__ __align__(16) unsigned char smem[MShape<T, N>::kLdsBytes];
    MArgs<T> A = A0;
    if (blockIdx.y) A = A1;
    myz_body<T, N>(A, blockIdx.x, smem);
}

template <typename T, int N>
__global__ __launch_bounds__((MShape<T, N>::kThreads)) void k_myz_batch(const MArgs<T>* __restrict__ descs)
{
    __shared__ __align__(16) unsigned char smem[MShape<T, N>::kLdsBytes];
    const MArgs<T> A = descs[blockIdx.y];
    if (A.skip) return;
    myz_body<T, N>(A, blockIdx.x, smem);
}

// ------------------------------------------------------------------ x pass --
// A wavefront per strip of columns; the strips of a workgroup share the
// matrices in LDS.
constexpr int kMXWaves = 4;

template <typename T, int N>
struct MXShape {
    static constexpr bool kStage = MShape<T, N>::kFragBytes >= 4096;  // below, each wave reads the tables itself
    static constexpr int kLdsBytes = kStage ? 2 * MShape<T, N>::kFragBytes : 16;
};

template <typename T, int N>
__device__ __forceinline__ void mx_body(const MXArgs<T>& A, unsigned bid, unsigned char* smem)
{
    using S = MShape<T, N>;
    constexpr int NC = S::NC;
    using Strip = MStrip<T, N>;
    const MLane<T, N> L;
    const int col = ((int)bid * kMXWaves + (int)(threadIdx.x >> 6)) * S::CPS + ((int)threadIdx.x & 15) / (16 / S::CPS);
    const bool act = col < A.ncols;
    Strip v, e, u;
    L.load(v, A.V + col, A.ncols, act);
    if (A.E) L.load(e, A.E + col, A.ncols, act);
    if (A.U) L.load(u, A.U + col, A.ncols, act);
    const T *ff = A.ff, *fh = A.fh;
    if constexpr (MXShape<T, N>::kStage) {
        using Quad = float __attribute__((ext_vector_type(4)));
        Quad* s4 = reinterpret_cast<Quad*>(smem);
        constexpr int kQuads = S::kFragBytes / 16;
        for (int i = (int)threadIdx.x; i < kQuads; i += 64 * kMXWaves) s4[i] = reinterpret_cast<const Quad*>(A.ff)[i];
        if (A.U)
            for (int i = (int)threadIdx.x; i < kQuads; i += 64 * kMXWaves) s4[kQuads + i] = reinterpret_cast<const Quad*>(A.fh)[i];
        __syncthreads();
        ff = reinterpret_cast<const T*>(smem);
        fh = reinterpret_cast<const T*>(smem + S::kFragBytes);
    }
    if (A.E) L.square(e);
    mdiffuse<N, NC>(v.v, ff);
    if (A.capV) L.store(v, A.capV + col, A.ncols, act);
    if (A.E) L.mul(v, e);
    L.store(v, A.V + col, A.ncols, act);
    if (!A.U) return;
    mdiffuse<N, NC>(u.v, fh);
    if (A.capU) L.store(u, A.capU + col, A.ncols, act);
    L.mul(u, e);
    mdiffuse<N, NC>(u.v, fh);
    L.store(u, A.U + col, A.ncols, act);
}

template <typename T, int N>
__global__ __launch_bounds__(64 * kMXWaves) void k_mx(MXArgs<T> A0, MXArgs<T> A1)
{
    __shared__ __align__(16) unsigned char smem[MXShape<T, N>::kLdsBytes];
    MXArgs<T> A = A0;
    if (blockIdx.y) A = A1;
    mx_body<T, N>(A, blockIdx.x, smem);
}

template <typename T, int N>
__global__ __launch_bounds__(64 * kMXWaves) void k_mx_batch(const MXArgs<T>* __restrict__ descs)
{
    __shared__ __align__(16) unsigned char smem[MXShape<T, N>::kLdsBytes];
    const MXArgs<T> A = descs[blockIdx.y];
    if (A.skip) return;
    mx_body<T, N>(A, blockIdx.x, smem);
}

// Plane sides (= ny = nz) of the yz pass and lengths of the x pass.
#define PFT_MPLANE_F32(X) X(8) X(12) X(16) X(20) X(24) X(32) X(40) X(48) X(64)
#define PFT_MPLANE_F64(X) X(8) X(12) X(16) X(20) X(24) X(32) X(40) X(48) X(64)
#define PFT_MX_F32(X) X(8) X(12) X(16) X(20) X(24) X(32) X(40) X(48) X(64) X(80) X(96)
#define PFT_MX_F64(X) X(8) X(12) X(16) X(20) X(24) X(32) X(40) X(48) X(64) X(80)

template <typename T>
bool mplane_supported(int n);
template <typename T>
bool mx_supported(int n);

// nsweeps 1 (a0) or 2: both sweeps' passes in one launch.
template <typename T>
hipError_t launch_myz(int n, const MArgs<T>& a0, const MArgs<T>& a1, int nsweeps, hipStream_t s);
template <typename T>
hipError_t launch_mx(int n, const MXArgs<T>& a0, const MXArgs<T>& a1, int nsweeps, hipStream_t s);
// The same over nrep argument sets of one shape in a device table.
template <typename T>
hipError_t launch_myz_batch(int n, int nplanes, const MArgs<T>* descs, int nrep, hipStream_t s);
template <typename T>
hipError_t launch_mx_batch(int n, int ncols, const MXArgs<T>* descs, int nrep, hipStream_t s);

}  // namespace pft
