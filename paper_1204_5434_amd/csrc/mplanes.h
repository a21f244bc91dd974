// Fused yz-plane pass of the Richardson split step, Eq. (12), on the matrix
// cores (mfma.h), the pass of planes.h:
//
//   U = Dz_{h/2} Dy_{h/2} U,  q' = (4 E4 U - V) / 3 (stored),
//   U = Dy_{h/2} Dz_{h/2} (E4 q'),  V = Dy_h Dz_h (E2 q')
//
// and the plain split step uses V alone.
//
// A wavefront holds a strip of columns of one plane with all their rows in
// registers; the plane goes through LDS three times, where the strips turn from
// columns (y in the rows) to rows (z in the rows) and back.
#pragma once

#include <hip/hip_runtime.h>

#include "mlines.h"

namespace pft {

template <typename T, int N>
struct MShape {
    static constexpr int NC = MStrip<T, N>::NC;
    static constexpr int CPS = MStrip<T, N>::CPS;
    // planes per workgroup: whole strips
    static constexpr int PW = (N % CPS == 0) ? 1 : (2 * N % CPS == 0) ? 2 : 4;
    static constexpr int kStrips = PW * N / CPS;
    static constexpr int kThreads = 64 * kStrips;
    static constexpr int RP = N + 1;  // odd pitch: strips of rows and of columns both spread over the banks
    // In LDS: the plane, then the four matrix tables of a pass.
    static constexpr int kPlaneBytes = PW * N * RP * (int)sizeof(cx<T>);
    static constexpr int kPlanePad = (kPlaneBytes + 15) / 16 * 16;
    static constexpr int kFragBytes = MSplit<N>::kFrag * (int)sizeof(T);
    static constexpr int kLdsBytes = kPlanePad + 4 * kFragBytes;
    static_assert(kLdsBytes <= 160 * 1024, "the plane and its tables must fit in LDS");
    // V and E are loaded before U's transforms: three strips, and the accumulators of
    // a product, in the registers of a lane at this workgroup size.
    static constexpr int kStripRegs = NC * (N / 4) * (int)sizeof(T) / 4;
    static_assert(4 * kStripRegs + 64 <= 512 / ((kStrips + 3) / 4), "three strips must fit the registers");
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

    // Matrix tables: slots 0 and 1 of LDS hold the y and z tables for h/2, slots 2
    // and 3 the z and y tables for h.
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
    auto diff = [&](Strip& x, int slot) { mdiffuse<N, NC>(x.v, static_cast<const T*>(fs + slot * kFrag)); };
    // turn a strip of columns into a strip of rows, and back
    auto turn = [&](Strip& x, bool to_rows) {
        const int wbase = pw * N * RP + (to_rows ? col : col * RP), ws = to_rows ? RP : 1;
        const int rbase = pw * N * RP + (to_rows ? col * RP : col), rs = to_rows ? 1 : RP;
        constexpr int R = MSplit<N>::R;
        __syncthreads();
        if constexpr (NC == 2) {
            cx<T>* s2 = reinterpret_cast<cx<T>*>(sh);
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
        } else {
            L.each([&](auto TI, auto I, int pt) {
                sh[2 * (wbase + pt * ws) + L.comp] = x.v[0][decltype(TI)::value * R + decltype(I)::value];
            });
            __syncthreads();
            L.each([&](auto TI, auto I, int pt) {
                x.v[0][decltype(TI)::value * R + decltype(I)::value] = sh[2 * (rbase + pt * rs) + L.comp];
            });
        }
    };

    Strip q, e;
    const bool rqm4 = A.scheme == kSchemeRQM4;
    // The tables are requested before the plane, so that they wait for nothing
    // else (memory answers a wavefront in order).
    const T* const fyh = A.has_prev ? A.fyh_p : A.fyh_n;
    const T* const fzh = A.has_prev ? A.fzh_p : A.fzh_n;
    Copy c0, c1, c2, c3;
    if (rqm4) {
        fetch(c0, fyh);
        fetch(c1, fzh);
    }
    if (A.has_next) {
        fetch(c2, A.fzf_n);
        fetch(c3, A.fyf_n);
    }
    auto tables_ready = [&]() {
        if (rqm4) {
            commit(c0, 0);
            commit(c1, 1);
        }
        if (A.has_next) {
            commit(c2, 2);
            commit(c3, 3);
        }
        __syncthreads();
    };
    if (A.has_prev && rqm4) {
        L.load(q, A.U + oc, N, act);
        Strip v;
        L.load_line(v, A.V + orow, act);
        L.load_line(e, A.Ep + orow, act);
        tables_ready();
        diff(q, 0);
        turn(q, true);
        diff(q, 1);
        if (A.hcap) L.store_line(q, A.hcap + orow, act);
        L.mul(q, e);
        L.combine(q, v);
    } else if (A.has_prev) {
        L.load_line(q, A.V + orow, act);
        L.load_line(e, A.Ep + orow, act);
        tables_ready();
        if (A.hcap) L.store_line(q, A.hcap + orow, act);
        L.mul(q, e);
        L.mul(q, e);
    } else {
        if (A.qin)
            L.load_line(q, A.qin + orow, act);
        else
            L.one(q);
        if (A.has_next) L.load_line(e, A.En + orow, act);
        tables_ready();
    }
    if (A.qout) L.store_line(q, A.qout + orow, act);
    if (!A.has_next) return;

    if (A.has_prev && A.En != A.Ep) L.load_line(e, A.En + orow, act);
    if (rqm4 && A.has_prev && (A.fyh_n != fyh || A.fzh_n != fzh)) {
        // the next step has another length
        fetch(c0, A.fyh_n);
        fetch(c1, A.fzh_n);
        __syncthreads();
        commit(c0, 0);
        commit(c1, 1);
        __syncthreads();
    }
    L.mul(q, e);
    Strip w = q;
    L.mul(w, e);
    if (rqm4) {
        diff(q, 1);
        turn(q, false);
        diff(q, 0);
        L.store(q, A.U + oc, N, act);
    }
    diff(w, 2);
    turn(w, false);
    diff(w, 3);
    L.store(w, A.V + oc, N, act);
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

// Plane sides (= ny = nz) of the yz pass.
#define PFT_MPLANE(X) X(8) X(12) X(16) X(20) X(24) X(32) X(40) X(48) X(64)

template <typename T>
bool mplane_supported(int n);

// nsweeps 1 (a0) or 2: both sweeps' passes in one launch.
template <typename T>
hipError_t launch_myz(int n, const MArgs<T>& a0, const MArgs<T>& a1, int nsweeps, hipStream_t s);
// The same over nrep argument sets of one shape in a device table.
template <typename T>
hipError_t launch_myz_batch(int n, int nplanes, const MArgs<T>* descs, int nrep, hipStream_t s);

}  // namespace pft
