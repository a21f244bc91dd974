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
    // The tables are requested before the plane, so that they wait for nothing
    // else (memory answers a wavefront in order).
    const T* const fyh = A.has_prev ? A.fyh_p : A.fyh_n;
    const T* const fzh = A.has_prev ? A.fzh_p : A.fzh_n;
    Copy c0, c1, c2, c3;
    if (rqm4) {
        if constexpr (S::kSlots == 4) {
            fetch(c0, fyh);
            fetch(c1, fzh);
        } else if constexpr (S::kSlots == 1) {
            fetch(c0, A.has_prev ? fyh : fzh);
        }
    }
    if constexpr (S::kSlots == 4) {
        if (A.has_next) {
            fetch(c2, A.fzf_n);
            fetch(c3, A.fyf_n);
        }
    }
    auto tables_ready = [&]() {
        if constexpr (S::kSlots > 0) {
            if (rqm4) commit(c0, 0);
            if constexpr (S::kSlots == 4) {
                if (rqm4) commit(c1, 1);
                if (A.has_next) {
                    commit(c2, 2);
                    commit(c3, 3);
                }
            }
            __syncthreads();
        }
    };
    if (A.has_prev && rqm4) {
        L.load(q, A.U + oc, N, act);
        Strip v;
        if constexpr (S::kEarly) {
            L.load_line(v, A.V + orow, act);
            L.load_line(e, A.Ep + orow, act);
        }
        tables_ready();
        diff(q, fyh, 0);
        turn(q, true, fzh);
        diff(q, fzh, 1);
        if (A.hcap) L.store_line(q, A.hcap + orow, act);
        if constexpr (!S::kEarly) L.load_line(e, A.Ep + orow, act);
        have_e = true;
        L.mul(q, e);
        if constexpr (!S::kEarly) L.load_line(v, A.V + orow, act);
        L.combine(q, v);
    } else if (A.has_prev) {
        L.load_line(q, A.V + orow, act);
        L.load_line(e, A.Ep + orow, act);
        have_e = true;
        tables_ready();
        if (A.hcap) L.store_line(q, A.hcap + orow, act);
        L.mul(q, e);
        L.mul(q, e);
    } else {
        if (A.qin)
            L.load_line(q, A.qin + orow, act);
        else
            L.one(q);
        if (A.has_next) {
            L.load_line(e, A.En + orow, act);
            have_e = true;
        }
        tables_ready();
    }
    if (A.qout) L.store_line(q, A.qout + orow, act);
    if (!A.has_next) return;

    if (A.has_prev && A.En != A.Ep) L.load_line(e, A.En + orow, act);
    if (rqm4 && A.has_prev) {
        // tables of a next step of another length (one slot: its first table)
        if constexpr (S::kSlots == 4) {
            if (A.fyh_n != fyh || A.fzh_n != fzh) {
                fetch(c0, A.fyh_n);
                fetch(c1, A.fzh_n);
                __syncthreads();
                commit(c0, 0);
                commit(c1, 1);
                __syncthreads();
            }
        } else if constexpr (S::kSlots == 1) {
            if (A.fzh_n != fzh) bring(A.fzh_n, 0);
        }
    }
    L.mul(q, e);
    Strip w = q;
    L.mul(w, e);
    if (rqm4) {
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
#define PFT_MPLANE_F32(X) X(8) X(12) X(16) X(20) X(24) X(32) X(40) X(48) X(64)
#define PFT_MPLANE_F64(X) X(8) X(12) X(16) X(20) X(24) X(32) X(40) X(48) X(64)

template <typename T>
bool mplane_supported(int n);

// nsweeps 1 (a0) or 2: both sweeps' passes in one launch.
template <typename T>
hipError_t launch_myz(int n, const MArgs<T>& a0, const MArgs<T>& a1, int nsweeps, hipStream_t s);
// The same over nrep argument sets of one shape in a device table.
template <typename T>
hipError_t launch_myz_batch(int n, int nplanes, const MArgs<T>* descs, int nrep, hipStream_t s);

}  // namespace pft
