// Axis passes of the split step on the matrix cores (mfma.h): the passes of
// kernels.h,
//
//   z : q' = (4 E4 Dz_{h/2} U - V) / 3 (stored), U = Dz_{h/2}(E4 q'), V = Dz_h(E2 q')
//   x : U = Dx_{h/2}(E2 Dx_{h/2} U), V = E2 Dx_h V
//   y : U = Dy_{h/2} U, V = Dy_h V, or U alone
//
// and those of the plain split step (V alone), on periodic axes and between
// walls (WALL; reflecting and absorbing differ by the table only).  A
// wavefront holds a strip of 16 columns with their whole lines: no barrier and
// no exchange.  The strips of a workgroup share the matrices through LDS, the
// smallest tables (below 4 KB) are read from the caches by each wavefront.
#pragma once

#include <hip/hip_runtime.h>

#include "mlines.h"

namespace pft {

// Arguments of a strided (x or y) pass over `ncols` columns, `width` contiguous
// ones per slab.
template <typename T>
struct MXArgs {
    int skip;        // batched launches: this replica has no work at this position
    int ncols, width;
    int64_t stride, slab_stride;
    cx<T>* U;        // NULL: not touched
    cx<T>* V;
    const cx<T>* E;  // E4 table of an x pass (NULL: diffusion alone)
    const T* fh;     // matrices for h/2 (U) and h (V)
    const T* ff;
    cx<T>* capU;     // reverse mode: U and V after their first diffusion
    cx<T>* capV;
};

// Wavefronts of a workgroup.  They share the tables, and a grid has as many
// workgroups as strips allow: two are quicker on few columns and slower on many,
// eight are slower on both (x pass of 48 points in complex float, us with 2 / 4 / 8:
// 1024 columns 5.4 / 5.9 / 8.5, 12288 columns 8.4 / 7.0 / 9.6; z pass of 64 points in
// complex double 7.4 / 8.7 / 11.6 and 16.5 / 17.3 / 14.4).
constexpr int kMXWaves = 4;

template <typename T, int N, bool WALL>
struct MXShape {
    static constexpr int kFrag = MSplit<N, WALL>::kFrag;
    static constexpr int kFragBytes = kFrag * (int)sizeof(T);
    // Tables of 4 KB and more go through LDS (us, read from the caches / staged, 4096
    // columns: z pass of 40 points in complex float 7.9 / 7.2, 80 points 18.5 / 14.3,
    // complex double 40 points 8.9 / 7.5, 80 points 18.1 / 13.6); of smaller ones some lose
    // and some gain (z pass of 24 points in complex double 4.7 / 4.9, in complex float 4.8 /
    // 4.6, of 48 points 10.2 / 8.8).
    static constexpr bool kStage = kFragBytes >= 4096;
    static constexpr int kLdsBytes = kStage ? 2 * kFragBytes : 16;
    // registers of a strip; long lines are compiled for two waves per SIMD (all 512
    // registers otherwise: 80 points in complex double, 12288 columns, us with the bound
    // / without: x 21.3 / 25.9, z 24.3 / 32.1; 96 points in complex float 14.1 / 14.5 and
    // 18.1 / 18.3; up to 64 points the bound changes 5% at most, either way)
    static constexpr int kStripRegs = MStrip<T, N>::NC * (N / 4) * (int)sizeof(T) / 4;
    static constexpr int kMinWaves = kStripRegs >= 40 ? 2 : 1;
    // every strip of a pass is loaded before its first product
    static_assert(kStripRegs < 64, "three strips must fit the registers");
};

// A table on its way to slot 0 or 1 of LDS: requested before the strip's own
// loads (memory answers a wavefront in order), written when it is there.
template <typename T, int N, bool WALL>
struct MTable {
    using S = MXShape<T, N, WALL>;
    using Quad = float __attribute__((ext_vector_type(4)));
    static constexpr int kQuads = S::kFragBytes / 16;
    static constexpr int kCopy = (kQuads + 64 * kMXWaves - 1) / (64 * kMXWaves);
    Quad r[kCopy];
    __device__ __forceinline__ void fetch(const T* f)
    {
        sfor<0, kCopy>([&](auto I) {
            const int i = decltype(I)::value * 64 * kMXWaves + (int)threadIdx.x;
            if (i < kQuads) r[decltype(I)::value] = reinterpret_cast<const Quad*>(f)[i];
        });
    }
    __device__ __forceinline__ void commit(unsigned char* smem, int slot) const
    {
        Quad* to = reinterpret_cast<Quad*>(smem + slot * S::kFragBytes);
        sfor<0, kCopy>([&](auto I) {
            const int i = decltype(I)::value * 64 * kMXWaves + (int)threadIdx.x;
            if (i < kQuads) to[i] = r[decltype(I)::value];
        });
    }
};

template <typename T, int N, bool WALL>
__device__ __forceinline__ void mx_body(const MXArgs<T>& A, unsigned bid, unsigned char* smem)
{
    using S = MXShape<T, N, WALL>;
    using Strip = MStrip<T, N>;
    constexpr int NC = Strip::NC, CPS = Strip::CPS;
    const MLane<T, N, WALL> L;
    const int c = ((int)bid * kMXWaves + (int)(threadIdx.x >> 6)) * CPS + ((int)threadIdx.x & 15) / (16 / CPS);
    const bool act = c < A.ncols;
    const int slab = A.width < A.ncols ? c / A.width : 0;
    const int64_t at = slab * A.slab_stride + (c - slab * A.width);
    Strip v, e, u;
    MTable<T, N, WALL> cf, ch;
    if constexpr (S::kStage) {
        if (A.V) cf.fetch(A.ff);
        if (A.U) ch.fetch(A.fh);
    }
    if (A.V) L.load(v, A.V + at, A.stride, act);
    if (A.E) L.load(e, A.E + at, A.stride, act);
    if (A.U) L.load(u, A.U + at, A.stride, act);
    const T *ff = A.ff, *fh = A.fh;
    if constexpr (S::kStage) {
        if (A.V) cf.commit(smem, 0);
        if (A.U) ch.commit(smem, 1);
        __syncthreads();
        ff = reinterpret_cast<const T*>(smem);
        fh = reinterpret_cast<const T*>(smem + S::kFragBytes);
    }
    if (A.E) L.square(e);
    if (A.V) {
        mdiffuse<N, NC, WALL>(v.v, ff);
        if (A.capV) L.store(v, A.capV + at, A.stride, act);
        if (A.E) L.mul(v, e);
        L.store(v, A.V + at, A.stride, act);
    }
    if (A.U) {
        mdiffuse<N, NC, WALL>(u.v, fh);
        if (A.capU) L.store(u, A.capU + at, A.stride, act);
        if (A.E) {
            L.mul(u, e);
            mdiffuse<N, NC, WALL>(u.v, fh);
        }
        L.store(u, A.U + at, A.stride, act);
    }
}

// One or two sweeps (blockIdx.y) per launch.
template <typename T, int N, bool WALL>
__global__ __launch_bounds__(64 * kMXWaves, (MXShape<T, N, WALL>::kMinWaves)) void k_mx(MXArgs<T> A0, MXArgs<T> A1)
{
    __shared__ __align__(16) unsigned char smem[MXShape<T, N, WALL>::kLdsBytes];
    MXArgs<T> A = A0;
    if (blockIdx.y) A = A1;
    mx_body<T, N, WALL>(A, blockIdx.x, smem);
}

template <typename T, int N, bool WALL>
__global__ __launch_bounds__(64 * kMXWaves, (MXShape<T, N, WALL>::kMinWaves)) void k_mx_batch(const MXArgs<T>* __restrict__ descs)
{
    __shared__ __align__(16) unsigned char smem[MXShape<T, N, WALL>::kLdsBytes];
    const MXArgs<T> A = descs[blockIdx.y];
    if (A.skip) return;
    mx_body<T, N, WALL>(A, blockIdx.x, smem);
}

template <typename T, int N, bool WALL>
__device__ __forceinline__ void mz_body(const MArgs<T>& A, unsigned bid, unsigned char* smem)
{
    using S = MXShape<T, N, WALL>;
    using Strip = MStrip<T, N>;
    constexpr int NC = Strip::NC, CPS = Strip::CPS;
    const MLane<T, N, WALL> L;
    const int line = ((int)bid * kMXWaves + (int)(threadIdx.x >> 6)) * CPS + ((int)threadIdx.x & 15) / (16 / CPS);
    const bool act = line < A.nlines;
    const int64_t at = (int64_t)line * N;
    const bool rqm4 = A.scheme == kSchemeRQM4;
    const T *ff = A.fzf_n, *fh = A.has_prev ? A.fzh_p : A.fzh_n;
    Strip q, e;
    bool have_e = false;  // has_prev, where the compiler sees it: tested itself, it costs 8 to 20 registers
    MTable<T, N, WALL> cf, ch;
    if constexpr (S::kStage) {
        if (rqm4) ch.fetch(fh);
        if (A.has_next) cf.fetch(ff);
    }
    auto tables_ready = [&]() {
        if constexpr (S::kStage) {
            if (rqm4) ch.commit(smem, 1);
            if (A.has_next) cf.commit(smem, 0);
            __syncthreads();
        }
    };
    if (A.has_prev) {
        Strip v;
        L.load_line(q, (rqm4 ? A.U : A.V) + at, act);
        if (rqm4) L.load_line(v, A.V + at, act);
        L.load_line(e, A.Ep + at, act);
        have_e = true;
        tables_ready();
        if (rqm4) mdiffuse<N, NC, WALL>(q.v, S::kStage ? reinterpret_cast<const T*>(smem + S::kFragBytes) : fh);
        if (A.hcap) L.store_line(q, A.hcap + at, act);
        L.mul(q, e);
        if (rqm4)
            L.combine(q, v);
        else
            L.mul(q, e);
    } else {
        if (A.qin)
            L.load_line(q, A.qin + at, act);
        else
            L.one(q);
        tables_ready();
    }
    if (A.qout) L.store_line(q, A.qout + at, act);
    if (!A.has_next) return;
    if (rqm4 && A.fzh_n != fh) {  // the next step has another length
        fh = A.fzh_n;
        if constexpr (S::kStage) {
            ch.fetch(fh);
            __syncthreads();
            ch.commit(smem, 1);
            __syncthreads();
        }
    }
    if constexpr (S::kStage) {
        ff = reinterpret_cast<const T*>(smem);
        fh = reinterpret_cast<const T*>(smem + S::kFragBytes);
    }
    if (!(have_e && A.En == A.Ep)) L.load_line(e, A.En + at, act);
    L.mul(q, e);
    Strip w = q;
    L.mul(w, e);
    if (rqm4) {
        mdiffuse<N, NC, WALL>(q.v, fh);
        L.store_line(q, A.U + at, act);
    }
    mdiffuse<N, NC, WALL>(w.v, ff);
    L.store_line(w, A.V + at, act);
}

template <typename T, int N, bool WALL>
__global__ __launch_bounds__(64 * kMXWaves, (MXShape<T, N, WALL>::kMinWaves)) void k_mz(MArgs<T> A0, MArgs<T> A1)
{
    __shared__ __align__(16) unsigned char smem[MXShape<T, N, WALL>::kLdsBytes];
    MArgs<T> A = A0;
    if (blockIdx.y) A = A1;
    mz_body<T, N, WALL>(A, blockIdx.x, smem);
}

template <typename T, int N, bool WALL>
__global__ __launch_bounds__(64 * kMXWaves, (MXShape<T, N, WALL>::kMinWaves)) void k_mz_batch(const MArgs<T>* __restrict__ descs)
{
    __shared__ __align__(16) unsigned char smem[MXShape<T, N, WALL>::kLdsBytes];
    const MArgs<T> A = descs[blockIdx.y];
    if (A.skip) return;
    mz_body<T, N, WALL>(A, blockIdx.x, smem);
}

// Line lengths with kernels: periodic, and between walls.
#define PFT_MLINE_F32(X) X(8) X(12) X(16) X(20) X(24) X(32) X(40) X(48) X(64) X(80) X(96)
#define PFT_MLINE_F64(X) X(8) X(12) X(16) X(20) X(24) X(32) X(40) X(48) X(64) X(80)
#define PFT_MWALL(X) X(8) X(12) X(16) X(20) X(24) X(32) X(40) X(48) X(64) X(80)

// The lengths are the same for strided and z passes.
template <typename T>
bool mline_supported(int n, bool wall);

// nsweeps 1 (a0) or 2: both sweeps' passes in one launch.
template <typename T>
hipError_t launch_mx(int n, bool wall, const MXArgs<T>& a0, const MXArgs<T>& a1, int nsweeps, hipStream_t s);
template <typename T>
hipError_t launch_mz(int n, bool wall, const MArgs<T>& a0, const MArgs<T>& a1, int nsweeps, hipStream_t s);
// The same over nrep argument sets of one shape in a device table.
template <typename T>
hipError_t launch_mx_batch(int n, bool wall, int ncols, const MXArgs<T>* descs, int nrep, hipStream_t s);
template <typename T>
hipError_t launch_mz_batch(int n, bool wall, int nlines, const MArgs<T>* descs, int nrep, hipStream_t s);

}  // namespace pft
