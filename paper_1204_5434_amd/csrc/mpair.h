// Fused yz pass of small planes (two copies in 64 KB of LDS) on the matrix cores: the
// pass of mplanes.h for planes that are not square, and between walls.
//
//   1. columns: U = Dy_{h/2} U into LDS
//   2. rows:    U = Dz_{h/2} U, q' = (4 E4 U - V) / 3 stored, then
//               Dz_{h/2}(E4 q') and Dz_h(E2 q') into the two planes of LDS
//   3. columns: U = Dy_{h/2} of the first, V = Dy_h of the second
//
// A wavefront takes strips of columns in steps 1 and 3 and strips of rows in
// step 2, so the two lengths meet only in LDS: one kernel holds every pair of
// lengths, its steps chosen by a switch on them.  The tables are read from the
// caches.
//
// For small grids, whose step is bound by launches and by the chain of one
// plane: two sweeps of 24 x 32 x 20 take 6.1 us (complex float) and 7.3 us
// (complex double) in one launch, against 14 us for the z and the two y passes.
// Longer lines lose to the separate passes (80 x 96 x 40 complex double 30.6
// against 52 us one after the other, but those of two sweeps overlap), and the
// registers of a row step with two tables in flight spill from 64 points on.
#pragma once

#include <hip/hip_runtime.h>

#include "mlines.h"

namespace pft {

constexpr int kPairWaves = 8;

// LDS of the two planes (pitch nz + 1: rows and columns both spread over the banks).
template <typename T>
constexpr int64_t pair_lds(int ny, int nz)
{
    return 2 * (int64_t)ny * (nz + 1) * (int64_t)sizeof(cx<T>);
}

// Lengths a kernel switches over; a row step of 64 points spills.
#define PFT_PAIR_LENGTHS(X) X(8) X(12) X(16) X(20) X(24) X(32) X(40) X(48)

template <typename T, int N, bool WALL>
__device__ __forceinline__ void pair_columns_in(const MArgs<T>& A, int plane, int nz, cx<T>* sh)
{
    using Strip = MStrip<T, N>;
    const MLane<T, N, WALL> L;
    const int waves = (int)(blockDim.x >> 6), pitch = nz + 1;
    for (int s = (int)(threadIdx.x >> 6); s * Strip::CPS < nz; s += waves) {
        const int col = s * Strip::CPS + ((int)threadIdx.x & 15) / (16 / Strip::CPS);
        const bool act = col < nz;
        Strip x;
        L.load(x, A.U + (int64_t)plane * N * nz + col, nz, act);
        mdiffuse<N, Strip::NC, WALL>(x.v, A.fyh_p);
        L.store(x, sh + col, pitch, act);
    }
}

template <typename T, int N, bool WALL>
__device__ __forceinline__ void pair_columns_out(const MArgs<T>& A, int plane, int nz, const cx<T>* sh)
{
    using Strip = MStrip<T, N>;
    const MLane<T, N, WALL> L;
    const int waves = (int)(blockDim.x >> 6), pitch = nz + 1;
    const int strips = (nz + Strip::CPS - 1) / Strip::CPS;
    const bool rqm4 = A.scheme == kSchemeRQM4;
    // strips of the second plane (V) first, then of the first (U)
    for (int t = (int)(threadIdx.x >> 6); t < (rqm4 ? 2 : 1) * strips; t += waves) {
        const bool second = t < strips;
        const int col = (second ? t : t - strips) * Strip::CPS + ((int)threadIdx.x & 15) / (16 / Strip::CPS);
        const bool act = col < nz;
        Strip x;
        L.load(x, sh + (second ? N * pitch : 0) + col, pitch, act);
        mdiffuse<N, Strip::NC, WALL>(x.v, second ? A.fyf_n : A.fyh_n);
        L.store(x, (second ? A.V : A.U) + (int64_t)plane * N * nz + col, nz, act);
    }
}

template <typename T, int N, bool WALL>
__device__ __forceinline__ void pair_rows(const MArgs<T>& A, int plane, int ny, cx<T>* sh)
{
    using Strip = MStrip<T, N>;
    constexpr int NC = Strip::NC, pitch = N + 1;
    const MLane<T, N, WALL> L;
    const int waves = (int)(blockDim.x >> 6);
    const bool rqm4 = A.scheme == kSchemeRQM4;
    bool first = true;
    for (int s = (int)(threadIdx.x >> 6); first || s * Strip::CPS < ny; s += waves) {
        const int row = s * Strip::CPS + ((int)threadIdx.x & 15) / (16 / Strip::CPS);
        const bool act = row < ny;
        const int64_t at = ((int64_t)plane * ny + row) * N;
        Strip q, e, v;
        if (A.has_prev) {
            // requested before the columns are waited for
            if (rqm4)
                L.load_line(v, A.V + at, act);
            else
                L.load_line(q, A.V + at, act);
            L.load_line(e, A.Ep + at, act);
        }
        if (first && A.has_prev && rqm4) __syncthreads();  // every column is in LDS
        first = false;
        if (s * Strip::CPS >= ny) break;
        if (A.has_prev && rqm4) {
            L.load(q, sh + row * pitch, 1, act);
            mdiffuse<N, NC, WALL>(q.v, A.fzh_p);
            if (A.hcap) L.store_line(q, A.hcap + at, act);
            L.mul(q, e);
            L.combine(q, v);
        } else if (A.has_prev) {
            if (A.hcap) L.store_line(q, A.hcap + at, act);
            L.mul(q, e);
            L.mul(q, e);
        } else if (A.qin) {
            L.load_line(q, A.qin + at, act);
        } else {
            L.one(q);
        }
        if (A.qout) L.store_line(q, A.qout + at, act);
        if (!A.has_next) continue;
        if (!(A.has_prev && A.En == A.Ep)) L.load_line(e, A.En + at, act);
        L.mul(q, e);
        Strip w = q;
        L.mul(w, e);
        if (rqm4) {
            mdiffuse<N, NC, WALL>(q.v, A.fzh_n);
            L.store(q, sh + row * pitch, 1, act);
        }
        mdiffuse<N, NC, WALL>(w.v, A.fzf_n);
        L.store(w, sh + (ny + row) * pitch, 1, act);
    }
}

template <typename T, bool WY, bool WZ>
__device__ __forceinline__ void pair_body(const MArgs<T>& A, int ny, int nz, int plane, cx<T>* sh)
{
    if (A.has_prev && A.scheme == kSchemeRQM4) {
        switch (ny) {
#define PFT_CASE(N) \
    case N: pair_columns_in<T, N, WY>(A, plane, nz, sh); break;
            PFT_PAIR_LENGTHS(PFT_CASE)
#undef PFT_CASE
        }
    }
    switch (nz) {
#define PFT_CASE(N) \
    case N: pair_rows<T, N, WZ>(A, plane, ny, sh); break;
        PFT_PAIR_LENGTHS(PFT_CASE)
#undef PFT_CASE
    }
    if (!A.has_next) return;
    __syncthreads();
    switch (ny) {
#define PFT_CASE(N) \
    case N: pair_columns_out<T, N, WY>(A, plane, nz, sh); break;
        PFT_PAIR_LENGTHS(PFT_CASE)
#undef PFT_CASE
    }
}

// One or two sweeps (blockIdx.y) per launch.
template <typename T, bool WY, bool WZ>
__global__ __launch_bounds__(64 * kPairWaves) void k_mpair(MArgs<T> A0, MArgs<T> A1, int ny, int nz)
{
    extern __shared__ __align__(16) unsigned char smem[];
    MArgs<T> A = A0;
    if (blockIdx.y) A = A1;
    pair_body<T, WY, WZ>(A, ny, nz, blockIdx.x, reinterpret_cast<cx<T>*>(smem));
}

template <typename T, bool WY, bool WZ>
__global__ __launch_bounds__(64 * kPairWaves) void k_mpair_batch(const MArgs<T>* __restrict__ descs, int ny, int nz)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const MArgs<T> A = descs[blockIdx.y];
    if (A.skip) return;
    pair_body<T, WY, WZ>(A, ny, nz, blockIdx.x, reinterpret_cast<cx<T>*>(smem));
}

// Whether a plane has the kernel.
inline bool pair_supported(int ny, int nz)
{
    auto has = [](int n) {
#define PFT_CASE(N) \
    if (n == N) return true;
        PFT_PAIR_LENGTHS(PFT_CASE)
#undef PFT_CASE
        return false;
    };
    return has(ny) && has(nz) && pair_lds<double>(ny, nz) <= 64 * 1024;
}

// nsweeps 1 (a0) or 2: both sweeps' passes in one launch.
template <typename T>
hipError_t launch_mpair(int ny, int nz, bool wy, bool wz, const MArgs<T>& a0, const MArgs<T>& a1, int nsweeps, hipStream_t s);
// The same over nrep argument sets of one shape in a device table.
template <typename T>
hipError_t launch_mpair_batch(int ny, int nz, bool wy, bool wz, int nplanes, const MArgs<T>* descs, int nrep, hipStream_t s);

}  // namespace pft
