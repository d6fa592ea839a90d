// Kernel templates of the x and y transforms of a 3-D problem in one pass: a
// block holds whole [ny][nx] planes in LDS, so that the spectrum makes one
// trip through memory where separate x and y passes make two.
//   k_plane_fwd - forward y then x transforms (after the contrast stencil);
//   k_plane_inv - inverse x then y transforms fused with the LS / BiCGSTAB
//                 epilogues and their FP64 partial inner products.
//
// Every axis length is a product R1 R2 of two radices, and an axis is two
// sweeps over the plane, in place: with n = R2 n1 + n2 and k = k1 + R1 k2,
//   A[k1][n2] = W_N^(n2 k1) sum_n1 x[R2 n1 + n2] W_R1^(n1 k1)   (sweep 1),
//   X[k1 + R1 k2] = sum_n2 A[k1][n2] W_R2^(n2 k2)                (sweep 2),
// both at positions R2 k1 + n2 (then R2 k1 + k2) of the axis.  The spectrum is
// left in that order, PlaneOrder, which the z pass maps to wavenumbers, and
// the inverse runs the sweeps backwards: no transform is ever reordered, and
// a transform costs one LDS round trip between its sweeps where the autosort
// passes of length-80 rows and length-40 columns took five together.  Work
// items (one butterfly each) are dealt to threads anew in every sweep: along x
// in the y sweeps, along y in the x sweeps, so that LDS accesses are
// contiguous or of odd stride (row stride nx + 1), and global accesses
// contiguous: the field is [y][x], the spectrum [x][y].
#pragma once

#include "fft_kernels.h"

FW_BEGIN
template <int NX, int NY>
struct PlaneShape {
    static constexpr int X1 = plane_radix(NX), X2 = NX / X1;
    static constexpr int Y1 = plane_radix(NY), Y2 = NY / Y1;
    static constexpr int RS = NX + 1;   // odd LDS row stride
    static constexpr int NP = NX * NY;
};

// One butterfly of radix R in place on R LDS elements STRIDE apart.
template <int R, bool INV, int STRIDE>
__device__ __forceinline__ void sweep_lds(cplx* p) {
    cplx v[R];
#pragma unroll
    for (int k = 0; k < R; ++k) v[k] = p[k * STRIDE];
    dft<R, INV>(v);
#pragma unroll
    for (int k = 0; k < R; ++k) p[k * STRIDE] = v[k];
}

// G planes per block (planes_per_sys is a multiple of G).
template <int NX, int NY>
__global__ __launch_bounds__(512) void k_plane_fwd(const cplx* __restrict__ in, cplx* __restrict__ out, int G,
                                                   int planes_per_sys, const SysState* __restrict__ st,
                                                   const cplx* __restrict__ twx, const cplx* __restrict__ twy) {
    using S = PlaneShape<NX, NY>;
    extern __shared__ cplx lds_dyn[];
    const int blk = xcd_remap(blockIdx.x, gridDim.x);
    const int plane0 = blk * G, nt = blockDim.x;
    if (st != nullptr && st[plane0 / planes_per_sys].status != ST_RUNNING) return;
    const cplx* src = in + (size_t)plane0 * S::NP;
    cplx* dst = out + (size_t)plane0 * S::NP;

    for (int i = threadIdx.x; i < G * S::Y2 * NX; i += nt) {   // y, sweep 1: from memory
        const int g = i / (S::Y2 * NX), r = i - g * (S::Y2 * NX), n2 = r / NX, x = r - n2 * NX;
        cplx v[S::Y1];
#pragma unroll
        for (int k = 0; k < S::Y1; ++k) v[k] = src[g * S::NP + (n2 + S::Y2 * k) * NX + x];
        dft<S::Y1, false>(v);
        twiddle_all<S::Y1, false>(v, twy, n2);
        cplx* p = lds_dyn + (g * NY + n2) * S::RS + x;
#pragma unroll
        for (int k = 0; k < S::Y1; ++k) p[S::Y2 * k * S::RS] = v[k];
    }
    __syncthreads();
    for (int i = threadIdx.x; i < G * S::Y1 * NX; i += nt) {   // y, sweep 2
        const int gk = i / NX, x = i - gk * NX;                // g Y1 + k1
        sweep_lds<S::Y2, false, S::RS>(lds_dyn + gk * S::Y2 * S::RS + x);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < G * S::X2 * NY; i += nt) {   // x, sweep 1
        const int g = i / (S::X2 * NY), r = i - g * (S::X2 * NY), n2 = r / NY, y = r - n2 * NY;
        cplx* p = lds_dyn + (g * NY + y) * S::RS + n2;
        cplx v[S::X1];
#pragma unroll
        for (int k = 0; k < S::X1; ++k) v[k] = p[S::X2 * k];
        dft<S::X1, false>(v);
        twiddle_all<S::X1, false>(v, twx, n2);
#pragma unroll
        for (int k = 0; k < S::X1; ++k) p[S::X2 * k] = v[k];
    }
    __syncthreads();
    for (int i = threadIdx.x; i < G * S::X1 * NY; i += nt) {   // x, sweep 2: to memory
        const int g = i / (S::X1 * NY), r = i - g * (S::X1 * NY), k1 = r / NY, y = r - k1 * NY;
        const cplx* p = lds_dyn + (g * NY + y) * S::RS + S::X2 * k1;
        cplx v[S::X2];
#pragma unroll
        for (int k = 0; k < S::X2; ++k) v[k] = p[k];
        dft<S::X2, false>(v);
        cplx* o = dst + g * S::NP + S::X2 * k1 * NY + y;
#pragma unroll
        for (int k = 0; k < S::X2; ++k) st_wt(o + k * NY, v[k]);
    }
}

// The inverse pass with the epilogues of k_rows that a run-time code selects
// (EPI_STORE, EPI_APPLY, EPI_BICG_V, EPI_BICG_T, EPI_TRUERES), one partial
// record per block.  The arithmetic of each epilogue is that of k_rows.
template <int NX, int NY>
__global__ __launch_bounds__(512) void k_plane_inv(const cplx* __restrict__ in, cplx* __restrict__ out,
                                                   const cplx* __restrict__ u, const cplx* __restrict__ aux,
                                                   double* __restrict__ partials, int epi, int G,
                                                   int planes_per_sys, SysState* __restrict__ st,
                                                   const cplx* __restrict__ twx, const cplx* __restrict__ twy) {
    using S = PlaneShape<NX, NY>;
    extern __shared__ cplx lds_dyn[];
    __shared__ double red[8 * kPartialNV];
    const int blk = xcd_remap(blockIdx.x, gridDim.x);
    const int plane0 = blk * G, nt = blockDim.x;
    const int sys = plane0 / planes_per_sys;
    if (st != nullptr && st[sys].status != ST_RUNNING) return;
    const size_t off = (size_t)plane0 * S::NP;
    const cplx* src = in + off;

    for (int i = threadIdx.x; i < G * S::X1 * NY; i += nt) {   // x, sweep 2 undone: from memory
        const int g = i / (S::X1 * NY), r = i - g * (S::X1 * NY), k1 = r / NY, y = r - k1 * NY;
        const cplx* s = src + g * S::NP + S::X2 * k1 * NY + y;
        cplx v[S::X2];
#pragma unroll
        for (int k = 0; k < S::X2; ++k) v[k] = s[k * NY];
        dft<S::X2, true>(v);
        cplx* p = lds_dyn + (g * NY + y) * S::RS + S::X2 * k1;
#pragma unroll
        for (int k = 0; k < S::X2; ++k) p[k] = v[k];
    }
    __syncthreads();
    for (int i = threadIdx.x; i < G * S::X2 * NY; i += nt) {   // x, sweep 1 undone
        const int g = i / (S::X2 * NY), r = i - g * (S::X2 * NY), n2 = r / NY, y = r - n2 * NY;
        cplx* p = lds_dyn + (g * NY + y) * S::RS + n2;
        cplx v[S::X1];
#pragma unroll
        for (int k = 0; k < S::X1; ++k) v[k] = p[S::X2 * k];
        twiddle_all<S::X1, true>(v, twx, n2);
        dft<S::X1, true>(v);
#pragma unroll
        for (int k = 0; k < S::X1; ++k) p[S::X2 * k] = v[k];
    }
    __syncthreads();
    for (int i = threadIdx.x; i < G * S::Y1 * NX; i += nt) {   // y, sweep 2 undone
        const int gk = i / NX, x = i - gk * NX;
        sweep_lds<S::Y2, true, S::RS>(lds_dyn + gk * S::Y2 * S::RS + x);
    }
    __syncthreads();
    const bool need_u = epi != EPI_STORE;
    const bool need_a = epi == EPI_BICG_V || epi == EPI_BICG_T || epi == EPI_TRUERES;
    double acc[kPartialNV] = {};
    for (int i = threadIdx.x; i < G * S::Y2 * NX; i += nt) {   // y, sweep 1 undone: the epilogue
        const int g = i / (S::Y2 * NX), r = i - g * (S::Y2 * NX), n2 = r / NX, x = r - n2 * NX;
        const size_t base = off + g * S::NP + n2 * NX + x;
        constexpr int R = S::Y1, ST = S::Y2 * NX;
        cplx uu[R], av[R];   // in flight during the butterfly
#pragma unroll
        for (int k = 0; k < R; ++k) {
            if (need_u) uu[k] = u[base + k * ST];
            if (need_a) av[k] = aux[base + k * ST];
        }
        const cplx* p = lds_dyn + (g * NY + n2) * S::RS + x;
        cplx v[R];
#pragma unroll
        for (int k = 0; k < R; ++k) v[k] = p[S::Y2 * k * S::RS];
        twiddle_all<R, true>(v, twy, n2);
        dft<R, true>(v);
        cplx* o = out + base;
        if (epi == EPI_STORE) {
#pragma unroll
            for (int k = 0; k < R; ++k) st_wt(o + k * ST, v[k]);
            continue;
        }
#pragma unroll
        for (int k = 0; k < R; ++k) v[k] = csub(uu[k], v[k]);   // A u
        if (epi == EPI_TRUERES) {
#pragma unroll
            for (int k = 0; k < R; ++k) v[k] = csub(av[k], v[k]);   // b - A u
        }
#pragma unroll
        for (int k = 0; k < R; ++k) st_wt(o + k * ST, v[k]);
        if (epi == EPI_BICG_V) {
#pragma unroll
            for (int k = 0; k < R; ++k) {
                const cplx a = av[k], w = v[k];
                acc[0] += (double)a.x * w.x + (double)a.y * w.y;
                acc[1] += (double)a.x * w.y - (double)a.y * w.x;
            }
        } else if (epi == EPI_TRUERES) {
#pragma unroll
            for (int k = 0; k < R; ++k) {
                const cplx w = v[k];
                acc[0] += (double)w.x * w.x + (double)w.y * w.y;
            }
        } else if (epi == EPI_BICG_T) {
#pragma unroll
            for (int k = 0; k < R; ++k) {
                const cplx w = v[k], q = uu[k], h = av[k];
                acc[0] += (double)w.x * q.x + (double)w.y * q.y;
                acc[1] += (double)w.x * q.y - (double)w.y * q.x;
                acc[2] += (double)w.x * w.x + (double)w.y * w.y;
                acc[3] += (double)q.x * q.x + (double)q.y * q.y;
                acc[4] += (double)h.x * q.x + (double)h.y * q.y;   // <r^, s>
                acc[5] += (double)h.x * q.y - (double)h.y * q.x;
                acc[6] += (double)h.x * w.x + (double)h.y * w.y;   // <r^, t>
                acc[7] += (double)h.x * w.y - (double)h.y * w.x;
            }
        }
    }
    if (!need_a) return;   // uniform: no records
    const int nb = planes_per_sys / G, bi = blk - sys * nb;
    block_sum_store<kPartialNV>(acc, red, partials + ((size_t)sys * nb + bi) * kPartialNV);
    // the iteration is complete up to its solution update
    if (epi == EPI_BICG_T && bi == 0 && threadIdx.x == 0) st[sys].iter += 1;
}

// Launches both passes of one (NX, NY).
template <int NX, int NY>
inline hipError_t plane_launch(int epi, const PlaneGeom& g, const cplx* in, cplx* out, const cplx* u,
                               const cplx* aux, double* part, int nplanes, int planes_per_sys, SysState* st,
                               const cplx* tw, hipStream_t s) {
    const cplx* twx = tw + twiddle_offset(NX);
    const cplx* twy = tw + twiddle_offset(NY);
    const dim3 grid((unsigned)(nplanes / g.G)), block((unsigned)(epi == PLANE_FWD ? g.threads : g.threads_inv));
    if (epi == PLANE_FWD) {
        hipError_t e = allow_lds(k_plane_fwd<NX, NY>, g.lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((k_plane_fwd<NX, NY>), grid, block, g.lds, s, in, out, g.G, planes_per_sys, st, twx, twy);
    } else {
        hipError_t e = allow_lds(k_plane_inv<NX, NY>, g.lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((k_plane_inv<NX, NY>), grid, block, g.lds, s, in, out, u, aux, part, epi, g.G,
                           planes_per_sys, st, twx, twy);
    }
    return hipGetLastError();
}

template <int NX, int NY>
inline hipError_t plane_try(int ny, int epi, const PlaneGeom& g, const cplx* in, cplx* out, const cplx* u,
                            const cplx* aux, double* part, int nplanes, int pps, SysState* st, const cplx* tw,
                            hipStream_t s, bool& hit) {
    if constexpr (plane_size_ok(NX, NY)) {
        if (ny == NY) {
            hit = true;
            return plane_launch<NX, NY>(epi, g, in, out, u, aux, part, nplanes, pps, st, tw, s);
        }
    }
    return hipSuccess;
}

// Every ny of one nx.
template <int NX>
inline hipError_t plane_any(int ny, int epi, const PlaneGeom& g, const cplx* in, cplx* out, const cplx* u,
                            const cplx* aux, double* part, int nplanes, int pps, SysState* st, const cplx* tw,
                            hipStream_t s) {
    bool hit = false;
    hipError_t e = hipSuccess;
#define FW_NY(N) \
    if (!hit) e = plane_try<NX, N>(ny, epi, g, in, out, u, aux, part, nplanes, pps, st, tw, s, hit);
    FW_NY(16) FW_NY(20) FW_NY(24) FW_NY(32) FW_NY(40) FW_NY(48) FW_NY(64) FW_NY(80) FW_NY(96) FW_NY(128) FW_NY(160)
    FW_NY(192) FW_NY(256)
#undef FW_NY
    return hit ? e : hipErrorInvalidValue;
}

FW_END
