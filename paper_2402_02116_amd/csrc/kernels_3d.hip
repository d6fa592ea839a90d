// Kernels of the 3-D, generally anisotropic LS solve, J and J* (the
// 21-constant form of eqs. decom, u_2 and dC; the six-strain vectors of the
// abbreviated subscript section; App. C for the VTI set):
//   k_stencil3        - contrast stencil b = w~^2 drho u + div_h(dC : E_h u) on
//                       [nsys][3][nz][ny][nx] fields, with the BiCGSTAB vector
//                       update of its input fused into the load (bicg.h);
//   k_axis            - FFT along y or z (a strided axis) in place;
//   k_green3          - the z transforms around the multiplication by the 3 x 3
//                       Green's tensor G_hat(k) = (Gamma(k) - rho0 w~^2 I)^-1;
//   k_point_sources3, k_gather3, k_scatter_conj3 - sources and receivers;
//   k_correlate3      - the adjoint correlation of eq. ad1 summed over
//                       systems in FP64.
// The x transforms are the row kernels of the 2-D path (rows of nx points), or
// with the y transforms the plane kernels (plane_kernels.h).
#include <algorithm>
#include <numeric>
#include <type_traits>

#include "bicg.h"
#include "fft_kernels.h"

FW_BEGIN
__device__ __forceinline__ int wrapm(int i, int n) {
    const int r = i % n;
    return r < 0 ? r + n : r;
}

// ------------------------------------------------------ contrast stencil --
// Number of stiffness maps of a parametrisation (the density map follows).
template <bool GEN>
struct Params3 { static constexpr int NS = GEN ? 21 : 5; };

// sigma = dC e for one cell: VTI maps (dC11, dC13, dC33, dC55, dC66), with
// dC12 = dC11 - 2 dC66, dC22 = dC11, dC23 = dC13, dC44 = dC55 (App. C), or
// the 21 constants of the upper triangle in row-major order.
template <bool GEN>
__device__ __forceinline__ void stress3(const real* m, int mstride, const cplx (&e)[6], cplx (&s)[6]) {
    if constexpr (!GEN) {
        const real c11 = m[0], c13 = m[mstride], c33 = m[2 * mstride], c55 = m[3 * mstride],
                   c66 = m[4 * mstride];
        const real c12 = c11 - 2.f * c66;
        s[0] = mkc(c11 * e[0].x + c12 * e[1].x + c13 * e[2].x, c11 * e[0].y + c12 * e[1].y + c13 * e[2].y);
        s[1] = mkc(c12 * e[0].x + c11 * e[1].x + c13 * e[2].x, c12 * e[0].y + c11 * e[1].y + c13 * e[2].y);
        s[2] = mkc(c13 * (e[0].x + e[1].x) + c33 * e[2].x, c13 * (e[0].y + e[1].y) + c33 * e[2].y);
        s[3] = cscale(e[3], c55);
        s[4] = cscale(e[4], c55);
        s[5] = cscale(e[5], c66);
    } else {
        real c[6][6];
        int p = 0;
#pragma unroll
        for (int i = 0; i < 6; ++i)
#pragma unroll
            for (int j = i; j < 6; ++j) {
                c[i][j] = m[p * mstride];
                c[j][i] = c[i][j];
                ++p;
            }
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            real sx = 0, sy = 0;
#pragma unroll
            for (int j = 0; j < 6; ++j) {
                sx += c[i][j] * e[j].x;
                sy += c[i][j] * e[j].y;
            }
            s[i] = mkc(sx, sy);
        }
    }
}

// A block owns a TX x TY x TZ tile of cells and loops over S systems of the
// same problem.  The stiffness contrast of the tile plus a 1-cell halo and the
// density of the tile go to LDS once.  Per system:
//   1. the input field (the vector update applied) on the tile plus a 2-cell
//      halo goes to LDS; own cells write the updated vectors;
//   2. the stress s' = dC e' (e' = raw central differences, 2 dx times the
//      Voigt strain) on the tile plus a 1-cell halo, in LDS;
//   3. b = w~^2 drho u + (1 / 4 dx^2) div'(s') on the tile.
// Tiles may overhang the grid: loads wrap periodically and only in-grid
// cells are written.
template <int TX, int TY, int TZ>
struct Tile3 {
    static constexpr int HX = TX + 4, HY = TY + 4, HZ = TZ + 4, HC = HX * HY * HZ;
    static constexpr int SX = TX + 2, SY = TY + 2, SZ = TZ + 2, SC = SX * SY * SZ;
    static constexpr int OC = TX * TY * TZ;
};

template <bool GEN, int TX, int TY, int TZ>
inline size_t stencil3_lds() {
    using T = Tile3<TX, TY, TZ>;
    return (size_t)(3 * T::HC + 6 * T::SC) * sizeof(cplx) +
           (size_t)(Params3<GEN>::NS * T::SC + T::OC) * sizeof(real);
}

template <int VM, bool GEN, int TX, int TY, int TZ>
__global__ __launch_bounds__(256) void k_stencil3(const cplx* __restrict__ u, const cplx* __restrict__ a1,
                                                  const cplx* __restrict__ a2, cplx* __restrict__ wout,
                                                  cplx* __restrict__ b, const real* __restrict__ maps, ProbDev3 pd,
                                                  int S, SysState* __restrict__ st, const double* __restrict__ part,
                                                  int np, cplx* __restrict__ rhat, const cplx* __restrict__ a3,
                                                  cplx* __restrict__ xio, cplx* __restrict__ rout) {
    using T = Tile3<TX, TY, TZ>;
    constexpr int NS = Params3<GEN>::NS;
    extern __shared__ __align__(16) unsigned char lds3[];
    cplx* su = reinterpret_cast<cplx*>(lds3);          // [3][HC]
    cplx* ss = su + 3 * T::HC;                           // [6][SC]
    real* sm = reinterpret_cast<real*>(ss + 6 * T::SC);  // [NS][SC], then rho [OC]
    __shared__ double red[4 * kPartialNV];
    __shared__ int s_status;

    const int nx = pd.nx, ny = pd.ny, nz = pd.nz;
    const size_t cells = (size_t)nx * ny * nz;
    const int ntx = (nx + TX - 1) / TX, nty = (ny + TY - 1) / TY;
    const int nsg = (pd.nsys + S - 1) / S;
    const int blk = xcd_remap(blockIdx.x, gridDim.x);
    const int tile = blk / nsg;
    const int sys0 = (blk - tile * nsg) * S;
    const int x0 = (tile % ntx) * TX, y0 = ((tile / ntx) % nty) * TY, z0 = (tile / (ntx * nty)) * TZ;
    auto gcell = [&](int dx_, int dy_, int dz_) -> size_t {
        return ((size_t)wrapm(z0 + dz_, nz) * ny + wrapm(y0 + dy_, ny)) * nx + wrapm(x0 + dx_, nx);
    };

    // contrast of the stress region and density of the tile
    for (int q = threadIdx.x; q < T::SC; q += 256) {
        const int sx = q % T::SX, sy = (q / T::SX) % T::SY, sz = q / (T::SX * T::SY);
        const size_t g = gcell(sx - 1, sy - 1, sz - 1);
#pragma unroll
        for (int p = 0; p < NS; ++p) sm[p * T::SC + q] = maps[(size_t)p * cells + g];
    }
    for (int o = threadIdx.x; o < T::OC; o += 256) {
        const int ox = o % TX, oy = (o / TX) % TY, oz = o / (TX * TY);
        sm[NS * T::SC + o] = maps[(size_t)NS * cells + gcell(ox, oy, oz)];
    }

    const real sc = pd.inv4dx2;
    for (int sys = sys0; sys < sys0 + S && sys < pd.nsys; ++sys) {
        if (st != nullptr) {
            // one read per block, broadcast: another block's writer may change
            // the word meanwhile, and every thread must take the same branch
            if (threadIdx.x == 0) s_status = st[sys].status;
            __syncthreads();
            const int stw = s_status;
            __syncthreads();
            if constexpr (VM == VM_PX) {
                if (!closing_enters(stw, kStampPx)) continue;
            } else {
                if (stw != ST_RUNNING) {
                    // the iteration's closing kernel is done: drop its tag
                    if (VM == VM_S && st_tag(stw) != 0 && tile == 0 && threadIdx.x == 0) st[sys].status = st_code(stw);
                    continue;
                }
            }
        }
        cplx c1 = mkc(0.f, 0.f), c2 = mkc(0.f, 0.f), c3 = mkc(0.f, 0.f);
        bool fresh = false;
        int step = SS_FULL;
        if constexpr (VM != VM_NONE) {
            step = stencil_scalars<VM>(st, sys, part, np, red, tile == 0 && threadIdx.x == 0, c1, c2, c3, fresh);
            if (step == SS_SKIP) continue;
        }
        const size_t so = (size_t)sys * 3 * cells;
        // VM_PX on an own cell: r = s - omega t, x += alpha p_old + omega s
        auto close_iteration = [&](size_t gi) {
            const cplx sv = u[so + gi], tv = a3[so + gi], pv = a1[so + gi];
            const cplx rv = close_r(sv, tv, c2);
            st_wt(rout + so + gi, rv);
            st_wt(xio + so + gi, close_x(xio[so + gi], pv, sv, c3, c2));
            if (fresh) st_wt(rhat + so + gi, rv);
        };
        if constexpr (VM == VM_PX) {
            if (step == SS_XONLY) {   // stopped: the last solution update only
                for (int o = threadIdx.x; o < T::OC; o += 256) {
                    const int ox = o % TX, oy = (o / TX) % TY, oz = o / (TX * TY);
                    if (x0 + ox >= nx || y0 + oy >= ny || z0 + oz >= nz) continue;
                    const size_t g = gcell(ox, oy, oz);
#pragma unroll
                    for (int c = 0; c < 3; ++c) close_iteration(c * cells + g);
                }
                continue;
            }
        }
        // input field value at index gi of this system (component offset included)
        auto field = [&](size_t gi) -> cplx {
            if constexpr (VM == VM_NONE) {
                return u[so + gi];
            } else if constexpr (VM == VM_P) {
                const cplx rv = u[so + gi];
                if (fresh) return rv;
                const cplx pv = a1[so + gi], vv = a2[so + gi];
                return cadd(rv, cmul(c1, csub(pv, cmul(c2, vv))));
            } else if constexpr (VM == VM_PX) {
                const cplx rv = close_r(u[so + gi], a3[so + gi], c2);
                if (fresh) return rv;
                const cplx pv = a1[so + gi], vv = a2[so + gi];
                return cadd(rv, cmul(c1, csub(pv, cmul(c2, vv))));
            } else {
                return csub(u[so + gi], cmul(c1, a1[so + gi]));
            }
        };
        __syncthreads();   // the previous system's reads of su / ss are done
        for (int h = threadIdx.x; h < T::HC; h += 256) {
            const int hx = h % T::HX, hy = (h / T::HX) % T::HY, hz = h / (T::HX * T::HY);
            const size_t g = gcell(hx - 2, hy - 2, hz - 2);
            const bool own = hx >= 2 && hx < TX + 2 && hy >= 2 && hy < TY + 2 && hz >= 2 && hz < TZ + 2 &&
                             x0 + hx - 2 < nx && y0 + hy - 2 < ny && z0 + hz - 2 < nz;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const size_t gi = c * cells + g;
                const cplx f = field(gi);
                su[c * T::HC + h] = f;
                if constexpr (VM != VM_NONE) {
                    if (own) {
                        st_wt(wout + so + gi, f);
                        if constexpr (VM == VM_P) {
                            if (fresh) st_wt(rhat + so + gi, f);   // p = r here
                        } else if constexpr (VM == VM_PX) {
                            close_iteration(gi);
                        }
                    }
                }
            }
        }
        __syncthreads();
        constexpr int DY = T::HX, DZ = T::HX * T::HY;
        for (int q = threadIdx.x; q < T::SC; q += 256) {
            const int sx = q % T::SX, sy = (q / T::SX) % T::SY, sz = q / (T::SX * T::SY);
            const int h = ((sz + 1) * T::HY + sy + 1) * T::HX + sx + 1;
            cplx d[3][3];   // d[c][j]: raw difference of component c along axis j
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const cplx* w = su + c * T::HC + h;
                d[c][0] = csub(w[1], w[-1]);
                d[c][1] = csub(w[DY], w[-DY]);
                d[c][2] = csub(w[DZ], w[-DZ]);
            }
            const cplx e[6] = {d[0][0], d[1][1], d[2][2], cadd(d[1][2], d[2][1]), cadd(d[0][2], d[2][0]),
                               cadd(d[0][1], d[1][0])};
            cplx s[6];
            stress3<GEN>(sm + q, T::SC, e, s);
#pragma unroll
            for (int i = 0; i < 6; ++i) ss[i * T::SC + q] = s[i];
        }
        __syncthreads();
        constexpr int EY = T::SX, EZ = T::SX * T::SY;
        for (int o = threadIdx.x; o < T::OC; o += 256) {
            const int ox = o % TX, oy = (o / TX) % TY, oz = o / (TX * TY);
            if (x0 + ox >= nx || y0 + oy >= ny || z0 + oz >= nz) continue;
            const int q = ((oz + 1) * T::SY + oy + 1) * T::SX + ox + 1;
            auto dd = [&](int i, int off) { return csub(ss[i * T::SC + q + off], ss[i * T::SC + q - off]); };
            // b_i = sum_j D_j sigma_ij, Voigt (xx, yy, zz, yz, xz, xy) = (0..5)
            const cplx bx = cadd(cadd(dd(0, 1), dd(5, EY)), dd(4, EZ));
            const cplx by = cadd(cadd(dd(5, 1), dd(1, EY)), dd(3, EZ));
            const cplx bz = cadd(cadd(dd(4, 1), dd(3, EY)), dd(2, EZ));
            const int h = ((oz + 2) * T::HY + oy + 2) * T::HX + ox + 2;
            const cplx wr = cscale(pd.w2, sm[NS * T::SC + o]);
            const size_t g = so + gcell(ox, oy, oz);
            st_wt(b + g, cadd(cmul(wr, su[h]), cscale(bx, sc)));
            st_wt(b + g + cells, cadd(cmul(wr, su[T::HC + h]), cscale(by, sc)));
            st_wt(b + g + 2 * cells, cadd(cmul(wr, su[2 * T::HC + h]), cscale(bz, sc)));
        }
    }
}

// The same stencil (plain: b of the input u) marching along z: a block owns
// a TX x TY column of cells over the z range [z0, z1) of one system and walks
// it plane by plane.  FULL: TX = nx, so that the column has halo rows only (a
// narrower one fetches a whole cache line for every two cells of its halo
// columns: with 16 x 16 columns at 80 x 40 the L1 fetched nine times the
// field from L2 and the pass waited on it; the halo columns in LDS are the
// row's own other end).  Each thread owns one cell of the column, and the
// first NH threads (in the rotated numbering below) also one cell of the
// halo: the NR cells next to the column, where the stress is needed too, then
// those at distance two (and the corners between them).
// LDS holds the input planes z+1 (for the x and y differences) and z (each
// thread's own cells), and the stress s' of plane z (all but s'_zz, which only
// the own z difference takes) and of z+1 as it is made.  Step z takes the
// input of plane z+2 at the thread's cells from registers, forms the stress of
// plane z+1 at the own and halo cells, then b on plane z, and puts plane z+2 in
// the place of plane z: one barrier per step.  The loop is unrolled by two, the
// period in which registers and LDS copies change roles, so that nothing is
// moved between registers; the next plane and its maps are in flight
// meanwhile.  Every input plane of the range is read once, plus three halo
// planes and the own column of a fourth.
// The BiCGSTAB update modes run as a streaming pass before it
// (launch_bicg_update): fused into this kernel they held one or two waves
// per SIMD.
template <int TX, int TY, bool FULL>
struct March3 {
    static constexpr int HX = TX + 4, HY = TY + 4, HP = HX * HY;   // input plane with halo 2
    static constexpr int SX = TX + 2, SY = TY + 2, SP = SX * SY;   // stress plane with halo 1
    static constexpr int NT = TX * TY;                             // one thread per own cell
    static constexpr int NR = FULL ? 2 * TX : 2 * (TX + TY);       // halo cells next to the column
    static constexpr int NH = FULL ? 4 * TX : 2 * NR + 4;          // halo cells of an input plane
    static constexpr int NL = 5;                                   // stress components in LDS
    // Copies of the stress planes: with one, a step waits a second time, for
    // the stress of plane z to be read before that of z+1 replaces it, but 1.4
    // times as many blocks fit in LDS (64^3 x 32: 133 -> 127 us, 128 x 128 x 64
    // x 4: 74 -> 65 us).  A block of five wavefronts puts two on one SIMD, so
    // that the registers allow two blocks at most, which fit with two copies
    // (80 x 40 x 32 x 100: 180 us, 187 with one).
    static constexpr int NB = NT / 64 == 5 ? 2 : 1;
};

template <int TX, int TY, bool FULL>
inline size_t march3_lds() {
    using M = March3<TX, TY, FULL>;
    return (size_t)(2 * 3 * M::HP + M::NB * M::NL * M::SP) * sizeof(cplx);
}

// Halo cell k of the column, relative to its first cell: those at distance 1,
// then 2 (rows above and below, and unless FULL columns left and right), then
// the corners between them.
template <int TX, int TY, bool FULL>
__device__ __forceinline__ void halo_cell(int k, int& x, int& y) {
    constexpr int NR = March3<TX, TY, FULL>::NR;
    if (!FULL && k >= 2 * NR) {
        x = (k & 1) ? TX : -1;
        y = (k & 2) ? TY : -1;
        return;
    }
    const int d = k < NR ? 1 : 2;
    k -= (d - 1) * NR;
    if (k < TX) {
        x = k;
        y = -d;
    } else if (FULL || k < 2 * TX) {
        x = k - TX;
        y = TY - 1 + d;
    } else if (k < 2 * TX + TY) {
        x = -d;
        y = k - 2 * TX;
    } else {
        x = TX - 1 + d;
        y = k - 2 * TX - TY;
    }
}

template <bool GEN, int TX, int TY, bool FULL>
__global__ __launch_bounds__(TX * TY, sizeof(real) == 8 ? 1 : GEN ? 3 : 4) void k_stencil3z(const cplx* __restrict__ u, cplx* __restrict__ b,
                                                       const real* __restrict__ maps, ProbDev3 pd, int ZC,
                                                       const SysState* __restrict__ st) {
    using M = March3<TX, TY, FULL>;
    static_assert(M::NH <= M::NT && M::NT % 64 == 0, "one halo cell per thread at most");
    constexpr int NS = Params3<GEN>::NS;
    extern __shared__ __align__(16) unsigned char lds3[];
    cplx* const sp = reinterpret_cast<cplx*>(lds3);   // input plane [2][3][HP]
    cplx* const ss = sp + 2 * 3 * M::HP;              // stress plane [2][NL][SP]: xx, yy, yz, xz, xy
    __shared__ int s_status;

    const int nx = pd.nx, ny = pd.ny, nz = pd.nz;
    const size_t cells = (size_t)nx * ny * nz;
    const int ntx = (nx + TX - 1) / TX, nty = (ny + TY - 1) / TY;
    // neighbouring blocks (on one XCD, resident together): the neighbouring
    // columns and z ranges of the same system, which read each other's cells
    // as their halos while those cache lines are still in the XCD's L2
    const int ncol = ntx * nty * ((nz + ZC - 1) / ZC);
    const int blk = xcd_remap(blockIdx.x, gridDim.x);
    const int sys = blk / ncol;
    const int col = blk - sys * ncol;
    const int x0 = (col % ntx) * TX, y0 = ((col / ntx) % nty) * TY, z0 = (col / (ntx * nty)) * ZC;
    const int z1 = min(z0 + ZC, nz);
    const int t = threadIdx.x;
    const int tx = t % TX, ty = t / TX;
    const bool own_xy = x0 + tx < nx && y0 + ty < ny;

    if (st != nullptr) {
        if (t == 0) s_status = st[sys].status;
        __syncthreads();
        if (s_status != ST_RUNNING) return;
    }
    // this system's vectors: uniform plane addresses and 32-bit offsets of the
    // thread's cells within a plane
    const cplx* __restrict__ us = u + (size_t)sys * 3 * cells;
    cplx* __restrict__ bs = b + (size_t)sys * 3 * cells;
    const uint32_t plane = (uint32_t)nx * (uint32_t)ny;
    // planes z0-2 .. z1+1 lie within one period of the axis
    auto zoff = [&](int z) -> size_t { return (size_t)((uint32_t)(z < 0 ? z + nz : (z >= nz ? z - nz : z)) * plane); };
    const uint32_t xy0 = (uint32_t)wrapm(y0 + ty, ny) * nx + wrapm(x0 + tx, nx);

    // the thread's halo cell; the wavefront with the extra stress differs from
    // block to block, so that these wavefronts spread over the SIMDs
    const int rt = ((t >> 6) + blk) % (M::NT / 64) * 64 + (t & 63);
    const bool has1 = rt < M::NH, st1 = rt < M::NR;
    int hx1 = 0, hy1 = 0;
    if (has1) halo_cell<TX, TY, FULL>(rt, hx1, hy1);
    // Every load of the march is unconditional, so that the compiler counts
    // the loads in flight exactly and waits for one step's while the next
    // step's travel (a load under a branch made every step wait for its own
    // prefetch): threads without a halo cell load their own cell again.
    const uint32_t xy1 = has1 ? (uint32_t)wrapm(y0 + hy1, ny) * nx + wrapm(x0 + hx1, nx) : xy0;
    const uint32_t xys = st1 ? xy1 : xy0;
    const int h0 = (ty + 2) * M::HX + tx + 2, h1 = (hy1 + 2) * M::HX + hx1 + 2;
    const int q0 = (ty + 1) * M::SX + tx + 1, q1 = (hy1 + 1) * M::SX + hx1 + 1;

    struct Cells {   // one plane of the input at the own and the halo cell
        cplx o[3], h[3];
    };
    auto load_own = [&](cplx (&r)[3], int z) {
        const cplx* p = us + zoff(z);
#pragma unroll
        for (int c = 0; c < 3; ++c) r[c] = (p + c * cells)[xy0];
    };
    auto load_cells = [&](Cells& r, int z) {
        load_own(r.o, z);
        const cplx* p = us + zoff(z);
#pragma unroll
        for (int c = 0; c < 3; ++c) r.h[c] = (p + c * cells)[xy1];
    };
    auto load_maps = [&](real (&m)[NS], int z, uint32_t xy) {
        const real* p = maps + zoff(z);
#pragma unroll
        for (int q = 0; q < NS; ++q) m[q] = (p + q * cells)[xy];
    };
    const real* rho = maps + (size_t)NS * cells;
    // s' = dC e' at position h of the LDS input plane w; z differences from
    // the planes below (lo) and above (hi)
    auto stress_at = [&](const cplx* w, const cplx (&lo)[3], const cplx (&hi)[3], const real (&m)[NS],
                         cplx (&sg)[6]) {
        cplx d[3][3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            d[c][0] = csub(w[c * M::HP + 1], w[c * M::HP - 1]);
            d[c][1] = csub(w[c * M::HP + M::HX], w[c * M::HP - M::HX]);
            d[c][2] = csub(hi[c], lo[c]);
        }
        const cplx e[6] = {d[0][0], d[1][1], d[2][2], cadd(d[1][2], d[2][1]), cadd(d[0][2], d[2][0]),
                           cadd(d[0][1], d[1][0])};
        stress3<GEN>(m, 1, e, sg);
    };
    // FULL: a row's two end cells are also the halo cells of its other end
    const bool end0 = FULL && (tx < 2 || tx >= TX - 2), end1 = FULL && (hx1 < 2 || hx1 >= TX - 2);
    const int o0 = tx < 2 ? TX : -TX, o1 = hx1 < 2 ? TX : -TX;
    auto put_plane = [&](int k, const Cells& f) {
        cplx* w = sp + k * 3 * M::HP;
#pragma unroll
        for (int c = 0; c < 3; ++c) w[c * M::HP + h0] = f.o[c];
        if (end0) {
#pragma unroll
            for (int c = 0; c < 3; ++c) w[c * M::HP + h0 + o0] = f.o[c];
        }
        if (has1) {
#pragma unroll
            for (int c = 0; c < 3; ++c) w[c * M::HP + h1] = f.h[c];
            if (end1) {
#pragma unroll
                for (int c = 0; c < 3; ++c) w[c * M::HP + h1 + o1] = f.h[c];
            }
        }
    };
    auto put_stress = [&](int k, int q, const cplx (&s)[6]) {
        cplx* w = ss + (M::NB == 2 ? k : 0) * M::NL * M::SP + q;
        w[0] = s[0];
        w[M::SP] = s[1];
        w[2 * M::SP] = s[3];
        w[3 * M::SP] = s[4];
        w[4 * M::SP] = s[5];
    };
    auto put_own_stress = [&](int k, const cplx (&s)[6]) {
        put_stress(k, q0, s);
        if (FULL && (tx == 0 || tx == TX - 1)) put_stress(k, q0 + o0, s);
    };
    struct ZStress {   // the own stress components whose z difference is taken
        cplx zz, yz, xz;
    };
    // the maps of the next stress plane, loaded a step ahead; the 21-constant
    // form loads them at the step instead (registers)
    constexpr int NM = GEN ? 1 : NS;
    struct Maps {
        real o[NM], h[NM], rho;
    };
    auto load_step_maps = [&](Maps& m, int z) {   // stress of plane z + 1, density of plane z
        if constexpr (!GEN) {
            load_maps(m.o, z + 1, xy0);
            load_maps(m.h, z + 1, xys);
        }
        m.rho = (rho + zoff(z))[xy0];
    };

    // the thread's cells of LDS input plane k
    auto get_own = [&](cplx (&r)[3], int k) {
#pragma unroll
        for (int c = 0; c < 3; ++c) r[c] = sp[(k * 3 + c) * M::HP + h0];
    };
    auto get_halo = [&](cplx (&r)[3], int k) {
#pragma unroll
        for (int c = 0; c < 3; ++c) r[c] = sp[(k * 3 + c) * M::HP + h1];
    };

    // ---- prologue: stress of plane z0-1 (own) and z0 (own and halo), input planes z0 and z0+1
    Cells fa, fb;     // planes z + 2 and z + 3
    ZStress sa, sb;   // own stress of planes z - 1 and z
    Maps ma, mb;
    {
        cplx fm2[3];
        Cells fm1, f0, f1;
        real m0[NS], m1[NS], mh[NS];
        load_cells(fm1, z0 - 1);
        load_cells(f0, z0);
        load_own(fm2, z0 - 2);
        load_maps(m0, z0 - 1, xy0);
        load_cells(f1, z0 + 1);
        load_maps(m1, z0, xy0);
        load_maps(mh, z0, xys);
        load_cells(fa, z0 + 2);
        load_step_maps(ma, z0);
        put_plane(0, fm1);
        put_plane(1, f0);
        __syncthreads();
        cplx s[6];
        stress_at(sp + h0, fm2, f0.o, m0, s);
        sa = ZStress{s[2], s[3], s[4]};
        stress_at(sp + 3 * M::HP + h0, fm1.o, f1.o, m1, s);
        sb = ZStress{s[2], s[3], s[4]};
        put_own_stress(0, s);
        if (st1) {
            stress_at(sp + 3 * M::HP + h1, fm1.h, f1.h, mh, s);
            put_stress(0, q1, s);
        }
        __syncthreads();
        put_plane(0, f1);
        __syncthreads();
    }

    const real sc = pd.inv4dx2;
    // step z (LDS copy K holds input plane z + 1 and stress plane z, the other
    // input plane z): c = input plane z + 2; d receives plane z + 3; old = own
    // stress of z - 1, replaced by that of z + 1
    auto plane_step = [&](auto kc, int z, const Cells& c, Cells& d, ZStress& old, Maps& m, Maps& mn) {
        constexpr int K = decltype(kc)::value;
        real mm[NS];   // 21 constants: this step's maps, issued before the next plane
        if constexpr (GEN) load_maps(mm, z + 1, xy0);
        load_cells(d, z + 3);   // at the end of the range: planes that exist but are not used
        load_step_maps(mn, z + 1);
        cplx a[3], s0[6];
        get_own(a, 1 - K);
        const cplx* w = sp + K * 3 * M::HP;
        if constexpr (GEN) stress_at(w + h0, a, c.o, mm, s0);
        else stress_at(w + h0, a, c.o, m.o, s0);
        const cplx* q = ss + (M::NB == 2 ? K : 0) * M::NL * M::SP + q0;
        auto dxy = [&](int i, int off) { return csub(q[i * M::SP + off], q[i * M::SP - off]); };
        const cplx bx = cadd(cadd(dxy(0, 1), dxy(4, M::SX)), csub(s0[4], old.xz));
        const cplx by = cadd(cadd(dxy(4, 1), dxy(1, M::SX)), csub(s0[3], old.yz));
        const cplx bz = cadd(cadd(dxy(3, 1), dxy(2, M::SX)), csub(s0[2], old.zz));
        const cplx wr = cscale(pd.w2, m.rho);
        cplx* o = bs + zoff(z);
        if (FULL || own_xy) {   // a FULL column does not overhang the grid
            st_wt(o + xy0, cadd(cmul(wr, a[0]), cscale(bx, sc)));
            st_wt(o + cells + xy0, cadd(cmul(wr, a[1]), cscale(by, sc)));
            st_wt(o + 2 * cells + xy0, cadd(cmul(wr, a[2]), cscale(bz, sc)));
        }
        old = ZStress{s0[2], s0[3], s0[4]};
        if constexpr (M::NB == 1) __syncthreads();   // the stress of plane z is read
        put_own_stress(1 - K, s0);
        if (st1) {
            cplx s1[6];
            get_halo(a, 1 - K);
            if constexpr (GEN) {
                load_maps(mm, z + 1, xy1);
                stress_at(w + h1, a, c.h, mm, s1);
            } else {
                stress_at(w + h1, a, c.h, m.h, s1);
            }
            put_stress(1 - K, q1, s1);
        }
        put_plane(1 - K, c);
        __syncthreads();
    };
    using K0 = std::integral_constant<int, 0>;
    using K1 = std::integral_constant<int, 1>;
    for (int z = z0; z < z1; z += 2) {   // ranges hold an even number of planes
        plane_step(K0{}, z, fa, fb, sa, ma, mb);
        plane_step(K1{}, z + 1, fb, fa, sb, mb, ma);
    }
}

template <bool GEN, int TX, int TY, bool FULL>
static hipError_t stencil3z_launch(const StencilArgs& a, const ProbDev3& pd, const SysState* st, hipStream_t s) {
    if (FULL && (pd.nx != TX || pd.ny % TY != 0)) return hipErrorInvalidValue;
    const int ntx = (pd.nx + TX - 1) / TX, nty = (pd.ny + TY - 1) / TY;
    if (pd.nz % 4 != 0) return hipErrorInvalidValue;   // every supported length is a multiple of four
    const size_t lds = march3_lds<TX, TY, FULL>();
    // z ranges of ZC planes (a multiple of four, at most 32) by the plane steps
    // one after the other: a range's steps, its start counted as four (three
    // halo planes and their latency), times the rounds in which the chip takes
    // the blocks (by LDS, and by the wavefronts per SIMD that the registers
    // allow with a block's first wavefront on the first SIMD).  The shortest
    // range within an eighth of the fewest steps, since the neighbours of a
    // short range's halos are resident with it (80 x 40 x 32 x 100: 175 us by
    // ranges of 16, 186 by 32); the fewest steps where a start loads 63 maps a
    // cell (21 constants at 50 systems: 132 us by 32, 157 by 16).  Few blocks,
    // against halving the range until there are 1024: 96 x 64 x 48 x 7
    // 39.8 -> 36 us, 80 x 40 x 32 x 1 14.8 -> 9.7 us.
    constexpr int kWaves = TX * TY / 64, kPerSimd = sizeof(real) == 8 ? 1 : GEN ? 3 : 4;
    const int bpc = std::max(1, std::min((int)(kMaxLds / (lds + 64)), kPerSimd / ((kWaves + 3) / 4)));
    auto steps = [&](int zc) -> long long {
        const long long nb = (long long)ntx * nty * ((pd.nz + zc - 1) / zc) * pd.nsys;
        return (nb + kCUs * bpc - 1) / (kCUs * bpc) * (zc + 4);
    };
    int ZC = std::min(pd.nz, 32);
    long long best = steps(ZC);
    for (int zc = ZC - 4; zc >= 4; zc -= 4) best = std::min(best, steps(zc));
    const long long limit = GEN ? best : best + best / 8;
    if (GEN) {
        while (steps(ZC) > limit) ZC -= 4;
    } else {
        for (ZC = 4; steps(ZC) > limit;) ZC += 4;
    }
    const long long blocks = (long long)ntx * nty * ((pd.nz + ZC - 1) / ZC) * pd.nsys;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    hipError_t e = allow_lds(k_stencil3z<GEN, TX, TY, FULL>, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_stencil3z<GEN, TX, TY, FULL>), dim3((unsigned)blocks), dim3(TX * TY), lds, s, a.u, a.b, a.maps,
                       pd, ZC, st);
    return hipGetLastError();
}

// Tile of the build: 8 x 8 x 4 cells (complex64), 4 x 4 x 4 (complex128,
// twice the bytes per value).
#ifdef FW_C128
constexpr int kT3X = 4, kT3Y = 4, kT3Z = 4;
#else
constexpr int kT3X = 8, kT3Y = 8, kT3Z = 4;
#endif

template <int VM, bool GEN>
static hipError_t stencil3_launch(const StencilArgs& a, const ProbDev3& pd, SysState* st, hipStream_t s) {
    const int ntiles = ((pd.nx + kT3X - 1) / kT3X) * ((pd.ny + kT3Y - 1) / kT3Y) * ((pd.nz + kT3Z - 1) / kT3Z);
    int S = 1;
    while (S < pd.nsys && (long long)ntiles * ((pd.nsys + 2 * S - 1) / (2 * S)) >= 2048) S *= 2;
    S = std::min(S, std::max(pd.nsys, 1));
    const int blocks = ntiles * ((pd.nsys + S - 1) / S);
    const size_t lds = stencil3_lds<GEN, kT3X, kT3Y, kT3Z>();
    hipError_t e = allow_lds(k_stencil3<VM, GEN, kT3X, kT3Y, kT3Z>, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_stencil3<VM, GEN, kT3X, kT3Y, kT3Z>), dim3(blocks), dim3(256), lds, s, a.u, a.a1, a.a2,
                       a.wout, a.b, a.maps, pd, S, st, a.part, a.np, a.rhat, a.a3, a.xio, a.rout);
    return hipGetLastError();
}

// Whether a grid takes the z-marching stencil: not one thinner than 8 cells
// in y, which takes the tiled kernel.
static bool march_ok(const ProbDev3& pd) { return pd.ny >= 8 && pd.nx >= 16; }

template <bool GEN>
static hipError_t stencil3z_any(const StencilArgs& a, const ProbDev3& pd, const SysState* st, hipStream_t s) {
#ifndef FW_C128
#define FW_FULL(X, Y) \
    if (pd.nx == X && pd.ny % Y == 0) return stencil3z_launch<GEN, X, Y, true>(a, pd, st, s);
    FW_FULL(16, 16) FW_FULL(24, 8) FW_FULL(32, 8) FW_FULL(40, 8) FW_FULL(48, 4) FW_FULL(64, 4) FW_FULL(80, 4)
    FW_FULL(96, 4) FW_FULL(128, 4)
#undef FW_FULL
#endif
    // 16 x 16 or 32 x 8 cells, whichever overhangs the grid less
    const long long q = (long long)((pd.nx + 15) / 16) * 16 * ((pd.ny + 15) / 16) * 16;
    const long long r = (long long)((pd.nx + 31) / 32) * 32 * ((pd.ny + 7) / 8) * 8;
    return q <= r ? stencil3z_launch<GEN, 16, 16, false>(a, pd, st, s)
                  : stencil3z_launch<GEN, 32, 8, false>(a, pd, st, s);
}

template <int VM, bool GEN>
static hipError_t stencil3_any(const StencilArgs& a, const ProbDev3& pd, SysState* st, hipStream_t s) {
    if (!march_ok(pd)) return stencil3_launch<VM, GEN>(a, pd, st, s);   // the tiled kernel, update fused
    StencilArgs p = a;
    if constexpr (VM != VM_NONE) {
        // the vector update as its own streaming pass, then the plain
        // z-marching stencil on the updated input (the marching kernel with
        // the update fused held one or two waves per SIMD: 206 against
        // 217 ms for the 80 x 40 x 32 x 100-system step)
        hipError_t e = launch_bicg_update(VM, a, 3LL * pd.nx * pd.ny * pd.nz, pd.nsys, st, s);
        if (e != hipSuccess) return e;
        p.u = a.wout;
    }
    return stencil3z_any<GEN>(p, pd, st, s);
}

template <bool GEN>
static hipError_t stencil3_vm(int vm, const StencilArgs& a, const ProbDev3& pd, SysState* st, hipStream_t s) {
    if (vm == VM_NONE) return stencil3_any<VM_NONE, GEN>(a, pd, st, s);
    if (vm == VM_P) return stencil3_any<VM_P, GEN>(a, pd, st, s);
    if (vm == VM_PX) return stencil3_any<VM_PX, GEN>(a, pd, st, s);
    return stencil3_any<VM_S, GEN>(a, pd, st, s);
}

hipError_t launch_stencil3(int vm, const StencilArgs& a, const ProbDev3& pd, SysState* st, hipStream_t s) {
    if (vm < 0 || vm > 3 || (vm != 0 && !st) || ((vm == VM_P || vm == VM_PX) && !a.rhat) ||
        (vm == VM_PX && (!a.a3 || !a.xio || !a.rout)) || (vm != VM_NONE && !a.wout))
        return hipErrorInvalidValue;
    return pd.params == kParamsGeneral ? stencil3_vm<true>(vm, a, pd, st, s) : stencil3_vm<false>(vm, a, pd, st, s);
}

// ------------------------------------------------------ strided axes -----
// Transforms along an axis of length N with stride S (the product of the
// faster dimensions): the data is [nslab][N][S], one slab per (system,
// component, outer index).  A block takes W adjacent columns of one slab;
// thread (t, c) holds positions t + T m of column c.
struct AxisLds {
    cplx* base;
    int stride, PL;
    __device__ __forceinline__ cplx& operator()(int f, int pos) const { return padded(f, lds_pad(pos)); }
    __device__ __forceinline__ cplx& padded(int f, int pp) const { return base[(f * PL + pp) * stride]; }
};

// out = gscale (Gamma' - ga I)^-1 b for the real symmetric scaled
// Christoffel matrix Gamma' (entries xx, yy, zz, yz, xz, xy), by the
// adjugate of the complex symmetric 3 x 3 matrix.
__device__ __forceinline__ void green_mul3(cplx (&b)[3], const real (&g)[6], cplx ga, real gscale) {
    const cplx mxx = mkc(g[0] - ga.x, -ga.y), myy = mkc(g[1] - ga.x, -ga.y), mzz = mkc(g[2] - ga.x, -ga.y);
    const real myz = g[3], mxz = g[4], mxy = g[5];
    const cplx axx = mkc(cmul(myy, mzz).x - myz * myz, cmul(myy, mzz).y);
    const cplx ayy = mkc(cmul(mxx, mzz).x - mxz * mxz, cmul(mxx, mzz).y);
    const cplx azz = mkc(cmul(mxx, myy).x - mxy * mxy, cmul(mxx, myy).y);
    const cplx axy = csub(mkc(mxz * myz, 0.f), cscale(mzz, mxy));
    const cplx axz = csub(mkc(mxy * myz, 0.f), cscale(myy, mxz));
    const cplx ayz = csub(mkc(mxy * mxz, 0.f), cscale(mxx, myz));
    const cplx det = cadd(cmul(mxx, axx), cadd(cscale(axy, mxy), cscale(axz, mxz)));
    const real s = gscale * green_rcp(det.x * det.x + det.y * det.y);
    const cplx inv = mkc(det.x * s, -det.y * s);
    const cplx gx = cmul(inv, b[0]), gy = cmul(inv, b[1]), gz = cmul(inv, b[2]);
    b[0] = cadd(cmul(axx, gx), cadd(cmul(axy, gy), cmul(axz, gz)));
    b[1] = cadd(cmul(axy, gx), cadd(cmul(ayy, gy), cmul(ayz, gz)));
    b[2] = cadd(cmul(axz, gx), cadd(cmul(ayz, gy), cmul(azz, gz)));
}

// Wavenumber of index i on an n-point axis: exact (dk * signed index) or the
// central-difference symbol sin(2 pi i / n) / dx.
__device__ __forceinline__ real axis_k(int i, int n, real dk, real dx, bool central) {
    const int si = fft_signed(i, n);
    return central ? rsinpi(2.0f * (real)si / (real)n) / dx : (real)si * dk;
}

template <int N, int P, bool INV>
__global__ __launch_bounds__(256) void k_axis(cplx* __restrict__ data, int S, int W, int slabs_per_sys,
                                              const SysState* __restrict__ st, const cplx* __restrict__ tw) {
    using FS = FftShape<N, P>;
    constexpr int T = FS::T;
    constexpr int PL = PaddedLen<N>::value;
    extern __shared__ cplx lds_dyn[];

    const int tid = threadIdx.x;
    const int c = tid % W, t = tid / W;
    const int ncb = S / W;
    const int blk = xcd_remap(blockIdx.x, gridDim.x);
    const int slab = blk / ncb;
    const int col = (blk - slab * ncb) * W + c;
    if (st != nullptr && st[slab / slabs_per_sys].status != ST_RUNNING) return;
    const bool active = t < T;
    cplx* base = data + (size_t)slab * N * S + col;

    cplx v[1][P];
#pragma unroll
    for (int m = 0; m < P; ++m) v[0][m] = active ? base[(size_t)(t + T * m) * S] : mkc(0.f, 0.f);
    AxisLds lds{active ? lds_dyn + c : lds_dyn + (size_t)PL * W, active ? W : 1, PL};
    fft_run<N, P, INV, 1>(v, active ? t : 0, tw, lds);
    if (active) {
#pragma unroll
        for (int m = 0; m < P; ++m) st_wt(base + (size_t)(t + T * m) * S, v[0][m]);
    }
}

// ------------------------------------------------------------- z pass -----
// z transforms of the three components of W columns, the 3 x 3 Green multiply
// and the inverse transforms, in place on [nsys][3][N][S].  As in the plane
// passes, N = R1 R2 and a transform is two sweeps in place in LDS:
//   1. a butterfly of radix R1 of one component per item, from memory;
//   2. the radix-R2 butterflies of all three components per item, the Green
//      multiply of the R2 wavenumbers k1 + R1 k2 it then holds, and the
//      inverse butterflies;
//   3. sweep 1 undone, to memory.
// Small radices in sweep 2 keep the three components of an item in few
// registers.  The terms of Gamma' without kz are formed once per column.
// Against all points of three components in one thread
// (two wavefronts per SIMD at 12 points): 32 points at 80 x 40 x 100 90 -> 83
// us (a read and a write of the field at the rate of a large copy take 96,
// part of it stays in the memory-side cache), 48 points at 96 x 64 x 7 35.5 ->
// 20.1 us, 64 points at 64 x 64 x 32 79 -> 61 us.
template <int N>
struct GreenShape {
    static constexpr int R2 = N < 128 ? 4 : 8, R1 = N / R2;
};

constexpr int kGreenThreads = sizeof(real) == 8 ? 256 : 512;   // complex128 needs the registers

template <int N, int W>
__global__ __launch_bounds__(kGreenThreads) void k_green3(cplx* __restrict__ data, int S, const SysState* __restrict__ st,
                                                const cplx* __restrict__ tw, ProbDev3 pd, PlaneOrder ord) {
    constexpr int R1 = GreenShape<N>::R1, R2 = GreenShape<N>::R2;
    extern __shared__ cplx lds_dyn[];   // [3][N][W]
    const int ncb = S / W, nt = blockDim.x;
    const int blk = xcd_remap(blockIdx.x, gridDim.x);
    const int sys = blk / ncb;
    if (st != nullptr && st[sys].status != ST_RUNNING) return;
    const int col0 = (blk - sys * ncb) * W;
    cplx* base = data + (size_t)sys * 3 * N * S + col0;

    for (int i = threadIdx.x; i < 3 * R2 * W; i += nt) {
        const int c = i % W, q = i / W, f = q / R2, n2 = q - f * R2;
        const cplx* s = base + ((size_t)f * N + n2) * S + c;
        cplx v[R1];
#pragma unroll
        for (int k = 0; k < R1; ++k) v[k] = s[(size_t)k * R2 * S];
        dft<R1, false>(v);
        twiddle_all<R1, false>(v, tw, n2);
        cplx* p = lds_dyn + (f * N + n2) * W + c;
#pragma unroll
        for (int k = 0; k < R1; ++k) p[k * R2 * W] = v[k];
    }
    __syncthreads();
    for (int i = threadIdx.x; i < R1 * W; i += nt) {
        const int c = i % W, k1 = i / W, col = col0 + c;
        cplx* p = lds_dyn + k1 * R2 * W + c;
        cplx v[3][R2];
#pragma unroll
        for (int f = 0; f < 3; ++f) {
#pragma unroll
            for (int k = 0; k < R2; ++k) v[f][k] = p[(f * N + k) * W];
            dft<R2, false>(v[f]);
        }
        int ix = col % pd.nx, iy = col / pd.nx;
        if (ord.planes) {   // column y + ny x of the positions R2 k1 + k2
            const int px = col / pd.ny, py = col - px * pd.ny;
            ix = px / ord.x2 + ord.x1 * (px % ord.x2);
            iy = py / ord.y2 + ord.y1 * (py % ord.y2);
        }
        const bool central = pd.symbol == 1;
        const real kx = axis_k(ix, pd.nx, pd.dk[0], pd.dx, central);
        const real ky = axis_k(iy, pd.ny, pd.dk[1], pd.dx, central);
        // products of two different components: 0 at an even axis's Nyquist index
        const real kxo = (pd.nx % 2 == 0 && ix == pd.nx / 2) ? 0.f : kx;
        const real kyo = (pd.ny % 2 == 0 && iy == pd.ny / 2) ? 0.f : ky;
        // The entries are summed in the order of mono, so that their rounding
        // (which a wavenumber near the slowness surface amplifies) does not
        // depend on the path: terms of a column that are the same for all of
        // its wavenumbers first, then those in kz; an orthotropic medium has
        // the latter in five entries only.
        const real kx2 = kx * kx, ky2 = ky * ky, kxy = kxo * kyo;
        real g0[6];
#pragma unroll
        for (int e = 0; e < 6; ++e) g0[e] = pd.gq[e][0] * kx2 + pd.gq[e][1] * ky2;
#pragma unroll
        for (int k = 0; k < R2; ++k) {
            const int iz = k1 + R1 * k;
            const real kz = axis_k(iz, N, pd.dk[2], pd.dx, central);
            const real kzo = (N % 2 == 0 && iz == N / 2) ? 0.f : kz;
            const real kz2 = kz * kz, kyz = kyo * kzo, kxz = kxo * kzo;
            real g[6];
            if (pd.ortho) {
#pragma unroll
                for (int e = 0; e < 3; ++e) g[e] = g0[e] + pd.gq[e][2] * kz2;
                g[3] = pd.gq[3][3] * kyz;
                g[4] = pd.gq[4][4] * kxz;
                g[5] = pd.gq[5][5] * kxy;
            } else {
#pragma unroll
                for (int e = 0; e < 6; ++e) {
                    real a = g0[e] + pd.gq[e][2] * kz2;
                    a += pd.gq[e][3] * kyz;
                    a += pd.gq[e][4] * kxz;
                    a += pd.gq[e][5] * kxy;
                    g[e] = a;
                }
            }
            cplx b3[3] = {v[0][k], v[1][k], v[2][k]};
            green_mul3(b3, g, pd.ga, pd.gscale);
            v[0][k] = b3[0];
            v[1][k] = b3[1];
            v[2][k] = b3[2];
            __builtin_amdgcn_sched_barrier(0);   // one point at a time: bounded registers
        }
#pragma unroll
        for (int f = 0; f < 3; ++f) {
            dft<R2, true>(v[f]);
#pragma unroll
            for (int k = 0; k < R2; ++k) p[(f * N + k) * W] = v[f][k];
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < 3 * R2 * W; i += nt) {
        const int c = i % W, q = i / W, f = q / R2, n2 = q - f * R2;
        const cplx* p = lds_dyn + (f * N + n2) * W + c;
        cplx v[R1];
#pragma unroll
        for (int k = 0; k < R1; ++k) v[k] = p[k * R2 * W];
        twiddle_all<R1, true>(v, tw, n2);
        dft<R1, true>(v);
        cplx* o = base + ((size_t)f * N + n2) * S + c;
#pragma unroll
        for (int k = 0; k < R1; ++k) st_wt(o + (size_t)k * R2 * S, v[k]);
    }
}

// Points per thread of the strided passes: radix-8 passes for 2^k, 12 for
// 3 * 2^k, 10 for 5 * 2^k.
int axis_points(int n) { return (n % 5 == 0) ? 10 : (n % 3 == 0) ? 12 : 8; }

#define FW_AXIS_SIZES(X) \
    X(16) X(20) X(24) X(32) X(40) X(48) X(64) X(80) X(96) X(128) X(160) X(192) X(256)

bool axis3_size_supported(int n) {
#define FW_IS(N) if (n == N) return true;
    FW_AXIS_SIZES(FW_IS)
#undef FW_IS
    return false;
}

template <int N, bool INV>
static hipError_t axis_launch(cplx* data, int S, int nslab, int slabs_per_sys, const SysState* st, const cplx* tw,
                              hipStream_t s) {
    constexpr int P = (N % 5 == 0) ? 10 : (N % 3 == 0) ? 12 : 8;
    constexpr int T = N / P;
    int W = 16;
    while (W > 1 && (W * T > 256 || S % W != 0)) W /= 2;
    const int threads = ((W * T + 63) / 64) * 64;
    const size_t lds = (size_t)(PaddedLen<N>::value * (W + 1)) * sizeof(cplx);
    hipError_t e = allow_lds(k_axis<N, P, INV>, lds);
    if (e != hipSuccess) return e;
    const long long blocks = (long long)nslab * (S / W);
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_axis<N, P, INV>), dim3((unsigned)blocks), dim3(threads), lds, s, data, S, W, slabs_per_sys,
                       st, tw + twiddle_offset(N));
    return hipGetLastError();
}

template <int N, int W>
static hipError_t green3_launch(cplx* data, int S, int nsys, const SysState* st, const cplx* tw, const ProbDev3& pd,
                                const PlaneOrder& ord, hipStream_t s) {
    using G = GreenShape<N>;
    const size_t lds = (size_t)3 * N * W * sizeof(cplx);
    hipError_t e = allow_lds(k_green3<N, W>, lds);
    if (e != hipSuccess) return e;
    const long long blocks = (long long)nsys * (S / W);
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    const int items = std::max(3 * G::R2 * W, G::R1 * W);
    const int threads = std::min(kGreenThreads, (items + 63) / 64 * 64);
    hipLaunchKernelGGL((k_green3<N, W>), dim3((unsigned)blocks), dim3(threads), lds, s, data, S, st,
                       tw + twiddle_offset(N), pd, ord);
    return hipGetLastError();
}

// 16 columns per block (a full cache line of each plane), 8 where those would
// leave LDS for two blocks per CU only or do not divide the plane, 4 for the
// lengths that are odd multiples of 4 on grids one cell thick.
template <int N>
static hipError_t green3_any(cplx* data, int S, int nsys, const SysState* st, const cplx* tw, const ProbDev3& pd,
                             const PlaneOrder& ord, hipStream_t s) {
    if constexpr ((size_t)3 * N * 16 * sizeof(cplx) <= kMaxLds / 3)
        if (S % 16 == 0) return green3_launch<N, 16>(data, S, nsys, st, tw, pd, ord, s);
    if (S % 8 == 0) return green3_launch<N, 8>(data, S, nsys, st, tw, pd, ord, s);
    if (S % 4 == 0) return green3_launch<N, 4>(data, S, nsys, st, tw, pd, ord, s);
    return hipErrorInvalidValue;
}

hipError_t launch_axis3(int mode, int n, cplx* data, int S, int nslab, int slabs_per_sys, const SysState* st,
                        const cplx* tw, const ProbDev3& pd, hipStream_t s, bool planes) {
    PlaneOrder ord{};
    if (planes) {
        if (!plane_size_ok(pd.nx, pd.ny)) return hipErrorInvalidValue;
        ord = PlaneOrder{1, plane_radix(pd.nx), pd.nx / plane_radix(pd.nx), plane_radix(pd.ny),
                         pd.ny / plane_radix(pd.ny)};
    }
#define FW_AX(N)                                                                                     \
    if (n == N) {                                                                                    \
        if (mode == AX_FWD) return axis_launch<N, false>(data, S, nslab, slabs_per_sys, st, tw, s);  \
        if (mode == AX_INV) return axis_launch<N, true>(data, S, nslab, slabs_per_sys, st, tw, s);   \
        if (mode == AX_GREEN) return green3_any<N>(data, S, nslab, st, tw, pd, ord, s);              \
    }
    FW_AXIS_SIZES(FW_AX)
#undef FW_AX
    return hipErrorInvalidValue;
}

// -------------------------------------------------------- x-y planes -----
// Planes per block: whole planes until the block has about 256 threads' work
// (a butterfly each) in its widest sweep.  Threads: up to 512, since a sweep's
// items rarely divide evenly (80 x 40 x 32 x 100, forward: 95 us by 512
// threads, 98 by 256, 320 or 384).  The inverse pass holds 118 registers, 16
// wavefronts per CU: blocks of four wavefronts where four of them fit in LDS
// (140 -> 135 us there; 48 x 48 x 64 x 9: 20.1 -> 17.6 us), else of eight
// (96 x 64 x 48 x 7: 24.2 us against 27.5 by four); five or six wavefronts
// leave a quarter of them unused (157 us).
PlaneGeom plane_geom(int nx, int ny, int planes_per_sys) {
    const int x1 = plane_radix(nx), y1 = plane_radix(ny);
    const int items = nx * ny / std::min(std::min(x1, nx / x1), std::min(y1, ny / y1));
    const size_t lds = (size_t)ny * (nx + 1) * sizeof(cplx);
    PlaneGeom g;
    g.G = std::max(1, std::min(256 / items, (int)(kPlaneLds / lds)));
    while (planes_per_sys % g.G != 0) --g.G;
    g.threads = std::min(512, ((g.G * items + 63) / 64) * 64);
    g.lds = g.G * lds;
    g.threads_inv = 4 * (g.lds + 1024) <= kMaxLds ? std::min(256, g.threads) : g.threads;
    return g;
}

hipError_t launch_plane_a(int, int, int, const PlaneGeom&, const cplx*, cplx*, const cplx*, const cplx*, double*, int,
                          int, SysState*, const cplx*, hipStream_t);
hipError_t launch_plane_b(int, int, int, const PlaneGeom&, const cplx*, cplx*, const cplx*, const cplx*, double*, int,
                          int, SysState*, const cplx*, hipStream_t);
hipError_t launch_plane_c(int, int, int, const PlaneGeom&, const cplx*, cplx*, const cplx*, const cplx*, double*, int,
                          int, SysState*, const cplx*, hipStream_t);

hipError_t launch_plane(int nx, int ny, int epi, const cplx* in, cplx* out, const cplx* u, const cplx* aux,
                        double* part, int nplanes, int planes_per_sys, SysState* st, const cplx* tw, hipStream_t s) {
    const bool rec = epi == EPI_BICG_V || epi == EPI_BICG_T || epi == EPI_TRUERES;
    if (!plane_size_ok(nx, ny) || nplanes < 1 || planes_per_sys < 1 || nplanes % planes_per_sys != 0 ||
        !(epi == PLANE_FWD || epi == EPI_STORE || epi == EPI_APPLY || rec) || !in || !out || in == out ||
        (epi >= EPI_APPLY && !u) || (rec && (!aux || !part)) || (epi == EPI_BICG_T && !st))
        return hipErrorInvalidValue;
    const PlaneGeom g = plane_geom(nx, ny, planes_per_sys);
    hipError_t e = launch_plane_a(nx, ny, epi, g, in, out, u, aux, part, nplanes, planes_per_sys, st, tw, s);
    if (e == hipErrorInvalidValue)
        e = launch_plane_b(nx, ny, epi, g, in, out, u, aux, part, nplanes, planes_per_sys, st, tw, s);
    if (e == hipErrorInvalidValue)
        e = launch_plane_c(nx, ny, epi, g, in, out, u, aux, part, nplanes, planes_per_sys, st, tw, s);
    return e;
}

// ---------------------------------------------------- sources, receivers --
// f must be zero on entry: one force per system, F / dx^3 at (ix, iy, iz).
__global__ void k_point_sources3(cplx* __restrict__ f, const int32_t* __restrict__ ixyz,
                                 const double* __restrict__ force, ProbDev3 pd) {
    const int sys = blockIdx.x * blockDim.x + threadIdx.x;
    if (sys >= pd.nsys) return;
    const size_t cells = (size_t)pd.nx * pd.ny * pd.nz;
    const size_t g = ((size_t)ixyz[3 * sys + 2] * pd.ny + ixyz[3 * sys + 1]) * pd.nx + ixyz[3 * sys];
    const double inv = 1.0 / ((double)pd.dx * (double)pd.dx * (double)pd.dx);
#pragma unroll
    for (int c = 0; c < 3; ++c) f[(size_t)sys * 3 * cells + c * cells + g] = mkc((real)(force[3 * sys + c] * inv), 0.f);
}

hipError_t launch_point_sources3(cplx* f, const int32_t* src_ixyz, const double* src_f, const ProbDev3& pd,
                                 hipStream_t s) {
    hipLaunchKernelGGL(k_point_sources3, dim3((pd.nsys + 63) / 64), dim3(64), 0, s, f, src_ixyz, src_f, pd);
    return hipGetLastError();
}

// d[sys][rec][c] = w[sys][c][iz][iy][ix]
__global__ void k_gather3(const cplx* __restrict__ w, cplx* __restrict__ d, const int32_t* __restrict__ rec,
                          int nrec, ProbDev3 pd) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= pd.nsys * nrec * 3) return;
    const int c = i % 3, rr = (i / 3) % nrec, sys = i / (3 * nrec);
    const size_t cells = (size_t)pd.nx * pd.ny * pd.nz;
    const size_t g = ((size_t)rec[3 * rr + 2] * pd.ny + rec[3 * rr + 1]) * pd.nx + rec[3 * rr];
    d[i] = w[(size_t)sys * 3 * cells + c * cells + g];
}

hipError_t launch_gather3(const cplx* w, cplx* d, const int32_t* rec, int nrec, const ProbDev3& pd, hipStream_t s) {
    const int total = pd.nsys * nrec * 3;
    hipLaunchKernelGGL(k_gather3, dim3((total + 255) / 256), dim3(256), 0, s, w, d, rec, nrec, pd);
    return hipGetLastError();
}

// f (zero on entry) += conj(d) at the receivers; one thread per (sys, c) walks
// the receivers in order, so repeated receivers add deterministically.
// f += R^T conj(d) with the receivers in the host's stable cell order (perm,
// run lengths glen): one thread per (system, run, component), each run
// summed in receiver order.
__global__ void k_scatter_conj3(const cplx* __restrict__ d, cplx* __restrict__ f, const int32_t* __restrict__ rec,
                                const int32_t* __restrict__ perm, const int32_t* __restrict__ glen, int nrec,
                                ProbDev3 pd) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (size_t)pd.nsys * nrec * 3) return;
    const int c = (int)(i % 3);
    const size_t q = i / 3;
    const int k = (int)(q % nrec), sys = (int)(q / nrec);
    const int n = glen[k];
    if (n == 0) return;
    const cplx* ds = d + (size_t)sys * nrec * 3 + c;
    const int r0 = perm[k];
    cplx acc = cconj(ds[3 * (size_t)r0]);
    for (int j = 1; j < n; ++j) acc = cadd(acc, cconj(ds[3 * (size_t)perm[k + j]]));
    const size_t cells = (size_t)pd.nx * pd.ny * pd.nz;
    cplx* fs = f + (size_t)sys * 3 * cells + c * cells;
    const size_t g = ((size_t)rec[3 * r0 + 2] * pd.ny + rec[3 * r0 + 1]) * pd.nx + rec[3 * r0];
    fs[g] = cadd(fs[g], acc);
}

hipError_t launch_scatter_conj3(const cplx* d, cplx* f, const int32_t* rec, const int32_t* perm,
                                const int32_t* glen, int nrec, const ProbDev3& pd, hipStream_t s) {
    const size_t total = (size_t)pd.nsys * nrec * 3;
    if (total == 0) return hipSuccess;
    hipLaunchKernelGGL(k_scatter_conj3, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, d, f, rec, perm, glen,
                       nrec, pd);
    return hipGetLastError();
}

// ------------------------------------------------------- correlation -----
// Per cell, summed over systems in FP64 (eq. ad1):
//   g_p   = -conj( sum_IJ e^a_I B^(p)_IJ e^b_J ) / (4 dx^2)   (raw differences e)
//   g_rho = conj( w~^2 sum_c u^a_c u^b_c ),
// for the VTI maps (C11, C13, C33, C55, C66) with App. C's B, or the 21
// constants with B^(IJ) = e_I e_J^T + e_J e_I^T (I != J), e_I e_I^T (I = J).
__device__ __forceinline__ void zacc(double& re, double& im, cplx a, cplx b, double w = 1.0) {
    re += w * ((double)a.x * b.x - (double)a.y * b.y);
    im += w * ((double)a.x * b.y + (double)a.y * b.x);
}

__device__ __forceinline__ void strain_raw3(const cplx* f, size_t cells, size_t c0, size_t xp, size_t xm, size_t yp,
                                            size_t ym, size_t zp, size_t zm, cplx (&e)[6]) {
    const cplx* ux = f;
    const cplx* uy = f + cells;
    const cplx* uz = f + 2 * cells;
    (void)c0;
    e[0] = csub(ux[xp], ux[xm]);
    e[1] = csub(uy[yp], uy[ym]);
    e[2] = csub(uz[zp], uz[zm]);
    e[3] = cadd(csub(uy[zp], uy[zm]), csub(uz[yp], uz[ym]));
    e[4] = cadd(csub(ux[zp], ux[zm]), csub(uz[xp], uz[xm]));
    e[5] = cadd(csub(ux[yp], ux[ym]), csub(uy[xp], uy[xm]));
}

template <bool GEN>
__global__ __launch_bounds__(256) void k_correlate3(const cplx* __restrict__ ua, const cplx* __restrict__ ub,
                                                    double2* __restrict__ g, ProbDev3 pd, int accumulate) {
    constexpr int NS = Params3<GEN>::NS;
    const int nx = pd.nx, ny = pd.ny, nz = pd.nz;
    const size_t cells = (size_t)nx * ny * nz;
    const size_t cell = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (cell >= cells) return;
    const int x = (int)(cell % nx), y = (int)((cell / nx) % ny), z = (int)(cell / ((size_t)nx * ny));
    auto at = [&](int xx, int yy, int zz) { return ((size_t)wrapm(zz, nz) * ny + wrapm(yy, ny)) * nx + wrapm(xx, nx); };
    const size_t xp = at(x + 1, y, z), xm = at(x - 1, y, z), yp = at(x, y + 1, z), ym = at(x, y - 1, z),
                 zp = at(x, y, z + 1), zm = at(x, y, z - 1);
    double acc[NS][2] = {};
    double rr = 0, ri = 0;
    for (int s = 0; s < pd.nsys; ++s) {
        const cplx* A = ua + (size_t)s * 3 * cells;
        const cplx* B = ub + (size_t)s * 3 * cells;
#pragma unroll
        for (int c = 0; c < 3; ++c) zacc(rr, ri, A[c * cells + cell], B[c * cells + cell]);
        cplx ea[6], eb[6];
        strain_raw3(A, cells, cell, xp, xm, yp, ym, zp, zm, ea);
        strain_raw3(B, cells, cell, xp, xm, yp, ym, zp, zm, eb);
        if constexpr (GEN) {
            int p = 0;
#pragma unroll
            for (int i = 0; i < 6; ++i)
#pragma unroll
                for (int j = i; j < 6; ++j) {
                    zacc(acc[p][0], acc[p][1], ea[i], eb[j]);
                    if (i != j) zacc(acc[p][0], acc[p][1], ea[j], eb[i]);
                    ++p;
                }
        } else {
            const cplx sa = cadd(ea[0], ea[1]), sb = cadd(eb[0], eb[1]);
            zacc(acc[0][0], acc[0][1], sa, sb);                                  // B^11
            zacc(acc[1][0], acc[1][1], sa, eb[2]);                               // B^13
            zacc(acc[1][0], acc[1][1], ea[2], sb);
            zacc(acc[2][0], acc[2][1], ea[2], eb[2]);                            // B^33
            zacc(acc[3][0], acc[3][1], ea[3], eb[3]);                            // B^55
            zacc(acc[3][0], acc[3][1], ea[4], eb[4]);
            zacc(acc[4][0], acc[4][1], ea[5], eb[5]);                            // B^66
            zacc(acc[4][0], acc[4][1], ea[0], eb[1], -2.0);
            zacc(acc[4][0], acc[4][1], ea[1], eb[0], -2.0);
        }
    }
    const double sc = (double)pd.inv4dx2;
    const double wr = pd.w2.x, wi = pd.w2.y;
#pragma unroll
    for (int p = 0; p <= NS; ++p) {
        double2* dst = g + (size_t)p * cells + cell;
        double ore, oim;
        if (p < NS) {
            ore = -acc[p][0] * sc;     // -conj(a) / (4 dx^2)
            oim = acc[p][1] * sc;
        } else {
            ore = wr * rr - wi * ri;   // conj(w~^2 rho)
            oim = -(wr * ri + wi * rr);
        }
        double2 o = accumulate ? *dst : double2{0.0, 0.0};
        o.x += ore;
        o.y += oim;
        *dst = o;
    }
}

hipError_t launch_correlate3(const cplx* ua, const cplx* ub, double2* g, const ProbDev3& pd, bool accumulate,
                             hipStream_t s) {
    const size_t cells = (size_t)pd.nx * pd.ny * pd.nz;
    const unsigned blocks = (unsigned)((cells + 255) / 256);
    if (pd.params == kParamsGeneral)
        hipLaunchKernelGGL(k_correlate3<true>, dim3(blocks), dim3(256), 0, s, ua, ub, g, pd, accumulate ? 1 : 0);
    else
        hipLaunchKernelGGL(k_correlate3<false>, dim3(blocks), dim3(256), 0, s, ua, ub, g, pd, accumulate ? 1 : 0);
    return hipGetLastError();
}

FW_END
