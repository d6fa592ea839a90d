// x-y plane passes of 3-D problems with nx in {20, 32, 48, 80} (plane_kernels.h).
#include "plane_kernels.h"

FW_BEGIN
hipError_t launch_plane_b(int nx, int ny, int epi, const PlaneGeom& g, const cplx* in, cplx* out, const cplx* u,
                          const cplx* aux, double* part, int nplanes, int pps, SysState* st, const cplx* tw,
                          hipStream_t s) {
#define FW_NX(N) \
    if (nx == N) return plane_any<N>(ny, epi, g, in, out, u, aux, part, nplanes, pps, st, tw, s);
    FW_NX(20) FW_NX(32) FW_NX(48) FW_NX(80)
#undef FW_NX
    return hipErrorInvalidValue;
}
FW_END
