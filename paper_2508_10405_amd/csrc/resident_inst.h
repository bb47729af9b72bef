// The resident kernels of one row count per lane (RES_BZ); one source file per
// value, so that they compile side by side.
#include "resident_adj.h"
#include "resident_fwd.h"

namespace lsrtm {

template <int CX>
static hipError_t launch_cx(int kind, int nblocks, size_t lds, hipStream_t st, const ResArgs& a, hipEvent_t e0,
                            hipEvent_t e1) {
    auto go = [&](auto k) {
        if (e0) hipExtLaunchKernelGGL(k, dim3(nblocks), dim3(RES_NT), lds, st, e0, e1, 0, a);
        else k<<<dim3(nblocks), dim3(RES_NT), lds, st>>>(a);
        return hipGetLastError();
    };
    switch (kind) {
    case R_BG: return go(k2r_fwd<RES_BZ, CX, R_BG>);
    case R_SEG: return go(k2r_fwd<RES_BZ, CX, R_SEG>);
    case R_BORN: return go(k2r_fwd<RES_BZ, CX, R_BORN>);
    case R_BORN_RC: return go(k2r_fwd<RES_BZ, CX, R_BORN_RC>);
    case R_ADJ: return go(k2r_adj<RES_BZ, CX>);
    default: return hipErrorInvalidValue;
    }
}

template <>
hipError_t launch_resident_bz<RES_BZ>(int kind, int cx, int nblocks, size_t lds, hipStream_t st, const ResArgs& a,
                                      hipEvent_t e0, hipEvent_t e1) {
    switch (cx) {
    case 1: return launch_cx<1>(kind, nblocks, lds, st, a, e0, e1);
    case 2: return launch_cx<2>(kind, nblocks, lds, st, a, e0, e1);
    case 3: return launch_cx<3>(kind, nblocks, lds, st, a, e0, e1);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace lsrtm
