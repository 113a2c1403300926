// Fused forward x-y kernels, double.
#include "plane.hpp"

namespace dds {

template <>
void launch_xy_fwd<double>(int Py, int M, const double* in, cplx<double>* out, int64_t nplanes, int ny, int nx, int64_t wx,
                       const cplx<double>* tw, hipStream_t s, int zp) {
    if (nplanes <= 0) return;
    check_plane_launch(nplanes, zp);
#define CALL(PYV, MV) plane_fwd_launch<double, PYV, MV>(in, out, nplanes, ny, nx, wx, tw, s, zp)
    switch (Py) {
        case 16: DDS_PLANE_M(16, CALL) break;
        case 32: DDS_PLANE_M(32, CALL) break;
        case 64: DDS_PLANE_M(64, CALL) break;
        case 128: DDS_PLANE_M(128, CALL) break;
        default: fail(DDSTRESS_E_INVALID, "plane lengths not covered by the fused x-y kernels");
    }
#undef CALL
    check_hip(hipGetLastError(), "fused forward x-y launch");
}

}  // namespace dds
