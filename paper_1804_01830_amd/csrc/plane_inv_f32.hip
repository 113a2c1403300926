// Fused inverse y-x kernels, float.
#include "plane.hpp"

namespace dds {

template <>
void launch_yx_inv<float>(int Py, int M, const cplx<float>* in, float* out, int64_t nplanes, int ny, int nx, int64_t wx,
                       const cplx<float>* tw, hipStream_t s, double* rowsq, int zp) {
    if (nplanes <= 0) return;
    check_plane_launch(nplanes, zp);
#define CALL(PYV, MV) plane_inv_launch<float, PYV, MV>(in, out, nplanes, ny, nx, wx, tw, s, rowsq, zp)
    switch (Py) {
        case 16: DDS_PLANE_M(16, CALL) break;
        case 32: DDS_PLANE_M(32, CALL) break;
        case 64: DDS_PLANE_M(64, CALL) break;
        case 128: DDS_PLANE_M(128, CALL) break;
        case 256:
            if (M != 128) fail(DDSTRESS_E_INVALID, "plane lengths not covered by the fused x-y kernels");
            CALL(256, 128);
            break;
        default: fail(DDSTRESS_E_INVALID, "plane lengths not covered by the fused x-y kernels");
    }
#undef CALL
    check_hip(hipGetLastError(), "fused inverse y-x launch");
}

}  // namespace dds
