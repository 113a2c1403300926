// Fused z kernels, register form.
#include "zreg.hpp"

namespace dds {

// The register form pays where several realisations share a staged tile.
// Measured at 128 x 128 x {8, 16, 32} and 64^3 against the best tile of the
// single-group form (us, register / single-group):
//   z length 16: three channels 21 / 20 at B = 4 (never taken); six 32 / 47 and nine 59 / 82 at B = 3, but 32 / 33
//                and 59 / 56 at B = 2
//   z length 32: three, six, nine channels 35 / 39, 74 / 99, 147 / 162 at B = 3; six 78 / 58 at B = 2
//   z length 64: three channels 168 / 157 at B = 6, 201 / 212 at B = 8 (but 429 / 425 for the whole evaluation,
//                where the pass follows the others), 278 / 303 at B = 12; six and nine 191 / 217 and 293 / 320 at B = 4
//   z length 128: three and six channels 63 / 72 and 122 / 145 at B = 4; nine 226 / 222 (never taken)
bool z_reg_applies(int N, int C, int B) {
    switch (N) {
        case 16: return C > 3 && B >= 3;
        case 32: return B >= 3;
        case 64: return B >= (C == 3 ? 12 : 4);
        case 128: return C < 9 && B >= 4;
        default: return false;
    }
}

int z_reg_tile(int N) { return 64 / z_reg_lanes(N); }

// As few rounds of up to four waves as the realisations need, evenly filled.
int z_reg_waves(int B) {
    const int rounds = (B + 3) / 4;
    return (B + rounds - 1) / rounds;
}

int z_reg_split(int N, int C) {
    const int vg = z_reg_vg(N, C);
    return vg > 0 ? 6 / vg : 1;
}

// The staged spectrum tile, and for eight lanes per column the twiddle table
// of both directions.
size_t z_reg_lds_bytes(int N, int C, int nkz) {
    const int lp = z_reg_lanes(N), vg = z_reg_vg(N, C);
    const size_t tile = (size_t)C * (vg > 0 ? vg : 6) * nkz * (64 / lp) * sizeof(float);
    return tile + (lp == 8 ? (size_t)2 * lane_tw_count<128, 8>() * lp * sizeof(cplx<float>) : 0);
}

void z_reg_dispatch(int N, int C, const cplx<float>* in, cplx<float>* out, const float* spec, const ZGeom& g,
                    const cplx<float>* tw, int64_t blocks, hipStream_t s) {
    if (!z_reg_applies(N, C, g.B)) fail(DDSTRESS_E_INVALID, "fused z register form: shape not covered");
    switch (N * 16 + C) {
        case 16 * 16 + 6: z_reg_launch<16, 6>(blocks, in, out, spec, g, tw, s); break;
        case 16 * 16 + 9: z_reg_launch<16, 9>(blocks, in, out, spec, g, tw, s); break;
        case 32 * 16 + 3: z_reg_launch<32, 3>(blocks, in, out, spec, g, tw, s); break;
        case 32 * 16 + 6: z_reg_launch<32, 6>(blocks, in, out, spec, g, tw, s); break;
        case 32 * 16 + 9: z_reg_launch<32, 9>(blocks, in, out, spec, g, tw, s); break;
        case 64 * 16 + 3: z_reg_launch<64, 3>(blocks, in, out, spec, g, tw, s); break;
        case 64 * 16 + 6: z_reg_launch<64, 6>(blocks, in, out, spec, g, tw, s); break;
        case 64 * 16 + 9: z_reg_launch<64, 9>(blocks, in, out, spec, g, tw, s); break;
        case 128 * 16 + 3: z_reg_launch<128, 3>(blocks, in, out, spec, g, tw, s); break;
        case 128 * 16 + 6: z_reg_launch<128, 6>(blocks, in, out, spec, g, tw, s); break;
        default: fail(DDSTRESS_E_INVALID, "fused z register form: shape not covered");
    }
}

}  // namespace dds
