// Transforms held in the registers of a few lanes of one wave: lane bits are
// exchanged with register-index bits instead of going through LDS.
#pragma once

#include "fft_device.hpp"

namespace dds {

// Exchange lane bit LB with the register-index bit that distinguishes a (0)
// from b (1): afterwards a lane whose bit is 1 holds in a what its partner
// held in b, and a lane whose bit is 0 holds in b what its partner held in a.
template <int LB>
__device__ __forceinline__ void lane_swap(unsigned& a, unsigned& b) {
    static_assert(LB >= 3 && LB <= 5, "lane bit");
    if constexpr (LB == 5) {
        const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
        a = r[0];
        b = r[1];
    } else if constexpr (LB == 4) {
        const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
        a = r[0];
        b = r[1];
    } else {
        // lanes 8..15 of each row take b from lane - 8, lanes 0..7 take a from lane + 8
        const int x = (int)a, y = (int)b;
        a = (unsigned)__builtin_amdgcn_update_dpp(x, y, 0x118, 0xf, 0xc, false);
        b = (unsigned)__builtin_amdgcn_update_dpp(y, x, 0x108, 0xf, 0x3, false);
    }
}
template <int LB>
__device__ __forceinline__ void lane_swap(float& a, float& b) {
    unsigned x = __float_as_uint(a), y = __float_as_uint(b);
    lane_swap<LB>(x, y);
    a = __uint_as_float(x);
    b = __uint_as_float(y);
}
template <int LB>
__device__ __forceinline__ void lane_swap(double& a, double& b) {
    unsigned xl = (unsigned)__double2loint(a), yl = (unsigned)__double2loint(b);
    unsigned xh = (unsigned)__double2hiint(a), yh = (unsigned)__double2hiint(b);
    lane_swap<LB>(xl, yl);
    lane_swap<LB>(xh, yh);
    a = __hiloint2double((int)xh, (int)xl);
    b = __hiloint2double((int)yh, (int)yl);
}
template <int LB, typename T>
__device__ __forceinline__ void lane_swap(cplx<T>& a, cplx<T>& b) {
    lane_swap<LB>(a.x, b.x);
    lane_swap<LB>(a.y, b.y);
}

// exp(-2 pi i k / 64) as the library's twiddle table holds it (long double
// cosine and sine rounded once; at a quarter turn the cosine of the long double
// nearest to pi / 2), so that compile-time twiddles give the same bits as
// table ones. The FP32 table equals these values rounded to float.
constexpr double kW64[64][2] = {
    {0x1p+0, -0x0p+0},    {0x1.fd88da3d12526p-1, -0x1.917a6bc29b42cp-4},
    {0x1.f6297cff75cbp-1, -0x1.8f8b83c69a60bp-3},    {0x1.e9f4156c62ddap-1, -0x1.294062ed59f06p-2},
    {0x1.d906bcf328d46p-1, -0x1.87de2a6aea963p-2},    {0x1.c38b2f180bdb1p-1, -0x1.e2b5d3806f63bp-2},
    {0x1.a9b66290ea1a3p-1, -0x1.1c73b39ae68c8p-1},    {0x1.8bc806b151741p-1, -0x1.44cf325091dd6p-1},
    {0x1.6a09e667f3bcdp-1, -0x1.6a09e667f3bcdp-1},    {0x1.44cf325091dd6p-1, -0x1.8bc806b151741p-1},
    {0x1.1c73b39ae68c8p-1, -0x1.a9b66290ea1a3p-1},    {0x1.e2b5d3806f63bp-2, -0x1.c38b2f180bdb1p-1},
    {0x1.87de2a6aea963p-2, -0x1.d906bcf328d46p-1},    {0x1.294062ed59f06p-2, -0x1.e9f4156c62ddap-1},
    {0x1.8f8b83c69a60bp-3, -0x1.f6297cff75cbp-1},    {0x1.917a6bc29b42cp-4, -0x1.fd88da3d12526p-1},
    {-0x1.d9cceba3f91f2p-66, -0x1p+0},    {-0x1.917a6bc29b42cp-4, -0x1.fd88da3d12526p-1},
    {-0x1.8f8b83c69a60bp-3, -0x1.f6297cff75cbp-1},    {-0x1.294062ed59f06p-2, -0x1.e9f4156c62ddap-1},
    {-0x1.87de2a6aea963p-2, -0x1.d906bcf328d46p-1},    {-0x1.e2b5d3806f63bp-2, -0x1.c38b2f180bdb1p-1},
    {-0x1.1c73b39ae68c8p-1, -0x1.a9b66290ea1a3p-1},    {-0x1.44cf325091dd6p-1, -0x1.8bc806b151741p-1},
    {-0x1.6a09e667f3bcdp-1, -0x1.6a09e667f3bcdp-1},    {-0x1.8bc806b151741p-1, -0x1.44cf325091dd6p-1},
    {-0x1.a9b66290ea1a3p-1, -0x1.1c73b39ae68c8p-1},    {-0x1.c38b2f180bdb1p-1, -0x1.e2b5d3806f63bp-2},
    {-0x1.d906bcf328d46p-1, -0x1.87de2a6aea963p-2},    {-0x1.e9f4156c62ddap-1, -0x1.294062ed59f06p-2},
    {-0x1.f6297cff75cbp-1, -0x1.8f8b83c69a60bp-3},    {-0x1.fd88da3d12526p-1, -0x1.917a6bc29b42cp-4},
    {-0x1p+0, 0x1.d9cceba3f91f2p-65},    {-0x1.fd88da3d12526p-1, 0x1.917a6bc29b42cp-4},
    {-0x1.f6297cff75cbp-1, 0x1.8f8b83c69a60bp-3},    {-0x1.e9f4156c62ddap-1, 0x1.294062ed59f06p-2},
    {-0x1.d906bcf328d46p-1, 0x1.87de2a6aea963p-2},    {-0x1.c38b2f180bdb1p-1, 0x1.e2b5d3806f63bp-2},
    {-0x1.a9b66290ea1a3p-1, 0x1.1c73b39ae68c8p-1},    {-0x1.8bc806b151741p-1, 0x1.44cf325091dd6p-1},
    {-0x1.6a09e667f3bcdp-1, 0x1.6a09e667f3bcdp-1},    {-0x1.44cf325091dd6p-1, 0x1.8bc806b151741p-1},
    {-0x1.1c73b39ae68c8p-1, 0x1.a9b66290ea1a3p-1},    {-0x1.e2b5d3806f63bp-2, 0x1.c38b2f180bdb1p-1},
    {-0x1.87de2a6aea963p-2, 0x1.d906bcf328d46p-1},    {-0x1.294062ed59f06p-2, 0x1.e9f4156c62ddap-1},
    {-0x1.8f8b83c69a60bp-3, 0x1.f6297cff75cbp-1},    {-0x1.917a6bc29b42cp-4, 0x1.fd88da3d12526p-1},
    {0x1.b1acd85d7d6bbp-63, 0x1p+0},    {0x1.917a6bc29b42cp-4, 0x1.fd88da3d12526p-1},
    {0x1.8f8b83c69a60bp-3, 0x1.f6297cff75cbp-1},    {0x1.294062ed59f06p-2, 0x1.e9f4156c62ddap-1},
    {0x1.87de2a6aea963p-2, 0x1.d906bcf328d46p-1},    {0x1.e2b5d3806f63bp-2, 0x1.c38b2f180bdb1p-1},
    {0x1.1c73b39ae68c8p-1, 0x1.a9b66290ea1a3p-1},    {0x1.44cf325091dd6p-1, 0x1.8bc806b151741p-1},
    {0x1.6a09e667f3bcdp-1, 0x1.6a09e667f3bcdp-1},    {0x1.8bc806b151741p-1, 0x1.44cf325091dd6p-1},
    {0x1.a9b66290ea1a3p-1, 0x1.1c73b39ae68c8p-1},    {0x1.c38b2f180bdb1p-1, 0x1.e2b5d3806f63bp-2},
    {0x1.d906bcf328d46p-1, 0x1.87de2a6aea963p-2},    {0x1.e9f4156c62ddap-1, 0x1.294062ed59f06p-2},
    {0x1.f6297cff75cbp-1, 0x1.8f8b83c69a60bp-3},    {0x1.fd88da3d12526p-1, 0x1.917a6bc29b42cp-4},
};
template <int L, int K, typename T>
__device__ __forceinline__ cplx<T> wconst() {
    constexpr int q = (K % L) * (64 / L);
    constexpr T c = (T)kW64[q][0], s = (T)kW64[q][1];
    return {c, s};
}

// Keeps the scheduler from interleaving more butterflies than registers hold
// (64 FP32 or 32 FP64 complex values per lane).
template <int E, typename T>
__device__ __forceinline__ void lane_fence() {
    if constexpr (E * sizeof(T) >= 256) __builtin_amdgcn_sched_barrier(0);
}

// Lanes per column, and twiddles of the lane stages (see col_fft).
template <int N>
constexpr int col_lanes() { return N == 16 ? 2 : 4; }
template <int N>
constexpr int col_tw_count() {
    return N == 16 ? 4 * 2 : N == 32 ? 2 * 3 * 4 : N == 64 ? 2 * 7 * 4 : N == 128 ? 4 * 7 * 2 + 16 * 4 : 16 * 3 * 4;
}
// Index (in 1 / N turns) of entry e of the twiddle table.
template <int N>
__device__ __forceinline__ int col_tw_index(int e) {
    if constexpr (N == 16) return (e & 1) + 2 * (e >> 1);
    else if constexpr (N == 64) return ((e & 3) + 4 * (e / 28)) * ((e >> 2) % 7 + 1);
    else if constexpr (N == 128) {
        if (e < 56) {                              // [g = k0b0 + 2 k0b2][r - 1][k0b1]
            const int g = e / 14, r = (e >> 1) % 7 + 1;
            return 2 * ((g & 1) + 2 * (e & 1) + 4 * (g >> 1)) * r;
        }
        return ((e - 56) & 3) + 4 * ((e - 56) >> 2);
    } else return ((e & 3) + 4 * (e / 12)) * ((e >> 2) % 3 + 1);      // 32, 256: [i][r - 1][p]
}

// First stage: radix 8 over registers a + S r (a < S), inputs from load(m)
// (upper half zero and not read with HZ).
template <int S, bool FWD, bool HZ, typename T, int E, class LOAD>
__device__ __forceinline__ void col_first(cplx<T> (&v)[E], LOAD&& load) {
#pragma unroll
    for (int a = 0; a < S; ++a) {
        cplx<T> t[8];
#pragma unroll
        for (int r = 0; r < (HZ ? 4 : 8); ++r) t[r] = load(a + S * r);
        if constexpr (HZ) dft8_hz<FWD>(t);
        else dft8<FWD>(t);
#pragma unroll
        for (int r = 0; r < 8; ++r) v[a + S * r] = t[r];
        lane_fence<E, T>();
    }
}
// Second stage of length 256: registers r + 8 k0, twiddles w64^(k0 r) (constants).
template <bool FWD, int K0, int R, typename T>
__device__ __forceinline__ void col_w64(cplx<T> (&t)[8]) {
    if constexpr (R < 8) {
        t[R] = twmul<FWD>(t[R], wconst<64, K0 * R, T>());
        col_w64<FWD, K0, R + 1>(t);
    }
}
template <bool FWD, int K0, typename T>
__device__ __forceinline__ void col_second256(cplx<T> (&v)[64]) {
    if constexpr (K0 < 8) {
        cplx<T> t[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) t[r] = v[r + 8 * K0];
        if constexpr (K0 > 0) col_w64<FWD, K0, 1>(t);
        dft8<FWD>(t);
#pragma unroll
        for (int r = 0; r < 8; ++r) v[r + 8 * K0] = t[r];
        lane_fence<64, T>();
        col_second256<FWD, K0 + 1>(v);
    }
}

// Transform of length N over LP = col_lanes<N>() lanes of a wave (the lane's
// top bits, p = lane / (64 / LP)), E = N / LP values per lane: the stages,
// twiddles and products of the Stockham transforms of element classes 8 and 16
// (radices 8, 2; 8, 4; 8, 8; 8, 8, 2; 8, 8, 4), so the same bits. load(m) gives
// row p + LP m of the input (m < E / 2 only with HZ); store(r0, dr, t) takes
// the rows p + r0 + dr k of the output, t[k], as soon as they are formed. tw:
// col_tw_index. Digits: N = 64: row d0 + 8 d1, p the low bits of d0; N = 128:
// row d0 + 2 d1 + 16 d2, p = d0 + 2 (d1's low bit); otherwise p = d0. An
// exchange swaps p's bits with the low bits of the first output digit k0.
template <int N, bool FWD, bool HZ, typename T, class LOAD, class STORE>
__device__ __forceinline__ void col_fft(cplx<T> (&v)[N / col_lanes<N>()], const cplx<T>* tw, int p, LOAD&& load,
                                        STORE&& store) {
    if constexpr (N == 16) {
        col_first<1, FWD, HZ>(v, load);
#pragma unroll
        for (int s = 0; s < 8; s += 2) lane_swap<5>(v[s], v[s + 1]);
#pragma unroll
        for (int h = 0; h < 4; ++h) {              // k0 = p + 2 h
            cplx<T> t[2] = {v[2 * h], twmul<FWD>(v[2 * h + 1], tw[2 * h + p])};
            dft2<FWD>(t);
            store(2 * h, 8, t);
        }
    } else if constexpr (N == 64) {
        col_first<2, FWD, HZ>(v, load);
        // register d0b2 + 2 k0 -> d0b2 + 2 (d0b0, d0b1) + 8 k0b2, lane (k0b0, k0b1)
#pragma unroll
        for (int s = 0; s < 16; ++s)
            if (!(s & 2)) lane_swap<4>(v[s], v[s + 2]);
#pragma unroll
        for (int s = 0; s < 16; ++s)
            if (!(s & 4)) lane_swap<5>(v[s], v[s + 4]);
#pragma unroll
        for (int h = 0; h < 2; ++h) {              // k0 = p + 4 h
            cplx<T> t[8];
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                t[r] = v[(r >> 2) + 2 * (r & 3) + 8 * h];
                if (r > 0) t[r] = twmul<FWD>(t[r], tw[(7 * h + r - 1) * 4 + p]);
            }
            dft8<FWD, col_apart<64>()>(t);
            store(4 * h, 8, t);
            lane_fence<16, T>();
        }
    } else if constexpr (N == 128) {
        col_first<4, FWD, HZ>(v, load);
        // register d1hi + 4 k0, lane bit 5 (d1's low bit) <-> k0b1
#pragma unroll
        for (int s = 0; s < 32; ++s)
            if (!(s & 8)) lane_swap<5>(v[s], v[s + 8]);
#pragma unroll
        for (int g = 0; g < 4; ++g) {              // k0 = k0b0 + 2 (lane bit 5) + 4 k0b2, g = k0b0 + 2 k0b2
            const int s0 = 4 * (g & 1) + 16 * (g >> 1);
            cplx<T> t[8];
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                t[r] = v[s0 + (r >> 1) + 8 * (r & 1)];
                if (r > 0) t[r] = twmul<FWD>(t[r], tw[(7 * g + r - 1) * 2 + (p >> 1)]);
            }
            dft8<FWD>(t);
#pragma unroll
            for (int r = 0; r < 8; ++r) v[s0 + (r >> 1) + 8 * (r & 1)] = t[r];      // k1 in d1's place
            lane_fence<32, T>();
        }
        // lane bit 4 (d0) <-> k0b0
#pragma unroll
        for (int s = 0; s < 32; ++s)
            if (!(s & 4)) lane_swap<4>(v[s], v[s + 4]);
#pragma unroll
        for (int i = 0; i < 16; ++i) {             // k0 + 8 k1 = p + 4 i, i = k0b2 + 2 k1
            const int k1 = i >> 1, s = 16 * (i & 1) + (k1 >> 1) + 8 * (k1 & 1);
            cplx<T> t[2] = {v[s], twmul<FWD>(v[s + 4], tw[56 + 4 * i + p])};
            dft2<FWD>(t);
            store(4 * i, 64, t);
            if (i % 4 == 3) lane_fence<32, T>();
        }
    } else {                                       // 32: radices 8, 4; 256: 8, 8, 4
        static_assert(N == 32 || N == 256, "length");
        constexpr int E = N / 4, S = E / 8;        // register (k1 +) S k0
        col_first<S, FWD, HZ>(v, load);
        if constexpr (N == 256) col_second256<FWD, 0>(v);
#pragma unroll
        for (int s = 0; s < E; ++s)
            if (!(s & S)) lane_swap<4>(v[s], v[s + S]);
#pragma unroll
        for (int s = 0; s < E; ++s)
            if (!(s & (2 * S))) lane_swap<5>(v[s], v[s + 2 * S]);
#pragma unroll
        for (int i = 0; i < E / 4; ++i) {          // k0 + 8 k1 = p + 4 i, i = k0b2 + 2 k1
            const int s = (i >> 1) + 4 * S * (i & 1);
            cplx<T> t[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                t[r] = v[s + S * r];
                if (r > 0) t[r] = twmul<FWD>(t[r], tw[(3 * i + r - 1) * 4 + p]);
            }
            dft4<FWD>(t);
            store(4 * i, E, t);
            lane_fence<E, T>();
        }
    }
}

}  // namespace dds
