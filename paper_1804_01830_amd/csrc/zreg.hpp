// Fused z pass, register form (FP32). Same work and the same bits as the
// single-group form of element class 4 (zfused.hpp), with no LDS exchange and
// no workgroup barrier between the stages of a transform: a column's N values
// live in the registers of LP lanes of one wave, E = N / LP per lane, and the
// digits a radix-4 (or final radix-2) stage combines are brought into one lane
// by exchanging lane bits with register-index bits (v_permlane32_swap,
// v_permlane16_swap: one instruction moves two registers; DPP for bit 3).
#pragma once

#include "ddstress_internal.hpp"
#include "lane_fft.hpp"
#include "zfused.hpp"

namespace dds {

// Radix-4 DFT over registers v[I0 + r S], r = 0..3 (r >= 2 zero with HZ).
template <bool FWD, bool HZ, int I0, int S, int E>
__device__ __forceinline__ void reg_dft4(cplx<float> (&v)[E]) {
    cplx<float> t[4];
    t[0] = v[I0];
    t[1] = v[I0 + S];
    if constexpr (!HZ) {
        t[2] = v[I0 + 2 * S];
        t[3] = v[I0 + 3 * S];
        dft4<FWD>(t);
    } else {
        dft4_hz<FWD>(t);
    }
    v[I0] = t[0];
    v[I0 + S] = t[1];
    v[I0 + 2 * S] = t[2];
    v[I0 + 3 * S] = t[3];
}

// Twiddles and radix-4 DFT of a stage whose previous digit is K0 (a constant)
// and whose first stage was radix 4: v[I0 + r S] *= w16^(K0 r), r = 1..3.
template <bool FWD, int K0, int I0, int S, int E>
__device__ __forceinline__ void reg_stage16(cplx<float> (&v)[E]) {
    if constexpr (K0 > 0) {
        v[I0 + S] = twmul<FWD>(v[I0 + S], wconst<16, K0, float>());
        v[I0 + 2 * S] = twmul<FWD>(v[I0 + 2 * S], wconst<16, 2 * K0, float>());
        v[I0 + 3 * S] = twmul<FWD>(v[I0 + 3 * S], wconst<16, 3 * K0, float>());
    }
    reg_dft4<FWD, false, I0, S>(v);
}

// Number of lane-dependent twiddles of one transform direction.
template <int N, int LP>
constexpr int lane_tw_count() {
    return N == 128 ? 20 : N == 64 ? 12 : N == 32 ? 10 : 3;
}

// Position of lane group p (the lane's upper bits, p < LP) of a column:
// register m holds row z = p + LP m of the input, spectrum row
// kz = k_low(p) + LP m, which the inverse starts from, and row
// z = zo_low(p) + LP m of its output (the lane bits are followed in lane_fft).
template <int N, int LP>
__device__ __forceinline__ int k_low(int p) {
    if constexpr (N == 128) return ((p & 1) << 2) | ((p & 6) >> 1);          // lane bits 3, 4, 5: k1lo, k0lo, k0hi
    else return p;
}
template <int N, int LP>
__device__ __forceinline__ int zo_low(int p) {
    if constexpr (N == 128) return ((p & 1) << 1) | ((p & 2) << 1) | ((p & 4) >> 2);  // j0hi, j1lo, j0lo
    else return p;
}

// Index (of 1 / N turns) of lane twiddle i of lane group p; dir 0 forward, 1 inverse.
template <int N, int LP>
__device__ __forceinline__ int lane_tw_index(int dir, int i, int p) {
    if constexpr (N == 64 && LP == 4) {             // w64^((k0 + 4 k1) r), k0 = p, k1 = i / 3, r = 1 + i % 3
        return (p + 4 * (i / 3)) * (1 + i % 3);
    } else if constexpr (N == 16 && LP == 4) {      // w16^(k0 r)
        return p * (1 + i);
    } else if constexpr (N == 32 && LP == 4) {
        const int k0lo = p & 1, k0hi = p >> 1;
        if (i < 6) return 2 * ((i / 3 + 2 * k0hi) * (1 + i % 3));    // stage 2: w16^(k0 r), k0lo = i / 3
        return k0lo + 2 * k0hi + 4 * (i - 6);                        // stage 3: w32^(k0 + 4 k1)
    } else {                                        // N == 128, LP == 8
        // lane bits of (k0lo, k0hi, k1lo): forward p bits 1, 2, 0; inverse 2, 0, 1
        const int k0 = dir ? ((p >> 2) | ((p & 1) << 1)) : p >> 1, k1lo = dir ? (p >> 1) & 1 : p & 1;
        if (i < 12) return 2 * ((k0 + 4 * (i / 3)) * (1 + i % 3));   // stage 3: w64^((k0 + 4 k1) r), k1 = i / 3
        const int q = i - 12;                                        // stage 4: w128^(k0 + 4 k1 + 16 k2), q = k1hi + 2 k2
        return k0 + 4 * k1lo + 8 * q;
    }
}

// One transform of length N over LP lanes (bits 3.. or 4.. of the lane up to
// bit 5), radix 4 with a final radix-2 stage where N is an odd power of two:
// the stages, twiddles and products of the Stockham transforms of element
// class 4, so the same bits. W(i) returns lane twiddle i (see lane_tw_index).
// HZ: registers m >= E / 2 of the input are zero and not read.
template <int N, int LP, bool FWD, bool HZ, int E, class TW>
__device__ __forceinline__ void lane_fft(cplx<float> (&v)[E], TW&& W) {
    static_assert(E * LP == N, "E elements per lane");
    if constexpr (N == 64 && LP == 4) {
        // z = d0 + 4 d1 + 16 d2: lane d0 (bits 4, 5), register d1 + 4 d2
        reg_dft4<FWD, HZ, 0, 4>(v); reg_dft4<FWD, HZ, 1, 4>(v); reg_dft4<FWD, HZ, 2, 4>(v); reg_dft4<FWD, HZ, 3, 4>(v);
        reg_stage16<FWD, 0, 0, 1>(v); reg_stage16<FWD, 1, 4, 1>(v); reg_stage16<FWD, 2, 8, 1>(v); reg_stage16<FWD, 3, 12, 1>(v);
        // register k1 + 4 k0, lane d0 -> register k1 + 4 d0, lane k0
#pragma unroll
        for (int i = 0; i < 8; ++i) lane_swap<5>(v[i], v[i + 8]);
#pragma unroll
        for (int i = 0; i < 16; ++i)
            if (!(i & 4)) lane_swap<4>(v[i], v[i + 4]);
#pragma unroll
        for (int k1 = 0; k1 < 4; ++k1)
#pragma unroll
            for (int r = 1; r < 4; ++r) v[k1 + 4 * r] = twmul<FWD>(v[k1 + 4 * r], W(3 * k1 + r - 1));
        reg_dft4<FWD, false, 0, 4>(v); reg_dft4<FWD, false, 1, 4>(v); reg_dft4<FWD, false, 2, 4>(v); reg_dft4<FWD, false, 3, 4>(v);
        // register k1 + 4 k2, lane k0: k = p + 4 m
    } else if constexpr (N == 16 && LP == 4) {
        // z = d0 + 4 d1: lane d0, register d1
        reg_dft4<FWD, HZ, 0, 1>(v);
        lane_swap<5>(v[0], v[2]); lane_swap<5>(v[1], v[3]);
        lane_swap<4>(v[0], v[1]); lane_swap<4>(v[2], v[3]);
#pragma unroll
        for (int r = 1; r < 4; ++r) v[r] = twmul<FWD>(v[r], W(r - 1));
        reg_dft4<FWD, false, 0, 1>(v);
    } else if constexpr (N == 32 && LP == 4) {
        // z = d0 + 2 d1 + 8 d2 (d0 one bit): lane bit 4 d0, bit 5 d1lo; register d1hi + 2 d2
        reg_dft4<FWD, HZ, 0, 2>(v); reg_dft4<FWD, HZ, 1, 2>(v);
        // register d1hi + 2 k0; lane bit 5 <-> k0hi: register d1hi + 2 k0lo + 4 d1lo
#pragma unroll
        for (int i = 0; i < 4; ++i) lane_swap<5>(v[i], v[i + 4]);
#pragma unroll
        for (int k0lo = 0; k0lo < 2; ++k0lo) {
            cplx<float> t[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                t[r] = v[(r >> 1) + 2 * k0lo + 4 * (r & 1)];
                if (r > 0) t[r] = twmul<FWD>(t[r], W(3 * k0lo + r - 1));
            }
            dft4<FWD>(t);
#pragma unroll
            for (int r = 0; r < 4; ++r) v[(r >> 1) + 2 * k0lo + 4 * (r & 1)] = t[r];
        }
        // register k1hi + 2 k0lo + 4 k1lo; lane bit 4 (d0) <-> k0lo
        lane_swap<4>(v[0], v[2]); lane_swap<4>(v[1], v[3]); lane_swap<4>(v[4], v[6]); lane_swap<4>(v[5], v[7]);
        cplx<float> o[8];
#pragma unroll
        for (int k1 = 0; k1 < 4; ++k1) {
            const int s = (k1 >> 1) + 4 * (k1 & 1);
            cplx<float> t[2] = {v[s], twmul<FWD>(v[s + 2], W(6 + k1))};
            dft2<FWD>(t);
            o[k1] = t[0];                                // k = p + 4 k1 + 16 k2
            o[k1 + 4] = t[1];
        }
#pragma unroll
        for (int m = 0; m < 8; ++m) v[m] = o[m];
    } else if constexpr (N == 128 && LP == 8) {
        // Forward: z = d0 + 2 d1 + 8 d2 + 32 d3 (d0 one bit), lane bit 3 d0, bits (4, 5) d1; register d2 + 4 d3.
        // Output: lane bit 3 k1lo, (4, 5) k0; register k1hi + 2 k2 + 8 k3. The inverse reads that order: its
        // d0 = k0lo (4), d1 = (k0hi, k1lo) (5, 3), and ends with j0 at (5, 3), j1lo at 4.
        constexpr int B0 = FWD ? 3 : 4, B1 = FWD ? 4 : 5, B2 = FWD ? 5 : 3;
        reg_dft4<FWD, HZ, 0, 4>(v); reg_dft4<FWD, HZ, 1, 4>(v); reg_dft4<FWD, HZ, 2, 4>(v); reg_dft4<FWD, HZ, 3, 4>(v);
        reg_stage16<FWD, 0, 0, 1>(v); reg_stage16<FWD, 1, 4, 1>(v); reg_stage16<FWD, 2, 8, 1>(v); reg_stage16<FWD, 3, 12, 1>(v);
        // register k1 + 4 k0, lane d1 -> register k1 + 4 d1, lane k0
#pragma unroll
        for (int i = 0; i < 8; ++i) lane_swap<B2>(v[i], v[i + 8]);
#pragma unroll
        for (int i = 0; i < 16; ++i)
            if (!(i & 4)) lane_swap<B1>(v[i], v[i + 4]);
#pragma unroll
        for (int k1 = 0; k1 < 4; ++k1)
#pragma unroll
            for (int r = 1; r < 4; ++r) v[k1 + 4 * r] = twmul<FWD>(v[k1 + 4 * r], W(3 * k1 + r - 1));
        reg_dft4<FWD, false, 0, 4>(v); reg_dft4<FWD, false, 1, 4>(v); reg_dft4<FWD, false, 2, 4>(v); reg_dft4<FWD, false, 3, 4>(v);
        // register k1 + 4 k2; lane bit B0 (d0) <-> k1lo
#pragma unroll
        for (int i = 0; i < 16; i += 2) lane_swap<B0>(v[i], v[i + 1]);
        cplx<float> o[16];
#pragma unroll
        for (int q = 0; q < 8; ++q) {                    // q = k1hi + 2 k2
            cplx<float> t[2] = {v[2 * q], twmul<FWD>(v[2 * q + 1], W(12 + q))};
            dft2<FWD>(t);
            o[q] = t[0];
            o[q + 8] = t[1];
        }
#pragma unroll
        for (int m = 0; m < 16; ++m) v[m] = o[m];
    }
}

// ----------------------------------------------------------------------------
// The kernel. A block's waves (2 to 4) share one tile of tk = 64 / LP
// consecutive kx columns at one ky (or a group of the Nyquist strip, see
// z_roles), whose spectrum is copied to LDS once ([c][v][kz][tk] as stored,
// y-mirror sign applied); wave w evaluates realisations b0 + w, b0 + w + waves,
// ... on its own, with no barrier after the copy. Lane p tk + c holds rows
// z = p + LP m of column c. ZM: only kz <= N / 2 is stored and register
// m >= E / 2 reads row N - kz. FR: all N / 2 rows are data (nz = N / 2), one
// row offset instead of one per register. SPLIT: the spectrum's tiles are narrower
// than the block's.
// VG = 0: the C channel spectra stay in registers and the six stress
// components are formed and transformed back one after the other. VG > 0: a
// block takes VG components, whose accumulators stay in registers while the
// channels pass through (6 / VG blocks per tile, neighbours in the launch, each
// transforming every channel: more arithmetic, half or a third of the staged
// tile).
//
// What bounds it: HBM. The pass reads 8 C and writes 48 bytes per data row of
// a column; the same loads and stores without any arithmetic take 400 us at
// 128 x 128 x 32, six channels, 16 realisations (4.05 TB/s; a plain copy
// reaches 4.8), the kernel 515 us, the grouped form it replaces 912 us; with
// three channels and 64 realisations 1.26 against 1.40 ms (single-group form). 128-byte row segments (16 columns) matter
// more than the arithmetic: eight columns a wave (LP = 8) need a fifth less of
// it at six channels and take 552 us, because their loads and stores alone
// take 503. Two waves per SIMD (up to 256 registers) cover what latency is
// left; three would spill the accumulators.
// ----------------------------------------------------------------------------
template <int N, int LP, int NC, bool ZM, int VG, bool FR, bool SPLIT>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
    k_z_reg(const cplx<float>* __restrict__ in, cplx<float>* __restrict__ out, const float* __restrict__ spec, ZGeom g,
            const cplx<float>* __restrict__ tw) {
    using T = float;
    constexpr int E = N / LP, EH = E / 2, TK = 64 / LP;
    constexpr int NKZ = ZM ? N / 2 + 1 : N;
    constexpr int TWC = lane_tw_count<N, LP>();
    constexpr bool TWR = LP == 4;                   // one twiddle set for both directions, in registers
    constexpr int PL = NKZ * TK;                    // values of one (c, v) plane of the tile
    extern __shared__ unsigned char smem_raw[];
    T* const s_l = reinterpret_cast<T*>(smem_raw);
    cplx<T>* const tw_l = reinterpret_cast<cplx<T>*>(smem_raw + (size_t)NC * (VG > 0 ? VG : 6) * PL * sizeof(T));
    const int lane = (int)threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int nw = (int)blockDim.x >> 6;
    const int c = lane % TK, p = lane / TK;
    constexpr int VS = VG > 0 ? 6 / VG : 1;         // blocks per tile
    constexpr int NV = VG > 0 ? VG : 6;             // components of this block: v0 .. v0 + NV - 1
    const int lb = z_logical_block(g, VS);
    const ZRoles ro = z_roles<T, SPLIT>(lb / VS, TK, c, g);
    const int v0 = (lb % VS) * NV;
    const NyquistRole nq = ro.nq;
    if (nq.skip_block) return;                      // uniform over the block, before any barrier
    const bool flip_y = ro.flip_y;
    const T* sp = spec + ((int64_t)ro.kyc * (SPLIT ? g.snt : g.ntiles) + ro.tile) * (int64_t)(NC * 6 * NKZ * (SPLIT ? g.stk : TK));
    const __amdgpu_buffer_rsrc_t srs = SPLIT ? split_rsrc(sp, ro, g) : make_rsrc(sp, (uint32_t)(NC * 6 * PL * sizeof(T)));
    // rows z < nz of the lane's column (others: reads give zero, stores are dropped)
    const cplx<T>* in_b = in + ro.in0;
    int r_off[FR ? 1 : EH];
    row_offsets<T, FR ? 1 : EH>(r_off, true, p, LP, ro.lane_in, (int)g.irs, g.nz, ro.in_bytes);
    const int r_step = LP * (int)g.irs * (int)sizeof(cplx<T>);
    const cplx<T>* out_b = out + ro.own0;
    const int zo = zo_low<N, LP>(p);
    int o_off[FR ? 1 : EH];
    row_offsets<T, FR ? 1 : EH>(o_off, nq.own, zo, LP, ro.lane_out, (int)g.ors, g.nz, ro.out_bytes);
    const int o_step = LP * (int)g.ors * (int)sizeof(cplx<T>);
    auto load_rho = [&](cplx<T> (&dst)[EH], int b, int ch) {
        const __amdgpu_buffer_rsrc_t rr = make_rsrc(in_b + (int64_t)(b * NC + ch) * g.iqs, ro.in_bytes);
#pragma unroll
        for (int m = 0; m < EH; ++m) dst[m] = buf_cplx<T>(rr, r_off[FR ? 0 : m], m * r_step);
    };
    // channels requested ahead: all of the next realisation's, or one channel
    // ahead of the transforms where registers are short
    constexpr int NB = VG == 0 && NC * EH <= 24 ? NC : 1;
    cplx<T> nxt[NB][EH];
    if (ro.b0 + w < ro.b1) {
#pragma unroll
        for (int ch = 0; ch < NB; ++ch) load_rho(nxt[ch], ro.b0 + w, ch);
    }
    // lane twiddles: registers, or an LDS table [direction][i][p]
    cplx<T> twr[TWR ? TWC : 1];
    if constexpr (TWR) {
#pragma unroll
        for (int i = 0; i < TWC; ++i) twr[i] = tw[N - 1 + lane_tw_index<N, LP>(0, i, p)];
    } else {
        for (int e = (int)threadIdx.x; e < 2 * TWC * LP; e += (int)blockDim.x) {
            const int pp = e % LP, i = (e / LP) % TWC, dir = e / (LP * TWC);
            tw_l[e] = tw[N - 1 + (lane_tw_index<N, LP>(dir, i, pp) & (N - 1))];
        }
    }
    {
        // 16-byte pieces of [c][v - v0][kz][tk], CH loads of a thread in flight (halves of
        // them where the spectrum's tiles are narrower)
        constexpr int P4 = PL / 4, n4 = NC * NV * P4, CH = 8;
        const int nt = (int)blockDim.x;
        for (int i0 = (int)threadIdx.x; i0 < n4; i0 += CH * nt) {
            uint4 piece[CH];
            if constexpr (!SPLIT) {
#pragma unroll
                for (int k = 0; k < CH; ++k) {
                    const int i = i0 + k * nt, q0 = i / P4, cv = (q0 / NV) * 6 + v0 + q0 % NV;
                    piece[k] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(
                                                             srs, (cv * P4 + i - q0 * P4) * 16, 0, 0));
                }
            } else {
#pragma unroll
                for (int k = 0; k < CH; ++k) {
                    const int i = i0 + k * nt, q0 = i / P4, cv = (q0 / NV) * 6 + v0 + q0 % NV, r = 4 * (i - q0 * P4);
                    const int row = (cv * NKZ + r / TK) * g.stk, cc = r % TK;
                    const uint2 lo = spec_half(srs, i < n4 ? (row + spec_col(g, split_part(ro, g), cc)) * 4 : kNoOffset);
                    const uint2 hi = spec_half(srs, i < n4 ? (row + spec_col(g, split_part(ro, g), cc + 2)) * 4 : kNoOffset);
                    piece[k] = {lo.x, lo.y, hi.x, hi.y};
                }
            }
#pragma unroll
            for (int k = 0; k < CH; ++k) {
                const int i = i0 + k * nt, q0 = i / P4, cv = (q0 / NV) * 6 + v0 + q0 % NV;
                if (i < n4) {
                    const uint32_t msk = sign_mask(flip_y && ((g.sgn_y >> (cv & 63)) & 1));
                    uint4 q = piece[k];
                    q.x ^= msk; q.y ^= msk; q.z ^= msk; q.w ^= msk;
                    *reinterpret_cast<uint4*>(s_l + 4 * i) = q;
                }
            }
        }
    }
    __syncthreads();
    // spectrum rows of register m: kz = kl + LP m, or the mirror row N - kz for m >= E / 2
    const int kl = k_low<N, LP>(p);
    const int s_lane = kl * TK + c, s_lane_m = (LP - kl) * TK + c;
    auto load_spec = [&](T (&dst)[E], int ch, int v) {
        const int base = (ch * NV + v - v0) * PL;
#pragma unroll
        for (int m = 0; m < E; ++m) {
            const bool mir = ZM && 2 * m >= E;
            const int off = base + (mir ? LP * (E - 1 - m) : LP * m) * TK;
            dst[m] = s_l[(mir ? s_lane_m : s_lane) + off];
        }
    };
    // acc += i S rho (staged values carry the y sign; the z sign of mirrored
    // rows is a bit flip by a wave-uniform mask)
    auto contract = [&](cplx<T> (&acc)[E], const T (&sv)[E], const cplx<T> (&rho)[E], int ch, int v) {
        const uint32_t mz = ZM ? sign_mask((g.sgn_z >> (ch * 6 + v)) & 1) : 0u;
#pragma unroll
        for (int m = 0; m < E; ++m) {
            const T s = (ZM && 2 * m >= E) ? flip_sign(sv[m], mz) : sv[m];
            acc[m].x -= s * rho[m].y;
            acc[m].y += s * rho[m].x;
        }
    };
    auto store = [&](const cplx<T> (&acc)[E], int b, int v) {
        const __amdgpu_buffer_rsrc_t orr = make_rsrc(out_b + (int64_t)(b * 6 + v) * g.oqs, ro.out_bytes);
#pragma unroll
        for (int m = 0; m < EH; ++m) buf_store_cplx<T>(orr, o_off[FR ? 0 : m], m * o_step, acc[m]);
        if (nq.mirror) {
            cplx<T>* dst = out + ro.mir + (int64_t)(b * 6 + v) * g.oqs;
#pragma unroll
            for (int m = 0; m < EH; ++m) {
                const int z = zo + LP * m;
                if (z < g.nz) dst[(int64_t)z * g.ors] = cconj(acc[m]);
            }
        }
    };
    int pt = p;
    auto twf = [&](int i) { if constexpr (TWR) return twr[i]; else return tw_l[i * LP + pt]; };
    auto twi = [&](int i) { if constexpr (TWR) return twr[i]; else return tw_l[(TWC + i) * LP + pt]; };

    for (int b = ro.b0 + w; b < ro.b1; b += nw) {
        // (the table reads stay inside the loop: held across it they would take the registers of a column)
        if constexpr (!TWR) asm volatile("" : "+v"(pt));
        if constexpr (VG == 0) {
            cplx<T> rho[NC][E];
#pragma unroll
            for (int ch = 0; ch < NC; ++ch) {
#pragma unroll
                for (int m = 0; m < EH; ++m) rho[ch][m] = nxt[NB == 1 ? 0 : ch][m];
                if constexpr (NB == 1) {
                    const bool last = ch + 1 == NC;
                    if (!last || b + nw < ro.b1) load_rho(nxt[0], last ? b + nw : b, last ? 0 : ch + 1);
                }
                lane_fft<N, LP, true, true>(rho[ch], twf);
            }
            if constexpr (NB > 1) {
                if (b + nw < ro.b1) {
#pragma unroll
                    for (int ch = 0; ch < NC; ++ch) load_rho(nxt[ch], b + nw, ch);
                }
            }
#pragma unroll 1
            for (int v = 0; v < 6; ++v) {
                cplx<T> acc[E];
#pragma unroll
                for (int m = 0; m < E; ++m) acc[m] = {T(0), T(0)};
#pragma unroll
                for (int ch = 0; ch < NC; ++ch) {
                    T sv[E];
                    load_spec(sv, ch, v);
                    contract(acc, sv, rho[ch], ch, v);
                }
                lane_fft<N, LP, false, false>(acc, twi);
                store(acc, b, v);
            }
        } else {
            cplx<T> acc[NV][E];
#pragma unroll
            for (int v = 0; v < NV; ++v)
#pragma unroll
                for (int m = 0; m < E; ++m) acc[v][m] = {T(0), T(0)};
#pragma unroll 1
            for (int ch = 0; ch < NC; ++ch) {
                cplx<T> cur[E];
#pragma unroll
                for (int m = 0; m < EH; ++m) cur[m] = nxt[0][m];
                const bool last = ch + 1 == NC;
                if (!last || b + nw < ro.b1) load_rho(nxt[0], last ? b + nw : b, last ? 0 : ch + 1);
                lane_fft<N, LP, true, true>(cur, twf);
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    T sv[E];
                    load_spec(sv, ch, v0 + v);
                    contract(acc[v], sv, cur, ch, v0 + v);
                }
            }
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                lane_fft<N, LP, false, false>(acc[v], twi);
                store(acc[v], b, v0 + v);
            }
        }
    }
}

// Lanes per column and component groups (0: the channel form) by z length and
// channels: the choices that fit 256 registers and an 80 KB tile (two blocks
// per CU).
constexpr int z_reg_lanes(int N) { return N <= 64 ? 4 : 8; }
constexpr int z_reg_vg(int N, int NC) {
    return N == 128 ? (NC == 3 ? 0 : 3) : N == 64 ? (NC == 3 ? 0 : NC == 6 ? 3 : 2) : N == 32 && NC == 9 ? 3 : 0;
}

template <int N, int NC>
void z_reg_launch(int64_t blocks, const cplx<float>* in, cplx<float>* out, const float* spec, const ZGeom& g,
                  const cplx<float>* tw, hipStream_t s) {
    constexpr int LP = z_reg_lanes(N);
    constexpr int VG = z_reg_vg(N, NC);
    const size_t lds = z_reg_lds_bytes(N, NC, g.nkz_s);
    if (lds > (size_t)80 * 1024 || blocks > 0x7fffffffLL)
        fail(DDSTRESS_E_UNSUPPORTED, "fused z register form: grid or spectrum tile too large");
    const dim3 grid((unsigned)blocks), block(64 * z_reg_waves(g.B));
    const bool full = g.nz == N / 2;                // every row of the unpadded half is a data row
#define DDS_Z_REG(ZMV, FRV, SPLITV)                                                                            \
    hipLaunchKernelGGL((k_z_reg<N, LP, NC, ZMV, VG, FRV, SPLITV>), grid, block, lds, s, in, out, spec, g, tw)
    if (g.stk != z_reg_tile(N)) {
        if (g.nkz_s < N) DDS_Z_REG(true, false, true);
        else DDS_Z_REG(false, false, true);
    } else if (g.nkz_s < N) {
        if (full) DDS_Z_REG(true, true, false);
        else DDS_Z_REG(true, false, false);
    } else {
        if (full) DDS_Z_REG(false, true, false);
        else DDS_Z_REG(false, false, false);
    }
#undef DDS_Z_REG
}

}  // namespace dds
