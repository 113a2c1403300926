// Fused x and y passes of planes that fit in LDS: the forward x
// (real-to-complex) and forward y before the fused z pass, and the inverse y
// and inverse x (complex-to-real) after it. Every (realisation, channel or
// component, z) plane is one work item; its intermediate plane (rows y < Ny, half
// spectra of M = Px/2 columns) stays in LDS and never travels to memory, and
// two launches with their gaps go.
//
// A block has M / 16 waves (at least one).
//   Rows (x): the threads take rows of M / EX lanes each; a row's lanes are
//   consecutive lanes of one wave and the row's LDS is its own, so its
//   transform and the split synchronise within the wave.
//   Columns (y): wave w owns the 16 columns 16 w .. 16 w + 15, four lanes a
//   column (two at Py = 16), E = Py / 4 rows per lane in registers, whose
//   stages exchange lane bits with register bits (col_fft): no LDS exchange, no
//   barrier; a wave's loads and stores are E accesses of four 128-byte (FP64:
//   256-byte) pieces.
// The two phases meet at one barrier per direction of the hand-over. The column
// kx = M (the Nyquist column) is transformed apart, inside the last wave. In
// the inverse of the largest planes (Py = 256, M = 128) it travels instead as
// the imaginary part of column 0, X[0] + i X[M]: both are Hermitian along ky
// (the z pass writes column M exactly Hermitian; column 0's rounding-level
// imaginary part is dropped), and the split takes the real and imaginary part
// as its two real inputs. Otherwise the arithmetic, and the bits, are those
// of the separate passes.
//
// Vector loads and stores complete in issue order for a wave's wait counter,
// so nothing here reads a twiddle from memory behind other traffic: all
// tables are copied to LDS at the start. Where a plane takes a CU's LDS for
// itself (Py = 256, M = 128) a block walks over planes and requests the next
// plane's data before the phase that does not need those registers; smaller
// planes take one block each, several per CU.
//
// What bounds them: HBM and the latency of a plane. At 128 x 128 x 32, eight
// realisations, the forward moves 253 MB in 63 us (4.0 TB/s; 1024 threads with
// LDS exchanges and a barrier per stage took 78), the inverse 508 MB in 159 us
// (169 before); one realisation, less than one plane per CU, 19.6 and 23.3 us
// (25.2, 25.3). Small planes: 64^3 FP32, four realisations, forward 17 us and
// inverse 36 us (separate passes 30, 55); FP64 29 and 78 us (47, 102).
//
// Planes of the spectra may be interleaved: plane p starts at
// (p / zp) zp Py wx + (p % zp) wx and its rows lie zp wx apart (zp = 1: each
// plane contiguous; zp = Nz: the ky-major layout of the z pass).
#pragma once

#include "ddstress_internal.hpp"
#include "lane_fft.hpp"

namespace dds {

template <typename T, int PY, int M>
struct PlaneShape {
    static constexpr int LP = col_lanes<PY>(), GC = 64 / LP, E = PY / LP;   // columns: lanes, per wave, rows per lane
    static constexpr int NW = M > GC ? M / GC : 1, NT = 64 * NW;  // waves, threads
    static constexpr int EX = M >= 64 && sizeof(T) == 4 ? 16 : 8;  // rows: elements per lane
    static constexpr int TCX = M / EX;                            // lanes per row
    static constexpr int RPP = NT / TCX;                          // rows per pass of the block
    static constexpr int RPW = 64 / TCX;                          // rows per wave
    // row stride and pad of a plane in LDS: element i of a row exchange at
    // i + (i >> 3), a row's spectrum at i; by the bank model of x_lds_layout
    // both, and the column accesses (16 consecutive values of 4 rows), are within
    // 17 percent of conflict-free
    static constexpr int LD = sizeof(T) == 4 && M == 128 ? 152 : sizeof(T) == 4 && M == 64 ? 76 : M + M / 8, SH = 3;
    static constexpr int TWN = col_tw_count<PY>();                // column twiddle table (LDS, complex)
    static constexpr int NYN = PY > RPW ? PY : RPW;               // Nyquist column scratch (complex)
};

// The tables of a block, in LDS: twy col_fft's lane twiddles, twx
// exp(-2 pi i k / M) then exp(-2 pi i k / P), k < M, and behind them
// exp(-2 pi i k / Py), k < Py, for the column M.
template <typename T, int PY, int M>
__device__ __forceinline__ void load_plane_tables(cplx<T>* twy, cplx<T>* twx, const cplx<T>* __restrict__ tw) {
    using S = PlaneShape<T, PY, M>;
    for (int e = (int)threadIdx.x; e < S::TWN; e += S::NT) twy[e] = tw[(PY - 1) + (col_tw_index<PY>(e) & (PY - 1))];
    for (int e = (int)threadIdx.x; e < PY; e += S::NT) twx[2 * M + e] = tw[(PY - 1) + e];
    for (int e = (int)threadIdx.x; e < 2 * M; e += S::NT) twx[e] = e < M ? tw[(M - 1) + e] : tw[(2 * M - 1) + (e - M)];
}

// HX: open x axis (nx <= M: the upper half of every packed row is zero).
// HY: open y axis (ny <= Py / 2: the upper half of every column is zero).
// PF: the block walks over planes and requests the next plane's rows ahead.
template <typename T, int PY, int M, bool HX, bool HY, bool PF>
__global__ void __launch_bounds__((PlaneShape<T, PY, M>::NT)) __attribute__((amdgpu_waves_per_eu(PlaneShape<T, PY, M>::NT > 512 ? 1 : 2)))
    k_xy_fwd(const T* __restrict__ in, cplx<T>* __restrict__ out, int64_t nplanes, int ny, int nx, int64_t wx,
             const cplx<T>* __restrict__ tw, int rows_arg, int pairs, int zp) {
    using S = PlaneShape<T, PY, M>;
    constexpr int EX = S::EX, TCX = S::TCX, E = S::E;
    constexpr int EL = HX && EX > 1 ? EX / 2 : EX;                // row elements that can be non-zero
    constexpr int RMAX = HY ? PY / 2 : PY;
    constexpr int NP = (RMAX + S::RPP - 1) / S::RPP;              // row passes
    constexpr int xld = S::LD;
    const int rows = rows_arg;                                    // rows held: ny rounded up to whole waves
    extern __shared__ unsigned char smem_raw[];
    cplx<T>* const pl = reinterpret_cast<cplx<T>*>(smem_raw);     // [rows][LD]
    cplx<T>* const nyq = pl + (size_t)(rows < RMAX ? rows + 4 : rows) * xld;   // column M: rows, then its exchanges
    cplx<T>* const twy = nyq + S::NYN;
    cplx<T>* const twx = twy + S::TWN;
    const int t = (int)threadIdx.x, w = __builtin_amdgcn_readfirstlane(t >> 6);
    load_plane_tables<T, PY, M>(twy, twx, tw);
    if (rows < RMAX)                                              // four spare rows of zeros stand for the rest
        for (int e = t; e < 4 * xld; e += S::NT) pl[rows * xld + e] = {T(0), T(0)};

    // A block that walks over planes re-derives its indices at each use:
    // otherwise their address arithmetic is kept in registers across the planes.
    auto fresh = [&]() {
        int q = t;
        if constexpr (PF) asm volatile("" : "+v"(q));
        return q;
    };
    const int yw = w * S::RPW;                                    // the wave's first row (of pass 0)
    const uint32_t in_bytes = (uint32_t)((int64_t)ny * nx * sizeof(T));
    // reals past a row's end, and rows past the plane's, take the plane's size as offset and read zero
    auto load_row = [&](cplx<T> (&r)[EL], int64_t plane, int tq, int pass) {
        const int jx = tq % TCX, y = tq / TCX + pass * S::RPP;
        const __amdgpu_buffer_rsrc_t src = make_rsrc(in + plane * (int64_t)ny * nx, in_bytes);
        const int row = y * nx, lim = y < ny ? nx : 0;
        if (pairs) {
#pragma unroll
            for (int m = 0; m < EL; ++m) {
                const int i0 = 2 * (jx + TCX * m);
                r[m] = buf_cplx<T>(src, i0 < lim ? (row + i0) * (int)sizeof(T) : (int)in_bytes, 0);
            }
        } else {
#pragma unroll
            for (int m = 0; m < EL; ++m) {
                const int i0 = 2 * (jx + TCX * m);
                r[m].x = buf_real<T>(src, i0 < lim ? (row + i0) * (int)sizeof(T) : (int)in_bytes, 0);
                r[m].y = buf_real<T>(src, i0 + 1 < lim ? (row + i0 + 1) * (int)sizeof(T) : (int)in_bytes, 0);
            }
        }
    };
    cplx<T> nxt[PF ? NP : 1][EL];
    int64_t plane = blockIdx.x;
    if constexpr (PF) {
#pragma unroll
        for (int q = 0; q < NP; ++q) load_row(nxt[q], plane, fresh(), q);
    }
    __syncthreads();                                              // the tables
    for (; plane < nplanes; plane += gridDim.x) {
        // 1. rows: reals in pairs, length-M transform, split into M + 1 outputs
#pragma unroll (PF ? NP : 1)
        for (int q = 0; q < NP; ++q) {
            if (yw + q * S::RPP < ny) {                           // whole waves
                const int tq = fresh(), jx = tq % TCX, y = tq / TCX + q * S::RPP;   // row y, lane jx of it
                if constexpr (!PF) load_row(nxt[0], plane, tq, q);
                cplx<T> reg[EX];
#pragma unroll
                for (int m = 0; m < EX; ++m) reg[m] = m < EL ? nxt[PF ? q : 0][m] : cplx<T>{T(0), T(0)};
                const RowPad lay{xld, S::SH};
                fft_regs<T, M, EX, true, (HX && EX > 1), true>(reg, pl, lay, y, jx, twx);
                stage_sync<true>();
#pragma unroll
                for (int m = 0; m < EX; ++m) pl[lay(jx + TCX * m, y)] = reg[m];
                stage_sync<true>();
                const T half = T(0.5);
                cplx<T> xs[EX];
#pragma unroll
                for (int m = 0; m < EX; ++m) {
                    const int k = jx + TCX * m;
                    const cplx<T> zk = pl[lay(k, y)];
                    const cplx<T> zm = cconj(pl[lay((M - k) & (M - 1), y)]);
                    const cplx<T> e = cadd(zk, zm);
                    const cplx<T> wd = cmul(twx[M + k], csub(zk, zm));    // W_P^k (Z[k] - conj Z[M-k])
                    xs[m] = {half * (e.x + wd.y), half * (e.y - wd.x)};   // e/2 - (i/2) wd
                }
                const cplx<T> z0 = pl[lay(0, y)];
                stage_sync<true>();                               // the row is read: its spectrum takes its place
#pragma unroll
                for (int m = 0; m < EX; ++m) pl[y * xld + jx + TCX * m] = xs[m];
                if (jx == 0) nyq[y] = {z0.x - z0.y, T(0)};
            }
        }
        __syncthreads();
        if constexpr (PF) {
            const int64_t np = plane + gridDim.x;
            if (np < nplanes) {
#pragma unroll
                for (int q = 0; q < NP; ++q) load_row(nxt[q], np, fresh(), q);
            }
        }
        // 2. columns (rows >= ny are zero)
        int rs = zp * (int)wx;                                    // (a group's offsets fit 32 bits)
        asm volatile("" : "+s"(rs));                              // (its multiples are not kept across planes)
        const uint32_t bytes = (uint32_t)(((int64_t)(PY - 1) * rs + M + 1) * (int64_t)sizeof(cplx<T>));
        const __amdgpu_buffer_rsrc_t dst =
            make_rsrc(out + (plane / zp) * zp * (int64_t)PY * wx + (plane % zp) * wx, bytes);
        {
            cplx<T> v[E];
            const int tq = fresh(), c = w * S::GC + tq % S::GC, p = (tq & 63) / S::GC;   // column c, lane p of it
            const int off = c < M ? (p * rs + c) * (int)sizeof(cplx<T>) : (int)bytes;
            const cplx<T>* col = pl + p * xld + (M >= S::GC || c < M ? c : 0);
            col_fft<PY, true, HY>(
                v, twy, p,
                [&](int m) { return col[(S::LP * m < rows ? S::LP * m : rows) * xld]; },   // rows ny and up hold zeros
                [&](int r0, int dr, const auto& r) {
#pragma unroll
                    for (int k = 0; k < (int)(sizeof(r) / sizeof(r[0])); ++k)
                        buf_store_cplx<T>(dst, off, (r0 + dr * k) * rs * (int)sizeof(cplx<T>), r[k]);
                });
        }
        if (w == S::NW - 1) {                                     // column M, in the last wave
            constexpr int EN = PY < 8 ? PY : 8, TN = PY / EN;     // TN <= 32 lanes
            const int ln = fresh() & 63, jn = ln % TN;
            cplx<T> r[EN];
#pragma unroll
            for (int m = 0; m < EN; ++m) {
                const int y = jn + TN * m;
                r[m] = y < ny ? nyq[y] : cplx<T>{T(0), T(0)};
            }
            fft_regs<T, PY, EN, true, HY, true, col_apart<PY>()>(r, nyq, ColMajor{1}, 0, jn, twx + 2 * M, ln < TN);
            const int off = ln < TN ? (jn * rs + M) * (int)sizeof(cplx<T>) : (int)bytes;
#pragma unroll
            for (int m = 0; m < EN; ++m) buf_store_cplx<T>(dst, off, TN * m * rs * (int)sizeof(cplx<T>), r[m]);
        }
        if constexpr (PF) __syncthreads();                        // the plane is read: the next one takes its LDS
    }
}

// PF as above: the next plane's columns are requested before the rows phase.
template <typename T, int PY, int M, bool HY, bool PF>
__global__ void __launch_bounds__((PlaneShape<T, PY, M>::NT)) __attribute__((amdgpu_waves_per_eu(PlaneShape<T, PY, M>::NT > 512 ? 1 : 2)))
    k_yx_inv(const cplx<T>* __restrict__ in, T* __restrict__ out, int64_t nplanes, int ny, int nx, int64_t wx,
             const cplx<T>* __restrict__ tw, int rows_arg, int pairs, double* __restrict__ rowsq, int zp) {
    using S = PlaneShape<T, PY, M>;
    constexpr int EX = S::EX, TCX = S::TCX, E = S::E;
    constexpr int RMAX = HY ? PY / 2 : PY;
    constexpr int NP = (RMAX + S::RPP - 1) / S::RPP;
    // Column M: packed as the imaginary part of column 0 (PF, wave 0, EN values
    // per lane on their way), or a transform of its own in the last wave (EN
    // values in each of TN lanes).
    constexpr int EN = PF ? PY / 64 : 8, TN = PY / 8;
    constexpr bool LATE = !PF && E * sizeof(T) >= 256;            // column M after the others: registers are short
    const int wm = PF ? 0 : S::NW - 1;
    constexpr int xld = S::LD;
    const int rows = rows_arg;                                    // rows held: ny rounded up to whole waves
    extern __shared__ unsigned char smem_raw[];
    cplx<T>* const pl = reinterpret_cast<cplx<T>*>(smem_raw);
    cplx<T>* const nyq = pl + (size_t)(rows < RMAX ? rows + 4 : rows) * xld;
    cplx<T>* const twy = nyq + S::NYN;
    cplx<T>* const twx = twy + S::TWN;
    const int t = (int)threadIdx.x, w = __builtin_amdgcn_readfirstlane(t >> 6);
    load_plane_tables<T, PY, M>(twy, twx, tw);
    auto fresh = [&]() {                                          // (see the forward)
        int q = t;
        if constexpr (PF) asm volatile("" : "+v"(q));
        return q;
    };
    const int yw = w * S::RPW;
    cplx<T> v[E], vm[EN];
    auto load_cols = [&](int64_t plane) {
        int rs = zp * (int)wx;                                    // (a group's offsets fit 32 bits)
        asm volatile("" : "+s"(rs));                              // (its multiples are not kept across planes)
        const __amdgpu_buffer_rsrc_t src =
            make_rsrc(in + (plane / zp) * zp * (int64_t)PY * wx + (plane % zp) * wx,
                      (uint32_t)(((int64_t)(PY - 1) * rs + M + 1) * (int64_t)sizeof(cplx<T>)));
        const int tq = fresh(), lane = tq & 63, c = w * S::GC + tq % S::GC, p = lane / S::GC;
        const int off = (p * rs + (c < M ? c : 0)) * (int)sizeof(cplx<T>);
#pragma unroll
        for (int a = 0; a < E / 8; ++a)                           // in the order the first stage takes them
#pragma unroll
            for (int m = a; m < E; m += E / 8) v[m] = buf_cplx<T>(src, off, S::LP * m * rs * (int)sizeof(cplx<T>));
        if (!LATE && w == wm) {
            constexpr int dm = PF ? 64 : TN;
            const int offm = (lane % dm * rs + M) * (int)sizeof(cplx<T>);
#pragma unroll
            for (int m = 0; m < EN; ++m) vm[m] = buf_cplx<T>(src, offm, dm * m * rs * (int)sizeof(cplx<T>));
        }
    };
    auto column_m = [&](cplx<T> (&r)[EN], int lane) {
        if constexpr (!PF) {
            const int jn = lane % TN;
            fft_regs<T, PY, EN, false, false, true, col_apart<PY>()>(r, nyq, ColMajor{1}, 0, jn, twx + 2 * M, lane < TN);
            stage_sync<true>();
            if (lane < TN) {
#pragma unroll
                for (int m = 0; m < EN; ++m) nyq[jn + TN * m] = r[m];
            }
        }
    };
    int64_t plane = blockIdx.x;
    if (plane < nplanes) load_cols(plane);
    __syncthreads();                                              // the tables
    for (; plane < nplanes; plane += gridDim.x) {
        // 1. columns
        const int tc = fresh(), lane = tc & 63, c = w * S::GC + tc % S::GC, p = lane / S::GC;
        if (w == wm) {
            if constexpr (PF) {
#pragma unroll
                for (int m = 0; m < EN; ++m) nyq[lane + 64 * m] = vm[m];
                stage_sync<true>();
                if (c == 0) {
#pragma unroll
                    for (int m = 0; m < E; ++m) {
                        const cplx<T> xm = nyq[p + S::LP * m];
                        v[m] = {v[m].x - xm.y, v[m].y + xm.x};
                    }
                }
            } else if constexpr (!LATE) {
                column_m(vm, lane);
            }
        }
        col_fft<PY, false, false>(
            v, twy, p, [&](int m) { return v[m]; },
            [&](int r0, int dr, const auto& r) {
#pragma unroll
                for (int k = 0; k < (int)(sizeof(r) / sizeof(r[0])); ++k)
                    if (r0 + dr * k < (HY ? PY / 2 : PY) && r0 + dr * k < rows && (M >= S::GC || c < M))
                        pl[(p + r0 + dr * k) * xld + c] = r[k];
            });
        if constexpr (LATE) {
            if (w == wm) {
                const int rs = zp * (int)wx;
                const cplx<T>* src = in + (plane / zp) * zp * (int64_t)PY * wx + (plane % zp) * wx + M;
                cplx<T> r[EN];
#pragma unroll
                for (int m = 0; m < EN; ++m) r[m] = src[(int64_t)(lane % TN + TN * m) * rs];
                column_m(r, lane);
            }
        }
        if constexpr (PF) {
            if (plane + gridDim.x < nplanes) load_cols(plane + gridDim.x);
        }
        __syncthreads();
        // 2. rows: split into Z', inverse x, nx reals
#pragma unroll 1
        for (int q = 0; q < NP; ++q) {
            if (yw + q * S::RPP >= ny) break;                     // whole waves
            const int tq = fresh(), jx = tq % TCX, y = tq / TCX + q * S::RPP;
            const bool ok = y < ny;
            cplx<T>* row = pl + y * xld;                          // (rows is a multiple of a wave's rows)
            cplx<T> reg[EX];
#pragma unroll
            for (int m = 0; m < EX; ++m) {
                const int k = jx + TCX * m;
                cplx<T> xk = row[k];
                cplx<T> xm = cconj(row[(M - k) & (M - 1)]);
                if (m == 0 && k == 0) {
                    if constexpr (PF) {                           // X[0] and X[M], both real, packed in column 0
                        xm = {xk.y, T(0)};
                        xk = {xk.x, T(0)};
                    } else {
                        xm = cconj(nyq[y]);
                    }
                }
                const cplx<T> e = cadd(xk, xm);
                const cplx<T> wd = twmul<false>(csub(xk, xm), twx[M + k]);   // exp(+2 pi i k/P) (X[k] - conj X[M-k])
                reg[m] = {e.x - wd.y, e.y + wd.x};                           // e + i wd
            }
            stage_sync<true>();                                   // the row is read: its LDS serves the exchanges
            fft_regs<T, M, EX, false, false, true>(reg, pl, RowPad{xld, S::SH}, y, jx, twx);
            const uint32_t out_bytes = (uint32_t)((int64_t)ny * nx * sizeof(T));
            const __amdgpu_buffer_rsrc_t dst = make_rsrc(out + plane * (int64_t)ny * nx, out_bytes);
            const int lim = ok ? nx : 0;                          // (stores at the plane's size are dropped)
            if (pairs) {
#pragma unroll
                for (int m = 0; m < EX; ++m) {
                    const int i0 = 2 * (jx + TCX * m);
                    buf_store_cplx<T>(dst, i0 < lim ? (y * nx + i0) * (int)sizeof(T) : (int)out_bytes, 0, reg[m]);
                }
            } else {
#pragma unroll
                for (int m = 0; m < EX; ++m) {
                    const int i0 = 2 * (jx + TCX * m);
                    buf_store_real(dst, i0 < lim ? (y * nx + i0) * (int)sizeof(T) : (int)out_bytes, 0, reg[m].x);
                    buf_store_real(dst, i0 + 1 < lim ? (y * nx + i0 + 1) * (int)sizeof(T) : (int)out_bytes, 0, reg[m].y);
                }
            }
            if (rowsq && ok) row_square_sum<T, EX, TCX>(reg, jx, nx, rowsq + plane * (int64_t)ny + y);
            stage_sync<true>();
        }
        if constexpr (PF) __syncthreads();                        // the rows are read: the next plane takes their LDS
    }
}

// LDS of a block: the rows held (whole waves of rows, and four spare ones when
// that is not every row), the Nyquist column, the tables.
template <typename T, int PY, int M>
size_t plane_lds_bytes(int rows, int rmax) {
    using S = PlaneShape<T, PY, M>;
    return ((size_t)(rows < rmax ? rows + 4 : rows) * S::LD + S::NYN + S::TWN + 2 * M + PY) * sizeof(cplx<T>);
}

constexpr size_t kPlaneLds = 160 * 1024;     // LDS of a CU on gfx950
constexpr int kCUs = 256;

// A launch holds less than 2^32 threads: whole groups of zp planes, at most 2^22
// planes of 512 threads at a time.
template <class F>
void for_plane_chunks(int64_t nplanes, int zp, F&& launch) {
    const int64_t chunk = std::max<int64_t>(1, (int64_t(1) << 22) / zp) * zp;
    for (int64_t first = 0; first < nplanes; first += chunk) launch(first, std::min(chunk, nplanes - first));
}

template <typename T, int PY, int M>
void plane_fwd_launch(const T* in, cplx<T>* out, int64_t nplanes, int ny, int nx, int64_t wx, const cplx<T>* tw,
                      hipStream_t s, int zp) {
    using S = PlaneShape<T, PY, M>;
    constexpr bool PF = sizeof(T) == 4 && PY == 256 && M == 128;
    const int rows = (int)round_up(ny, S::RPW);
    const size_t lds = plane_lds_bytes<T, PY, M>(rows, ny <= PY / 2 ? PY / 2 : PY);
    if (lds > kPlaneLds || ny < 1 || ny > (PY < 256 ? PY : PY / 2) || nx < 1 || nx > 2 * M)
        fail(DDSTRESS_E_INVALID, "plane does not fit the fused forward x-y kernel");
    const int pairs = (reinterpret_cast<uintptr_t>(in) % sizeof(cplx<T>) == 0 && nx % 2 == 0) ? 1 : 0;
    for_plane_chunks(nplanes, zp, [&](int64_t first, int64_t np) {
        const dim3 grid((unsigned)(PF && np > kCUs ? kCUs : np)), block(S::NT);
        const T* src = in + first * ny * nx;
        cplx<T>* dst = out + first * PY * wx;
#define DDS_FWD(HXV, HYV)                                                                                          \
        hipLaunchKernelGGL((k_xy_fwd<T, PY, M, HXV, HYV, (PF && HYV)>), grid, block, lds, s, src, dst, np, ny, nx, wx, \
                           tw, rows, pairs, zp)
        if (ny <= PY / 2) {
            if (nx <= M) DDS_FWD(true, true);
            else DDS_FWD(false, true);
        } else if constexpr (PY < 256) {                              // (a full plane of 256 rows does not fit)
            if (nx <= M) DDS_FWD(true, false);
            else DDS_FWD(false, false);
        }
#undef DDS_FWD
    });
}

template <typename T, int PY, int M>
void plane_inv_launch(const cplx<T>* in, T* out, int64_t nplanes, int ny, int nx, int64_t wx, const cplx<T>* tw,
                      hipStream_t s, double* rowsq, int zp) {
    using S = PlaneShape<T, PY, M>;
    constexpr bool PF = sizeof(T) == 4 && PY == 256 && M == 128;
    const int rows = (int)round_up(ny, S::RPW);
    const size_t lds = plane_lds_bytes<T, PY, M>(rows, ny <= PY / 2 ? PY / 2 : PY);
    if (lds > kPlaneLds || ny < 1 || ny > (PY < 256 ? PY : PY / 2) || nx < 1 || nx > 2 * M)
        fail(DDSTRESS_E_INVALID, "plane does not fit the fused inverse y-x kernel");
    const int pairs = (reinterpret_cast<uintptr_t>(out) % sizeof(cplx<T>) == 0 && nx % 2 == 0) ? 1 : 0;
    for_plane_chunks(nplanes, zp, [&](int64_t first, int64_t np) {
        const dim3 grid((unsigned)(PF && np > kCUs ? kCUs : np)), block(S::NT);
        const cplx<T>* src = in + first * PY * wx;
        T* dst = out + first * ny * nx;
        double* sums = rowsq ? rowsq + first * ny : nullptr;
        if (ny <= PY / 2)
            hipLaunchKernelGGL((k_yx_inv<T, PY, M, true, PF>), grid, block, lds, s, src, dst, np, ny, nx, wx, tw, rows,
                               pairs, sums, zp);
        else if constexpr (PY < 256)
            hipLaunchKernelGGL((k_yx_inv<T, PY, M, false, false>), grid, block, lds, s, src, dst, np, ny, nx, wx, tw,
                               rows, pairs, sums, zp);
    });
}

// Every plane shape of precision T: F<PY, M>(...) for the given lengths.
#define DDS_PLANE_M(PYV, CALL)                  \
    switch (M) {                                \
        case 8: CALL(PYV, 8); break;            \
        case 16: CALL(PYV, 16); break;          \
        case 32: CALL(PYV, 32); break;          \
        case 64: CALL(PYV, 64); break;          \
        case 128: CALL(PYV, 128); break;        \
        default: fail(DDSTRESS_E_INVALID, "plane lengths not covered by the fused x-y kernels"); \
    }

}  // namespace dds
