// Fused single-pass separable tile, shared by the per-image and batched kernels.
#pragma once
#include "icl_device.hpp"
#include "tile_stage.hpp"

namespace icl {

// ------------------------------------------------------------------ fused tile (also used by the batched kernel)
// Geometry of one fused tile for radius R.
template <int R, int TH, int CX> struct SepTile {
    static constexpr int TW = 64 * CX;           // output columns
    static constexpr int RA = (R + 3) & ~3;      // column halo rounded up to whole float4s
    static constexpr int LW = TW + 2 * RA;       // staged input row length (floats)
    static constexpr int NR = TH + 2 * R;        // staged input rows
    static constexpr int LDS_FLOATS = NR * LW + NR * TW;
};

// Row pass over a staged tile: in_s [NR][LW] -> t_s [NR][TW], four columns per item.
// UNR > 0 caps the unrolling of the item loop (a trip count known at compile time is
// otherwise unrolled whole, with every item's window in registers at once).
template <int R, int TH, int CX, int UNR = 0>
__device__ __forceinline__ void sep_row_pass(const float* __restrict__ in_s, float* __restrict__ t_s,
                                             const float* __restrict__ tx) {
    using G = SepTile<R, TH, CX>;
    constexpr int TW = G::TW, RA = G::RA, LW = G::LW, NR = G::NR, G4 = TW / 4;
    auto item = [&](int idx) {
        const int rr = idx / G4, g = idx - rr * G4;
        float win[4 + 2 * RA];
#pragma unroll
        for (int m = 0; m < (4 + 2 * RA) / 4; ++m) {
            const v4f v = lds4(&in_s[rr * LW + 4 * g + 4 * m]);
            win[4 * m] = v.x; win[4 * m + 1] = v.y; win[4 * m + 2] = v.z; win[4 * m + 3] = v.w;
        }
        float o[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i <= 2 * R; ++i) {
            const float h = tx[i];
#pragma unroll
            for (int p = 0; p < 4; ++p) o[p] = fmaf(h, win[RA - R + p + i], o[p]);
        }
        lds4(&t_s[rr * TW + 4 * g], mk4(o[0], o[1], o[2], o[3]));
    };
    if constexpr (UNR > 0) {
#pragma unroll UNR
        for (int idx = threadIdx.x; idx < NR * G4; idx += 256) item(idx);
    } else {
        for (int idx = threadIdx.x; idx < NR * G4; idx += 256) item(idx);
    }
}

// Column pass: lane owns 4 adjacent columns (group g of TW/4) and PYC consecutive rows;
// the t_s rows it needs are read as float4, and the 4 outputs of a row are stored as one
// vector wherever they all lie in the image.
// GROUP > 0 fences the schedule every GROUP staged rows, so that at most GROUP rows' reads are
// in registers at a time (a kernel that must fit a register budget).
template <class T, int R, int TH, int CX, int GROUP = 0>
__device__ __forceinline__ void sep_col_pass(const float* __restrict__ t_s, void* __restrict__ dst, size_t dp, int W,
                                             int H, const float* __restrict__ ty, int x0, int y0) {
    using G = SepTile<R, TH, CX>;
    constexpr int TW = G::TW, G4 = TW / 4, RPI = 256 / G4, PYC = TH / RPI;
    static_assert(PYC * RPI == TH, "tile rows must split evenly over the row groups");
    const int g = threadIdx.x % G4, rg = threadIdx.x / G4;
    const float* col = t_s + (rg * PYC) * TW + 4 * g;
    // each staged row is read once and added into every output row it feeds
    v4f acc[PYC];
#pragma unroll
    for (int py = 0; py < PYC; ++py) acc[py] = mk4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int m = 0; m < PYC + 2 * R; ++m) {
        if (GROUP > 0 && m > 0 && m % GROUP == 0) __builtin_amdgcn_sched_barrier(0);
        const v4f v = lds4(col + m * TW);
#pragma unroll
        for (int py = 0; py < PYC; ++py) {
            const int j = m - py;
            if (j < 0 || j > 2 * R) continue;
            const float c = ty[j];
            acc[py].x = fmaf(c, v.x, acc[py].x);
            acc[py].y = fmaf(c, v.y, acc[py].y);
            acc[py].z = fmaf(c, v.z, acc[py].z);
            acc[py].w = fmaf(c, v.w, acc[py].w);
        }
    }
    const int x = x0 + 4 * g;
#pragma unroll
    for (int py = 0; py < PYC; ++py) {
        const int y = y0 + rg * PYC + py;
        if (y >= H) break;
        const size_t row = (size_t)y * dp;
        const v4f a = acc[py];
        if (x + 4 <= W) {
            store4<T>(dst, row + (size_t)x * T::size, a);
        } else {
            if (x < W) store_px<T>(dst, row + (size_t)x * T::size, a.x);
            if (x + 1 < W) store_px<T>(dst, row + (size_t)(x + 1) * T::size, a.y);
            if (x + 2 < W) store_px<T>(dst, row + (size_t)(x + 2) * T::size, a.z);
            if (x + 3 < W) store_px<T>(dst, row + (size_t)(x + 3) * T::size, a.w);
        }
    }
}

// Computes one TW x TH output tile whose top-left output pixel is (x0, y0), staging
// directly (no prefetch).  `lds` holds SepTile::LDS_FLOATS floats.
template <class T, int R, int TH, int CX>
__device__ __forceinline__ void sep_tile_body(const void* __restrict__ src, size_t sp, void* __restrict__ dst,
                                              size_t dp, int W, int H, const float* __restrict__ tx,
                                              const float* __restrict__ ty, int x0, int y0, float* __restrict__ lds,
                                              Border bd = {}) {
    using G = SepTile<R, TH, CX>;
    constexpr int RA = G::RA, LW = G::LW, NR = G::NR;
    float* in_s = lds;             // [NR][LW]
    float* t_s = lds + NR * LW;    // [NR][TW]
    Stage<T, NR, LW> st;           // every load is issued before any is written to LDS
    st.load(src, sp, W, H, x0 - RA, y0 - R);
    st.store(in_s, W, H, bd);
    __syncthreads();
    sep_row_pass<R, TH, CX>(in_s, t_s, tx);
    __syncthreads();
    sep_col_pass<T, R, TH, CX>(t_s, dst, dp, W, H, ty, x0, y0);
}

}  // namespace icl
