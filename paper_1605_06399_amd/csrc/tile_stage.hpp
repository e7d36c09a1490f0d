// Persistent tile machinery shared by the stencil kernels.
//
// A staged tile is NR rows x LW columns of float32 (LW a multiple of 4) whose
// top-left element is image pixel (gx0, gy0).  Stage<> loads it from global
// memory into registers (float4 per slot, 256 lanes), so the loads of the NEXT
// tile can be in flight while the current one is computed from LDS, and then
// writes the registers to LDS.  Reads outside the image follow the boundary: clamp or a
// constant (Border).
#pragma once
#include <type_traits>

#include "icl_device.hpp"

namespace icl {

// Columns x .. x + 3 of a row (x a multiple of 4, on either side of the row's ends too) read through the
// clamp, in two parts that need no branch: a vector load from the nearest position inside the row, then
// its elements moved to where they belong.  Rows of fewer than 4 pixels are read pixel by pixel.
template <class T>
__device__ __forceinline__ v4f load4_clamped(const void* __restrict__ src, size_t row, int W, int x) {
    if (W >= 4) return load4<T>(src, row + (size_t)min(max(x, 0), W - 4) * T::size);
    v4f v;
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = load_px<T>(src, row + (size_t)clampi(x + q, W) * T::size);
    return v;
}
__device__ __forceinline__ v4f fix4_clamped(v4f v, int W, int x) {
    if (W < 4) return v;
    const int d = x - min(max(x, 0), W - 4);   // right of the row's end: element q is the loaded q + d, at most the last
    if (d >= 4 || (d & 2 && d > 0)) v = mk4(v.z, v.w, v.w, v.w);
    if (d >= 4 || (d & 1 && d > 0)) v = mk4(v.y, v.z, v.w, v.w);
    if (d < 0) v = mk4(v.x, v.x, v.x, v.x);    // left of column 0: d <= -4
    return v;
}
// The elements of columns x .. x + 3 of row y that lie outside the image replaced by c.
__device__ __forceinline__ v4f outside4(v4f v, int W, int H, int x, int y, float c) {
    const bool row = y < 0 || y >= H;
#pragma unroll
    for (int q = 0; q < 4; ++q)
        if (row || x + q < 0 || x + q >= W) v[q] = c;
    return v;
}

template <class T, int NR, int LW>
struct Stage {
    static constexpr int C4 = LW / 4;
    static constexpr int N = (NR * C4 + 255) / 256;
    v4f v[N];
    int gx = 0, gy = 0;   // top-left pixel of the loaded tile (gx = -1: a constant fill)

    // Load the tile with top-left pixel (gx0, gy0), gx0 a multiple of 4.  Only loads: nothing here waits
    // for one, so a tile can be in flight while another is computed.
    __device__ __forceinline__ void load(const void* __restrict__ src, size_t sp, int W, int H, int gx0, int gy0) {
        gx = gx0;
        gy = gy0;
        // A tile that lies inside the image (the work-group's usual case) takes straight vector loads.
        if (inside(W, H)) {
#pragma unroll
            for (int k = 0; k < N; ++k) {
                const int idx = (int)threadIdx.x + 256 * k;
                if (N * 256 != NR * C4 && idx >= NR * C4) break;
                const int rr = idx / C4, c4 = idx - rr * C4;
                v[k] = load4<T>(src, (size_t)(gy0 + rr) * sp + (size_t)(gx0 + 4 * c4) * T::size);
            }
            return;
        }
        // A tile at the image's edge does the same from clamped addresses, and store() puts the pixels in
        // their places (a branch per chunk would make the compiler wait on each load in turn: 57 against
        // 44 us on a 256^3 volume, half of whose 64-column tiles are at an edge).
#pragma unroll
        for (int k = 0; k < N; ++k) {
            const int idx = (int)threadIdx.x + 256 * k;
            if (N * 256 != NR * C4 && idx >= NR * C4) break;
            const int rr = idx / C4, c4 = idx - rr * C4;
            v[k] = load4_clamped<T>(src, (size_t)clampi(gy0 + rr, H) * sp, W, gx0 + 4 * c4);
        }
    }

    // Every element the constant c (a whole staged region outside the image): stored as it is.
    __device__ __forceinline__ void fill(float c) {
#pragma unroll
        for (int k = 0; k < N; ++k) v[k] = mk4(c, c, c, c);
        gx = -1;
    }

    // Write the loaded tile to LDS.  bd: the boundary (clamp or a constant).
    __device__ __forceinline__ void store(float* __restrict__ s, int W, int H, Border bd = {}) const {
        const bool edge = gx != -1 && !inside(W, H);
#pragma unroll
        for (int k = 0; k < N; ++k) {
            const int idx = (int)threadIdx.x + 256 * k;
            if (N * 256 != NR * C4 && idx >= NR * C4) break;
            const int rr = idx / C4, c4 = idx - rr * C4;
            v4f e = v[k];
            if (edge) {
                const int x = gx + 4 * c4, y = gy + rr;
                e = fix4_clamped(e, W, x);
                if (bd.constant) e = outside4(e, W, H, x, y, bd.value);
            }
            lds4(&s[rr * LW + 4 * c4], e);
        }
    }

    __device__ __forceinline__ bool inside(int W, int H) const {
        return gx >= 0 && gx + LW <= W && gy >= 0 && gy + NR <= H;
    }
};

// Tile t of a tiles_x-wide row-major tiling -> top-left output pixel.
__device__ __forceinline__ void tile_origin(int t, int tiles_x, int tw, int th, int& x0, int& y0) {
    const int ty = t / tiles_x;
    x0 = (t - ty * tiles_x) * tw;
    y0 = ty * th;
}

// First tile of this block in a persistent walk (stride gridDim.x).  With a grid that
// is a multiple of 8, consecutive tiles of each round go to one XCD, so tiles sharing
// halo rows meet in the same L2.
__device__ __forceinline__ int first_tile() { return (int)xcd_remap(blockIdx.x, gridDim.x); }

// Persistent schedule over a tiles_x x tiles_y grid (tiles numbered row-major) that keeps
// halo reuse inside one L2: the grid is cut into 8 column bands, one per XCD (gfx950
// places work-group b on XCD b % 8), and the blocks of an XCD walk their band row by
// row.  A tile's upper neighbour was therefore processed on the same XCD shortly before,
// and the halo rows they share are served from that XCD's L2 rather than HBM.
struct BandWalk {
    int tiles_x, bx0, bw, nband, slot, nslots;
    __device__ __forceinline__ BandWalk(int tx, int ty) : tiles_x(tx) {
        const int g = (int)gridDim.x;
        // one band per XCD; fewer when the grid or the tile row is too small, so every
        // band owns at least one block and one column (every tile is covered exactly once)
        int nb = g < 8 ? g : 8;
        nb = nb < tx ? nb : tx;
        const int x = (int)blockIdx.x % nb;
        slot = (int)blockIdx.x / nb;
        nslots = g / nb + (x < g % nb ? 1 : 0);
        bx0 = x * tx / nb;
        bw = (x + 1) * tx / nb - bx0;
        nband = bw * ty;
    }
    // k-th tile of this block, or -1 when its band is exhausted
    __device__ __forceinline__ int tile(int k) const {
        const int j = k * nslots + slot;
        if (j >= nband) return -1;
        const int row = j / bw;
        return row * tiles_x + bx0 + (j - row * bw);
    }
};

}  // namespace icl

namespace icl {

// Staged tile whose shape is known only at run time (NR <= NRMAX rows, LW = 4*C4 <= 128
// columns), as in a batch whose images have different radii.  The 256 lanes form 8 rows
// x 32 float4 columns, so no division by the runtime row length is needed.
template <class T, int NRMAX>
struct RStage {
    static constexpr int K = (NRMAX + 7) / 8;
    static constexpr bool BF = std::is_same<T, BF16>::value;
    v4f v[K];
    bool raw = false;   // bfloat16 fast path: v[k].x, .y hold the four packed values, unpacked at store

    // vec: rows 4-pixel aligned in memory (gx0 a multiple of 4)
    __device__ __forceinline__ void load(const void* __restrict__ src, size_t sp, int W, int H, int gx0, int gy0,
                                         int NR, int C4, bool vec) {
        const int c4 = threadIdx.x & 31, ry = threadIdx.x >> 5;
        if (c4 >= C4) return;
        const int x = gx0 + 4 * c4;
        raw = false;
        // inside the image: straight vector loads, all in flight together (bfloat16 stays
        // packed until the LDS store, which keeps the registers of the walk in check)
        if (vec && gx0 >= 0 && gx0 + 4 * C4 <= W && gy0 >= 0 && gy0 + NR <= H) {
            raw = BF;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int rr = ry + 8 * k;
                if (rr >= NR) break;
                const size_t off = (size_t)(gy0 + rr) * sp + (size_t)x * T::size;
                if constexpr (BF) {
                    const v2u u = *reinterpret_cast<const v2u*>(static_cast<const char*>(src) + off);
                    v[k].x = __uint_as_float(u.x);
                    v[k].y = __uint_as_float(u.y);
                } else {
                    v[k] = load4<T>(src, off);
                }
            }
            return;
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int rr = ry + 8 * k;
            if (rr >= NR) break;
            v[k] = load4_clamped<T>(src, (size_t)clampi(gy0 + rr, H) * sp, W, x);
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if (ry + 8 * k >= NR) break;
            v[k] = fix4_clamped(v[k], W, x);
        }
    }

    __device__ __forceinline__ void store(float* __restrict__ s, int NR, int C4) const {
        const int c4 = threadIdx.x & 31, ry = threadIdx.x >> 5;
        if (c4 >= C4) return;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int rr = ry + 8 * k;
            if (rr >= NR) break;
            v4f e = v[k];
            if (BF && raw) {
                const unsigned a = __float_as_uint(v[k].x), b = __float_as_uint(v[k].y);
                e = mk4(__uint_as_float(a << 16), __uint_as_float(a & 0xffff0000u), __uint_as_float(b << 16),
                        __uint_as_float(b & 0xffff0000u));
            }
            lds4(&s[rr * 4 * C4 + 4 * c4], e);
        }
    }
};

}  // namespace icl
