// Harris corner response (ImageCL paper, Section 6: Harris corner detection,
// a Sobel kernel (Table 4) followed by a Harris kernel that reads the gradient
// images as Images (Table 5), so window reads clamp on the gradient images).
//
//   Ix = sum s[j] d[i] src(x+i, y+j),  Iy = sum d[j] s[i] src(x+i, y+j)
//        s = (1,2,1), d = (-1,0,1)
//   Sxx = sum_{j,i} g[j] g[i] Ix^2(x+i, y+j)   (Syy from Iy^2, Sxy from Ix*Iy)
//   R   = Sxx*Syy - Sxy^2 - k*(Sxx+Syy)^2
//
// Variants
//   plain_split   : the paper's two kernels with naive mapping: Sobel writes Ix, Iy
//                   (float32, workspace), the Harris kernel reads them with a
//                   clamped 2-D window loop.  16 B/px of HBM beyond in/out.
//   fused_t{TH}   : one pass per 64 x TH tile.  The image tile with a (1 + rg) halo
//                   is staged in LDS; gradients are evaluated at the clamped
//                   positions of the (64+2rg) x (TH+2rg) gradient region (which is
//                   exactly "window reads clamp on the gradient image"), their
//                   products go to LDS, and the separable window runs as a row pass
//                   into LDS and a column pass in registers.  8 B/px of HBM.
//   stream_t{TH}  : one wave per 248-column strip and TH rows, walking down the rows
//                   with everything in registers (one float4 image load per lane and
//                   row, neighbour columns by DPP lane shifts, rings of prefetched image
//                   rows and of pending output rows).  16-byte aligned rows, W >= 256.
//   strips_t{TH}  : the same strips for rows of any alignment and any width.
#include "harris_strip.hpp"
#include "icl_device.hpp"
#include "icl_internal.hpp"
#include "tile_stage.hpp"

namespace icl {
namespace {

// ------------------------------------------------------------------ plain split
__global__ __launch_bounds__(256) void sobel_plain(const float* __restrict__ src, size_t sp, float* __restrict__ ix,
                                                   float* __restrict__ iy, int W, int H) {
    const int x = blockIdx.x * 16 + threadIdx.x % 16;
    const int y = blockIdx.y * 16 + threadIdx.x / 16;
    if (x >= W || y >= H) return;
    const float s[3] = {1.f, 2.f, 1.f}, d[3] = {-1.f, 0.f, 1.f};
    float gx = 0.f, gy = 0.f;
    for (int j = -1; j <= 1; ++j) {
        const float* row = reinterpret_cast<const float*>(reinterpret_cast<const char*>(src) +
                                                          (size_t)clampi(y + j, H) * sp);
        for (int i = -1; i <= 1; ++i) {
            const float p = row[clampi(x + i, W)];
            gx += s[j + 1] * d[i + 1] * p;
            gy += d[j + 1] * s[i + 1] * p;
        }
    }
    ix[(size_t)y * W + x] = gx;
    iy[(size_t)y * W + x] = gy;
}

__global__ __launch_bounds__(256) void harris_window_plain(const float* __restrict__ ix, const float* __restrict__ iy,
                                                           float* __restrict__ resp, size_t rp, int W, int H,
                                                           const float* __restrict__ g, int rg, float k) {
    const int x = blockIdx.x * 16 + threadIdx.x % 16;
    const int y = blockIdx.y * 16 + threadIdx.x / 16;
    if (x >= W || y >= H) return;
    float a = 0.f, b = 0.f, c = 0.f;
    for (int j = -rg; j <= rg; ++j)
        for (int i = -rg; i <= rg; ++i) {
            const size_t q = (size_t)clampi(y + j, H) * W + clampi(x + i, W);
            const float w = g[j + rg] * g[i + rg];
            const float gx = ix[q], gy = iy[q];
            a += w * gx * gx;
            b += w * gy * gy;
            c += w * gx * gy;
        }
    float* out = reinterpret_cast<float*>(reinterpret_cast<char*>(resp) + (size_t)y * rp);
    out[x] = harris_response(a, b, c, k);
}

hipError_t launch_plain(const HarrisArgs& a) {
    float* ix = static_cast<float*>(a.ws);
    float* iy = ix + (size_t)a.W * a.H;
    dim3 grid((a.W + 15) / 16, (a.H + 15) / 16);
    hipLaunchKernelGGL(sobel_plain, grid, dim3(256), 0, a.st, a.src, a.sp, ix, iy, a.W, a.H);
    hipLaunchKernelGGL(harris_window_plain, grid, dim3(256), 0, a.st, ix, iy, a.resp, a.rp, a.W, a.H, a.g, a.rg, a.k);
    return hipGetLastError();
}

bool supports_plain(const HarrisArgs& a) {
    return a.ws != nullptr && a.wsb >= harris_workspace(a.W, a.H) && a.rg >= 0 && a.rg <= ICL_MAX_WINDOW_RADIUS;
}

// ------------------------------------------------------------------ fused tile
template <int RG, int TH> struct HTile {
    static constexpr int TW = 64;
    static constexpr int HX = RG + 1;                 // image halo rows / cols needed
    static constexpr int HXA = (HX + 3) & ~3;         // column halo rounded to float4
    static constexpr int IW = TW + 2 * HXA;           // staged image row length
    static constexpr int IR = TH + 2 * HX;            // staged image rows
    static constexpr int GW = TW + 2 * RG;            // gradient region
    static constexpr int GH = TH + 2 * RG;
    static constexpr int PY = TH / 4;
    static constexpr int REGION1 = (IR * IW > 3 * GH * TW) ? IR * IW : 3 * GH * TW;   // image, later h
    static constexpr int LDS_FLOATS = REGION1 + 3 * GH * GW;
};

template <int RG, int TH>
__global__ __launch_bounds__(256) void harris_fused(const float* __restrict__ src, size_t sp, float* __restrict__ resp,
                                                    size_t rp, int W, int H, const float* __restrict__ g, float k,
                                                    int tiles_x, int vec_ok) {
    using G = HTile<RG, TH>;
    constexpr int TW = G::TW, HX = G::HX, HXA = G::HXA, IW = G::IW, IR = G::IR, GW = G::GW, GH = G::GH,
                  PY = G::PY;
    __shared__ __attribute__((aligned(16))) float lds[G::LDS_FLOATS];
    float* img = lds;                      // [IR][IW], dead after the gradient stage
    float* hs = lds;                       // [3][GH][TW] row-pass sums (reuses img)
    float* abc = lds + G::REGION1;         // [3][GH][GW] products Ix^2, Iy^2, Ix*Iy
    const int tid = threadIdx.x;
    const unsigned t = xcd_remap(blockIdx.x, gridDim.x);
    const int tx = (int)(t % (unsigned)tiles_x);
    const int x0 = tx * TW;
    const int y0 = (int)(t / (unsigned)tiles_x) * TH;

    // 1. stage image rows y0-HX .. y0+TH+HX-1, columns x0-HXA .. x0+TW+HXA-1 (clamped)
    // every load is issued before the LDS writes (a load-then-write loop would wait on each)
    if (vec_ok && x0 - HXA >= 0 && x0 + TW + HXA <= W) {
        constexpr int C4 = IW / 4, NCH = IR * C4, PER = (NCH + 255) / 256;
        v4f v[PER];
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int idx = tid + 256 * i;
            if (NCH % 256 != 0 && idx >= NCH) break;
            const int rr = idx / C4, c4 = idx - rr * C4;
            const int y = clampi(y0 - HX + rr, H);
            v[i] = *reinterpret_cast<const v4f*>(reinterpret_cast<const char*>(src) + (size_t)y * sp +
                                                 (size_t)(x0 - HXA + 4 * c4) * 4);
        }
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int idx = tid + 256 * i;
            if (NCH % 256 != 0 && idx >= NCH) break;
            const int rr = idx / C4, c4 = idx - rr * C4;
            lds4(&img[rr * IW + 4 * c4], v[i]);
        }
    } else {
        constexpr int NE = IR * IW, PER = (NE + 255) / 256;
        float v[PER];
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int idx = tid + 256 * i;
            if (NE % 256 != 0 && idx >= NE) break;
            const int rr = idx / IW, c = idx - rr * IW;
            const int y = clampi(y0 - HX + rr, H);
            const int x = clampi(x0 - HXA + c, W);
            v[i] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(src) + (size_t)y * sp + (size_t)x * 4);
        }
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int idx = tid + 256 * i;
            if (NE % 256 != 0 && idx >= NE) break;
            img[idx] = v[i];
        }
    }
    __syncthreads();

    // 2. gradients at the clamped position of every gradient-region pixel, then products
    for (int idx = tid; idx < GH * GW; idx += 256) {
        const int gr = idx / GW, gc = idx - gr * GW;
        const int cy = clampi(y0 - RG + gr, H), cx = clampi(x0 - RG + gc, W);
        const float* p = &img[(cy - (y0 - HX)) * IW + (cx - (x0 - HXA))];
        const float a00 = p[-IW - 1], a01 = p[-IW], a02 = p[-IW + 1];
        const float a10 = p[-1], a12 = p[1];
        const float a20 = p[IW - 1], a21 = p[IW], a22 = p[IW + 1];
        const float ix = (a02 - a00) + 2.f * (a12 - a10) + (a22 - a20);
        const float iy = (a20 - a00) + 2.f * (a21 - a01) + (a22 - a02);
        abc[idx] = ix * ix;
        abc[GH * GW + idx] = iy * iy;
        abc[2 * GH * GW + idx] = ix * iy;
    }
    __syncthreads();

    // 3. window row pass over the three product images
    for (int idx = tid; idx < GH * TW; idx += 256) {
        const int gr = idx / TW, c = idx - gr * TW;
        float sa = 0.f, sb = 0.f, sc = 0.f;
#pragma unroll
        for (int i = 0; i <= 2 * RG; ++i) {
            const float w = g[i];
            const int q = gr * GW + c + i;
            sa = fmaf(w, abc[q], sa);
            sb = fmaf(w, abc[GH * GW + q], sb);
            sc = fmaf(w, abc[2 * GH * GW + q], sc);
        }
        hs[idx] = sa;
        hs[GH * TW + idx] = sb;
        hs[2 * GH * TW + idx] = sc;
    }
    __syncthreads();

    // 4. window column pass and response: lane owns column lx, rows ly*PY .. ly*PY+PY-1
    const int lx = tid & 63, ly = tid >> 6;
    float va[PY + 2 * RG], vb[PY + 2 * RG], vc[PY + 2 * RG];
#pragma unroll
    for (int m = 0; m < PY + 2 * RG; ++m) {
        const int q = (ly * PY + m) * TW + lx;
        va[m] = hs[q];
        vb[m] = hs[GH * TW + q];
        vc[m] = hs[2 * GH * TW + q];
    }
    const int x = x0 + lx;
#pragma unroll
    for (int py = 0; py < PY; ++py) {
        float sa = 0.f, sb = 0.f, sc = 0.f;
#pragma unroll
        for (int j = 0; j <= 2 * RG; ++j) {
            const float w = g[j];
            sa = fmaf(w, va[py + j], sa);
            sb = fmaf(w, vb[py + j], sb);
            sc = fmaf(w, vc[py + j], sc);
        }
        const int y = y0 + ly * PY + py;
        if (x < W && y < H)
            reinterpret_cast<float*>(reinterpret_cast<char*>(resp) + (size_t)y * rp)[x] = harris_response(sa, sb, sc, k);
    }
}

template <int RG, int TH>
hipError_t launch_fused_R(const HarrisArgs& a) {
    using G = HTile<RG, TH>;
    const int tiles_x = (a.W + G::TW - 1) / G::TW;
    const int tiles_y = (a.H + TH - 1) / TH;
    const int vec_ok = ((uintptr_t)a.src % 16 == 0) && (a.sp % 16 == 0);
    hipLaunchKernelGGL((harris_fused<RG, TH>), dim3(tiles_x * tiles_y), dim3(256), 0, a.st, a.src, a.sp, a.resp, a.rp,
                       a.W, a.H, a.g, a.k, tiles_x, vec_ok);
    return hipGetLastError();
}

// ------------------------------------------------------------------ streaming strips
// One wave per strip of 248 output columns and TH rows.  Lane l holds the four image columns
// xs-4+4l .. xs-1+4l; lanes 1..62 own the strip's outputs, lanes 0 and 63 only supply the left and right
// halo (3 columns suffice: Sobel 1 + window radius <= 3 = 4).  The wave walks down the window rows: per
// row it loads one float4 of the image per lane (a ring of rows in flight), gets the neighbouring columns
// by DPP lane shifts, forms the three products and their horizontal window sum, and adds that row into a
// ring of 2r+1 pending output rows; the oldest completes and is written each step.  No LDS tile, no
// barrier; bound by HBM (8 B/px) on large images and by the length of a wave's chain of rows on small ones.
//
// Rows on 16 bytes of W >= 256: strip 0 is the left band of 4 columns, strips 1 .. n start at 4 + 248 (s - 1),
// and those after them are the right remainder; the bands take the tile kernel's order of the Ix sum, so that
// every column has the bits that it has always had.  Other images: strips at 248 s, all in the tile kernel's
// order.  Strips and row blocks that reach past the image are the border set and come first in the launch.
// As two launches (strips, then the bands through the tile kernel) the second had too few waves to
// fill the chip.  r = 2, defaults before and now: 8192^2 154 -> 134 us, 3000 x 2000 37 -> 21, 1920 x 1080 32 -> 13,
// 700 x 600 26 -> 11; 6001 x 5000 (rows off 16 bytes, tiles before) 118 -> 66.
constexpr int HS_COLS = 248;   // output columns per strip (62 lanes x 4)
constexpr int HS_XL = 4;       // the left band where the strips start on 16 bytes

// TILE: the interior strips take the tile kernel's order of the Ix sum (and strip 1 starts at 248)
template <int RG, int TH, bool TILE>
__global__ __launch_bounds__(64, TH <= 8 ? 2 : RG <= 1 ? 4 : 3) void harris_strips(
    const float* __restrict__ src, size_t sp, float* __restrict__ resp, size_t rp, int W, int H,
    const float* __restrict__ g, float k, StripRegion rg_, int nborder) {
    constexpr int NW = 2 * RG + 1;   // window taps = ring of pending output rows
    constexpr int D = NW;
    constexpr int K = TH + 2 * RG;   // window rows walked
    constexpr int MI = D >= 5 ? D : (D == 3 ? 6 : 5);   // image-row ring
    constexpr int X1 = TILE ? HS_COLS : HS_XL;          // where strip 1 starts
    const int lane = threadIdx.x;
    int strip, rb;
    const bool interior = (int)blockIdx.x >= nborder;
    if (interior) {
        const unsigned i = blockIdx.x - (unsigned)nborder;
        strip = rg_.s_lo + (int)(i % (unsigned)rg_.ni());
        rb = rg_.b_lo + (int)(i / (unsigned)rg_.ni());
    } else {
        rg_.border_item((int)blockIdx.x, strip, rb);
    }
    const int y0 = rb * TH;
    const int xs = strip > 0 ? X1 + (strip - 1) * HS_COLS : 0;
    const int c = xs - 4 + 4 * lane;   // first image column of this lane
    float gw[NW];
#pragma unroll
    for (int j = 0; j < NW; ++j) gw[j] = g[j];
    v4f acc[D][3];
#pragma unroll
    for (int u = 0; u < D; ++u) acc[u][0] = acc[u][1] = acc[u][2] = mk4(0.f, 0.f, 0.f, 0.f);
    auto add = [&](v4f (&a)[3], float w, v4f qa, v4f qb, v4f qc) {
        a[0] = fma4(w, qa, a[0]);
        a[1] = fma4(w, qb, a[1]);
        a[2] = fma4(w, qc, a[2]);
    };
    auto response = [&](v4f (&a)[3]) {   // and clears the sums
        const v4f r = mk4(harris_response(a[0].x, a[1].x, a[2].x, k), harris_response(a[0].y, a[1].y, a[2].y, k),
                          harris_response(a[0].z, a[1].z, a[2].z, k), harris_response(a[0].w, a[1].w, a[2].w, k));
        a[0] = a[1] = a[2] = mk4(0.f, 0.f, 0.f, 0.f);
        return r;
    };
    char* out_col = reinterpret_cast<char*>(resp) + (ptrdiff_t)c * 4;

    if (interior) {
        // every read in bounds, nothing clamped.  Window row kk is gradient row y0 - r + kk, whose Sobel
        // reads image rows y0 - r - 1 + kk + {0, 1, 2}.  The walk is unrolled completely: ring slots, row
        // ranges and prefetch bounds are constants, no branch.
        const char* col = reinterpret_cast<const char*>(src) + (size_t)c * 4;
        auto image_row = [&](int y) { return *reinterpret_cast<const v4f_any*>(col + (size_t)y * sp); };
        const int ybase = y0 - RG - 1;
        const bool writer = lane >= 1 && lane <= 62;
        v4f img[MI];
#pragma unroll
        for (int i = 0; i < MI; ++i) img[i] = image_row(ybase + i);
        v4f hd[3];
        if constexpr (TILE) {
            hd[0] = row_difference(img[0]);
            hd[1] = row_difference(img[1]);
        }
        static_for<K>([&](auto k_c) __attribute__((always_inline)) {
            constexpr int kk = decltype(k_c)::value;
            v4f pa, pb, pc;
            if constexpr (TILE) {
                hd[(kk + 2) % 3] = row_difference(img[(kk + 2) % MI]);
                sobel_products_rows(hd[kk % 3], hd[(kk + 1) % 3], hd[(kk + 2) % 3], img[kk % MI], img[(kk + 2) % MI], pa,
                                    pb, pc);
            } else {
                sobel_products(img[kk % MI], img[(kk + 1) % MI], img[(kk + 2) % MI], pa, pb, pc);
            }
            const v4f qa = hwin<RG>(pa, gw), qb = hwin<RG>(pb, gw), qc = hwin<RG>(pc, gw);
            if constexpr (kk + MI <= K + 1) img[kk % MI] = image_row(ybase + kk + MI);
#pragma unroll
            for (int j = 0; j < NW; ++j)
                if (kk - j >= 0 && kk - j < TH) add(acc[(kk - j) % D], gw[j], qa, qb, qc);
            if constexpr (kk >= 2 * RG) {
                const v4f r = response(acc[(kk - 2 * RG) % D]);
                if (writer) *reinterpret_cast<v4f_any*>(out_col + (size_t)(y0 + kk - 2 * RG) * rp) = r;
            }
        });
        return;
    }

    // border strips and row blocks: loads at clamped columns; the products of columns outside the image are
    // replaced by those of the nearest column inside (window reads clamp on the gradient images)
    const bool tile = TILE || strip < rg_.s_lo || strip > rg_.s_hi;   // the order of the Ix sum
    const int xe = min(W, X1 + strip * HS_COLS);                      // columns up to the next strip's first
    const bool left = xs < 4, right = xs + 252 > W;
    const int l1 = (W - 1 - (xs - 4)) >> 2, e1 = (W - 1 - (xs - 4)) & 3;   // lane and element of column W - 1
    auto clamp_cols = [&](v4f p) -> v4f {
        if (left) {   // xs = 0: column 0 is lane 1's first
            const float v0 = lane_value(p.x, 1);
            if (lane == 0) p = mk4(v0, v0, v0, v0);
        }
        if (right) {
            const float sel = e1 == 0 ? p.x : (e1 == 1 ? p.y : (e1 == 2 ? p.z : p.w));
            const float v1 = lane_value(sel, l1 > 63 ? 63 : l1);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (c + q >= W) p[q] = v1;
        }
        return p;
    };
    // image row y, read clamped; its pixels are put in place where they are used, so that loads stay in flight
    auto image_row = [&](int y) { return load4_clamped<F32>(src, (size_t)clampi(y, H) * sp, W, c); };
    auto px = [&](v4f v) { return fix4_clamped(v, W, c); };
    auto wrow = [&](int kk) { return clampi(y0 - RG + kk, H); };
    v4f qa, qb, qc;
    auto products = [&](v4f ra, v4f rbw, v4f rc) {
        v4f pa, pb, pc;
        if (tile) sobel_products_rows(row_difference(ra), row_difference(rbw), row_difference(rc), ra, rc, pa, pb, pc);
        else sobel_products(ra, rbw, rc, pa, pb, pc);
        qa = hwin<RG>(clamp_cols(pa), gw);
        qb = hwin<RG>(clamp_cols(pb), gw);
        qc = hwin<RG>(clamp_cols(pc), gw);
    };
    // ring slot i % MI: image row y0 - 1 - r + i, which window row kk reads at i = kk, kk + 1, kk + 2 where its
    // gradient row is its own (a repeated gradient row keeps the last products)
    auto ring_row = [&](int i) { return image_row(y0 - 1 - RG + i); };
    static_assert(MI % D == 0, "a step's ring slots are constants");
    const int g0 = wrow(0);
    v4f img[MI];
#pragma unroll
    for (int i = 0; i < MI; ++i) img[i] = ring_row(i);
    if (y0 - RG >= 0 && y0 - RG <= H - 1) products(px(img[0]), px(img[1]), px(img[2 % MI]));
    else products(px(image_row(g0 - 1)), px(image_row(g0)), px(image_row(g0 + 1)));
    for (int kb = 0; kb < K; kb += MI) {
        static_for<MI>([&](auto u_c) __attribute__((always_inline)) {
            constexpr int u = decltype(u_c)::value;
            const int kk = kb + u;
            if (kk >= K) return;
            if (kk > 0 && wrow(kk) != wrow(kk - 1)) products(px(img[u]), px(img[(u + 1) % MI]), px(img[(u + 2) % MI]));
            img[u] = ring_row(kk + MI);
#pragma unroll
            for (int j = 0; j < NW; ++j)
                if (kk - j >= 0 && kk - j < TH) add(acc[((u - j) % D + D) % D], gw[j], qa, qb, qc);
            if (kk >= 2 * RG) {
                const v4f r = response(acc[((u - 2 * RG) % D + D) % D]);
                const int y = y0 + kk - 2 * RG;
                if (y >= H || lane < 1 || lane > 62) return;
                float* o = reinterpret_cast<float*>(out_col + (size_t)y * rp);
                if (c + 4 <= xe) {
                    *reinterpret_cast<v4f_any*>(o) = r;
                } else {
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (c + q < xe) o[q] = r[q];
                }
            }
        });
    }
}

bool supports_stream(const HarrisArgs& a) {
    return a.rg >= 0 && a.rg <= 3 && a.W >= HS_XL + HS_COLS + 4 && (uintptr_t)a.src % 16 == 0 && a.sp % 16 == 0 &&
           (uintptr_t)a.resp % 16 == 0 && a.rp % 16 == 0;
}

template <int RG, int TH, bool TILE>
hipError_t launch_strips_R(const HarrisArgs& a) {
    constexpr int X1 = TILE ? HS_COLS : HS_XL;
    StripRegion r{};
    r.nstrips = a.W <= X1 ? 1 : 1 + (a.W - X1 + HS_COLS - 1) / HS_COLS;
    r.nblocks = (a.H + TH - 1) / TH;
    if ((long long)r.nstrips * r.nblocks > 0x7fffffffLL) return hipErrorInvalidValue;
    // interior strips s >= 1: X1 + (s - 1) * 248 + 252 <= W (columns xs-4 .. xs+251 inside)
    r.s_lo = 1;
    r.s_hi = a.W >= X1 + 252 ? 1 + (a.W - X1 - 252) / HS_COLS : 0;
    // interior row blocks b: b TH >= r + 1 and b TH + TH + r <= H - 1
    r.b_lo = (RG + 1 + TH - 1) / TH;
    const int top = a.H - 1 - RG - TH;
    r.b_hi = top >= 0 ? top / TH : -1;
    hipLaunchKernelGGL((harris_strips<RG, TH, TILE>), dim3((unsigned)(r.nstrips * r.nblocks)), dim3(64), 0, a.st, a.src,
                       a.sp, a.resp, a.rp, a.W, a.H, a.g, a.k, r, (int)r.border());
    return hipGetLastError();
}

template <int TH, bool TILE>
hipError_t launch_strips(const HarrisArgs& a) {
    switch (a.rg) {
        case 0: return launch_strips_R<0, TH, TILE>(a);
        case 1: return launch_strips_R<1, TH, TILE>(a);
        case 2: return launch_strips_R<2, TH, TILE>(a);
        case 3: return launch_strips_R<3, TH, TILE>(a);
        default: return hipErrorInvalidValue;
    }
}

template <int TH>
hipError_t launch_stream(const HarrisArgs& a) { return launch_strips<TH, false>(a); }

// rows of any alignment and images of any width
template <int TH>
hipError_t launch_any(const HarrisArgs& a) {
    return supports_stream(a) ? launch_strips<TH, false>(a) : launch_strips<TH, true>(a);
}

template <int TH>
hipError_t launch_fused(const HarrisArgs& a) {
    switch (a.rg) {
        case 0: return launch_fused_R<0, TH>(a);
        case 1: return launch_fused_R<1, TH>(a);
        case 2: return launch_fused_R<2, TH>(a);
        case 3: return launch_fused_R<3, TH>(a);
        default: return hipErrorInvalidValue;
    }
}

bool supports_fused(const HarrisArgs& a) { return a.rg >= 0 && a.rg <= 3; }

const Variant<HarrisArgs> kHarris[] = {
    {"plain_split", supports_plain, launch_plain},
    {"fused_t16", supports_fused, launch_fused<16>},
    {"fused_t32", supports_fused, launch_fused<32>},
    {"fused_t8", supports_fused, launch_fused<8>},
    {"stream_t64", supports_stream, launch_stream<64>},
    {"stream_t32", supports_stream, launch_stream<32>},
    {"stream_t16", supports_stream, launch_stream<16>},
    {"stream_t12", supports_stream, launch_stream<12>},
    {"strips_t16", supports_fused, launch_any<16>},
    {"strips_t12", supports_fused, launch_any<12>},
    {"strips_t8", supports_fused, launch_any<8>},
    {"strips_t4", supports_fused, launch_any<4>},
};

}  // namespace

size_t harris_workspace(int W, int H) { return 2 * (size_t)W * (size_t)H * sizeof(float); }

const Variant<HarrisArgs>* harris_variants(int* count) {
    *count = (int)(sizeof(kHarris) / sizeof(kHarris[0]));
    return kHarris;
}

// The tile kernel below 256 columns and, for rows off 16 bytes, below 1024 waves of 16-row strips (its 4 waves
// share a tile, so a small image is done sooner: 1919 x 1081, r = 2, 12.1 us against 12.7 in strips of 4 rows; 3001 x
// 2001 27 against 21 in strips of 8; 6001 x 5000 115 against 66).  Aligned rows keep to strips at every size, as
// the two kernels round differently.  Strips of 12 or 16 rows where they give four waves per SIMD, 8 or 4 rows on smaller
// images: a wave is one chain of TH + 2 r rows.  r = 2, strips of 32 / 16 / 8 / 4 rows, us: 8192^2 132 / 134 / 148 / 182,
// 5000 x 4000 63 / 47 / 50 / -, 4000 x 3000 50 / 37 / 35 / 36, 3000 x 2000 43 / 28 / 21 / 23, 1920 x 1080 39 / 24 / 16 / 13;
// 16 / 12 rows at 8192^2: r = 3 156 / 165, r = 1 128 / 123.
int harris_default(const HarrisArgs& a) {
    if (!supports_fused(a)) return 0;
    const long long waves = (long long)(1 + a.W / HS_COLS) * ((a.H + 15) / 16);
    if (!supports_stream(a) && (a.W < 256 || waves < 1024)) return 1;
    return waves >= 4096 ? (a.rg >= 2 ? 8 : 9) : waves >= 1024 ? 10 : 11;
}

}  // namespace icl
