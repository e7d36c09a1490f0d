// 2-D correlation of unsigned char images on the matrix cores (radius 1 .. 7), exact.
//
// Along x a window is a product with a banded (Toeplitz) tap matrix; v_mfma_i32_16x16x64_i8 takes the
// 32-pixel windows of two image rows at once.  A wave owns 256 output columns: 16 chunks n of 16 columns.
// For tap rows (2t, 2t + 1) and the row pair (q, q + 1)
//   D[m][n] += sum_k T_t[m][k] X_q[k][n],   X_q[32 h + p][n] = src(xs + 16 n - 8 + p, q + h) - 128,
//   T_t[m][32 h + p] = w[2t + h][p - m - 8 + r]   (0 outside the taps)
// is the part of output row q + r - 2t, columns xs + 16 n + m, that the pair gives through the two tap
// rows.  Lane n + 16 g holds the 16 bytes of row q + g / 2 at column xs + 16 n - 8 + 16 (g % 2): one
// 16-byte load per lane and row, no LDS and no conversion but the sign flip, and the operand serves all
// r + 1 tap row pairs.  The tap operands stay in registers; the pending output rows move from one
// accumulator to the next as the wave walks down (rows of one parity share a set).
//
// Exactness: w = 256 wh + wl with wl in -128 .. 127 and wh = (w - wl) / 256 in -128 .. 128, two int32
// sums.  A tap from 32640 up has wh = 128: then wh is held as 127 + 1, the 1s in a third operand (a
// branch for the whole wave).  The sums start at 128 sum(w) (the pixels are taken off by 128) and the rounding bias;
// int32 wraps, and the result fits (r <= 7), so it is exact whatever wraps on the way.
//
// Bound: memory up to r = 3 (46 us at 8192^2, r = 2, of which a copy of the bytes takes 27), the products
// beyond (2 (r + 1) of 16 cycles per 256 pixels).  The dot-product strips issue 24 vector instructions per
// pixel there.  Per call at 8192^2, strips / here: r = 1 44 / 44 us, 2 56 / 46, 3 85 / 50, 4 122 / 68;
// plain / here: r = 5 3370 / 72, r = 7 5940 / 90.  At 512^2 both sit at the call's own 10 us.
// Strips at the image's left and right edge first cost twice a step of the others and set the kernel's end
// (52 us): they read past the row's ends and mask, and only the image's first and last rows shift bytes.
#include "icl_device.hpp"
#include "icl_internal.hpp"
#include "u8_rows.hpp"

namespace icl {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef v4i v4i_any __attribute__((aligned(1)));
typedef uint32_t u32_any __attribute__((aligned(1)));

constexpr int UW = U8_COLS;   // output columns of a wave
constexpr int UT = 14;        // words of a padded tap row
constexpr int uq(int r, bool inside) { return inside ? (r == 2 ? 6 : 8) : r == 2 ? 2 : 4; }   // input rows in flight
constexpr int waves_per_simd(int r) { return r <= 2 ? 4 : r == 3 ? 3 : 2; }   // the register budget

// Sixteen bytes loaded from the clamped column cb, moved to stand for columns c .. c + 15 (fill where
// outside the row): whole words first, then the bytes of the odd part.
__device__ __forceinline__ v4i bytes_fix(v4i v, int c, int cb, uint32_t fill) {
    const int d = c - cb;
    if (d > 0) {
        const int w = min(d, 16) >> 2;
        uint32_t e[8] = {(uint32_t)v.x, (uint32_t)v.y, (uint32_t)v.z, (uint32_t)v.w, fill, fill, fill, fill};
        uint32_t o[5];
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            o[i] = fill;
#pragma unroll
            for (int k = 0; k <= 4; ++k)
                if (w == k && i + k < 8) o[i] = e[i + k];
        }
        const uint32_t b = d < 16 ? d & 3 : 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = (int)__builtin_amdgcn_alignbyte(o[i + 1], o[i], b);
    } else if (d < 0) {   // only the first strip's first chunk: 8 columns left of the image
        v = v4i{(int)fill, (int)fill, v.x, v.y};
    }
    return v;
}

// INSIDE: every column the wave reads or writes lies in the image, so a step has no branch: the loads and
// stores are counted exactly, and a wait for a row leaves the later rows and the stores in flight.
template <int R, bool EXTRA, bool INSIDE>
__device__ __forceinline__ void u8_walk(const uint8_t* __restrict__ src, size_t sp, uint8_t* __restrict__ dst, size_t dp,
                                        int W, int H, const uint32_t (*__restrict__ wl)[2 * R + 2][UT], int tsum, int shift,
                                        int bias, int cmode, int cval, int tail, int xs, int y0, int rows) {
    constexpr int NP = R + 1, PARTS = EXTRA ? 3 : 2;
    const int lane = (int)threadIdx.x & 63, n = lane & 15, g = lane >> 4, half = g >> 1;
    const int K = rows + 2 * R;
    const int c = u8_col(xs, n, g), cb = min(max(c, 0), W - 16);
    const unsigned rowoff = half ? (unsigned)sp : 0u;
    // Rows whose columns left of 0 or right of W - 1 could lie outside the image's memory (its first row and its last
    // ones): an edge strip reads those from clamped columns, all others straight, into the padding or neighbour rows.
    auto guarded = [&](int k) { return u8_guarded(y0 - R + k, tail); };
    auto load_row = [&](int k) -> v4i {   // row pair y0 - R + k, read clamped: this lane's row of it
        const int q = y0 - R + k;
        const uint8_t* row = src + (size_t)u8_row(q, H) * sp;
        const unsigned off = q >= 0 && q + 1 < H ? rowoff : 0u;
        if constexpr (INSIDE) return *reinterpret_cast<const v4i_any*>(row + (off + (unsigned)c));
        return *reinterpret_cast<const v4i_any*>(row + u8_lane(q, H, tail, rowoff, c, cb));
    };
    const int ce = c < 0 ? 0 : W - 1;   // the column that stands for those outside
    auto load_end = [&](int k) -> uint32_t {
        const int q = y0 - R + k;
        return src[(size_t)clampi(q, H) * sp + (q >= 0 && q + 1 < H ? rowoff : 0u) + (unsigned)ce];
    };
    constexpr int UQ = uq(R, INSIDE);
    v4i ring[UQ];
    uint32_t ends[INSIDE ? 1 : UQ];
#pragma unroll
    for (int i = 0; i < UQ; ++i) {
        ring[i] = load_row(i);
        if constexpr (!INSIDE) ends[i] = load_end(i);
    }
    v4i keep;   // an edge strip's bytes that lie in the image
    if constexpr (!INSIDE) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            uint32_t m = 0;
#pragma unroll
            for (int b = 0; b < 4; ++b) m |= (c + 4 * i + b >= 0 && c + 4 * i + b < W ? 255u : 0u) << (8 * b);
            keep[i] = (int)m;
        }
    }
    // tap operands: lane (m = lane % 16, g) holds T_t[m][16 g .. 16 g + 15], low and high parts: 16 bytes of the
    // padded tap row from byte 16 (g % 2) - m + 16 on
    v4i a[PARTS][NP];
    const int tb = 16 * (g & 1) - n + 16;
#pragma unroll
    for (int t = 0; t < NP; ++t)
#pragma unroll
        for (int i = 0; i < PARTS; ++i) {
            const uint32_t* w = &wl[i][2 * t + half][tb >> 2];
#pragma unroll
            for (int e = 0; e < 4; ++e) a[i][t][e] = (int)__builtin_amdgcn_alignbyte(w[e + 1], w[e], tb & 3);
        }
    const int init = bias + 128 * tsum;
    const v4i first = v4i{init, init, init, init}, zero = v4i{0, 0, 0, 0};
    v4i sl[2][NP], sh[2][NP];   // low and high sums of the pending rows, by the parity of the step
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int t = 0; t < NP; ++t) sl[p][t] = sh[p][t] = zero;
    auto mm = [](v4i x, v4i y, v4i z) { return __builtin_amdgcn_mfma_i32_16x16x64_i8(x, y, z, 0, 0, 0); };
    const int xo = xs + 4 * lane;
    const int from = 4 * ((lane >> 2) + 16 * (lane & 3));   // the lane whose sums hold columns xo .. xo + 3
    const uint32_t cfill = (uint32_t)cval * 0x01010101u;
    static_assert(UQ % 2 == 0, "the parity of a step is that of its ring slot");
    for (int kb = 0; kb < K; kb += UQ) {
        static_for<UQ>([&](auto s_c) __attribute__((always_inline)) {
            constexpr int s = decltype(s_c)::value, p = s & 1;
            const int k = kb + s;
            v4i x = ring[s];
            ring[s] = load_row(k + UQ);
            const int q = y0 - R + k;
            auto outside = [&]() {   // rows outside the image
                if (cmode && (q < 0 || q + 1 >= H)) {
                    const bool out = q + half < 0 || q + half >= H;
#pragma unroll
                    for (int i = 0; i < 4; ++i) x[i] = out ? (int)cfill : x[i];
                }
            };
            if constexpr (INSIDE) {
                outside();
            } else {
                const uint32_t fill = cmode ? cfill : ends[s] * 0x01010101u;
                ends[s] = load_end(k + UQ);
                if (guarded(k)) {   // they are guarded
                    x = bytes_fix(x, c, cb, fill);
                    outside();
                } else {
                    x = (x & keep) | (v4i{(int)fill, (int)fill, (int)fill, (int)fill} & ~keep);
                }
            }
            x ^= (int)0x80808080;
#pragma unroll
            for (int t = NP - 1; t >= 0; --t) {
                sl[p][t] = mm(a[0][t], x, t > 0 ? sl[p][t > 0 ? t - 1 : 0] : first);
                sh[p][t] = mm(a[1][t], x, t > 0 ? sh[p][t > 0 ? t - 1 : 0] : zero);
            }
            if constexpr (EXTRA) {
#pragma unroll
                for (int t = 0; t < NP; ++t) sh[p][t] = mm(a[2][t], x, sh[p][t]);
            }
            if (!INSIDE && (k < 2 * R || k >= K)) return;
            // pair step k ends output row k - 2 R: its last pair is rows (k, k + 1) with tap row 2 R (+ a zero row)
            const v4i hi = sh[p][NP - 1], lo = sl[p][NP - 1];
            uint32_t o = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int v = (int)(((uint32_t)hi[i] << 8) + (uint32_t)lo[i]);
                int b = min(max(v >> shift, 0), 255);
                asm volatile("" : "+v"(b));   // keeps the pack in full 32-bit operations
                o |= (uint32_t)b << (8 * i);
            }
            o = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)o);
            const int y = y0 + k - 2 * R;
            if constexpr (INSIDE) {
                // a descriptor of size 0 drops the store of a step that ends no row of the segment
                const Rsrc rs = make_rsrc(dst + (size_t)max(y, 0) * dp, k >= 2 * R && k < K ? (unsigned)W : 0u);
                __builtin_amdgcn_raw_buffer_store_b32(o, rs, xo, 0, 0);
            } else {
                uint8_t* out = dst + (size_t)y * dp + xo;
                if (xo + 4 <= W) {
                    *reinterpret_cast<u32_any*>(out) = o;
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (xo + i < W) out[i] = (uint8_t)(o >> (8 * i));
                }
            }
        });
    }
}

template <int R>
__global__ __launch_bounds__(256, waves_per_simd(R)) void conv2d_u8_mfma_k(const uint8_t* __restrict__ src, size_t sp,
                                                        uint8_t* __restrict__ dst, size_t dp, int W, int H,
                                                        const int16_t* __restrict__ taps, int shift, int nstrips,
                                                        int nitems, int TH, int words, int tail, int cmode, int cval) {
    constexpr int N = 2 * R + 1;
    // the taps' low, high and extra parts as bytes at 24 - r .. 24 + r of each row, zeros around; row N is zero
    __shared__ uint32_t wl[3][N + 1][UT];
    __shared__ int sums[2];
    if (threadIdx.x < 2) sums[threadIdx.x] = 0;
    for (int i = (int)threadIdx.x; i < 3 * (N + 1) * UT; i += 256) (&wl[0][0][0])[i] = 0;
    __syncthreads();
    for (int i = (int)threadIdx.x; i < N * N; i += 256) {
        const int w = (int)taps[i], j = i / N, at = 24 - R + i - j * N;
        const int lo = (int)(int8_t)(w & 255), hi = (w - lo) >> 8;
        reinterpret_cast<uint8_t*>(wl[0][j])[at] = (uint8_t)lo;
        reinterpret_cast<uint8_t*>(wl[1][j])[at] = (uint8_t)min(hi, 127);
        reinterpret_cast<uint8_t*>(wl[2][j])[at] = hi > 127 ? 1 : 0;
        atomicAdd(&sums[0], w);
        if (hi > 127) atomicOr(&sums[1], 1);
    }
    __syncthreads();
    const int tsum = sums[0];
    const int item = __builtin_amdgcn_readfirstlane((int)(xcd_remap(blockIdx.x, gridDim.x) * 4 + (threadIdx.x >> 6)));
    if (item >= nitems) return;
    const int seg = item / nstrips, xs = (item - seg * nstrips) * UW, y0 = seg * TH;
    const int bias = shift > 0 ? 1 << (shift - 1) : 0, rows = min(TH, H - y0);
    if (__builtin_amdgcn_readfirstlane(sums[1]))
        u8_walk<R, true, false>(src, sp, dst, dp, W, H, wl, tsum, shift, bias, cmode, cval, tail, xs, y0, rows);
    else if (words && u8_inside(xs, W))
        u8_walk<R, false, true>(src, sp, dst, dp, W, H, wl, tsum, shift, bias, cmode, cval, tail, xs, y0, rows);
    else
        u8_walk<R, false, false>(src, sp, dst, dp, W, H, wl, tsum, shift, bias, cmode, cval, tail, xs, y0, rows);
}

template <int R>
hipError_t launch_R(const U8Args& a) {
    const int nstrips = (a.W + UW - 1) / UW;
    const int slots = 4 * device_cus() * waves_per_simd(R);   // resident waves
    const int want = slots / nstrips > 1 ? slots / nstrips : 1;
    int th = (a.H + want - 1) / want;
    if (th < 8) th = 8;
    const long long items = (long long)nstrips * ((a.H + th - 1) / th);
    if (items > 0x7fffffffLL - 4) return hipErrorInvalidValue;
    // buffer stores of whole words: the destination's rows start on one
    const int words = (uintptr_t)a.dst % 4 == 0 && a.dp % 4 == 0;
    hipLaunchKernelGGL(conv2d_u8_mfma_k<R>, dim3(grid_pad8((items + 3) / 4)), dim3(256), 0, a.st, a.src, a.sp, a.dst,
                       a.dp, a.W, a.H, a.taps, a.shift, nstrips, (int)items, th, words,
                       u8_tail(a.W, a.H, (unsigned)a.sp), a.cmode, a.cval);
    return hipGetLastError();
}

}  // namespace

bool supports_conv2d_u8_mfma(const U8Args& a) { return a.r >= 1 && a.r <= 7 && a.W >= 16 && a.sp < ((size_t)1 << 31); }

hipError_t launch_conv2d_u8_mfma(const U8Args& a) {
    switch (a.r) {
        case 1: return launch_R<1>(a);
        case 2: return launch_R<2>(a);
        case 3: return launch_R<3>(a);
        case 4: return launch_R<4>(a);
        case 5: return launch_R<5>(a);
        case 6: return launch_R<6>(a);
        case 7: return launch_R<7>(a);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace icl
