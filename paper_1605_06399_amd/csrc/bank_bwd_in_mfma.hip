// Input gradient of the filter bank on the matrix cores, float32 operands carried exactly (radius 3 and 4, up to 16
// filters), where the FMA tiles are bound by vector issue (F (2r+1)^2 FMAs per pixel).
//
//   z[u] = sum_f sum_k w[f,k] gy0[f, u - k],   gy0: gy extended by zero; the border pixels, onto which clamped
//   positions fold, are rewritten by bank_bwd_edge.
//
// A wave owns 128 columns and walks down the rows of gy.  Row y reaches the 2r + 1 output rows y - r .. y + r: they
// are the rows m of one product (v_mfma_f32_16x16x32_bf16)
//   D[m][p] += sum_{t,f} A[m][(t,f)] B[(t,f)][p],   A[m][(t,f)] = w[f, u_m - y, r - t],
//   B[(t,f)][p] = gy[f, y, x_p - r + t],            K = 2 taps x 16 filters, r + 1 pairs of taps,
// where output row u sits in D's row u mod (2r + 1), so that finished rows leave and new ones enter without moving the
// others: the tap operand rotates instead, read each row from a table in LDS with one row per w[., ky, .].  The 16
// pixels of a product are 8 apart (x_p = x0 + 8 p + g, g = 0 .. 7 one accumulator each), so that the operand of
// (g, pair t) depends on g + t alone: 8 + 2r loads of LDS serve 8 (r + 1) products, and a lane's 8 sums of a row are 8
// consecutive pixels.  Rows of gy are loaded a row ahead, a lane having 4 pixels of 8 filters, and written to LDS as
// records of one pixel's 8 filters; each wave has its own, so there is no barrier.
//
// Bound by the matrix cores: 32 x 16 x 1024^2, r = 4, takes 1.09e12 operations of them (9 of 16 rows of D and 9 of 10
// taps of the pairs are of use, six products per pair of operands) in 0.83 ms = 1.31 PFLOP/s, with 2.3 GB of gy read
// meanwhile; the FMA tiles took 1.11 ms.  Two waves per SIMD (one alone issues these products at half rate); the operands
// of the next products are loaded under these (0.84 against 0.86 without).  The split of the next row between the
// products instead of between the rows spilled and was slower (0.90).
//
// Precision: v = v1 + v2 + v3 exactly, each part the bfloat16 nearest to what is left (8 significant bits and a sign
// each, float32 has 24); products of parts are exact in float32.  v1 w1, v1 w2, v2 w1, v2 w2, v1 w3, v3 w1 are kept, what
// is left out is below 2^-26 |v w|.  v1 w1 is summed apart from the smaller ones.
// gy and w are split after a scaling by 2^24, which is exact, and the sums scaled back: the last bit of the smallest
// float32 (2^-149) is then a normal bfloat16, so that no operand below 2^104 loses bits in its split (unscaled, one below
// 2^-110 did: gy 1e-37 under taps of 1e12 erred by 3e-4 of the result, float32 FMAs by 7e-7).  The scaling costs a
// multiplication per staged value (1.5 % of the kernel); scaling back within the caller's factor and no test for small
// sums give more than that back (with the border 898 us unscaled, 880 so).
// Infinite, NaN or overflowing values turn every sum that meets them in a zero of A, or in the split, into a NaN, and
// scaled sums from 2^80 on are infinite: sums that are not finite are taken again by FMAs.
#include "icl_device.hpp"
#include "icl_internal.hpp"
#include "tile_stage.hpp"

namespace icl {
namespace {

typedef __bf16 b8 __attribute__((ext_vector_type(8)));
typedef __bf16 b2 __attribute__((ext_vector_type(2)));
typedef float f8 __attribute__((ext_vector_type(8)));
typedef float f2 __attribute__((ext_vector_type(2)));

template <class P, class V>
__device__ __forceinline__ P part(V& rest) {   // the leading bfloat16 of each element, taken off it
    const P p = __builtin_convertvector(rest, P);
    rest -= __builtin_convertvector(p, V);
    return p;
}

constexpr int BM_COLS = 128;   // columns of a wave
constexpr float BM_UP = 0x1p24f, BM_DOWN = 0x1p-48f;   // the operands' scale, and the sums' back
constexpr int BM_F = 16;       // filters of a product

template <int R> struct BmLds {
    static constexpr int N = 2 * R + 1, NJ = R + 1;
    static constexpr int ROW = NJ * 64 + 32;        // table: bytes of one tap row (pair, quarter wave, 8 filters), padded
    static constexpr int TAB = (N + 1) * ROW;       // and one row of zeros for D's unused rows
    static constexpr int PHASE = 18 * 16;           // records of pixels 8 idx + phase, idx 0 .. 17
    static constexpr int HALF = 8 * PHASE, PART = 2 * HALF, WAVE = 3 * PART;
    static constexpr int BYTES = 3 * TAB + 4 * WAVE;
};

typedef const float __attribute__((address_space(1))) gmem_t;
typedef const float __attribute__((address_space(4))) taps_t;   // read by scalar loads
typedef const v4f_any __attribute__((address_space(1))) gmem4_t;

template <class P>
__device__ __forceinline__ P* uniform(P* p) {
    const unsigned long long a = (unsigned long long)p;
    return reinterpret_cast<P*>((unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)(a >> 32)) << 32 |
                                (unsigned)__builtin_amdgcn_readfirstlane((int)a));
}

// A wave's lanes read back what others of them have written.
__device__ __forceinline__ void own_writes() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// Rows u0 .. u1 - 1 of a wave's columns times the caller's factor.
__device__ __attribute__((noinline)) void bwd_in_times(float* gxn, int W, int x0, int u0, int u1, float factor) {
#pragma unroll 1
    for (int u = u0; u < u1; ++u)
        for (int x = x0 + ((int)threadIdx.x & 63); x < min(x0 + BM_COLS, W); x += 64) gxn[(size_t)u * W + x] *= factor;
}

// The pixels of rows u0 .. u1 that a wave has written as not finite, taken again by FMAs over the pixels of
// gy in the image.
// A lane has two pixels, which share the 2r + 2 values of a row of gy; the loads of three rows are in flight together, and
// a wave whose sums are all NaN has nothing left to add.  A function of its own, called when the walk is over: within the
// walk its registers spilled.  32 x 16 x 1024^2, r = 4, all pixels: one at a time within the walk 261 ms; so, NaN or
// infinite gradients 1.1 ms (the FMA tiles 1.1) and finite sums past 2^80, which run to their end, 13 (1.3), waiting for
// the nine rows that each output row reads again.
template <int R>
__device__ __attribute__((noinline)) void bwd_in_again(const float* gyn_, const float* w_, float* gxn_, int F_, int H_, int W_,
                                                       int x0_, int u0_, int u1_, float sc) {
    constexpr int N = 2 * R + 1, NV = N + 1, GROUPS = (N + 2) / 3;
    gmem_t* gyn = (gmem_t*)uniform(gyn_);
    taps_t* w = (taps_t*)uniform(w_);
    float* gxn = uniform(gxn_);
    const int F = __builtin_amdgcn_readfirstlane(F_), H = __builtin_amdgcn_readfirstlane(H_),
              W = __builtin_amdgcn_readfirstlane(W_), u0 = __builtin_amdgcn_readfirstlane(u0_),
              u1 = __builtin_amdgcn_readfirstlane(u1_);
    const int x = __builtin_amdgcn_readfirstlane(x0_) + 2 * ((int)threadIdx.x & 63);
    const bool inside = __ballot(x < R || x + 2 + R > W) == 0;
    unsigned cols = 0;   // bit i: column x - r + i lies in the image
#pragma unroll
    for (int i = 0; i < NV; ++i) cols |= (unsigned)(x - R + i >= 0 && x - R + i < W) << i;
#pragma unroll 1
    for (int u = u0; u <= u1; ++u) {
        float* o = gxn + (size_t)u * W + x;
        const bool r0 = x < W && !(fabsf(o[0]) < __builtin_inff()), r1 = x + 1 < W && !(fabsf(o[1]) < __builtin_inff());
        if (__ballot(r0 || r1) == 0) continue;
        f2 acc = {0.f, 0.f};
#pragma unroll 1
        for (int e = 0; e < F * GROUPS; ++e) {
            const int f = e / GROUPS, j0 = 3 * (e - f * GROUPS);
            taps_t* wf = w + ((size_t)f * N + j0) * N;
            float v[3][NV];
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                gmem_t* row = gyn + ((size_t)f * H + clampi(u + R - j0 - j, H)) * W;
                if (inside) {
                    const v4f a = *(gmem4_t*)(row + x - R), b = *(gmem4_t*)(row + x - R + 4);
#pragma unroll
                    for (int i = 0; i < 4; ++i) v[j][i] = a[i], v[j][4 + i] = b[i];
#pragma unroll
                    for (int i = 8; i < NV; ++i) v[j][i] = row[x - R + i];
                } else {
#pragma unroll
                    for (int i = 0; i < NV; ++i) v[j][i] = row[clampi(x - R + i, W)];
                }
            }
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                if (j0 + j >= N || u + R - j0 - j < 0 || u + R - j0 - j >= H) continue;
                if (inside) {
#pragma unroll
                    for (int i = 0; i < N; ++i) {
                        acc[0] = fmaf(wf[j * N + i], v[j][2 * R - i], acc[0]);
                        acc[1] = fmaf(wf[j * N + i], v[j][2 * R - i + 1], acc[1]);
                    }
                } else {
                    asm volatile("" : "+v"(cols));   // its bits are tested here, not kept as 2r + 2 lane masks
#pragma unroll
                    for (int i = 0; i < N; ++i) {
                        const float t = wf[j * N + i];
                        if (cols >> (2 * R - i) & 1) acc[0] = fmaf(t, v[j][2 * R - i], acc[0]);
                        if (cols >> (2 * R - i + 1) & 1) acc[1] = fmaf(t, v[j][2 * R - i + 1], acc[1]);
                    }
                }
            }
            if (__ballot((r0 && acc[0] == acc[0]) || (r1 && acc[1] == acc[1])) == 0) break;
        }
        if (r0) o[0] = sc * acc[0];
        if (r1) o[1] = sc * acc[1];
    }
}

template <int R>
__global__ __launch_bounds__(256, 2) void bank_bwd_in_mfma_k(const float* __restrict__ gy, const float* __restrict__ w,
                                                             float* __restrict__ gx, int F, int H, int W, int strips,
                                                             int nblk, int th, int items,
                                                             const float* __restrict__ scale) {
    static_assert(R == 3 || R == 4, "the window starts on 3 or 4 columns left of the strip (fix4_clamped)");
    using L = BmLds<R>;
    constexpr int N = L::N, NJ = L::NJ;
    __shared__ __attribute__((aligned(16))) char lds[L::BYTES];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;

    // the tap table: row j, pair jj, quarter q, filter i of a half: w[8 (q & 1) + i, j, 2 r - 2 jj - (q >> 1)]
    for (int e = threadIdx.x; e < (N + 1) * NJ * 4; e += 256) {
        const int j = e / (NJ * 4), jj = (e >> 2) % NJ, q = e & 3, t = 2 * jj + (q >> 1);
        f8 v;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int f = 8 * (q & 1) + i;
            v[i] = (j < N && t < N && f < F) ? BM_UP * w[((size_t)f * N + j) * N + 2 * R - t] : 0.f;
        }
        char* o = lds + j * L::ROW + jj * 64 + q * 16;
        *reinterpret_cast<b8*>(o) = part<b8>(v);
        *reinterpret_cast<b8*>(o + L::TAB) = part<b8>(v);
        *reinterpret_cast<b8*>(o + 2 * L::TAB) = part<b8>(v);
    }
    char* rec = lds + 3 * L::TAB + wave * L::WAVE;
    if (lane < 48) {   // the records past the last staged pixel (met by a zero tap only)
        const v4f z = mk4(0.f, 0.f, 0.f, 0.f);
        *reinterpret_cast<v4f*>(rec + lane * L::PHASE + 17 * 16) = z;
    }
    __syncthreads();
    const int item = (int)blockIdx.x * 4 + wave;
    if (item >= items) return;   // no barrier from here on
    const int per = strips * nblk, n = item / per, rem = item - n * per, rb = rem / strips, strip = rem - rb * strips;
    const int u0 = rb * th, u1 = min(H, u0 + th);
    const int x0 = strip * BM_COLS, xs = x0 - R;
    // the sums' scaling back goes into the caller's factor; one that this would make subnormal is applied when the walk
    // is over (a second multiplication in the walk cost 1.5 % of the kernel)
    const float factor = scale ? *scale : 1.f;
    const bool after = factor != 0.f && !(fabsf(factor) >= 0x1p-78f);
    const float sc = after ? 1.f : factor, down = sc * BM_DOWN;
    const size_t hw = (size_t)H * W;
    const float* gyn = gy + (size_t)n * F * hw;
    float* gxn = gx + (size_t)n * hw;

    // staging: a lane's 4 pixels from column cx of the 8 filters of half fh, and 2 filters of one of the 8 columns
    // after those 128.  Filters past F read the last one (their taps are zero).
    const int fh = lane >> 5, c4 = lane & 31, cx = xs + 4 * c4;
    const int ex = xs + BM_COLS + (lane & 7), ef = 2 * (lane >> 3);
    const bool edge = xs < 0 || xs + BM_COLS + 8 > W;
    const float* p[8];
    const float* pe[2];
#pragma unroll
    for (int i = 0; i < 8; ++i) p[i] = gyn + (size_t)min(8 * fh + i, F - 1) * hw + min(max(cx, 0), W - 4);
#pragma unroll
    for (int i = 0; i < 2; ++i) pe[i] = gyn + (size_t)min(ef + i, F - 1) * hw + clampi(ex, W);
    char* wr = rec + fh * L::HALF + 4 * (c4 & 1) * L::PHASE + (c4 >> 1) * 16;
    char* we = rec + (lane >> 5) * L::HALF + (lane & 7) * L::PHASE + 16 * 16 + ((lane >> 3) & 3) * 4;
    v4f v[8];
    f2 ve;
    auto fetch = [&](int y) __attribute__((always_inline)) {
        const size_t o = (size_t)y * W;
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = *reinterpret_cast<const v4f_any*>(p[i] + o);
        ve[0] = pe[0][o];
        ve[1] = pe[1][o];
    };
    auto stage = [&]() __attribute__((always_inline)) {
        if (edge) {   // gy is zero outside the image
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = outside4(fix4_clamped(v[i], W, cx), W, 1, cx, 0, 0.f);
            if (ex >= W) ve[0] = ve[1] = 0.f;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            f8 a;
#pragma unroll
            for (int i = 0; i < 8; ++i) a[i] = BM_UP * v[i][e];
            *reinterpret_cast<b8*>(wr + e * L::PHASE) = part<b8>(a);
            *reinterpret_cast<b8*>(wr + e * L::PHASE + L::PART) = part<b8>(a);
            *reinterpret_cast<b8*>(wr + e * L::PHASE + 2 * L::PART) = __builtin_convertvector(a, b8);
        }
        ve *= BM_UP;
        *reinterpret_cast<b2*>(we) = part<b2>(ve);
        *reinterpret_cast<b2*>(we + L::PART) = part<b2>(ve);
        *reinterpret_cast<b2*>(we + 2 * L::PART) = __builtin_convertvector(ve, b2);
    };

    const int m = lane & 15, q = lane >> 4, par = q >> 1;
    v4f hi[8], lo[8];   // v1 w1, and the smaller products
#pragma unroll
    for (int g = 0; g < 8; ++g) hi[g] = lo[g] = mk4(0.f, 0.f, 0.f, 0.f);
    const char* rd = rec + (q & 1) * L::HALF + m * 16;
    const char* rda = rd + par * L::PHASE;                          // pixel 8 p + s + par, s & 7 < 7
    const char* rdb = rd + par * (16 - 7 * L::PHASE);               // s & 7 = 7: par steps into the next record

    // b: D's row of output row y - r
    auto products = [&](int b) __attribute__((always_inline)) {
        const int j = m < N ? (m >= b ? m - b : m - b + N) : N;
        const char* ta = lds + j * L::ROW + q * 16;
        b8 a[3][NJ];
#pragma unroll
        for (int jj = 0; jj < NJ; ++jj)
#pragma unroll
            for (int k = 0; k < 3; ++k) a[k][jj] = *reinterpret_cast<const b8*>(ta + k * L::TAB + jj * 64);
        b8 x[2][2][3];   // the operands of s = 2 i, 2 i + 1 and of the next two, whose loads run under these products
        auto operands = [&](auto i_c) __attribute__((always_inline)) {
            constexpr int i = decltype(i_c)::value;
            static_for<2>([&](auto o_c) __attribute__((always_inline)) {
                constexpr int o = decltype(o_c)::value, s = 2 * i + o;
                const char* r = ((s & 7) == 7 ? rdb : rda) + (s & 7) * L::PHASE + (s >> 3) * 16;
#pragma unroll
                for (int k = 0; k < 3; ++k) x[i & 1][o][k] = *reinterpret_cast<const b8*>(r + k * L::PART);
            });
        };
        operands(std::integral_constant<int, 0>{});
        static_for<4 + R>([&](auto i_c) __attribute__((always_inline)) {
            constexpr int i = decltype(i_c)::value;
            if constexpr (i + 1 < 4 + R) operands(std::integral_constant<int, i + 1>{});
            __builtin_amdgcn_sched_barrier(0);
#define ICL_BM_PRODUCT(ACC, KA, KX)                                                                                      \
    _Pragma("unroll") for (int o = 0; o < 2; ++o) _Pragma("unroll") for (int jj = 0; jj < NJ; ++jj) {                    \
        const int g = 2 * (i - jj) + o;                                                                                  \
        if (g >= 0 && g < 8)                                                                                             \
            ACC[g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[KA][jj], x[i & 1][o][KX], ACC[g], 0, 0, 0);               \
    }
            ICL_BM_PRODUCT(lo, 2, 0)
            ICL_BM_PRODUCT(hi, 0, 0)
            ICL_BM_PRODUCT(lo, 1, 0)
            ICL_BM_PRODUCT(lo, 1, 1)
            ICL_BM_PRODUCT(lo, 0, 1)
            ICL_BM_PRODUCT(lo, 0, 2)
#undef ICL_BM_PRODUCT
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    int bad0 = H, bad1 = -1;   // the first and the last row with a sum that may not be finite
    // output row u, complete in D's row b: the quarter of the wave that holds it writes 8 pixels per lane and clears it
    auto emit = [&](int u, int b, bool write) __attribute__((always_inline)) {
        float o[8];
        const bool mine = q == (b >> 2);
        static_for<4>([&](auto r_c) __attribute__((always_inline)) {
            constexpr int r = decltype(r_c)::value;
            if ((b & 3) == r) {
#pragma unroll
                for (int g = 0; g < 8; ++g) {
                    o[g] = hi[g][r] + lo[g][r];
                    hi[g][r] = mine ? 0.f : hi[g][r];
                    lo[g][r] = mine ? 0.f : lo[g][r];
                }
            }
        });
        if (!write) return;
        const int x = x0 + 8 * m;
        float big = 0.f;   // a NaN or an infinity stays in the sum
#pragma unroll
        for (int g = 0; g < 8; ++g) big += fabsf(o[g]);
        if (__ballot(mine && !(big < __builtin_inff()))) {
            bad0 = min(bad0, u);
            bad1 = u;
        }
        if (!mine) return;
        float* out = gxn + (size_t)u * W + x;
        if (x + 8 <= W) {
            *reinterpret_cast<v4f_any*>(out) = down * mk4(o[0], o[1], o[2], o[3]);
            *reinterpret_cast<v4f_any*>(out + 4) = down * mk4(o[4], o[5], o[6], o[7]);
        } else {
#pragma unroll
            for (int g = 0; g < 8; ++g)
                if (x + g < W) out[g] = down * o[g];
        }
    };

    const int ya = max(0, u0 - R), yb = min(H - 1, u1 - 1 + R);
    int b = (ya - R - u0 + 2 * N) % N, bp = 0;
    fetch(ya);
    for (int y = ya;; ++y) {
        const int u = y - 1 - R;   // the row that the step before completed
        if (y <= yb) stage();
        if (y > ya) emit(u, bp, u >= u0);
        if (u >= u1 - 1) break;
        if (y <= yb) {
            fetch(min(y + 1, yb));
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            products(b);
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
        bp = b;
        b = b + 1 == N ? 0 : b + 1;
    }
    if (bad1 < 0 && !after) return;
    if (bad1 >= 0) {
        own_writes();
        bwd_in_again<R>(gyn, w, gxn, F, H, W, x0, bad0, bad1, sc);
    }
    if (after) {
        own_writes();
        bwd_in_times(gxn, W, x0, u0, u1, factor);
    }
}

template <int R>
hipError_t launch_R(const BankArgs& a) {
    const int strips = (a.w + BM_COLS - 1) / BM_COLS;
    const long long per = (long long)a.n * strips;
    // rows per wave: the split into row blocks whose rounds of resident waves (two per SIMD) walk the fewest rows
    const long long resident = 8 * device_cus();
    const int most = (a.h + 15) / 16;
    int nblk = 1;
    long long best = -1;
    for (int k = 1; k <= most && k <= 256; ++k) {
        const int th = (a.h + k - 1) / k;
        const long long rounds = (per * k + resident - 1) / resident, cost = rounds * (th + 2 * R);
        if (best < 0 || cost < best) best = cost, nblk = k;
        if (rounds > 16) break;
    }
    const int th = (a.h + nblk - 1) / nblk;
    nblk = (a.h + th - 1) / th;
    const long long items = per * nblk;
    if (items > 0x7ffffff0LL) return hipErrorInvalidValue;
    hipLaunchKernelGGL(bank_bwd_in_mfma_k<R>, dim3((unsigned)((items + 3) / 4)), dim3(256), 0, a.st, a.a, a.b, a.out, a.f,
                       a.h, a.w, strips, nblk, th, (int)items, a.scale);
    return hipGetLastError();
}

}  // namespace

bool supports_bank_bwd_in_mfma(const BankArgs& a) { return (a.r == 3 || a.r == 4) && a.f <= BM_F && a.w >= 8; }

// every pixel but the folds at the border
hipError_t launch_bank_bwd_in_mfma(const BankArgs& a) { return a.r == 3 ? launch_R<3>(a) : launch_R<4>(a); }

}  // namespace icl
