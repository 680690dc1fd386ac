// The classifier's heavy layer (3x3, 32 -> 64 channels) and its gradients on
// MFMA, operands staged in LDS.
//
// Every input value takes part in nine taps.  A workgroup copies a band of
// rows to LDS once with 16-byte loads (the next band's loads are in flight
// while it computes) and its waves read the taps' fragments from there, at
// fixed offsets from one address per lane; pixels lie at strides of 80 or 144
// bytes instead of 64 or 128, so that neighbouring pixels start in other
// banks.  Reading the nine taps from memory instead, each wave one block of 16
// pixels ahead, waited on those loads.  26 x 26 images, before and now: forward
// of 1024 57 and 36 us (the 120 MB it moves take 25), input gradient of 256 50
// and 19 us, weight gradient of 256 41 us (64 x 64 tiles transposed on the way
// into LDS) and 21 us.
#include "conv_lds.hpp"

namespace tdp {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

constexpr int kCi = 32, kCo = 64;
constexpr int kXStride = kCi * 2 + 16;  // bytes of an input pixel in LDS
constexpr int kYStride = kCo * 2 + 16;  // bytes of an output pixel in LDS

__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {  // round to nearest even
    const f32x2 v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

__device__ __forceinline__ bool bf16_positive(uint32_t h) { return __uint_as_float(h << 16) > 0.f; }

// p / d for p * d < 2^22 and p < 2^10, with inv = ceil(2^22 / d).
__device__ __forceinline__ int div_small(int p, uint32_t inv) { return (int)(((uint32_t)p * inv) >> 22); }
uint32_t inv_small(int d) { return ((1u << 22) + d - 1) / d; }

// ------------------------------------------------------------- forward
// D[co][pixel] = sum_{tap, ci} W[co][tap][ci] x[pixel + tap][ci], taken
// transposed so that a lane ends up with eight consecutive channels of one
// pixel (weight row i of block j holds channel (i / 4) * 8 + j * 4 + i % 4 of
// the wave's half) and stores them as 16 bytes.  Four waves: two halves of
// the channels times two sets of pixel blocks; 72 registers of weights each.
constexpr int kFwdThreads = 256;
constexpr int kFwdMaxPx = 376;  // input pixels of a band

// MANY: bands of several images.
template <bool MANY>
__global__ __launch_bounds__(kFwdThreads, 2) void conv_fwd_kernel(const uint16_t* __restrict__ x,
                                                                  const uint16_t* __restrict__ w,
                                                                  const float* __restrict__ bias, int B, int H, int W,
                                                                  int relu, int rows, int bands, int imgs, int items,
                                                                  uint32_t inv_wo, uint32_t inv_ho,
                                                                  uint16_t* __restrict__ y) {
    constexpr int kLoads = (kFwdMaxPx * 4 + kFwdThreads - 1) / kFwdThreads;
    __shared__ __attribute__((aligned(16))) unsigned char s_x[2][kFwdMaxPx * kXStride];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int half = wave & 1, set = wave >> 1, q = lane >> 4;
    const int Ho = H - 2, Wo = W - 2;
    bf16x8 wf[9][2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int i = lane & 15, co = half * 32 + (i >> 2) * 8 + j * 4 + (i & 3);
#pragma unroll
        for (int k = 0; k < 9; ++k) wf[k][j] = *(const bf16x8*)&w[(co * 9 + k) * kCi + q * 8];
    }
    f32x4 bv[2];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) bv[j][r] = bias ? bias[half * 32 + q * 8 + j * 4 + r] : 0.f;
    u32x4 pre[kLoads];
    // the band of item it: output rows [oy0, oy0 + r), input rows [oy0, oy0 + r + 2) of image b, or, where
    // whole images fit (one band each), of ni images from b
    auto band = [&](int it, int& b, int& oy0, int& r, int& ni) {
        const int q = it / bands;
        b = MANY ? q * imgs : q;
        oy0 = (it - q * bands) * rows;
        r = Ho - oy0 < rows ? Ho - oy0 : rows;
        ni = !MANY ? 1 : B - b < imgs ? B - b : imgs;
    };
    auto fetch = [&](int it) {
        int b, oy0, r, ni;
        band(it, b, oy0, r, ni);
        const u32x4* src = (const u32x4*)(x + ((int64_t)b * H + oy0) * W * kCi);
        const int n = ni * (r + 2) * W * 4;
#pragma unroll
        for (int k = 0; k < kLoads; ++k) {
            const int i = k * kFwdThreads + t;
            pre[k] = src[i < n ? i : n - 1];
        }
    };
    auto stage = [&](int it, unsigned char* buf) {
        int b, oy0, r, ni;
        band(it, b, oy0, r, ni);
        const int n = ni * (r + 2) * W * 4;
#pragma unroll
        for (int k = 0; k < kLoads; ++k) {
            const int i = k * kFwdThreads + t;
            if (i < n) *(u32x4*)&buf[(i >> 2) * kXStride + (i & 3) * 16] = pre[k];
        }
    };
    int it = blockIdx.x, cur = 0;
    fetch(it);
    stage(it, s_x[0]);
    lds_barrier();
    for (; it < items; it += gridDim.x, cur ^= 1) {
        const int next = it + gridDim.x;
        if (next < items) fetch(next);
        int b, oy0, r, ni;
        band(it, b, oy0, r, ni);
        const int npx = ni * r * Wo;
        uint16_t* yo = y + ((int64_t)b * Ho + oy0) * Wo * kCo + half * 32 + q * 8;
        const unsigned char* buf = s_x[cur];
        for (int blk = set; blk * 16 < npx; blk += 2) {
            const int p = blk * 16 + (lane & 15), pc = p < npx ? p : npx - 1;
            // output row, counted over the band's images, and the input row it starts at (two more per image)
            const int oy = div_small(pc, inv_wo), iy = MANY ? oy + 2 * div_small(oy, inv_ho) : oy;
            const unsigned char* a = buf + (iy * W + pc - oy * Wo) * kXStride + q * 16;
            bf16x8 f[9];
#pragma unroll
            for (int k = 0; k < 9; ++k) f[k] = *(const bf16x8*)(a + ((k / 3) * W + k % 3) * kXStride);
            f32x4 acc[2] = {bv[0], bv[1]};
#pragma unroll
            for (int k = 0; k < 9; ++k)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[k][j], f[k], acc[j], 0, 0, 0);
            if (relu)
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[j][e] = acc[j][e] < 0.f ? 0.f : acc[j][e];
            if (p < npx)
                *(uint4*)&yo[p * kCo] = make_uint4(pack_bf16(acc[0][0], acc[0][1]), pack_bf16(acc[0][2], acc[0][3]),
                                                   pack_bf16(acc[1][0], acc[1][1]), pack_bf16(acc[1][2], acc[1][3]));
        }
        if (next < items) stage(next, s_x[cur ^ 1]);
        lds_barrier();
    }
}

// ------------------------------------------------------ input gradient
// D[ci][pixel] = sum_{tap, co} W[co][tap][ci] dy[pixel - tap][co].  The band's
// dy rows lie in LDS at the input's row width with two zero pixels in front of
// each row and zero rows above and below the image, so that a tap is a fixed
// distance from the pixel and nothing is tested.  Four waves: two blocks of 16
// input channels times two sets of pixel blocks (a wave with all 32 channels
// reads LDS half as often but spills its 144 registers of weights: 27 us for
// 256 images against 19); the workgroups of a CU cover each other's staging.
constexpr int kDgThreads = 256;
constexpr int kDgMaxPx = 290;  // three workgroups per CU
constexpr int kDgPerCU = 3;
constexpr int kDgLoads = (kDgMaxPx * 8 + kDgThreads - 1) / kDgThreads;

template <bool MANY>
__global__ __launch_bounds__(kDgThreads, kDgPerCU) void conv_dgrad_kernel(const uint16_t* __restrict__ dy,
                                                                   const uint16_t* __restrict__ w,
                                                                   const uint16_t* __restrict__ mask, int B, int H, int W,
                                                                   int rows, int bands, int imgs, int items,
                                                                   uint32_t inv_wo, uint32_t inv_ho,
                                                                   uint16_t* __restrict__ dx) {
    constexpr int kBuf = kDgMaxPx * kYStride > kCo * 9 * kCi * 2 ? kDgMaxPx * kYStride : kCo * 9 * kCi * 2;
    __shared__ __attribute__((aligned(16))) unsigned char s_y[kBuf];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int half = wave & 1, set = wave >> 1, q = lane >> 4;
    const int Ho = H - 2, Wo = W - 2;
    // weights through LDS: the eight output channels of one (tap, ci) are strided
    for (int i = t; i < kCo * 9 * kCi / 8; i += kDgThreads) ((uint4*)s_y)[i] = ((const uint4*)w)[i];
    __syncthreads();
    bf16x8 wf[9][2];
    {
        const uint16_t* s_w = (const uint16_t*)s_y;
        const int ci = half * 16 + (lane & 15);
#pragma unroll
        for (int k = 0; k < 9; ++k)
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
                uint32_t e[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int co = kb * 32 + q * 8 + 2 * c;
                    e[c] = (uint32_t)s_w[(co * 9 + k) * kCi + ci] | ((uint32_t)s_w[((co + 1) * 9 + k) * kCi + ci] << 16);
                }
                wf[k][kb] = __builtin_bit_cast(bf16x8, u32x4{e[0], e[1], e[2], e[3]});
            }
    }
    __syncthreads();
    for (int i = t; i < kDgMaxPx * kYStride / 16; i += kDgThreads) ((uint4*)s_y)[i] = make_uint4(0, 0, 0, 0);
    const int row_pieces = Wo * 8;  // 16-byte pieces of a dy row
    for (int it = blockIdx.x; it < items; it += gridDim.x) {
        const int q2 = it / bands, b = MANY ? q2 * imgs : q2, iy0 = (it - q2 * bands) * rows;
        const int ni = !MANY ? 1 : B - b < imgs ? B - b : imgs;
        {
            // the dy rows of a band of one image, from two above it, those outside the image as zeros; or all of
            // several images, each behind two rows that stay zero
            const u32x4* src = (const u32x4*)(dy + (int64_t)b * Ho * Wo * kCo);
            const int first = MANY ? 0 : (iy0 - 2) * row_pieces, total = ni * Ho * row_pieces;
            const int pieces = MANY ? total : (rows + 2) * row_pieces;
            u32x4 pre[kDgLoads];
#pragma unroll
            for (int k = 0; k < kDgLoads; ++k) {
                const int i = first + k * kDgThreads + t;
                const bool in = i >= 0 && i < total;
                const u32x4 v = src[in ? i : 0];
                pre[k] = in ? v : u32x4{0, 0, 0, 0};
            }
            lds_barrier();  // the last band has been read
#pragma unroll
            for (int k = 0; k < kDgLoads; ++k) {
                const int i = k * kDgThreads + t, row = div_small(i >> 3, inv_wo);
                const int at = row * W + (i >> 3) - row * Wo + (MANY ? 2 + 2 * div_small(row, inv_ho) : 0) * W;
                if (i < pieces) *(u32x4*)&s_y[(at + 2) * kYStride + (i & 7) * 16] = pre[k];
            }
            lds_barrier();
        }
        const int npx = ni * (H - iy0 < rows ? H - iy0 : rows) * W;
        const int64_t out = ((int64_t)b * H + iy0) * W * kCi + half * 16 + q * 4;
        auto mask_of = [&](int blk) {  // the mask is read one block ahead
            const int p = blk * 16 + (lane & 15);
            return mask && p < npx ? *(const uint2*)&mask[out + p * kCi] : make_uint2(0x3F803F80u, 0x3F803F80u);
        };
        uint2 mk = mask_of(set);
        for (int blk = set; blk * 16 < npx; blk += 2) {
            const uint2 mk2 = mask_of(blk + 2);
            const int p = blk * 16 + (lane & 15), pc = p < npx ? p : npx - 1;
            const unsigned char* a = s_y + pc * kYStride + q * 16;
            f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
            for (int k = 0; k < 9; ++k)
#pragma unroll
                for (int kb = 0; kb < 2; ++kb) {
                    const bf16x8 f = *(const bf16x8*)(a + ((2 - k / 3) * W + 2 - k % 3) * kYStride + kb * 64);
                    acc[kb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[k][kb], f, acc[kb], 0, 0, 0);
                }
            float v[4];
            const uint32_t mh[4] = {mk.x & 0xFFFFu, mk.x >> 16, mk.y & 0xFFFFu, mk.y >> 16};
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = bf16_positive(mh[r]) ? acc[0][r] + acc[1][r] : 0.f;
            if (p < npx) *(uint2*)&dx[out + p * kCi] = make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]));
            mk = mk2;
        }
    }
}

// ----------------------------------------------------- weight gradient
// dw[co][tap][ci] = sum over output pixels of dy[pixel][co] x[pixel + tap][ci]:
// the reduction runs over pixels, the slow dimension of both operands, so the
// fragments are read with the LDS transpose load (each group of 16 lanes reads
// four pixels' 16 channels and gets four pixels of one channel per lane).  A
// workgroup takes one tap row ky and a share of the bands; its eight waves are
// two halves of the output channels times four sets of 32-pixel steps, whose
// sums are added in LDS, then to dw with one float32 atomic per weight and
// workgroup.  The three tap rows of a share are 8 k workgroups apart, so that
// they read the same band through one XCD's L2.
constexpr int kWgThreads = 512;
constexpr int kWgMaxOut = 576;  // output pixels of a band
constexpr int kWgMaxIn = 624;   // input pixels under one tap row
constexpr int kWgShares = 85;   // 3 x 85 workgroups: one per CU (133 KB of LDS each)
// Each share adds its sums to all of dw with atomics, so small batches take few:
// both gradients of 6 and 12 images of 26 x 26 take 15.2 and 17.0 us with shares
// of 288 pixels or more, 15.0 and 17.7 with 192, 16.0 and 20.8 with 96, 19.3 and
// 19.9 with as many shares as there are rows and CUs for.
constexpr int kWgMinPx = 288;

__device__ __forceinline__ s16x4 read_tr(const unsigned char* p) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)p);
}

__device__ __forceinline__ bf16x8 join_tr(s16x4 lo, s16x4 hi) {
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

template <bool MANY>
__global__ __launch_bounds__(kWgThreads) void conv_wgrad_kernel(const uint16_t* __restrict__ x,
                                                                const uint16_t* __restrict__ dy, int B, int H, int W,
                                                                int rows, int bands, int imgs, int items, int shares,
                                                                int share_step, uint32_t inv_wo, uint32_t inv_in,
                                                                float* dw, float* db) {
    constexpr int kYLoads = kWgMaxOut * 8 / kWgThreads, kXLoads = (kWgMaxIn * 4 + kWgThreads - 1) / kWgThreads;
    // one more pixel of each: zeros, read in the place of pixels past the band
    __shared__ __attribute__((aligned(16))) unsigned char s_y[(kWgMaxOut + 1) * kYStride];
    __shared__ __attribute__((aligned(16))) unsigned char s_x[(kWgMaxIn + 1) * kXStride];
    __shared__ float s_db[kWgThreads / kWave][kCo];
    const int share = blockIdx.x % share_step, ky = blockIdx.x / share_step;
    if (share >= shares) return;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int half = wave & 1, set = wave >> 1, g = lane >> 4, l16 = lane & 15;
    const int Ho = H - 2, Wo = W - 2;
    if (t < kYStride / 16) *(uint4*)&s_y[kWgMaxOut * kYStride + t * 16] = make_uint4(0, 0, 0, 0);
    if (t < kXStride / 16) *(uint4*)&s_x[kWgMaxIn * kXStride + t * 16] = make_uint4(0, 0, 0, 0);
    u32x4 py[kYLoads], px[kXLoads];
    // output rows of the band of item it, over its images (several only where each is one band)
    auto band_rows = [&](int it, int& b, int& oy0) {
        const int q = it / bands;
        b = MANY ? q * imgs : q;
        oy0 = (it - q * bands) * rows;
        return (!MANY ? 1 : B - b < imgs ? B - b : imgs) * (Ho - oy0 < rows ? Ho - oy0 : rows);
    };
    auto fetch = [&](int it) {
        int b, oy0;
        const int r = band_rows(it, b, oy0);
        const u32x4* ys = (const u32x4*)(dy + ((int64_t)b * Ho + oy0) * Wo * kCo);
        const u32x4* xs = (const u32x4*)(x + ((int64_t)b * H + oy0 + ky) * W * kCi);
        const int ny = r * Wo * 8, nx = r * W * 4;
#pragma unroll
        for (int k = 0; k < kYLoads; ++k) {
            const int i = k * kWgThreads + t;
            py[k] = ys[i < ny ? i : ny - 1];
        }
#pragma unroll
        for (int k = 0; k < kXLoads; ++k) {
            const int i = k * kWgThreads + t < nx ? k * kWgThreads + t : nx - 1;
            // two rows lie between the images' rows under the tap
            px[k] = xs[MANY ? i + div_small(i >> 2, inv_in) * 2 * W * 4 : i];
        }
    };
    float bsum[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};  // this thread's eight channels of dy
    f32x4 acc[2][3][2];
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int kx = 0; kx < 3; ++kx)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[c][kx][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    fetch(share);
    for (int it = share; it < items; it += shares) {
        int b, oy0;
        const int r = band_rows(it, b, oy0);
        const int npx = r * Wo, ny = npx * 8, nx = r * W * 4;
        lds_barrier();
#pragma unroll
        for (int k = 0; k < kYLoads; ++k) {
            const int i = k * kWgThreads + t;
            if (i < ny) {
                *(u32x4*)&s_y[(i >> 3) * kYStride + (i & 7) * 16] = py[k];
                if (ky == 0) {
                    const uint32_t u[4] = {py[k].x, py[k].y, py[k].z, py[k].w};
#pragma unroll
                    for (int h = 0; h < 4; ++h) {
                        bsum[2 * h] += __uint_as_float(u[h] << 16);
                        bsum[2 * h + 1] += __uint_as_float(u[h] & 0xFFFF0000u);
                    }
                }
            }
        }
#pragma unroll
        for (int k = 0; k < kXLoads; ++k) {
            const int i = k * kWgThreads + t;
            if (i < nx) *(u32x4*)&s_x[(i >> 2) * kXStride + (i & 3) * 16] = px[k];
        }
        lds_barrier();
        if (it + shares < items) fetch(it + shares);
        for (int m0 = set * 32; m0 < npx; m0 += 128) {
            const unsigned char *ya[2], *xa[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int m = m0 + g * 8 + h * 4 + (l16 >> 2);
                const int oy = div_small(m, inv_wo);
                const bool in = m < npx;
                ya[h] = s_y + (in ? m : kWgMaxOut) * kYStride + half * 64 + (l16 & 3) * 8;
                // past the band every tap reads the zero pixel
                xa[h] = s_x + (in ? oy * W + m - oy * Wo : kWgMaxIn) * kXStride + (l16 & 3) * 8;
            }
            const int dx0 = m0 + g * 8 + (l16 >> 2) < npx ? kXStride : 0;
            const int dx1 = m0 + g * 8 + 4 + (l16 >> 2) < npx ? kXStride : 0;
            bf16x8 a[2];
#pragma unroll
            for (int c = 0; c < 2; ++c) a[c] = join_tr(read_tr(ya[0] + c * 32), read_tr(ya[1] + c * 32));
#pragma unroll
            for (int kx = 0; kx < 3; ++kx)
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const bf16x8 f = join_tr(read_tr(xa[0] + kx * dx0 + j * 32), read_tr(xa[1] + kx * dx1 + j * 32));
#pragma unroll
                    for (int c = 0; c < 2; ++c)
                        acc[c][kx][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[c], f, acc[c][kx][j], 0, 0, 0);
                }
        }
    }
    // the four sets' sums, [co][kx][ci], in the buffer of dy
    float* s_sum = (float*)s_y;
    for (int s = 0; s < 4; ++s) {
        __syncthreads();
        if (set != s) continue;
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int kx = 0; kx < 3; ++kx)
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int co = half * 32 + c * 16 + g * 4 + e;
                        float* p = &s_sum[(co * 3 + kx) * kCi + j * 16 + l16];
                        *p = s == 0 ? acc[c][kx][j][e] : *p + acc[c][kx][j][e];
                    }
    }
    if (ky == 0 && db) {
#pragma unroll
        for (int k = 0; k < 8; ++k) {
#pragma unroll
            for (int off = 8; off < 64; off <<= 1) bsum[k] += __shfl_xor(bsum[k], off, kWave);
            if (lane < 8) s_db[wave][lane * 8 + k] = bsum[k];
        }
    }
    __syncthreads();
    for (int i = t; i < kCo * 3 * kCi; i += kWgThreads) {
        const int co = i / (3 * kCi), rest = i - co * 3 * kCi;
        atomicAdd(&dw[(co * 9 + ky * 3) * kCi + rest], s_sum[i]);
    }
    if (ky == 0 && db && t < kCo) {
        float v = 0.f;
#pragma unroll
        for (int k = 0; k < kWgThreads / kWave; ++k) v += s_db[k][t];
        atomicAdd(&db[t], v);
    }
}

// Rows of a band: as many as fit, spread evenly, and few enough that `want`
// workgroups have work.
int band_rows(int total, int most, int B, int want) {
    const int bands = (int)std::max<int64_t>(ceil_div(total, most), std::min<int64_t>(ceil_div(want, B), total));
    return (int)ceil_div(total, bands);
}

// Images of a band, where each is one band and `most` fit: few enough that
// `want` workgroups have work.  With one image a band whatever its size a
// workgroup waited for the loads of each: 700K pixels in images of 5 x 5, weight
// gradient 793 us, 35 so, 60 by the 64 x 64 tiles; forward 70, 21, 23; input
// gradient 75, 41, 90; 16 x 16, weight gradient 133, 92, 112.
int band_images(int bands, int most, int B, int want) {
    return bands > 1 ? 1 : std::max(std::min(most, B / want), 1);
}

}  // namespace

bool conv_fwd_32_64(const uint16_t* x, const uint16_t* w, const float* bias, int B, int H, int W, int relu,
                    uint16_t* y, hipStream_t s) {
    const int most = std::min(kFwdMaxPx / W - 2, H - 2);
    if (most < 1) return false;
    const int rows = band_rows(H - 2, most, B, 2 * kCUs), bands = (int)ceil_div(H - 2, rows);
    const int imgs = band_images(bands, kFwdMaxPx / (H * W), B, 2 * kCUs);
    const int64_t items = ceil_div(B, imgs) * bands;
    if (items >= (1ll << 30)) return false;
    const auto kernel = imgs > 1 ? conv_fwd_kernel<true> : conv_fwd_kernel<false>;
    kernel<<<(unsigned)std::min<int64_t>(items, 2 * kCUs), kFwdThreads, 0, s>>>(
        x, w, bias, B, H, W, relu, rows, bands, imgs, (int)items, inv_small(W - 2), inv_small(H - 2), y);
    return true;
}

bool conv_dgrad_64_32(const uint16_t* dy, const uint16_t* w, const uint16_t* mask, int B, int H, int W, uint16_t* dx,
                      hipStream_t s) {
    const int most = std::min((kDgMaxPx - 2) / W - 2, H);
    if (most < 1) return false;
    // a workgroup first brings the weights through LDS: small calls take at most one per CU
    const int rows = band_rows(H, most, B, kCUs / B * B), bands = (int)ceil_div(H, rows);
    const int imgs = band_images(bands, ((kDgMaxPx - 2) / W - 2) / H, B + kCUs - 1, kCUs);
    const int64_t items = ceil_div(B, imgs) * bands;
    if (items >= (1ll << 30)) return false;
    const auto kernel = imgs > 1 ? conv_dgrad_kernel<true> : conv_dgrad_kernel<false>;
    kernel<<<(unsigned)std::min<int64_t>(items, kDgPerCU * kCUs), kDgThreads, 0, s>>>(
        dy, w, mask, B, H, W, rows, bands, imgs, (int)items, inv_small(W - 2), inv_small(H - 2), dx);
    return true;
}

bool conv_wgrad_32_64(const uint16_t* x, const uint16_t* dy, int B, int H, int W, float* dw, float* db, hipStream_t s) {
    const int most = std::min(std::min(kWgMaxOut / (W - 2), kWgMaxIn / W), H - 2);
    if (most < 1) return false;
    // bands: as many as there are shares of at least kWgMinPx pixels, one each
    const int64_t shares_px = std::min<int64_t>(std::max<int64_t>((int64_t)B * (H - 2) * (W - 2) / kWgMinPx, 1), kWgShares);
    const int rows = band_rows(H - 2, most, 1, (int)std::max<int64_t>(shares_px / B, 1)), bands = (int)ceil_div(H - 2, rows);
    const int imgs = band_images(bands, std::min(kWgMaxOut / ((H - 2) * (W - 2)), kWgMaxIn / ((H - 2) * W)), B, (int)shares_px);
    const int64_t items = ceil_div(B, imgs) * bands;
    if (items >= (1ll << 30)) return false;
    // every share the same number of bands, but for the last ones
    const int shares = (int)ceil_div(items, ceil_div(items, (int64_t)kWgShares));
    const int step = (int)ceil_div(shares, 8) * 8;
    const auto kernel = imgs > 1 ? conv_wgrad_kernel<true> : conv_wgrad_kernel<false>;
    kernel<<<3 * step, kWgThreads, 0, s>>>(x, dy, B, H, W, rows, bands, imgs, (int)items, shares, step, inv_small(W - 2),
                                           inv_small((H - 2) * W), dw, db);
    return true;
}

}  // namespace tdp
