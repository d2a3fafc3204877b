// Depthwise conv2d, NHWC, fp32, on the vector ALUs: a bandwidth-bound kernel,
// one per decision trace.
//
// Schedule (Table 2 primitives of arXiv 2205.13603):
//   split   oh -> I0..I3, ow -> J0..J3, c -> C0..C3 (index ((x0*F1+x1)*F2+x2)*F3+x3)
//   reorder i0 j0 c0 | i2 j2 c2 | i1 j1 c1 | i3 j3 | kh kw | c3
//   bind    fuse(i0,j0,c0) -> blockIdx.x (c fastest), fuse(i2,j2,c2) -> threadIdx.x (c fastest:
//           neighbouring lanes touch neighbouring channels of one pixel = coalesced)
//   reorder (REORDER 2): workgroup order grouped per XCD
//   vectorize c3 (4 or 2 channels per load/store when 4 or 2 divides C3)
//   cache-read (CACHE_READ 1): the workgroup's input halo tile is staged in LDS, zero padded
//   unroll  the kh,kw tap loops (UNROLL_K1 == 0: fully, with the I3 x J3 output patch sharing one
//           register copy of its input patch; 1: rolled, every tap re-reads its input)
#include "common.h"

#ifndef STRIP
#define STRIP 0
#endif
#if STRIP
// Strips (STRIP S > 0; the host's rule is dw_strip() in ms_interp.cpp): images whose extents have no small divisor but 2,
// so that no perfect tile gives a thread a compact output patch.  A thread makes S x S output pixels of one channel;
// threads count the channels first, then the strips of the image, and the last strips of a row or column are masked.
// What bounds the general kernel there is the L1: a 1 x 29 patch of one thread reads 6 values per output, lane groups of 16
// channels read half lines, and its 188 registers leave one workgroup per compute unit.  The halo costs no branch: a
// buffer load beyond the image's bytes returns zero, and pixels outside the image ask for such an offset.
// 57 x 57 x 144, stride 2, batch 128: 83.2 -> 60.7 us with inputs that change from launch to launch (57.1 with results streamed), 75.1 -> 50.4 with inputs
// that stay; with those, of one channel 4 x 4 was the fastest (2 x 4: 53.1,
// 6 x 6: 51.4, 8 x 8: 64.3), 2 and 4 channels per thread read more lines per output (2 x 4 of 2: 55.6, of 4: 49.8 but
// 327 against 300 us on 112 x 112 x 32, stride 1).
constexpr int SP_H = (STRIP - 1) * CV_STRIDE + CV_KH, SP_W = (STRIP - 1) * CV_STRIDE + CV_KW; // input patch of a strip
constexpr int S_OH = (CV_OH + STRIP - 1) / STRIP, S_OW = (CV_OW + STRIP - 1) / STRIP;           // strips of an image
constexpr unsigned S_GROUPS = (S_OH * S_OW * CV_C + STRIP_THREADS - 1) / STRIP_THREADS;          // workgroups of an image: gridDim.x
constexpr int IMG_BYTES = CV_H * CV_W * CV_C * 4;

// Results of 4 MiB and more are streamed (200 launches measured on both sides; 57 x 57 x 144, stride 2, batch 128: 56.8 us, plain 60.2).
// Not where small filters of stride 1 leave a pixel less than three lines and part of one: neighbouring pixels share lines, which
// streaming wavefronts write in pieces, with few loads to hide it (3 x 3, 57 x 57 x 24, batch 49: 9.85 us, 8.67 plain; 57 x 57 x 72, batch 257:
// 129 and 120; 104 channels and more, or 5 x 5: within 5 % either way, 1 and 2 % faster in the mean).  Around the size of the eight L2s,
// 32 MiB, streaming pays all the same: kept there, results are written back when nothing else runs any more (57 x 57 x 72, batch 33, 31 MB:
// 13.1 us, 19.2 plain; at 60 MB either side wins by up to 9 %).
constexpr long OUT_BYTES = (long)CV_N * CV_OH * CV_OW * CV_C * 4;
constexpr bool SHARED_LINES = CV_STRIDE == 1 && CV_KH * CV_KW < 25 && CV_C % 32 != 0 && CV_C < 96;
constexpr bool STREAM = stream_from(OUT_BYTES) <= 1 && (!SHARED_LINES || (OUT_BYTES >= 20000000 && OUT_BYTES <= 100000000));

extern "C" __global__ void __launch_bounds__(STRIP_THREADS)
ms_kernel(const void *__restrict__ x_, const void *__restrict__ w_, const void *__restrict__ unused_, void *__restrict__ y_, int instances)
{
    (void)unused_;
    int z = blockIdx.z * gridDim.y + blockIdx.y; // instance * N + n
    int wg = blockIdx.x;
    {
        // Workgroup order grouped per XCD: strips that share input rows meet in one L2 (18 x 66 x 66 x 328, stride 1, 6678 workgroups: 52 us in
        // the order of launch, 31.7).  In one run for each XCD, or, from about 90 MB of images on, in runs of 32: the last-level cache no longer
        // holds those for the next launch, and eight places far apart are read from HBM more slowly than one (154 x 33 x 33 x 208: one run
        // 67.1 us, in the order of launch 64.0, runs of 32 62.1; 29 x 112 x 112 x 152, 5 x 5: 137, 131, 126; below, short runs share fewer rows:
        // 17 x 65 x 65 x 288, 5 x 5, 83 MB: 33.8, 55.1, 35.1; 55 x 32 x 32 x 272, 61 MB: 18.2, 26.2, 19.6).  Multiples of 8 keep one run:
        // images that have just been written are in part still in that cache, where eight places meet more of them (57 x 57 x 144, stride 2,
        // batch 128, first pass on new images: 71 us, runs of 32 85; again and again 57.2 and 55.1).
        // Divisions by a constant: by gridDim.x a launch of 4 us took 0.3 to 0.9 longer.
        const unsigned images = gridDim.y * gridDim.z, total = S_GROUPS * images, f = wg + S_GROUPS * z;
        const unsigned g = total % 8 && images > 90000000u / IMG_BYTES ? xcd_run<32>(f, total) : xcd_run<0>(f, total);
        wg = (int)(g % S_GROUPS);
        z = (int)(g / S_GROUPS);
    }
    if (z >= instances * CV_N) return;
    const int item = wg * STRIP_THREADS + threadIdx.x;
    if (item >= S_OH * S_OW * CV_C) return;
    const int c = item % CV_C, ow = item / CV_C % S_OW * STRIP, oh = item / (CV_C * S_OW) * STRIP;
    const float *X = (const float *)x_ + (long)z * (CV_H * CV_W * CV_C);
    const float *__restrict__ Wt = (const float *)w_ + (long)(z / CV_N) * CV_KH * CV_KW * CV_C + c;
    float *__restrict__ Y = (float *)y_ + (long)z * CV_OH * CV_OW * CV_C + c;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(X), 0, IMG_BYTES, 0x00020000);

    float x[SP_H][SP_W], w[CV_KH][CV_KW];
#pragma unroll
    for (int ph = 0; ph < SP_H; ++ph)
#pragma unroll
        for (int pw = 0; pw < SP_W; ++pw) {
            const int ih = oh * CV_STRIDE - CV_PAD + ph, iw = ow * CV_STRIDE - CV_PAD + pw;
            const bool in = (unsigned)ih < (unsigned)CV_H && (unsigned)iw < (unsigned)CV_W;
            x[ph][pw] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, in ? ((ih * CV_W + iw) * CV_C + c) * 4 : IMG_BYTES, 0, 0));
        }
#pragma unroll
    for (int kh = 0; kh < CV_KH; ++kh)
#pragma unroll
        for (int kw = 0; kw < CV_KW; ++kw) w[kh][kw] = Wt[(kh * CV_KW + kw) * CV_C];
#pragma unroll
    for (int a = 0; a < STRIP; ++a)
#pragma unroll
        for (int b = 0; b < STRIP; ++b) {
            float acc = 0.f;
#pragma unroll
            for (int kh = 0; kh < CV_KH; ++kh)
#pragma unroll
                for (int kw = 0; kw < CV_KW; ++kw) acc += x[a * CV_STRIDE + kh][b * CV_STRIDE + kw] * w[kh][kw];
            if (oh + a < CV_OH && ow + b < CV_OW) {
                float *y = Y + ((oh + a) * CV_OW + ow + b) * CV_C;
                if constexpr (STREAM) store_stream(y, acc);
                else *y = acc;
            }
        }
}
#else
constexpr int BOH = I1 * I2 * I3;
constexpr int BOW = J1 * J2 * J3;
constexpr int BC = C1 * C2 * C3;
constexpr int VC = C3 % 4 == 0 ? 4 : (C3 % 2 == 0 ? 2 : 1); // channels per memory instruction
constexpr int NV = C3 / VC;
constexpr int TIH = (BOH - 1) * CV_STRIDE + CV_KH;  // input halo tile of a workgroup
constexpr int TIW = (BOW - 1) * CV_STRIDE + CV_KW;
constexpr int PH = (I3 - 1) * CV_STRIDE + CV_KH;    // input patch of one I3 x J3 output patch
constexpr int PW = (J3 - 1) * CV_STRIDE + CV_KW;

typedef vec_t<float, VC> cv_t;

__device__ __forceinline__ cv_t zero_cv()
{
    cv_t z;
#pragma unroll
    for (int q = 0; q < VC; ++q) z.v[q] = 0.f;
    return z;
}

// input pixel (ih, iw), channels [c, c+VC): zero outside the image
__device__ __forceinline__ cv_t load_x(const float *__restrict__ X, int ih, int iw, int c)
{
    if (ih >= 0 && ih < CV_H && iw >= 0 && iw < CV_W) return *reinterpret_cast<const cv_t *>(X + ((long)ih * CV_W + iw) * CV_C + c);
    return zero_cv();
}

extern "C" __global__ void __launch_bounds__(NTHREADS)
ms_kernel(const void *__restrict__ x_, const void *__restrict__ w_, const void *__restrict__ unused_, void *__restrict__ y_, int instances)
{
    (void)unused_;
    int z = blockIdx.z * gridDim.y + blockIdx.y; // instance * N + n
    int wg = blockIdx.x;
#if REORDER == 2
    // undo the round-robin of workgroups over the 8 XCDs (workgroup f of the launch goes to XCD f mod 8):
    // neighbouring tiles, which share halo rows and columns, then sit behind the same L2
    {
        constexpr int G = I0 * J0 * C0;
        const long total = (long)G * gridDim.y * gridDim.z;
        if (total % 8 == 0) {
            const long f = wg + (long)G * z;
            const long g = (f % 8) * (total / 8) + f / 8;
            wg = (int)(g % G);
            z = (int)(g / G);
        }
    }
#endif
    if (z >= instances * CV_N) return;
    const float *__restrict__ X = (const float *)x_ + (long)z * CV_H * CV_W * CV_C;
    const float *__restrict__ Wt = (const float *)w_ + (long)(z / CV_N) * CV_KH * CV_KW * CV_C;
    float *__restrict__ Y = (float *)y_ + (long)z * CV_OH * CV_OW * CV_C;

    const int c0 = wg % C0, j0 = (wg / C0) % J0, i0 = wg / (C0 * J0);
    const int tid = threadIdx.x;
    const int tc = tid % C2, tj = (tid / C2) % J2, ti = tid / (C2 * J2);

#if CACHE_READ
    __shared__ __attribute__((aligned(16))) float tile[TIH * TIW * BC];
    {
        const int ih0 = i0 * BOH * CV_STRIDE - CV_PAD, iw0 = j0 * BOW * CV_STRIDE - CV_PAD;
        constexpr int CV_PER_PIX = BC / VC;
        constexpr int TOTAL = TIH * TIW * CV_PER_PIX;
        for (int idx = tid; idx < TOTAL; idx += NTHREADS) {
            const int cv = idx % CV_PER_PIX, pix = idx / CV_PER_PIX;
            const int pw = pix % TIW, ph = pix / TIW;
            // channels of the tile are stored in block order: local channel lc <-> global c0*BC + lc
            *reinterpret_cast<cv_t *>(&tile[(ph * TIW + pw) * BC + cv * VC]) = load_x(X, ih0 + ph, iw0 + pw, c0 * BC + cv * VC);
        }
    }
    __syncthreads();
#endif

#pragma unroll 1
    for (int r1 = 0; r1 < I1; ++r1)
#pragma unroll 1
        for (int q1 = 0; q1 < J1; ++q1)
#pragma unroll 1
            for (int s1 = 0; s1 < C1; ++s1) {
                const int ohl = (r1 * I2 + ti) * I3, owl = (q1 * J2 + tj) * J3, cl = (s1 * C2 + tc) * C3; // block-local
                const int oh = i0 * BOH + ohl, ow = j0 * BOW + owl, c = c0 * BC + cl;
#pragma unroll 1
                for (int v = 0; v < NV; ++v) {
                    const int cc = c + v * VC, ccl = cl + v * VC;
                    (void)ccl;
                    cv_t acc[I3][J3];
#pragma unroll
                    for (int a = 0; a < I3; ++a)
#pragma unroll
                        for (int b = 0; b < J3; ++b) acc[a][b] = zero_cv();
#if UNROLL_K1 == 0
                    // taps unrolled: one register copy of the input patch serves the whole output patch
                    cv_t w[CV_KH][CV_KW], x[PH][PW];
#pragma unroll
                    for (int kh = 0; kh < CV_KH; ++kh)
#pragma unroll
                        for (int kw = 0; kw < CV_KW; ++kw) w[kh][kw] = *reinterpret_cast<const cv_t *>(Wt + (kh * CV_KW + kw) * CV_C + cc);
#pragma unroll
                    for (int ph = 0; ph < PH; ++ph)
#pragma unroll
                        for (int pw = 0; pw < PW; ++pw) {
#if CACHE_READ
                            x[ph][pw] = *reinterpret_cast<const cv_t *>(&tile[((ohl * CV_STRIDE + ph) * TIW + owl * CV_STRIDE + pw) * BC + ccl]);
#else
                            x[ph][pw] = load_x(X, oh * CV_STRIDE - CV_PAD + ph, ow * CV_STRIDE - CV_PAD + pw, cc);
#endif
                        }
#pragma unroll
                    for (int a = 0; a < I3; ++a)
#pragma unroll
                        for (int b = 0; b < J3; ++b)
#pragma unroll
                            for (int kh = 0; kh < CV_KH; ++kh)
#pragma unroll
                                for (int kw = 0; kw < CV_KW; ++kw)
#pragma unroll
                                    for (int q = 0; q < VC; ++q)
                                        acc[a][b].v[q] += x[a * CV_STRIDE + kh][b * CV_STRIDE + kw].v[q] * w[kh][kw].v[q];
#else
#pragma unroll 1
                    for (int kh = 0; kh < CV_KH; ++kh)
#pragma unroll 1
                        for (int kw = 0; kw < CV_KW; ++kw) {
                            const cv_t w = *reinterpret_cast<const cv_t *>(Wt + (kh * CV_KW + kw) * CV_C + cc);
#pragma unroll
                            for (int a = 0; a < I3; ++a)
#pragma unroll
                                for (int b = 0; b < J3; ++b) {
#if CACHE_READ
                                    const cv_t x = *reinterpret_cast<const cv_t *>(
                                        &tile[(((ohl + a) * CV_STRIDE + kh) * TIW + (owl + b) * CV_STRIDE + kw) * BC + ccl]);
#else
                                    const cv_t x = load_x(X, (oh + a) * CV_STRIDE - CV_PAD + kh, (ow + b) * CV_STRIDE - CV_PAD + kw, cc);
#endif
#pragma unroll
                                    for (int q = 0; q < VC; ++q) acc[a][b].v[q] += x.v[q] * w.v[q];
                                }
                        }
#endif
#pragma unroll
                    for (int a = 0; a < I3; ++a)
#pragma unroll
                        for (int b = 0; b < J3; ++b)
                            *reinterpret_cast<cv_t *>(Y + ((long)(oh + a) * CV_OW + ow + b) * CV_C + cc) = acc[a][b];
                }
            }
}
#endif // STRIP
