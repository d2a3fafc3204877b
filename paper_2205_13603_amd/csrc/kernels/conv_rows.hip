// First-layer convolution (2-D or 3-D, 1 to 4 channels per pixel, + bias + ReLU) on the CDNA4 matrix cores, straight
// from image rows; which variants run here says conv_rows() in ms_interp.cpp.
//
// What bounds the im2col form of such a layer is its loader: a matrix-core operand of 8 k values crosses taps and rows,
// so every value is a 2-byte load with its own index arithmetic.  Here the reduction is laid out by filter rows: for one
// filter plane kd, the KW * Cin elements that a filter row meets are contiguous in an image row, and a lane's 8 k values
// are one 16-byte piece ("chunk") of them.  A run takes CPR chunks of 8; the lane groups of an intrinsic take two
// consecutive chunks of the whole plane, which need not belong to the same filter row, so that only runs are padded
// (7 x 3 channels: 22 of 24) and not k steps.
//
// A workgroup makes CR_WAVES x TM x 32 consecutive pixels of one output plane for CR_TN x 32 output channels.  Per
// filter plane it stages the image rows that its pixels meet (where a row is several tiles long, SPAN, only the columns
// of those rows) and the plane's weights in LDS, and while it multiplies
// them the next plane's rows and weights are on their way into registers.  Filter planes outside the input are skipped.
// A wavefront holds TM x CR_TN accumulator tiles: LDS reads 8 * (TM + TN) clocks per k step on each of four SIMDs
// against 32 * TM * TN of the matrix cores.  The code object may hold two kernels: TM for one instance, chosen to spread it over
// the chip, and a larger one for launches whose instances fill it.
// Inputs changing from launch to launch, before (im2col loader) and now: 8 x 16 x 224 x 224 x 3 -> 64, 7 x 7 x 7, stride 2 in
// fp16: 573 -> 127 us (835 TFLOP/s); 128 x 224 x 224 x 3 -> 64, 7 x 7: 117 -> 72.5 us (3.4 TB/s),
// 62 with results streamed past the caches (4.0 TB/s).
#include "common.h"

typedef _Float16 h8_t __attribute__((ext_vector_type(8)));
typedef __bf16 b8_t __attribute__((ext_vector_type(8)));
typedef short tr4_t __attribute__((ext_vector_type(4)));
typedef float accv_t __attribute__((ext_vector_type(16)));
typedef unsigned u4_t __attribute__((ext_vector_type(4)));

constexpr int TN = CR_TN, NT = CR_WAVES * 64;
constexpr int BN = TN * 32, JB = DIM_N / BN;              // output channels of a workgroup, column blocks
constexpr int OHW = CV_OH * CV_OW;
constexpr int LEAD = CV_PAD * CV_CIN % 2;                 // runs start at even elements: 4-byte LDS reads
constexpr int RUN = CV_KW * CV_CIN, CPR = (LEAD + RUN + 7) / 8; // elements of a filter row, its chunks
constexpr int NCH = CV_KH * CPR, STEPS = (NCH + 1) / 2;   // chunks of a filter plane, matrix-core steps of two chunks
constexpr int ROW_E = CV_W * CV_CIN, CPW = ROW_E / 8;     // elements of an image row, its 16-byte vectors
static_assert(ROW_E % 8 == 0 && CV_STRIDE * CV_CIN % 2 == 0 && DIM_N % BN == 0, "whole vectors per row, even pixel steps");

// LDS: image rows with their zero columns, then the weights row-major, rows padded by 32 bytes for the transposing reads
constexpr int LHALO = ((CV_PAD * CV_CIN + LEAD) * 2 + 15) / 16 * 16;
constexpr int ORG = LHALO - (CV_PAD * CV_CIN + LEAD) * 2; // byte of pixel 0's run in its row
constexpr int RMB = BN * 2 + 32;                          // bytes of a weight row
constexpr int WT_B = STEPS * 16 * RMB;
constexpr int SROW = BN * (int)sizeof(out_t) + 16, STG_B = CR_WAVES * 32 * SROW; // staged output rows, 32 per wavefront
constexpr int cr_gcd(int a, int b) { return b ? cr_gcd(b, a % b) : a; }
constexpr int AL = cr_gcd(16, cr_gcd(ORG, CV_STRIDE * CV_CIN * 2)); // alignment of a fragment in its row

// What depends on the tile: TM 32-pixel tiles per wavefront; SPAN: a workgroup keeps to one output row and stages the columns
// that its pixels meet, not whole image rows.
template <int TM, bool SPAN> struct tile_t {
    static constexpr int PX = CR_WAVES * TM * 32;         // output pixels of a workgroup
    static constexpr int TPR = (CV_OW + PX - 1) / PX, TILES = SPAN ? CV_OH * TPR : (OHW + PX - 1) / PX;
    static constexpr int READ_END = ORG + ((SPAN ? PX : CV_OW) - 1) * CV_STRIDE * CV_CIN * 2 + CPR * 16, IMG_END = SPAN ? 0 : LHALO + ROW_E * 2;
    static constexpr int PRS = ((READ_END > IMG_END ? READ_END : IMG_END) + 15) / 16 * 16;
    static constexpr int P_OUT_ = PX % CV_OW == 0 ? PX / CV_OW : (CV_OW + PX - 2) / CV_OW + 1;
    static constexpr int P_OUT = SPAN ? 1 : P_OUT_ < CV_OH ? P_OUT_ : CV_OH; // output rows that a workgroup can touch
    static constexpr int PR = (P_OUT - 1) * CV_STRIDE + CV_KH; // input rows
    static constexpr int PATCH_B = PR * PRS;
    static constexpr int LDS_B = PATCH_B + WT_B > STG_B ? PATCH_B + WT_B : STG_B;
    static constexpr int SV = SPAN ? PRS / 16 : CPW;      // staged vectors of an image row
    static constexpr int XI = (PR * SV + NT - 1) / NT;    // staged vectors of the image rows per thread
};

// X, W and Y are aligned to their elements only: 16 bytes at any address
struct __attribute__((packed, aligned(2))) raw16_t {
    u4_t v;
};
constexpr int WROWS = CV_KH * RUN, WCB = BN / 8;          // weight rows of a filter plane, 16-byte vectors of one
constexpr int WI = (WROWS * WCB + NT - 1) / NT;

// byte of chunk c relative to a pixel's run; the chunk behind the last one (odd counts) meets zero weights and is masked
constexpr int koff(int c, int prs) { return c < NCH ? c / CPR * prs + c % CPR * 16 : koff(c - 1, prs); }
// bits of dword d of chunk c that belong to the run: the others are neighbours, which may be infinite or NaN
constexpr unsigned kmask(int c, int d)
{
    unsigned m = 0;
    for (int h = 0; h < 2; ++h) {
        const int q = c % CPR * 8 + d * 2 + h;
        if (c < NCH && q >= LEAD && q < LEAD + RUN) m |= 0xffffu << (16 * h);
    }
    return m;
}

__device__ __forceinline__ accv_t mfma(const u4_t &a, const u4_t &b, accv_t c)
{
#if IN_DT == DT_F16
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(h8_t, a), __builtin_bit_cast(h8_t, b), c, 0, 0, 0);
#else
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(b8_t, a), __builtin_bit_cast(b8_t, b), c, 0, 0, 0);
#endif
}

template <class T> struct stage_t {
    u4_t x[T::XI], w[WI];
};

template <int TM, bool SPAN, class T = tile_t<TM, SPAN>>
__device__ __forceinline__ void stage_fetch(stage_t<T> &st, const in_t *__restrict__ plane, const in_t *__restrict__ wt, int ih_lo, int v_lo, int tid)
{
#pragma unroll
    for (int i = 0; i < T::XI; ++i) {
        const int idx = i * NT + tid, row = idx / T::SV, ih = ih_lo + row, col = (SPAN ? v_lo : 0) + idx % T::SV;
        const bool ok = (unsigned)ih < (unsigned)CV_H && row < T::PR && (!SPAN || (unsigned)col < (unsigned)CPW);
        // vectors outside the image read the plane's first one (always there) and become zero
        const u4_t v = reinterpret_cast<const raw16_t *>(plane + (ok ? ih * ROW_E + col * 8 : 0))->v;
        st.x[i] = ok ? v : u4_t{0, 0, 0, 0};
    }
#pragma unroll
    for (int i = 0; i < WI; ++i) {
        const int idx = i * NT + tid;
        if (WROWS * WCB % NT == 0 || idx < WROWS * WCB) st.w[i] = reinterpret_cast<const raw16_t *>(wt + (long)(idx / WCB) * DIM_N + idx % WCB * 8)->v;
    }
}

template <int TM, bool SPAN, class T = tile_t<TM, SPAN>>
__device__ __forceinline__ void stage_commit(const stage_t<T> &st, char *__restrict__ patch, char *__restrict__ wts, int tid)
{
#pragma unroll
    for (int i = 0; i < T::XI; ++i) {
        const int idx = i * NT + tid;
        if (T::PR * T::SV % NT == 0 || idx < T::PR * T::SV)
            *reinterpret_cast<u4_t *>(patch + idx / T::SV * T::PRS + (SPAN ? 0 : LHALO) + idx % T::SV * 16) = st.x[i];
    }
#pragma unroll
    for (int i = 0; i < WI; ++i) {
        const int idx = i * NT + tid, r = idx / WCB;
        if (WROWS * WCB % NT == 0 || idx < WROWS * WCB)
            *reinterpret_cast<u4_t *>(wts + (r / RUN * CPR * 8 + LEAD + r % RUN) * RMB + idx % WCB * 16) = st.w[i];
    }
}

template <int TM, bool SPAN>
__device__ __forceinline__ void image_rows(const void *__restrict__ x_, const void *__restrict__ w_, const void *__restrict__ bias_, void *__restrict__ y_, int instances)
{
    typedef tile_t<TM, SPAN> T;
    constexpr int PX = T::PX, TPR = T::TPR, TILES = T::TILES, PRS = T::PRS, PATCH_B = T::PATCH_B;
    __shared__ __attribute__((aligned(16))) char smem[T::LDS_B];
    int wg = blockIdx.x, z = blockIdx.z * gridDim.y + blockIdx.y; // z = instance
    {
        // Workgroup order grouped per XCD: tiles that share input rows and planes meet in one L2 (5 x 8 x 160 x 160 x 4 -> 32, 7 x 7 x 7: 24.6 us
        // in the order of launch, 22.1).  Planes are shared furthest apart, in one run for each XCD; rows in runs of 32 (114 x 96 x 96 x 3 -> 64,
        // 5 x 5: 9.7 us in the order of launch, 10.1 in one run, 9.4 in runs of 32; 103 x 96 x 96 x 4 -> 96, 3 x 3: 12.6, 11.5, 11.2).
        // 2-D launches that the chip holds at once, two workgroups per compute unit, load all their rows at the same time and keep the
        // order of launch (5 x 224 x 224 x 3 -> 96, 3 x 3, 490 workgroups: 5.35 us, 5.65 in runs).
        // Divisions by a constant: by gridDim.x a launch of 5 us took 0.2 to 0.7 longer.
        constexpr unsigned GROUPS = JB * CV_OD * TILES * CV_N; // of an instance: gridDim.x
        const unsigned total = GROUPS * gridDim.y * gridDim.z, f = wg + GROUPS * z;
        const unsigned g = CV_OD > 1 ? xcd_run<0>(f, total) : total <= 512 ? f : xcd_run<32>(f, total);
        wg = (int)(g % GROUPS);
        z = (int)(g / GROUPS);
    }
    if (z >= instances) return;
    const int jb = wg % JB, od = wg / JB % CV_OD, tile = wg / (JB * CV_OD) % TILES, n = wg / (JB * CV_OD * TILES);
    const int tid = threadIdx.x, lane = tid % 64, wave = tid / 64, lrow = lane % 32, lgrp = lane / 32;
    const int p0 = SPAN ? tile / TPR * CV_OW + tile % TPR * PX : tile * PX, oh_lo = p0 / CV_OW, ih_lo = oh_lo * CV_STRIDE - CV_PAD_H;
    const int p_end = SPAN ? (oh_lo + 1) * CV_OW : OHW;        // end of the pixels that a workgroup stores
    const int v_lo = tile % TPR * (PX * CV_STRIDE * CV_CIN / 8) - LHALO / 16; // SPAN: first staged vector of an image row
    const in_t *X = (const in_t *)x_ + (long)z * A_INST + (long)n * CV_D * CV_H * ROW_E;
    const in_t *Wt = (const in_t *)w_ + (long)z * B_INST + jb * BN;
    char *patch = smem, *wts = smem + PATCH_B;

    // filter planes that lie inside the input
    const int id0 = CV_D > 1 || CV_KD > 1 ? od * CV_STRIDE - CV_PAD : 0;
    const int kd_lo = id0 < 0 ? -id0 : 0, kd_hi = CV_D - id0 < CV_KD ? CV_D - id0 : CV_KD;

    stage_t<T> st;
    if (kd_lo < kd_hi) stage_fetch<TM, SPAN>(st, X + (long)(id0 + kd_lo) * CV_H * ROW_E, Wt + (long)kd_lo * WROWS * DIM_N, ih_lo, v_lo, tid);
    // zero columns of the image rows and padding rows of the weights: written once, no plane overwrites them
    for (int i = tid; i < (PATCH_B + WT_B) / 16; i += NT) *reinterpret_cast<u4_t *>(smem + i * 16) = u4_t{0, 0, 0, 0};

    accv_t acc[TM][TN];
    int pix[TM];
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) {
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) acc[tm][tn] = accv_t{};
        int p = p0 + (wave * TM + tm) * 32 + lrow;
        p = p < p_end ? p : p_end - 1; // pixels behind the last one repeat it and are not stored
        pix[tm] = SPAN ? ORG + (p - p0) * (CV_STRIDE * CV_CIN * 2)
                          : (p / CV_OW - oh_lo) * CV_STRIDE * PRS + ORG + p % CV_OW * (CV_STRIDE * CV_CIN * 2);
    }
    const int li = lane % 16;
    const char *wl = wts + (lgrp * 8 + li / 4) * RMB + lrow / 16 * 32 + li % 4 * 8;

#pragma unroll 1
    for (int kd = kd_lo; kd < kd_hi; ++kd) {
        __syncthreads();
        stage_commit<TM, SPAN>(st, patch, wts, tid);
        __syncthreads();
        if (kd + 1 < kd_hi) stage_fetch<TM, SPAN>(st, X + (long)(id0 + kd + 1) * CV_H * ROW_E, Wt + (long)(kd + 1) * WROWS * DIM_N, ih_lo, v_lo, tid);
#pragma unroll
        for (int s = 0; s < STEPS; ++s) {
            u4_t fa[TM], fb[TN];
#pragma unroll
            for (int tn = 0; tn < TN; ++tn) {
                union {
                    u4_t u;
                    tr4_t h[2];
                } b;
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    b.h[h] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) tr4_t *)(wl + (s * 16 + h * 4) * RMB + tn * 64));
                fb[tn] = b.u;
            }
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) {
                const unsigned *src = reinterpret_cast<const unsigned *>(
                    __builtin_assume_aligned(patch + (pix[tm] + lgrp * (koff(2 * s + 1, PRS) - koff(2 * s, PRS)) + koff(2 * s, PRS)), AL));
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    const unsigned m0 = kmask(2 * s, d), m1 = kmask(2 * s + 1, d);
                    fa[tm][d] = m0 == ~0u && m1 == ~0u ? src[d] : src[d] & (lgrp ? m1 : m0);
                }
            }
#pragma unroll
            for (int tm = 0; tm < TM; ++tm)
#pragma unroll
                for (int tn = 0; tn < TN; ++tn) acc[tm][tn] = mfma(fb[tn], fa[tm], acc[tm][tn]);
        }
    }

    // epilogue: + bias, ReLU, one rounding; a wavefront turns 32 pixels at a time in its own LDS rows and stores whole rows
    __syncthreads();
    out_t *Y = (out_t *)y_ + (((long)z * CV_N + n) * CV_OD + od) * OHW * DIM_N + jb * BN;
    char *stg = smem + wave * 32 * SROW;
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) {
#pragma unroll
        for (int tn = 0; tn < TN; ++tn)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int col = tn * 32 + 8 * g + 4 * lgrp;
                vec_t<out_t, 4> o;
#if HAS_BIAS
                const vec_t<float, 4> bias = *reinterpret_cast<const vec_t<float, 4> *>((const float *)bias_ + (long)z * DIM_N + jb * BN + col);
#endif
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float v = acc[tm][tn][4 * g + e];
#if HAS_BIAS
                    v += bias.v[e];
#endif
#if RELU
                    v = v > 0 ? v : 0;
#endif
                    o.v[e] = from_acc(v);
                }
                *reinterpret_cast<vec_t<out_t, 4> *>(stg + lrow * SROW + col * (int)sizeof(out_t)) = o;
            }
        __builtin_amdgcn_wave_barrier();
        constexpr int OV = 16 / sizeof(out_t), OCB = BN / OV; // 16-byte vectors of a row
        const int pw = p0 + (wave * TM + tm) * 32;
#pragma unroll
        for (int i = 0; i < 32 * OCB / 64; ++i) {
            const int idx = i * 64 + lane, r = idx / OCB, c = idx % OCB;
            const u4_t v = *reinterpret_cast<const u4_t *>(stg + r * SROW + c * 16);
            if (pw + r < p_end) store_stream(Y + (long)(pw + r) * DIM_N + c * OV, v);
        }
        __builtin_amdgcn_wave_barrier();
    }
    (void)bias_;
}

// Wavefronts of a SIMD that the registers are to leave room for.  Tiles of 2 x 3 intrinsics with little on its way come out at 126 to 130 of
// the 128 registers that four of them share, by accident of the compiler: 231 x 64 x 64 x 3 -> 96, 5 x 5 with 130 13.3 us, with 128 12.6.
template <int TM, bool SPAN> constexpr int rows_waves()
{
    return TM * TN == 6 && CV_KD == 1 && TM * TN * 16 + (tile_t<TM, SPAN>::XI + WI) * 4 <= 128 ? 4 : 2;
}

extern "C" __global__ void __launch_bounds__(NT, (rows_waves<CR_TM, CR_SPAN>()))
ms_kernel(const void *__restrict__ x_, const void *__restrict__ w_, const void *__restrict__ bias_, void *__restrict__ y_, int instances)
{
    image_rows<CR_TM, CR_SPAN>(x_, w_, bias_, y_, instances);
}

#if CR_MANY_TM
// the larger tile of launches over many instances; which launches take it says image_rows_many() in ms_interp.cpp
extern "C" __global__ void __launch_bounds__(NT, (rows_waves<CR_MANY_TM, CR_MANY_SPAN>()))
ms_kernel_many(const void *__restrict__ x_, const void *__restrict__ w_, const void *__restrict__ bias_, void *__restrict__ y_, int instances)
{
    image_rows<CR_MANY_TM, CR_MANY_SPAN>(x_, w_, bias_, y_, instances);
}
#endif
