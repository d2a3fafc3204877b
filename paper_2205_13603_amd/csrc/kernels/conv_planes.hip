// First-layer convolution (2-D or 3-D, 1 to 4 channels per pixel, + bias + ReLU) on the CDNA4 matrix cores, persistent workgroups
// over filter planes; which launches run here says takes_fill() in ms_interp.cpp, and conv_rows.hip has the layout of runs and
// chunks and takes the others.
//
// A filter plane's image rows and weights are loaded straight into LDS, so that no register holds data on its way and a step's
// fragments are read while the step before it is multiplied.  Two workgroups of four wavefronts share a compute unit: one loads
// a plane or writes results while the other multiplies.  The next tile's first plane is requested ahead of a tile's results,
// which leave through trades between lanes (no LDS) as whole lines.
// What bounds it: LDS reads, 0.75 clocks per clock of the matrix cores, and the rounds of tiles, which differ in their planes:
// 8 x 16 x 224 x 224 x 3 -> 64, 7 x 7 x 7, stride 2 in fp16: 122 -> 102 us, 52 of them products, 57 LDS; 128 x 224 x 224 x 3 -> 64, 7 x 7:
// 62 -> 53.5 us (4.6 TB/s).  Two stages under one workgroup of eight wavefronts
// took 104 and 57.
#include "common.h"

typedef _Float16 h8_t __attribute__((ext_vector_type(8)));
typedef __bf16 b8_t __attribute__((ext_vector_type(8)));
typedef short tr4_t __attribute__((ext_vector_type(4)));
typedef float accv_t __attribute__((ext_vector_type(16)));
typedef float f4_t __attribute__((ext_vector_type(4)));
typedef unsigned u4_t __attribute__((ext_vector_type(4)));
typedef unsigned u2_t __attribute__((ext_vector_type(2)));

constexpr int TM = CR_TM, TN = CR_TN, NW = CR_WAVES, NT = NW * 64;
constexpr int BN = TN * 32, JB = DIM_N / BN;              // output channels of a workgroup, column blocks
constexpr int OHW = CV_OH * CV_OW, PX = NW * TM * 32;     // output pixels of a plane, of a workgroup
constexpr int TILES = (OHW + PX - 1) / PX;
// the layout of runs and chunks is that of conv_rows.hip
constexpr int LEAD = CV_PAD * CV_CIN % 2;
constexpr int RUN = CV_KW * CV_CIN, CPR = (LEAD + RUN + 7) / 8;
constexpr int NCH = CV_KH * CPR, STEPS = (NCH + 1) / 2;
constexpr int ROW_E = CV_W * CV_CIN, ROW_B = ROW_E * 2, WROWS = CV_KH * RUN;
static_assert(ROW_E % 8 == 0 && CV_STRIDE * CV_CIN % 2 == 0 && DIM_N % BN == 0 && sizeof(out_t) == 2 && TN <= 2, "see conv_planes()");
constexpr int up(int n, int d) { return (n + d - 1) / d; }
constexpr int LHALO = up((CV_PAD * CV_CIN + LEAD) * 2, 16) * 16;
constexpr int ORG = LHALO - (CV_PAD * CV_CIN + LEAD) * 2; // byte of pixel 0's run in its row
constexpr int READ_END = ORG + (CV_OW - 1) * CV_STRIDE * CV_CIN * 2 + CPR * 16, IMG_END = LHALO + ROW_B;
constexpr int PRS = up(READ_END > IMG_END ? READ_END : IMG_END, 16) * 16, SV = PRS / 16; // bytes of a staged row, its 16-byte units
constexpr int P_OUT_ = PX % CV_OW == 0 ? PX / CV_OW : (CV_OW + PX - 2) / CV_OW + 1, P_OUT = P_OUT_ < CV_OH ? P_OUT_ : CV_OH;
constexpr int PR = (P_OUT - 1) * CV_STRIDE + CV_KH;       // input rows of a tile
constexpr int NPI = up(PR * SV, 64), UB = BN / 8, NWI = up(STEPS * 16 * UB, 64); // load instructions: rows, weights (1 KiB each)
constexpr int PATCH_B = NPI * 1024, WT_B = NWI * 1024, STAGE_B = PATCH_B + WT_B;
constexpr int LP = up(NPI, NW), LW = up(NWI, NW);         // of a wavefront, at most
constexpr int BIAS_AT = STAGE_B, LDS_B = BIAS_AT + (HAS_BIAS ? 2048 : 0);
static_assert(LDS_B == CR_LDS, "the host's count of LDS");
constexpr int cr_gcd(int a, int b) { return b ? cr_gcd(b, a % b) : a; }
constexpr int AL = cr_gcd(16, cr_gcd(ORG, CV_STRIDE * CV_CIN * 2)); // alignment of a fragment in its row
constexpr int ROW_BYTES_W = BN * 2;
// 32-byte granules (16 columns) of a weight row XOR-swizzled by the row, so that the transposing reads of 4 rows x 2 granules meet all banks
constexpr int NGRAN = BN / 16, GBLK = NGRAN % 8 == 0 ? 8 : NGRAN & -NGRAN;
__device__ __forceinline__ constexpr int swz_w(int k) { return ((k / (8 / GBLK)) % (GBLK / 2) * 2 + k / 8 % 2) * 2; }

constexpr int koff(int c) { return c < NCH ? c / CPR * PRS + c % CPR * 16 : koff(c - 1); }
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

struct tile_id {
    int inst, n, od, tile, jb, kd_lo, kd_hi;              // filter planes [kd_lo, kd_hi) lie inside the input
};
__device__ __forceinline__ tile_id decode(long f, long total)
{
    f = f % 8 * (total / 8) + (f % 8 < total % 8 ? f % 8 : total % 8) + f / 8; // tiles of one XCD follow each other: they share input rows and planes
    constexpr int G = JB * CV_OD * TILES * CV_N;
    const int g = (int)(f % G);
    tile_id t;
    t.inst = (int)uniform((unsigned)(f / G));
    t.jb = (int)uniform(g % JB);
    // output planes apart: a workgroup's tiles are of several, and planes at the ends of the depth meet fewer filter planes
    t.tile = (int)uniform(g / JB % TILES);
    t.od = (int)uniform(g / (JB * TILES) % CV_OD);
    t.n = (int)uniform(g / (JB * TILES * CV_OD));
    const int id0 = CV_D > 1 || CV_KD > 1 ? t.od * CV_STRIDE - CV_PAD : 0;
    t.kd_lo = id0 < 0 ? -id0 : 0;
    t.kd_hi = CV_D - id0 < CV_KD ? CV_D - id0 : CV_KD;
    if (t.kd_lo >= t.kd_hi) t.kd_lo = t.kd_hi = 0;
    return t;
}

extern "C" __global__ void __launch_bounds__(NT, 2)
ms_kernel(const void *__restrict__ x_, const void *__restrict__ w_, const void *__restrict__ bias_, void *__restrict__ y_, int instances)
{
    const int tid = threadIdx.x, lane = tid % 64, wave = __builtin_amdgcn_readfirstlane(tid / 64), lrow = lane % 32, lgrp = lane / 32;
    __shared__ __attribute__((aligned(1024))) char lds[LDS_B];
    lds_char *const lds3 = (lds_char *)lds;
    const long total = (long)JB * CV_OD * TILES * CV_N * instances, first = blockIdx.x, stride = gridDim.x;
    if (first >= total) return;
    const int my_tiles = (int)((total - first + stride - 1) / stride);

    // ---- loads of a filter plane: the cursor is plane lk of tile lt; past the end the last plane is requested again
    unsigned poff[LP], woff[LW];
#pragma unroll
    for (int j = 0; j < LP; ++j) {
        const int idx = (j * NW + wave) * 64 + lane, row = idx / SV, at = idx % SV * 16 - LHALO;
        poff[j] = row < PR && at >= 0 && at < ROW_B ? (unsigned)(row * ROW_B + at) : OUTSIDE;
    }
#pragma unroll
    for (int j = 0; j < LW; ++j) {
        const int idx = (j * NW + wave) * 64 + lane, k = idx / UB, c = (idx % UB) ^ swz_w(k), q = k % (CPR * 8) - LEAD, kh = k / (CPR * 8);
        woff[j] = kh < CV_KH && q >= 0 && q < RUN ? (unsigned)(((kh * RUN + q) * DIM_N + c * 8) * 2) : OUTSIDE;
    }
    int li = 0, lk = 0, half = 0;
    tile_id lt = decode(first, total);
    lk = lt.kd_lo;
    auto request = [&]() {
        const int id = CV_D > 1 || CV_KD > 1 ? lt.od * CV_STRIDE - CV_PAD + lk : 0;
        const int ih_lo = (int)((unsigned)(lt.tile * PX) / CV_OW) * CV_STRIDE - CV_PAD_H;
        // a tile without a plane inside the input reads plane 0 and multiplies nothing
        const char *plane = (const char *)x_ + ((long)lt.inst * A_INST + ((long)lt.n * CV_D + (id < 0 || id >= CV_D ? 0 : id)) * (CV_H * ROW_E)) * 2;
        const rsrc_t xb = buffer_at(plane, CV_H * ROW_B);
        const rsrc_t wb = buffer_at((const char *)w_ + ((long)lt.inst * B_INST + (long)lk * (WROWS * DIM_N) + lt.jb * BN) * 2);
        const unsigned toff = uniform((unsigned)(ih_lo * ROW_B));
#pragma unroll
        for (int j = 0; j < LW; ++j) {
            const int i = j * NW + wave;
            if (NWI % NW == 0 || i < NWI) gather_lds16(wb, woff[j], lds3 + PATCH_B + i * 1024);
        }
#pragma unroll
        for (int j = 0; j < LP; ++j) {
            const int i = j * NW + wave;
            if (NPI % NW == 0 || i < NPI) gather_lds16(xb, poff[j] + toff, lds3 + i * 1024);
        }
#if HAS_BIAS
        if (wave == 0 && lk == lt.kd_lo) // with a tile's first plane
            gather_lds16(buffer_at((const char *)bias_ + ((long)lt.inst * DIM_N + lt.jb * BN) * 4, BN * 4), (unsigned)lane * 16, lds3 + BIAS_AT + half * 1024);
#endif
        if (lk + 1 < lt.kd_hi) ++lk;
        else if (li + 1 < my_tiles) {
            ++li;
            half ^= 1;
            lt = decode(first + (long)li * stride, total);
            lk = lt.kd_lo;
        }
    };

    accv_t acc[TM][TN];
    int pix[TM];
    const int l16 = lane % 16, tr_row = lgrp * 8 + l16 / 4;
    const int wl = PATCH_B + tr_row * ROW_BYTES_W + l16 % 4 * 8;
    int wcol[TN];
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) wcol[tn] = wl + (((tn * 2 + lrow / 16) * 2) ^ swz_w(tr_row)) * 16;

    request();
    DL_WAIT_VM(0);
    __builtin_amdgcn_s_barrier();
    constexpr int STORES = TM * TN * 2;
#pragma unroll 1
    for (int ti = 0; ti < my_tiles; ++ti) {
        const tile_id t = decode(first + (long)ti * stride, total);
        const int p0 = t.tile * PX, oh_lo = (int)((unsigned)p0 / CV_OW);
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
#pragma unroll
            for (int tn = 0; tn < TN; ++tn) {
                accv_t sum = {};
#if HAS_BIAS
#pragma unroll
                for (int g = 0; g < 4; ++g) {             // sums start from the bias
                    const f4_t b = *(const __attribute__((address_space(3))) f4_t *)(lds3 + BIAS_AT + (ti & 1) * 1024 + (tn * 32 + 8 * g + 4 * lgrp) * 4);
#pragma unroll
                    for (int e = 0; e < 4; ++e) sum[4 * g + e] = b[e];
                }
#endif
                acc[tm][tn] = sum;
            }
            int p = p0 + (wave * TM + tm) * 32 + lrow;
            p = p < OHW ? p : OHW - 1; // pixels behind the last one repeat it and are not stored
            pix[tm] = (p / CV_OW - oh_lo) * CV_STRIDE * PRS + ORG + p % CV_OW * (CV_STRIDE * CV_CIN * 2);
        }
        const int planes = t.kd_hi > t.kd_lo ? t.kd_hi - t.kd_lo : 1;
#pragma unroll 1
        for (int kd = 0; kd < planes; ++kd) {
            const bool last = kd + 1 == planes;
            if (t.kd_lo < t.kd_hi) {
                // the fragments of a step are read, as they lie, while the one before it is multiplied
                u4_t fa[2][TM], fb[2][TN];
                auto read = [&](int s) {
#pragma unroll
                    for (int tn = 0; tn < TN; ++tn) {
                        union {
                            u4_t u;
                            tr4_t h[2];
                        } b;
#pragma unroll
                        for (int h = 0; h < 2; ++h)
                            b.h[h] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) tr4_t *)(lds3 + wcol[tn] + (s * 16 + h * 4) * ROW_BYTES_W));
                        fb[s % 2][tn] = b.u;
                    }
#pragma unroll
                    for (int tm = 0; tm < TM; ++tm) {
                        typedef unsigned piece_t __attribute__((ext_vector_type(4), aligned(AL)));
                        fa[s % 2][tm] = *(const __attribute__((address_space(3))) piece_t *)(lds3 + (pix[tm] + lgrp * (koff(2 * s + 1) - koff(2 * s)) + koff(2 * s)));
                    }
                };
                read(0);
#pragma unroll
                for (int s = 0; s < STEPS; ++s) {
                    __builtin_amdgcn_sched_barrier(0);
                    if (s + 1 < STEPS) read(s + 1);
#pragma unroll
                    for (int tm = 0; tm < TM; ++tm) {
                        u4_t a = fa[s % 2][tm];
#pragma unroll
                        for (int d = 0; d < 4; ++d) {
                            const unsigned m0 = kmask(2 * s, d), m1 = kmask(2 * s + 1, d);
                            if (m0 != ~0u || m1 != ~0u) a[d] &= lgrp ? m1 : m0;
                        }
#pragma unroll
                        for (int tn = 0; tn < TN; ++tn) acc[tm][tn] = mfma(fb[s % 2][tn], a, acc[tm][tn]);
                    }
#pragma unroll
                    for (int m = 0; m < TM * TN; ++m) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0); // a product, two reads
                        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            // everybody has read the plane: the next may come
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_barrier();
            request();
            __builtin_amdgcn_sched_barrier(0);
            if (last) {
                // results: + bias, ReLU, one rounding.  A lane has 4 channels of every 8 of a pixel; trades between lanes leave it with 8
                // channels in a row, and a store with whole lines
                out_t *const Y = (out_t *)y_ + (((long)t.inst * CV_N + t.n) * CV_OD + t.od) * ((long)OHW * DIM_N) + t.jb * BN;
#pragma unroll
                for (int tm = 0; tm < TM; ++tm) {
                    u4_t q[TN][2];                        // pixels of half a tile: channels tn * 32 + lane / 16 % 2 * 16 + lgrp * 8 on
#pragma unroll
                    for (int tn = 0; tn < TN; ++tn) {
                        unsigned o[4][2];
#pragma unroll
                        for (int g = 0; g < 4; ++g) {
                            o[g][0] = finish(acc[tm][tn][4 * g], acc[tm][tn][4 * g + 1]);
                            o[g][1] = finish(acc[tm][tn][4 * g + 2], acc[tm][tn][4 * g + 3]);
                        }
                        u4_t p[2];
#pragma unroll
                        for (int g = 0; g < 2; ++g) {
                            const u2_t lo = __builtin_amdgcn_permlane32_swap(o[2 * g][0], o[2 * g + 1][0], false, false);
                            const u2_t hi = __builtin_amdgcn_permlane32_swap(o[2 * g][1], o[2 * g + 1][1], false, false);
                            p[g] = u4_t{lo[0], hi[0], lo[1], hi[1]}; // channels tn * 32 + g * 16 + lgrp * 8 on
                        }
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const u2_t r = __builtin_amdgcn_permlane16_swap(p[0][e], p[1][e], false, false);
                            q[tn][0][e] = r[0];           // pixels 0 to 15 of the tile
                            q[tn][1][e] = r[1];           // 16 to 31
                        }
                    }
                    const int pw = p0 + (wave * TM + tm) * 32;
                    auto put = [&](int px, int ch, const u4_t &v) {
                        if (pw + px < OHW) store_stream(Y + (long)(pw + px) * DIM_N + ch, v);
                    };
                    const int ch = lane / 16 % 2 * 16 + lgrp * 8;
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        if constexpr (TN == 2) {
                            u4_t a, b;
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                a[e] = __builtin_amdgcn_update_dpp(q[0][h][e], q[1][h][e], 0x128, 0xf, 0xc, false); // row_ror:8 into lanes 8 to 15
                                b[e] = __builtin_amdgcn_update_dpp(q[1][h][e], q[0][h][e], 0x128, 0xf, 0x3, false); // and into lanes 0 to 7
                            }
                            put(h * 16 + lane % 8, lane / 8 % 2 * 32 + ch, a);
                            put(h * 16 + 8 + lane % 8, lane / 8 % 2 * 32 + ch, b);
                        } else {
                            put(h * 16 + lane % 16, ch, q[0][h]);
                        }
                    }
                }
            }
            // the next plane has landed; behind it only this tile's stores, where every wavefront issued them all
            __builtin_amdgcn_sched_barrier(0);
            if (last && p0 + (wave + 1) * (TM * 32) <= OHW) DL_WAIT_VM(STORES);
            else DL_WAIT_VM(0);
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    DL_WAIT_VM(0); // the re-loads past the end must land before the workgroup's LDS is released
    (void)bias_;
}
