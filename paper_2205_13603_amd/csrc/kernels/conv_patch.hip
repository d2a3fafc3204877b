// Convolution of stride 1 (conv2d or transposed, + bias + ReLU; whole 32-channel groups) on the CDNA4 matrix cores from input
// patches in LDS; which launches run here says takes_fill() in ms_interp.cpp.
//
// A tile is rows of one image (or whole images) by BN output channels.  Its reduction runs over chunks of 32 input channels: the
// chunk's patch, zero border included, is loaded straight into LDS once and read under every tap, while the next chunk's is on
// its way; the weights of one filter column come in a ring of three stages.  A step is one filter column: with a wavefront's
// tile R rows high, a lane's fragment of an input row is read once for the up to TH output rows that meet it, so that LDS reads
// of a step are R + TH - 1 fragments of pixels and TH * TN of weights for R * TH * TN products (56 x 56 x 64 -> 64 on 7 rows and 4
// column tiles: 63 clocks of LDS, at 128 bytes each, per 100 of the matrix cores, 164 where a tap reads its own fragments).
// One wavefront of the workgroup issues all loads and counts them; the others multiply and store, and never wait for memory:
// the counter of loads and stores runs down in issue order, and behind a tile's streamed stores a load would wait for HBM.
// What bounds it: the two wavefronts of a SIMD run through a step's first fragment reads and a tile's results at nearly the same
// time, one waiting for the other no further than the rings allow.  56 x 56 x 64 -> 64 x 512 in fp16: 126 us, 42 % matrix-core busy
// at 2.15 GHz; without products 102, without patch loads 108, without stores 110; 143 before, from weights and patches resident
// under helper wavefronts.  48 x 48 x 96 -> 32, batch 440: 180 -> 71; 32 x 32 x 256 -> 32, dilation 2, batch 144: 86 -> 34.
#include "common.h"

typedef _Float16 h8_t __attribute__((ext_vector_type(8)));
typedef __bf16 b8_t __attribute__((ext_vector_type(8)));
typedef short tr4_t __attribute__((ext_vector_type(4)));
typedef float accv_t __attribute__((ext_vector_type(4)));
typedef unsigned u4_t __attribute__((ext_vector_type(4)));
typedef unsigned u2_t __attribute__((ext_vector_type(2)));

constexpr int TH = CS_TH, TW = CS_TW, DIL = CS_DIL;
constexpr int OH = CS_PH_H, OW = CS_PH_W, CHUNKS = CS_C / 32, PIXEL_B = CS_C * 2;
constexpr int up(int n, int d) { return (n + d - 1) / d; }
// 16 pixels of an intrinsic: CW columns of BANDS rows; a wavefront: R rows of such strips, TN x 16 channels
constexpr int CW = CP_CW, BANDS = 16 / CW, R = CP_R, TN = CP_TN, WR = CP_WR, WJ = CP_WJ, WS = up(OW, CW);
constexpr int NW = WS * WR * WJ, NT = (NW + 1) * 64, BN = WJ * TN * 16, JB = DIM_N / BN;
// a tile: BANDS x WR x R rows of one image, or, where R is a whole one, BANDS x WR images
constexpr bool WHOLE = CP_WHOLE;
constexpr int ROWS = WHOLE ? OH : BANDS * WR * R, IMGS = WHOLE ? BANDS * WR : 1;
static_assert(!WHOLE || R == OH, "whole images");
static_assert(CS_C % 32 == 0 && DIM_N % BN == 0 && TW >= 2 && TN % 2 == 0 && sizeof(in_t) == 2 && sizeof(out_t) == 2, "see conv_patch()");
constexpr int TPI = WHOLE ? 1 : up(OH, ROWS), GROUPS = up(CS_N, IMGS); // tiles of an image, groups of IMGS images
constexpr int P_H = ROWS + (TH - 1) * DIL;                             // patch rows of an image
constexpr int P_W0 = OW + (TW - 1) * DIL, P_W = CW == 4 ? P_W0 | 1 : P_W0; // patch columns (odd: see swz)
constexpr int BAND_ROWS = WHOLE ? P_H : WR * R, WR_ROWS = WHOLE ? BANDS * P_H : R; // patch rows between bands, wavefronts
constexpr int SLOTS = IMGS * P_H * P_W, NPI = up(SLOTS, 16), PATCH_B = NPI * 1024; // 64-byte slots, load instructions, bytes
constexpr int W_ROW = BN * 2, CB = BN / 8;                // weights of a step: TH x 32 k-rows of BN columns
constexpr int NWI = TH * 32 * W_ROW / 1024, W_B = NWI * 1024;
// patch loads ahead of filter column kw's: they are spread over all slots of a chunk but the last
constexpr int share(int kw) { return kw >= TW - 1 ? NPI : NPI * kw / (TW - 1); }
constexpr int WST = 3;                            // stages of weights
constexpr int W_AT = 2 * PATCH_B, BIAS_AT = W_AT + WST * W_B, FLAGS_AT = BIAS_AT + (HAS_BIAS ? 2 * 1024 : 0), LDS_B = FLAGS_AT + 128;
static_assert(NW <= 15 && NPI + NWI <= 192, "flags, registers of the loads' addresses");
static_assert(LDS_B == CP_LDS && NT == CP_THREADS, "the host's counts");

// The four 16-byte units of a slot are XOR-swizzled by the column: LDS serves 8 pixels x 2 units at once, which
// are 8 slots in a row, or (CW 4) 4 of one band and 4 of the next, an odd number of slots away
__device__ __forceinline__ constexpr int swz(int col) { return CW == 4 ? (col & 1) * 2 + (col >> 1 & 1) : col >> 1 & 3; }
// weights: 32-byte granules (16 columns) of a k-row swizzled by the row, for the transposing reads
constexpr int NGRAN = BN / 16, GBLK = NGRAN % 8 == 0 ? 8 : NGRAN & -NGRAN;
__device__ __forceinline__ constexpr int swz_w(int k) { return GBLK < 2 ? 0 : ((k / (8 / GBLK)) % (GBLK > 1 ? GBLK / 2 : 1) * 2 + k / 8 % 2) * 2; }

__device__ __forceinline__ accv_t mfma(const u4_t &a, const u4_t &b, accv_t c)
{
#if IN_DT == DT_F16
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8_t, a), __builtin_bit_cast(h8_t, b), c, 0, 0, 0);
#else
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(b8_t, a), __builtin_bit_cast(b8_t, b), c, 0, 0, 0);
#endif
}

struct tile_id {
    int inst, n0, row0, jb;                               // instance, first image, first output row, column block
};
__device__ __forceinline__ tile_id decode(long f, long total)
{
    f = f % 8 * (total / 8) + (f % 8 < total % 8 ? f % 8 : total % 8) + f / 8; // tiles of one XCD follow each other: they share patch rows
    constexpr int G = JB * TPI * GROUPS;
    const int g = (int)(f % G), t = g / JB;
    return {(int)uniform((unsigned)(f / G)), (int)uniform(t / TPI * IMGS), (int)uniform(t % TPI * ROWS), (int)uniform(g % JB)};
}
// first input row and column of the patch of output pixel (0, 0): a transposed convolution of stride 1 reads its taps backwards
constexpr int ROW_0 = CS_TR ? CS_PAD_H - (TH - 1) : -CS_PAD_H, COL_0 = CS_TR ? CS_PAD_W - (TW - 1) : -CS_PAD_W;

constexpr int vm_cap(int n) { return n > 63 ? 63 : n; }
#define INLINE __attribute__((always_inline))
template <int N> struct int_c {
    static constexpr int value = N;
};
template <class F, int N> __device__ __forceinline__ void all_steps(F &step, int_c<N> n)
{
    step(n);
    if constexpr (N + 1 < TW) all_steps(step, int_c<N + 1>{});
}

extern "C" __global__ void __launch_bounds__(NT, up(CP_PER_CU * (NW + 1), 4))
ms_kernel(const void *__restrict__ x_, const void *__restrict__ w_, const void *__restrict__ bias_, void *__restrict__ y_, int instances)
{
    const int tid = threadIdx.x, lane = tid % 64, wave = __builtin_amdgcn_readfirstlane(tid / 64);
    __shared__ __attribute__((aligned(1024))) char lds[LDS_B];
    lds_char *const lds3 = (lds_char *)lds;

    const long total = (long)JB * TPI * GROUPS * instances, first = blockIdx.x, stride = gridDim.x;
    if (first >= total) return;
    const long my_tiles = (total - first + stride - 1) / stride;

    // Progress is told through words in LDS, not barriers: `ready` counts the steps whose operands have landed, done[w] the steps
    // that wavefront w has read.  The loads' wavefront waits for every done[w], the others for `ready`; both only grow, and every
    // wavefront runs the same number of steps.
    typedef __attribute__((address_space(3))) int lds_int;
    lds_int *const ready = (lds_int *)((__attribute__((address_space(3))) char *)lds + FLAGS_AT), *const done = ready + 16;
    if (tid < 32) ready[tid] = 0;
    __syncthreads();

    if (wave == NW) {
        // ---- the wavefront that loads.  Patches: the cursor is chunk pc of tile pt, going into buffer pb; past the end the last chunk
        // is requested again
        long pt = 0;
        int pc = 0, pb = 0;
        rsrc_t prs;
        unsigned ptoff = 0, poff[NPI];
        int cs = lane / 4 % P_W, pr = lane / 4 / P_W;     // column and row of the lane's slot, 16 slots further on from load to load
#pragma unroll
        for (int i = 0; i < NPI; ++i) {
            const int img = WHOLE ? pr / P_H : 0, iw = cs + COL_0, ih = pr - img * P_H + (WHOLE ? ROW_0 : 0);
            const bool ok = pr < IMGS * P_H && cs < P_W0 && (unsigned)iw < (unsigned)CS_W && (!WHOLE || (unsigned)ih < (unsigned)CS_H);
            poff[i] = ok ? (unsigned)(((img * CS_H + ih) * CS_W + iw) * PIXEL_B + ((lane % 4) ^ swz(cs)) * 16) : OUTSIDE;
            cs += 16 % P_W;
            pr += 16 / P_W;
            if (cs >= P_W) {
                cs -= P_W;
                ++pr;
            }
        }
        auto patch_at = [&]() INLINE {
            const tile_id t = decode(first + pt * stride, total);
            const int images = WHOLE && CS_N - t.n0 < IMGS ? CS_N - t.n0 : IMGS;
            const char *base = (const char *)x_ + ((long)t.inst * CS_N + t.n0) * (CS_H * CS_W * (long)PIXEL_B) + pc * 64;
            prs = buffer_at(base, (unsigned)(images * (CS_H * CS_W * PIXEL_B) - pc * 64));
            ptoff = WHOLE ? 0u : uniform((unsigned)((t.row0 + ROW_0) * (CS_W * PIXEL_B)));
        };
        auto next_patch = [&]() INLINE {
            pb ^= 1;
            if (pc + 1 < CHUNKS) ++pc;
            else if (pt + 1 < my_tiles) {
                pc = 0;
                ++pt;
            }
            patch_at();
        };
        // weights: step (wc, wtw) of tile wt, into stage ws
        long wt = 0;
        int wc = 0, wtw = 0, ws = 0;
        const char *wtile, *wbase;
        unsigned woff[NWI];
        constexpr int TAP_K = TW * CS_C;                  // k-rows between two taps of a filter column
#pragma unroll
        for (int i = 0; i < NWI; ++i) {
            const int e = i * 64 + lane, k = e / CB, c = (e % CB) ^ swz_w(k % 32);
            woff[i] = (unsigned)(((k / 32 * TAP_K + k % 32) * DIM_N + c * 8) * 2);
        }
        auto weights_at = [&]() INLINE {
            wbase = wtile + (long)(wtw * CS_C + wc * 32) * (DIM_N * 2);
        };
        auto weights_tile = [&]() INLINE {
            const tile_id t = decode(first + wt * stride, total);
            wtile = (const char *)w_ + ((long)t.inst * B_INST + t.jb * BN) * 2;
            weights_at();
        };
        auto load_weights = [&]() INLINE {
#pragma unroll
            for (int i = 0; i < NWI; ++i) load_lds16_to(wbase, woff[i], uniform((unsigned)(size_t)(lds3 + W_AT + ws * W_B + i * 1024)));
            ws = ws + 1 == WST ? 0 : ws + 1;
            if (++wtw < TW) return weights_at();
            if (wc + 1 < CHUNKS) {
                wtw = 0;
                ++wc;
                return weights_at();
            }
            if (wt + 1 < my_tiles) {
                wtw = wc = 0;
                ++wt;
                return weights_tile();
            }
            --wtw; // behind the last step: again
        };
        long bt = 0;
        int bh = 0;
        auto load_bias = [&]() INLINE { // of tile bt, into half bh
#if HAS_BIAS
            const tile_id t = decode(first + bt * stride, total);
            const char *b = (const char *)bias_ + ((long)t.inst * DIM_N + t.jb * BN) * 4;
            gather_lds16(buffer_at(b, BN * 4), (unsigned)lane * 16, lds3 + BIAS_AT + bh * 1024);
            if (bt + 1 < my_tiles) ++bt;
            bh ^= 1;
#endif
        };
        patch_at();
        weights_tile();
        load_bias();
#pragma unroll
        for (int i = 0; i < NPI; ++i) gather_lds16(prs, poff[i] + ptoff, lds3 + pb * PATCH_B + i * 1024);
        next_patch();
#pragma unroll
        for (int s = 0; s < WST - 1; ++s) load_weights();
        DL_WAIT_VM(vm_cap(NWI));
        asm volatile("" ::: "memory");
        *(volatile lds_int *)ready = 1;

        int s = 0;
        // the loads behind step s - 1: weights WST - 1 steps ahead, a share of the next patch, in the first step of a tile the next bias
        auto slot = [&](auto kw_, bool first_chunk) INLINE {
            constexpr int kw = decltype(kw_)::value, lo = share(kw), hi = share(kw + 1);
            while (__builtin_amdgcn_ballot_w64(lane < NW && ((volatile lds_int *)done)[lane < NW ? lane : 0] < s)) __builtin_amdgcn_s_sleep(1);
            asm volatile("" ::: "memory");
            if (kw == 0 && first_chunk) load_bias();
            load_weights();
#pragma unroll
            for (int i = lo; i < hi; ++i) gather_lds16(prs, poff[i] + ptoff, lds3 + pb * PATCH_B + i * 1024);
            if (kw == TW - 2) next_patch();
            // Landed by now: the weights of step s + 1 and, behind the last step of a chunk, the next patch.  Loads land in order, and
            // behind the weights of step s + 1 there are the patch's share of the last slot and all of this one
            __builtin_amdgcn_sched_barrier(0);
            DL_WAIT_VM(vm_cap(NWI + (kw == TW - 1 ? 0 : hi - (kw ? share(kw - 1) : 0))));
            asm volatile("" ::: "memory");
            ++s;
            *(volatile lds_int *)ready = s + 1;
        };
#pragma unroll 1
        for (int ti = 0; ti < (int)my_tiles; ++ti)
#pragma unroll 1
            for (int c = 0; c < CHUNKS; ++c) {
                auto f = [&](auto kw) INLINE { slot(kw, c == 0); };
                all_steps(f, int_c<0>{});
            }
        DL_WAIT_VM(0); // the re-loads past the end must land before the workgroup's LDS is released
        return;
    }

    // ---- the wavefronts that multiply
    const int wj = wave % WJ, wr = wave / WJ % WR, wst = wave / (WJ * WR), lrow = lane % 16, lgrp = lane / 16;
    int qa[TW], rb[TN];
    int col = wst * CW + lrow % CW;
    col = col < OW ? col : OW - 1; // pixels behind the last one of a row are not stored
#pragma unroll
    for (int kw = 0; kw < TW; ++kw) {
        const int cs = col + (CS_TR ? TW - 1 - kw : kw * DIL);
        qa[kw] = ((lrow / CW * BAND_ROWS + wr * WR_ROWS) * P_W + cs) * 64 + (lgrp ^ swz(cs)) * 16;
    }
    const int li = lane % 16, tr_row = lgrp * 8 + li / 4;
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) rb[tn] = W_AT + tr_row * W_ROW + (((wj * TN + tn) * 2) ^ swz_w(tr_row)) * 16 + li % 4 * 8;

    accv_t acc[R][TN];
    // sums start from the bias
    auto start_acc = [&](int at) INLINE {
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
            accv_t bias = {};
#if HAS_BIAS
            bias = *(const __attribute__((address_space(3))) accv_t *)(lds3 + BIAS_AT + at * 1024 + ((wj * TN + tn) * 16 + lgrp * 4) * 4);
#endif
#pragma unroll
            for (int r = 0; r < R; ++r) acc[r][tn] = bias;
        }
    };
    int rd = 0, rp = 0;
    constexpr int ROWS_IN = R + (TH - 1) * DIL;           // input rows that the wavefront's tile meets
    int seen = 0, s = 0;          // what `ready` said last, step
    // One step, the taps of filter column kw: an input row is read once for all output rows that meet it, two rows ahead of its
    // products.
    auto step = [&](auto kw_) INLINE {
        constexpr int kw = decltype(kw_)::value;
        while (seen <= s) {
            seen = __builtin_amdgcn_readfirstlane(*(volatile lds_int *)ready);
            if (seen <= s) __builtin_amdgcn_s_sleep(1);
        }
        asm volatile("" ::: "memory");
        u4_t fb[TH][TN], fa[3];
        auto read_a = [&](int i) INLINE { return *(const __attribute__((address_space(3))) u4_t *)(lds3 + (qa[kw] + rp) + i * (P_W * 64)); };
        fa[0] = read_a(0);
#pragma unroll
        for (int q = 0; q < TH; ++q) {
            const int kh = CS_TR ? TH - 1 - q : q;
            if (q == TH / 2 && ROWS_IN > 1) fa[1] = read_a(1);
#pragma unroll
            for (int tn = 0; tn < TN; ++tn) {
                union {
                    u4_t u;
                    tr4_t h[2];
                } b;
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    b.h[h] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                        (__attribute__((address_space(3))) tr4_t *)(lds3 + (rb[tn] + rd * W_B) + (kh * 32 + h * 4) * W_ROW));
                fb[kh][tn] = b.u;
            }
        }
#pragma unroll
        for (int i = 0; i < ROWS_IN; ++i) {
            if (i + 2 < ROWS_IN) fa[(i + 2) % 3] = read_a(i + 2);
#pragma unroll
            for (int q = 0; q < TH; ++q) {
                const int r = i - q * DIL, kh = CS_TR ? TH - 1 - q : q;
                if (r < 0 || r >= R) continue;
#pragma unroll
                for (int tn = 0; tn < TN; ++tn) acc[r][tn] = mfma(fb[kh][tn], fa[i % 3], acc[r][tn]);
            }
        }
        asm volatile("" ::: "memory");
        ++s;
        if (lane == 0) *(volatile lds_int *)(done + wave) = s;
        rd = rd + 1 == WST ? 0 : rd + 1;
    };
#pragma unroll 1
    for (int ti = 0; ti < (int)my_tiles; ++ti) {
        const tile_id t = decode(first + ti * stride, total);
        while (seen <= s) {
            seen = __builtin_amdgcn_readfirstlane(*(volatile lds_int *)ready);
            if (seen <= s) __builtin_amdgcn_s_sleep(1);
        }
        asm volatile("" ::: "memory");
        start_acc(ti & 1);
#pragma unroll 1
        for (int c = 0; c < CHUNKS; ++c) {
            all_steps(step, int_c<0>{});
            rp = PATCH_B - rp;
        }
        // ---- results: ReLU, one rounding.  A lane has 4 channels of every 16; neighbouring lane groups trade them for those of
        // the next 16, so that each stores 8 channels at once
        const int rows = OH - t.row0 < ROWS ? OH - t.row0 : ROWS, images = CS_N - t.n0 < IMGS ? CS_N - t.n0 : IMGS; // inside the image, the stack
        out_t *const Y = (out_t *)y_ + (((long)t.inst * CS_N + t.n0) * OH + t.row0) * (OW * DIM_N) + t.jb * BN + wj * (TN * 16);
        const int chan = lgrp % 2 * 16 + lgrp / 2 * 8;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            unsigned o[TN][2];
#pragma unroll
            for (int tn = 0; tn < TN; ++tn)
#pragma unroll
                for (int h = 0; h < 2; ++h) o[tn][h] = finish(acc[r][tn][2 * h], acc[r][tn][2 * h + 1]);
            u4_t v[TN / 2];                               // channels tn * 32 + chan on
#pragma unroll
            for (int tn = 0; tn < TN; tn += 2) {
                const u2_t lo = __builtin_amdgcn_permlane16_swap(o[tn][0], o[tn + 1][0], false, false);
                const u2_t hi = __builtin_amdgcn_permlane16_swap(o[tn][1], o[tn + 1][1], false, false);
                v[tn / 2] = u4_t{lo[0], hi[0], lo[1], hi[1]};
            }
            // 64 channels: pixels 0 to 7 and 8 to 15 trade halves, so that a store covers whole lines
            if constexpr (TN == 4) {
                u4_t a, b;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    a[e] = __builtin_amdgcn_update_dpp(v[0][e], v[1][e], 0x128, 0xf, 0xc, false); // row_ror:8 into lanes 8 to 15
                    b[e] = __builtin_amdgcn_update_dpp(v[1][e], v[0][e], 0x128, 0xf, 0x3, false); // and into lanes 0 to 7
                }
                v[0] = a;
                v[1] = b;
            }
#pragma unroll
            for (int h = 0; h < TN / 2; ++h) {
                const int p = TN == 4 ? h * 8 + lrow % 8 : lrow, band = p / CW, ow = wst * CW + p % CW;
                const int img = WHOLE ? wr * BANDS + band : 0, row = WHOLE ? r : (band * WR + wr) * R + r;
                out_t *const dst = Y + (((img * OH + row) * OW + ow) * DIM_N + chan + (TN == 4 ? lrow / 8 * 32 : h * 32));
                if (ow < OW && row < rows && img < images) store_stream(dst, v[h]);
            }
        }
    }
    (void)bias_;
}
