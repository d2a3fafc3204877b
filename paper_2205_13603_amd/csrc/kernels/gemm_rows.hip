// Product of up to 128 rows with a row-major matrix (a decoding step) on the CDNA4 matrix cores; which launches run here says
// takes_fill() in ms_interp.cpp.
//
// The wavefronts of a workgroup split the reduction of its tile and add their sums up in LDS at the end, so that nothing waits
// for a barrier before, and every wavefront keeps whole blocks of 64 k values in flight in its registers.
// What bounds it: the address lookups of a compute unit's loads, one per clock for four lanes, whatever they load; next the
// misses that its L1 keeps in flight, from HBM.  So every lane loads 16 bytes and four lanes 64 bytes that follow each other: lines of
// B as they lie, their columns dealt out by trades between lanes; lines of A by way of LDS (loaded as fragments, from 16 rows at
// once, they took four times the lookups: 48 x 6720 x 4096 23.8 us, 19.0 so; 96 x 1728 x 3072 10.0 and 7.4; tiles of 32 columns with 8-byte loads: 32 x 2048 x 2816
// 7.65, 7.13 so).
// Against nests whose workgroups stage 256 k values under barriers: 48 x 4096 x 2048 in fp16 8.25 -> 6.9 us (2.8 at the rate of a copy, 3.5
// any launch), 128 x 6720 x 2048 in bf16 43.6 -> 9.7, 16 x 5440 x 2304 9.7 -> 7.1, 128 x 8192 x 4096 57 -> 26 (2.9 TB/s).
#include "common.h"

typedef _Float16 h8_t __attribute__((ext_vector_type(8)));
typedef __bf16 b8_t __attribute__((ext_vector_type(8)));
typedef float f4_t __attribute__((ext_vector_type(4)));
typedef unsigned u4_t __attribute__((ext_vector_type(4)));

constexpr int MT = FR_MT, NC = FR_NC, NW = FR_WAVES, R = MT * 16, C = NC * 16;
constexpr int RT = DIM_M / R, CT = DIM_N / C, TILES = RT * CT;
constexpr int KB = DIM_K / 64, PER = (KB + NW - 1) / NW; // k blocks, of a wavefront at most
constexpr int D = FR_DEPTH < PER ? FR_DEPTH : PER;       // blocks in flight
constexpr int rows_per_pass()                            // 16-row tiles whose partial sums are in LDS at a time
{
    int g = MT;
    while (MT % g || NW * g * NC * 1024 > FR_LDS) --g;
    return g;
}
constexpr int G = rows_per_pass();
static_assert(DIM_M % R == 0 && DIM_N % C == 0 && DIM_K % 64 == 0 && sizeof(in_t) == 2, "see few_rows()");
static_assert(NW * G * NC * 1024 <= FR_LDS && NW * MT * 2048 <= FR_LDS, "the host's count of LDS");

// Lane 16 q + UL t + u: load r of B brings columns 8 u ... of k value 16 q + 2 NC t + r; after the trades the lane holds columns 8 u + NC t ... of all
// 16 k values of q
constexpr int UL = NC * 2;
struct block {
    u4_t a[MT][2];    // row 8 h + lane / 8 of a tile, 16-byte chunk lane % 8 of its line (swizzled by the row)
    u4_t b[2 * NC];
};

__device__ __forceinline__ f4_t mfma(const u4_t &a, const u4_t &b, f4_t c)
{
#if IN_DT == DT_F16
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8_t, a), __builtin_bit_cast(h8_t, b), c, 0, 0, 0);
#else
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(b8_t, a), __builtin_bit_cast(b8_t, b), c, 0, 0, 0);
#endif
}

__device__ __forceinline__ void request(block &x, const in_t *a, const in_t *b, int kb)
{
#pragma unroll
    for (int r = 0; r < 2 * NC; ++r) x.b[r] = *(const u4_t *)(b + (unsigned)(kb * 64 + r) * (unsigned)SB_K);
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int h = 0; h < 2; ++h) x.a[m][h] = *(const u4_t *)(a + (unsigned)((m * 16 + h * 8) * SA_I + kb * 64));
}

// `keep`, in the banks of four lanes of `BANKS` the value of `from` that a rotation of 16 lanes brings
template <int ROTATE, int BANKS> __device__ __forceinline__ unsigned trade(unsigned keep, unsigned from)
{
    return __builtin_amdgcn_update_dpp(keep, from, ROTATE, 0xf, BANKS, false);
}

// Fragments of A that other lanes of the wavefront have stored: LDS serves a wavefront in order, and the compiler may not tell these
// addresses from those of the stores, ahead or behind (see `fragments`)
__device__ __forceinline__ void multiply(const block &x, char *own, int lane, const int (&from)[2], f4_t (&acc)[MT][NC])
{
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int h = 0; h < 2; ++h) *(u4_t *)(own + (m * 2 + h) * 1024 + lane * 16) = x.a[m][h];
    // trades between lanes 8 and 4 apart: each keeps NC of the 8 columns, for 16 k values
    unsigned v[16][NC / 2];
#pragma unroll
    for (int r = 0; r < 2 * NC; ++r) {
        unsigned own_half[2], other[2];
#pragma unroll
        for (int d = 0; d < 2; ++d) {
            own_half[d] = trade<0x128, 0xc>(x.b[r][d], x.b[r][d + 2]);
            other[d] = trade<0x128, 0x3>(x.b[r][d + 2], x.b[r][d]);
        }
        if constexpr (NC == 4) {
#pragma unroll
            for (int d = 0; d < 2; ++d) v[r][d] = own_half[d], v[r + 8][d] = other[d];
        } else {
            v[r][0] = trade<0x124, 0xa>(own_half[0], own_half[1]);
            v[r + 4][0] = trade<0x12c, 0x5>(own_half[1], own_half[0]);
            v[r + 8][0] = trade<0x124, 0xa>(other[0], other[1]);
            v[r + 12][0] = trade<0x12c, 0x5>(other[1], other[0]);
        }
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        u4_t f[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int d = 0; d < 4; ++d)
                f[c][d] = __builtin_amdgcn_perm(v[h * 8 + 2 * d + 1][c / 2], v[h * 8 + 2 * d][c / 2], c % 2 ? 0x07060302u : 0x05040100u);
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            const u4_t a = *(const u4_t *)(own + m * 2048 + from[h]);
#pragma unroll
            for (int c = 0; c < NC; ++c) acc[m][c] = mfma(a, f[c], acc[m][c]);
        }
    }
}

extern "C" __global__ __launch_bounds__(NW * 64, (NW + 3) / 4) void ms_kernel(const in_t *__restrict__ A, const in_t *__restrict__ B, const void *, out_t *__restrict__ Y, int)
{
    __shared__ __attribute__((aligned(16))) char lds[FR_LDS];
    const int inst = blockIdx.z * gridDim.y + blockIdx.y;
    // tiles of one XCD follow each other, those of the same columns first: they share lines of B in its L2
    const int xcd = blockIdx.x % 8, tile = xcd * (TILES / 8) + (xcd < TILES % 8 ? xcd : TILES % 8) + blockIdx.x / 8;
    const int rt = tile % RT, ct = tile / RT;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64, l = lane % 16, q = lane / 16;
    A += (size_t)inst * A_INST + (unsigned)(rt * R * SA_I);
    B += (size_t)inst * B_INST + (unsigned)(ct * C);
    Y += (size_t)inst * DIM_M * DIM_N;
    const int row = lane / 8, chunk = lane % 8 ^ row, t = l / UL, u = l % UL;
    const in_t *a = A + (unsigned)(row * SA_I + chunk * 8), *b = B + ((unsigned)(q * 16 + t * 2 * NC) * (unsigned)SB_K + u * 8);
    char *own = lds + wave * MT * 2048;
    // where a lane's fragments start, opaque: stores and loads of the exchange then stay in order for the compiler too.  (A fence with a barrier
    // of the wavefront orders all loads along with them: 48 x 4096 x 2048 7.08 us, 6.90 so; 32 x 5824 x 1792 6.37 and 6.04.)
    int fragments[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        fragments[h] = l * 128 + ((2 * q + h) ^ (l % 8)) * 16;
        asm("" : "+v"(fragments[h]));
    }
    const int lo = wave * KB / NW, n = (wave + 1) * KB / NW - lo;
    const int turn = n ? ct % n : 0; // columns start at different blocks of A: 48 x 4096 x 2048 7.7 us without, 6.9
    f4_t acc[MT][NC];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int c = 0; c < NC; ++c) acc[m][c] = f4_t{0, 0, 0, 0};
    block x[D];
    auto at = [&](int s) __attribute__((always_inline)) {
        const int k = lo + s + turn - (s + turn < n ? 0 : n);
        return k < KB ? k : 0; // a step past the last one multiplies nothing
    };
#pragma unroll
    for (int d = 0; d < D; ++d) request(x[d], a, b, at(d));
    constexpr int MAIN = (PER / D - 1) * D, TAIL = PER - MAIN;
    for (int s = 0; s < MAIN; s += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            multiply(x[d], own, lane, fragments, acc);
            request(x[d], a, b, at(s + d + D));
        }
    }
#pragma unroll
    for (int e = 0; e < TAIL; ++e) {
        if (KB % NW == 0 || e < TAIL - 1 || n == PER) multiply(x[e % D], own, lane, fragments, acc);
        if (e + D < TAIL) request(x[e % D], a, b, at(MAIN + e + D));
    }
    // partial sums of the wavefronts, groups of NC columns
    typedef vec_t<float, NC> sum_t;
    sum_t *part = (sum_t *)lds;
#pragma unroll
    for (int p = 0; p < MT / G; ++p) {
        __syncthreads();
#pragma unroll
        for (int m = 0; m < G; ++m)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                sum_t v;
#pragma unroll
                for (int c = 0; c < NC; ++c) v.v[c] = acc[p * G + m][c][r];
                part[((wave * G + m) * 4 + r) * 64 + lane] = v;
            }
        __syncthreads();
        // rows 4 q + r of tile m
        for (int s = wave; s < G * 4; s += NW) {
            sum_t y = part[s * 64 + lane];
#pragma unroll
            for (int w = 1; w < NW; ++w) {
                const sum_t v = part[(w * G * 4 + s) * 64 + lane];
#pragma unroll
                for (int c = 0; c < NC; ++c) y.v[c] += v.v[c];
            }
            vec_t<out_t, NC> o;
#pragma unroll
            for (int c = 0; c < NC; ++c) o.v[c] = from_acc(y.v[c]);
            const int row = rt * R + (p * G + s / 4) * 16 + q * 4 + s % 4;
            *(vec_t<out_t, NC> *)(Y + (size_t)row * DIM_N + ct * C + u * 8 + t * NC) = o;
        }
    }
}
