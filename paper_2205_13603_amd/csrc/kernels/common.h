// Shared by every kernel template (spliced in before run-time compilation).
// Everything that depends on the schedule arrives as a -D constant.

#define DT_F32 0
#define DT_F16 1
#define DT_BF16 2
#define DT_I8 3
#define DT_I32 4
#define DT_F8E4M3 5 // input of the matrix-core kernels only: bit patterns, never converted in software

typedef _Float16 half_t;

template <int DT> struct dt_traits;
template <> struct dt_traits<DT_F32> { typedef float type; };
template <> struct dt_traits<DT_F16> { typedef half_t type; };
template <> struct dt_traits<DT_BF16> { typedef unsigned short type; };
template <> struct dt_traits<DT_I8> { typedef signed char type; };
template <> struct dt_traits<DT_I32> { typedef int type; };
template <> struct dt_traits<DT_F8E4M3> { typedef unsigned char type; };

typedef dt_traits<IN_DT>::type in_t;
typedef dt_traits<OUT_DT>::type out_t;

#if IN_DT == DT_I8
typedef int acc_t;
#else
typedef float acc_t;
#endif

// A naturally aligned group of N elements: loads and stores of it become one
// memory instruction of N*sizeof(T) bytes.
template <typename T, int N> struct __attribute__((aligned(sizeof(T) * N))) vec_t {
    T v[N];
};

__device__ __forceinline__ float bf16_to_float(unsigned short b) { return __uint_as_float((unsigned)b << 16); }

// round to nearest even; NaN stays NaN.  The conversion is the hardware's (one instruction per pair of values):
// spelled out in integer arithmetic with its NaN test it costs a branch per element, and an epilogue of 128
// values per lane then shows in the run time of a tile
__device__ __forceinline__ unsigned short float_to_bf16(float f) { return __builtin_bit_cast(unsigned short, (__bf16)f); }

__device__ __forceinline__ acc_t to_acc(in_t x)
{
#if IN_DT == DT_BF16
    return bf16_to_float(x);
#else
    return (acc_t)x;
#endif
}

// the single rounding from the accumulator to the output type
__device__ __forceinline__ out_t from_acc(acc_t x)
{
#if OUT_DT == DT_BF16
    return float_to_bf16(x);
#else
    return (out_t)x;
#endif
}

#if defined(RELU) && (OUT_DT == DT_F16 || OUT_DT == DT_BF16)
// ReLU and the one rounding of two sums
__device__ __forceinline__ unsigned finish(float x, float y)
{
#if OUT_DT == DT_F16
    // the rounding keeps signs: ReLU on the rounded pair is ReLU ahead of the rounding (NaN becomes 0 either way)
    typedef _Float16 h2_t __attribute__((ext_vector_type(2)));
    typedef float f2_t __attribute__((ext_vector_type(2)));
    h2_t v = __builtin_convertvector((f2_t{x, y}), h2_t);
#if RELU
    v = __builtin_elementwise_max(v, h2_t{0, 0});
#endif
    return __builtin_bit_cast(unsigned, v);
#else
#if RELU
    // the middle of (v, 0, infinity), one instruction (NaN becomes 0); a maximum would first quiet v
    x = __builtin_amdgcn_fmed3f(x, 0.f, __builtin_inff());
    y = __builtin_amdgcn_fmed3f(y, 0.f, __builtin_inff());
#endif
    typedef __bf16 b2_t __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(unsigned, (b2_t{(__bf16)x, (__bf16)y}));
#endif
}
#endif

// Hardware deals workgroups to the XCDs in turn, XCD f % 8 gets workgroup f.  The place of f in an order in which each XCD receives
// runs of neighbours: of RUN workgroups, the last eight runs as long as each other but for one; RUN 0: one run for each XCD.
template <unsigned RUN> __device__ __forceinline__ unsigned xcd_run(unsigned f, unsigned total)
{
    unsigned from = 0, part = total;
    if (RUN) {
        from = f / (RUN * 8) * (RUN * 8);
        part = total - from < RUN * 8 ? total - from : RUN * 8;
    }
    const unsigned at = f - from, xcd = at % 8, left = part % 8;
    return from + xcd * (part / 8) + (xcd < left ? xcd : left) + at / 8;
}

#ifdef I0 // kernels built from the factors of a trace
// Workgroup -> (z, i0, j0): z = instance * batch + batch index, (i0, j0) = the two outer spatial loops.
// REORDER 0: i outer.  1: j outer.  2: i outer, after a permutation of the launch-wide workgroup
// id that undoes the round-robin of workgroups over the 8 XCDs: the hardware sends workgroup f
// (x fastest, then y, z) to XCD f mod 8, so id (f mod 8) * (total / 8) + f / 8 makes the workgroups
// one XCD receives consecutive in (z, i0, j0) order; tiles that share operand panels, and whole
// instances, then sit behind one L2.
// Batched products whose rows are split into several tiles do so under REORDER 0 and 1 too where the launch writes more than the L2s
// hold: tiles whose rows are no whole lines then join them in one L2, and tiles of one product find its operands there
// (12 x 416 x 416 x 128 x 71 in fp16: 139 -> 124 us; 16 x 432 x 432 x 32 x 42 in bf16: 81 -> 65; 8 x 448 x 128 x 448 x 75: 118 -> 100).  Launches below lose a little to
// the arithmetic (12 x 384 x 384 x 32 x 2: 4.1 and 4.4); tiles of whole rows lose to the order (8 x 320 x 32 x 320, 233 instances: 99.9 in that
// of launch, 106.7; 19 of 21 such sizes by 0.4 to 6 %).
// RFACTOR > 1 (matrix-core kernels): RFACTOR consecutive workgroups share one output tile, workgroup ks
// of them reduces over the ks-th run of k0 steps.
#ifndef RFACTOR
#define RFACTOR 1
#endif
__device__ __forceinline__ void block_to_tile(int &z, int &i0, int &j0, int &ks)
{
    constexpr int G = I0 * J0 * RFACTOR;
    int wg = blockIdx.x;
    z = blockIdx.z * gridDim.y + blockIdx.y;
#if defined(DIM_B) && !IS_CONV
    constexpr bool JOIN = REORDER < 2 && DIM_B > 1 && J0 > 1;
#else
    constexpr bool JOIN = false;
#endif
    if constexpr (REORDER >= 2 || JOIN) {
        const int nz = gridDim.y * gridDim.z;
        const long total = (long)G * nz;
        bool permute = total % 8 == 0;
#if defined(DIM_B) && !IS_CONV
        if (JOIN) permute = permute && nz >= (32l << 20) / ((long)DIM_M * DIM_N * (int)sizeof(out_t));
#endif
        if (permute) {
            const long f = wg + (long)G * z;
            const long g = (f % 8) * (total / 8) + f / 8;
            wg = (int)(g % G);
            z = (int)(g / G);
        }
    }
    ks = wg % RFACTOR;
    wg /= RFACTOR;
#if REORDER == 1
    j0 = wg / I0;
    i0 = wg % I0;
#else
    i0 = wg / J0;
    j0 = wg % J0;
#endif
}
#endif

// A value of 2, 4, 8 or 16 bytes to global memory past the caches' replacement order: results that nothing on this compute unit
// reads again.  A launch whose stores stay in the L2s writes them back at its end, when nothing else runs any more.
// `dst` need only be aligned to 2 bytes: the hardware stores vectors at any address.
template <class T> __device__ __forceinline__ void store_stream(void *dst, const T &v)
{
    typedef unsigned u4 __attribute__((ext_vector_type(4), aligned(2)));
    typedef unsigned u2 __attribute__((ext_vector_type(2), aligned(2)));
    typedef unsigned u1 __attribute__((aligned(2)));
    static_assert(sizeof(T) == 2 || sizeof(T) == 4 || sizeof(T) == 8 || sizeof(T) == 16, "one memory instruction");
    if constexpr (sizeof(T) == 16) __builtin_nontemporal_store(__builtin_bit_cast(u4, v), reinterpret_cast<u4 *>(dst));
    else if constexpr (sizeof(T) == 8) __builtin_nontemporal_store(__builtin_bit_cast(u2, v), reinterpret_cast<u2 *>(dst));
    else if constexpr (sizeof(T) == 4) __builtin_nontemporal_store(__builtin_bit_cast(unsigned, v), reinterpret_cast<u1 *>(dst));
    else __builtin_nontemporal_store(__builtin_bit_cast(unsigned short, v), reinterpret_cast<unsigned short *>(dst));
}
// From how many instances on a launch writes so much that streaming pays: one L2's worth.  Below, the write-back at the end costs
// nothing and the caches join the pieces of a line (softmax 896 x 1456 in bf16: 3.40 us, 3.48 streamed; 16 x 64 x 64 scores x 3:
// 2.25, 2.45).
constexpr int stream_from(long bytes_per_instance) { return (int)(((4l << 20) + bytes_per_instance - 1) / bytes_per_instance); }

// ---- loads straight into LDS
//
// 16 bytes per lane from `base` (wave-uniform) + `voff` to `dst` (wave-uniform) + 16 * lane.  Written as assembly so that the
// compiler does not see a write to LDS: before every LDS read behind the builtin it waits until all such loads have landed
// (one s_waitcnt vmcnt(0) per k step, which drains the ring).  No register is written; the landing of a load is waited for by
// count (DL_WAIT_VM) and published by a barrier.  M0 holds the LDS address.
// A scalar register that a vector instruction has written (v_readfirstlane, or v_readlane where the compiler spilled it) takes
// five wait states before a vector-memory instruction may read it.  The compiler keeps this rule for its own loads but does not
// see one inside the asm, so the asm keeps it: a plain load reads a copy made by the scalar unit, which no rule delays, and a
// gather spends the wait on its own index arithmetic (bf16 4096^3: 97.1 us, 98.6 with s_nop 3 instead, 96.4 without any wait;
// transposed 16 x 16 x 256 -> 128, 4 x 4, batch 64: 20.6, 21.0, 20.5).  M0 takes one wait state before the load.
// Operands of the loads below that have to sit in scalar registers: equal in all lanes by construction, but the compiler keeps
// some of them (a base chosen by a wave's number, an LDS address of a deep ring) in vector registers and then rejects the asm.
__device__ __forceinline__ unsigned uniform(unsigned x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ unsigned long uniform(const char *p)
{
    const unsigned long a = (unsigned long)p;
    return (unsigned long)uniform((unsigned)(a >> 32)) << 32 | uniform((unsigned)a);
}
__device__ __forceinline__ unsigned lds_address(const char *p) { return uniform((unsigned)(size_t)(const __attribute__((address_space(3))) char *)p); }
__device__ __forceinline__ void load_lds16_to(const char *base, unsigned voff, unsigned dst)
{
    unsigned long copy;
    asm volatile("s_mov_b32 m0, %1\n\ts_mov_b64 %0, %3\n\tglobal_load_lds_dwordx4 %2, %0"
                 : "=&s"(copy) : "s"(dst), "v"(voff), "s"(uniform(base)) : "memory", "m0");
}
__device__ __forceinline__ void load_lds16(const char *base, unsigned voff, const char *dst) { load_lds16_to(base, voff, lds_address(dst)); }

// The same from a buffer at `base`: `voff` per lane, `soff` wave-uniform.  Lanes that ask for OUTSIDE write zeros (a range-checked
// load beyond the buffer returns zero, into LDS too).
constexpr unsigned OUTSIDE = 0x80000000u;
typedef unsigned rsrc_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ rsrc_t buffer_at(const char *base, unsigned bytes = 0x7ffffff0u)
{
    const unsigned long b = uniform(base);
    return {(unsigned)b, (unsigned)(b >> 32) & 0xffffu, uniform(bytes), 0x00020000u};
}
typedef __attribute__((address_space(3))) char lds_char;
__device__ __forceinline__ void gather_lds16(const rsrc_t &buffer, unsigned voff, const lds_char *dst)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                 : : "s"(uniform((unsigned)(size_t)dst)), "v"(voff), "s"(buffer) : "memory", "m0");
}
__device__ __forceinline__ void gather_lds16(const char *base, unsigned voff, unsigned soff, const char *dst)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 : : "s"(lds_address(dst)), "v"(voff), "s"(buffer_at(base)), "s"(uniform(soff)) : "memory", "m0");
}
// voff where all bits of `want` are set in `have`, else OUTSIDE.  A mask in VCC takes two wait states before it is read.
__device__ __forceinline__ void gather_lds16(const char *base, unsigned voff, unsigned have, unsigned want, unsigned soff, const char *dst)
{
    unsigned at;
    asm volatile("s_mov_b32 m0, %1\n\tv_and_b32 %0, %3, %4\n\tv_cmp_eq_u32 vcc, %0, %4\n\tv_mov_b32 %0, 0x80000000\n\t"
                 "s_nop 0\n\tv_cndmask_b32 %0, %0, %2, vcc\n\tbuffer_load_dwordx4 %0, %5, %6 offen lds"
                 : "=&v"(at) : "s"(lds_address(dst)), "v"(voff), "v"(have), "v"(want), "s"(buffer_at(base)), "s"(uniform(soff)) : "memory", "m0", "vcc");
}
// wait until at most `n` of this wavefront's vector-memory operations are outstanding
#define DL_WAIT_VM(n) __builtin_amdgcn_s_waitcnt((((n) & 15) | (((n) >> 4) << 14) | (7 << 4) | (15 << 8)))
