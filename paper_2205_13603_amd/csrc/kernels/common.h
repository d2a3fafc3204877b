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

#ifdef I0 // kernels built from the factors of a trace
// Workgroup -> (z, i0, j0): z = instance * batch + batch index, (i0, j0) = the two outer spatial loops.
// REORDER 0: i outer.  1: j outer.  2: i outer, after a permutation of the launch-wide workgroup
// id that undoes the round-robin of workgroups over the 8 XCDs: the hardware sends workgroup f
// (x fastest, then y, z) to XCD f mod 8, so id (f mod 8) * (total / 8) + f / 8 makes the workgroups
// one XCD receives consecutive in (z, i0, j0) order; tiles that share operand panels, and whole
// instances, then sit behind one L2.
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
#if REORDER >= 2
    const int nz = gridDim.y * gridDim.z;
    const long total = (long)G * nz;
    if (total % 8 == 0) {
        const long f = wg + (long)G * z;
        const long g = (f % 8) * (total / 8) + f / 8;
        wg = (int)(g % G);
        z = (int)(g / G);
    }
#endif
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
