// Exercises variant handles and launches (ms_runtime.cpp) on the CPU, under -fsanitize=address,undefined: the HIP calls are
// replaced by a bookkeeping of which device holds which module, the compiler by an empty code object.  What it checks is
// when a call builds, loads or unloads a kernel.  Exit status 0 = every check held.
#include "../../paper_2205_13603_amd/csrc/ms_internal.h"

#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <set>
#include <string>

#define CHECK(x)                                                               \
    do {                                                                       \
        if (!(x)) {                                                            \
            fprintf(stderr, "%s:%d: CHECK failed: %s (last error: %s)\n", __FILE__, __LINE__, #x, ms_last_error()); \
            exit(1);                                                           \
        }                                                                      \
    } while (0)

static int g_device, g_compiled, g_moved, g_launched; // moved: modules loaded or unloaded
static std::set<std::pair<void *, int>> g_modules;   // and the device each is on
static char g_workspace[256];

namespace ms {
int32_t jit_get_code(const KernelSpec &, uint64_t, std::vector<char> **out)
{
    static std::vector<char> code(16);
    ++g_compiled;
    *out = &code;
    return MS_OK;
}
} // namespace ms

extern "C" {
hipError_t hipGetDevice(int *d) { return *d = g_device, hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t *p, int)
{
    memset(p, 0, sizeof *p);
    strcpy(p->gcnArchName, "gfx950");
    p->sharedMemPerBlock = 160 << 10;
    p->multiProcessorCount = 256;
    return hipSuccess;
}
hipError_t hipModuleLoadData(hipModule_t *m, const void *)
{
    *m = (hipModule_t)malloc(1);
    g_modules.insert({*m, g_device});
    ++g_moved;
    return hipSuccess;
}
hipError_t hipModuleUnload(hipModule_t m)
{
    for (int d = 0; d < 2; ++d) g_modules.erase({m, d});
    free(m);
    ++g_moved;
    return hipSuccess;
}
// the module itself stands for its functions
hipError_t hipModuleGetFunction(hipFunction_t *f, hipModule_t m, const char *) { return *f = (hipFunction_t)m, hipSuccess; }
hipError_t hipModuleLaunchKernel(hipFunction_t f, unsigned, unsigned, unsigned, unsigned, unsigned, unsigned, unsigned, hipStream_t, void **, void **)
{
    CHECK(g_modules.count({(void *)f, g_device})); // a kernel of a module that is loaded on this device
    ++g_launched;
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *) { return *p = g_workspace, hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *) { return hipErrorUnknown; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipErrorUnknown; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipErrorUnknown; }
hipError_t hipEventElapsedTime(float *, hipEvent_t, hipEvent_t) { return hipErrorUnknown; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipErrorUnknown; }
hipError_t hipGetLastError(void) { return hipErrorUnknown; }
hipError_t hipDeviceGetAttribute(int *, hipDeviceAttribute_t, int) { return hipErrorUnknown; }
const char *hipGetErrorString(hipError_t) { return "stub"; }
}

static bool two_kernels(ms_variant *v)
{
    int32_t one = 0, many = 0;
    CHECK(ms_variant_launch_shape(v, 1, nullptr, &one, nullptr) == MS_OK && ms_variant_launch_shape(v, 64, nullptr, &many, nullptr) == MS_OK);
    return one != many;
}

// a variant on `body` and, for products, with another kernel for one instance than for many
static ms_variant *build(const ms_op_desc &d, int32_t body)
{
    ms_op *op = nullptr;
    ms_space space;
    ms_variant *v = nullptr;
    CHECK(ms_op_create(&d, &op) == MS_OK && ms_space_describe(op, MS_SPACE_DEFAULT, &space) == MS_OK);
    for (int n = 0; n < 4000 && !v; ++n) {
        ms_trace t;
        ms_variant_params p;
        if (ms_trace_sample_valid(op, &space, 5, n, 1000, &t) == MS_OK && ms_trace_validate(op, &space, &t, &p) == MS_OK && p.body == body)
            CHECK(ms_variant_build(op, &space, &t, &v) == MS_OK);
        if (v && body == MS_BODY_DOUBLE_STEPS && !two_kernels(v)) {
            ms_variant_destroy(v);
            v = nullptr;
        }
    }
    CHECK(v);
    ms_op_destroy(op);
    return v;
}

int main()
{
    alignas(16) char tensor[64];
    const void *aligned[3] = {tensor, tensor, tensor}, *off[3] = {tensor + 2, tensor, tensor};
    void *out[1] = {tensor};
    int moved, compiled, launched;

    // ---- a product with a kernel of its own for few tiles
    ms_op_desc d;
    memset(&d, 0, sizeof d);
    d.kind = MS_OP_GEMM;
    d.in_dtype = d.out_dtype = MS_F16;
    d.dims[0] = d.dims[1] = d.dims[2] = 1024;
    ms_variant *v = build(d, MS_BODY_DOUBLE_STEPS);
    CHECK(ms_variant_launch_static(v, aligned, out, 1, nullptr) == MS_ERR_BAD_ARG); // not prepared
    CHECK(ms_variant_prepare(v) == MS_OK);
    moved = g_moved;
    for (int32_t n : {1, 64}) CHECK(ms_variant_launch_static(v, aligned, out, n, nullptr) == MS_OK);
    CHECK(g_moved == moved);
    // a launch on another device may load there, a static launch back here may not
    for (int32_t n : {1, 64}) {
        g_device = 1;
        CHECK(ms_variant_launch(v, aligned, out, nullptr, n, nullptr) == MS_OK);
        g_device = 0;
        moved = g_moved;
        launched = g_launched;
        for (int32_t m : {1, 64}) {
            const int32_t rc = ms_variant_launch_static(v, aligned, out, m, nullptr);
            CHECK(rc == MS_OK || rc == MS_ERR_BAD_ARG);
            CHECK(g_launched - launched == (rc == MS_OK));
            CHECK(g_moved == moved);
            launched = g_launched;
        }
        // set-up on the device again, and both kernels are there again
        CHECK(ms_variant_prepare(v) == MS_OK);
        moved = g_moved;
        for (int32_t m : {1, 64}) CHECK(ms_variant_launch_static(v, aligned, out, m, nullptr) == MS_OK);
        CHECK(g_moved == moved);
    }
    ms_variant_destroy(v);
    // the first launch on a device loads all a later one of any number of instances needs
    v = build(d, MS_BODY_DOUBLE_STEPS);
    CHECK(ms_variant_launch(v, aligned, out, nullptr, 1, nullptr) == MS_OK);
    moved = g_moved;
    CHECK(ms_variant_launch(v, aligned, out, nullptr, 64, nullptr) == MS_OK && ms_variant_launch(v, aligned, out, nullptr, 1, nullptr) == MS_OK);
    CHECK(g_moved == moved);
    ms_variant_destroy(v);

    // ---- a gathered convolution: operands off 16-byte boundaries run the nest
    memset(&d, 0, sizeof d);
    d.kind = MS_OP_CONV2D_NHWC;
    d.in_dtype = d.out_dtype = MS_F16;
    d.stride = d.pad = d.has_bias = 1;
    d.dims[0] = 8;
    d.dims[1] = d.dims[2] = 16;
    d.dims[3] = 64;
    d.dims[4] = 128;
    d.dims[5] = d.dims[6] = 3;
    v = build(d, MS_BODY_CONV_STEPS);
    CHECK(ms_variant_launch(v, aligned, out, nullptr, 1, nullptr) == MS_OK);
    moved = g_moved;
    compiled = g_compiled;
    CHECK(ms_variant_launch_static(v, off, out, 1, nullptr) == MS_ERR_BAD_ARG); // the nest is not there yet
    CHECK(g_moved == moved && g_compiled == compiled);
    CHECK(ms_variant_prepare(v) == MS_OK);
    moved = g_moved;
    compiled = g_compiled;
    CHECK(ms_variant_launch_static(v, off, out, 1, nullptr) == MS_OK && ms_variant_launch_static(v, aligned, out, 1, nullptr) == MS_OK);
    CHECK(g_moved == moved && g_compiled == compiled);
    g_device = 1;
    CHECK(ms_variant_launch(v, off, out, nullptr, 1, nullptr) == MS_OK);
    g_device = 0;
    moved = g_moved;
    CHECK(ms_variant_launch_static(v, off, out, 1, nullptr) == MS_ERR_BAD_ARG && ms_variant_launch_static(v, aligned, out, 1, nullptr) == MS_OK);
    CHECK(g_moved == moved);
    ms_variant_destroy(v);
    CHECK(g_modules.empty());
    printf("launch checks ok\n");
    return 0;
}
