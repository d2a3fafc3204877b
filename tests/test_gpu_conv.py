"""GPU parity of implicit-GEMM conv2d + bias + ReLU (config C3) against the CPU oracle."""
import numpy as np
import pytest

from oracle import compare, oracle as O
from paper_2205_13603_amd import binding as B, inputs as I
from gpu_util import run_variant, run_variant_distinct, run_variant_offset
from test_gpu_gemm_mfma import traces_covering_intrinsics, F16_INTRINS

pytestmark = pytest.mark.gpu


def test_c3_conv_bias_relu():
    """Config C3: 1x56x56x64 -> 64, 3x3 s1 p1, bias + ReLU, fp16 in/out, fp32 accumulate."""
    X, W, bias = I.c3(seed=0)
    ref = O.conv2d_nhwc(X, W, bias=bias, relu=True, stride=1, pad=1)
    assert (ref == 0).mean() > 0.05, "ReLU must be active on part of the output"
    op = B.conv2d_op(1, 56, 56, 64, 64, 3, 3, stride=1, pad=1)
    space = op.space()
    for n, t in enumerate(traces_covering_intrinsics(op, space, 0, 4, F16_INTRINS)):
        print("trace", n, t.decisions(), flush=True)
        got = run_variant(op, space, t, [X, W, bias], "f16", (1, 56, 56, 64))
        if got is None:
            continue
        compare.assert_float_close(got, ref, compare.RTOL_HALF, "C3 trace %d" % n)


@pytest.mark.parametrize("stride,pad,k,relu,has_bias", [(2, 1, 3, True, True), (1, 0, 1, False, False), (2, 3, 7, True, True),
                                                       (1, 2, 5, False, True)])
def test_conv_other_geometries_exact(stride, pad, k, relu, has_bias):
    """Strides, paddings and kernel sizes beyond C3; batch 2; 2 instances; integer-valued inputs make
    the fp32 accumulation exact, so the fp32 output must equal the oracle exactly."""
    N, H, W_, Cin, Cout = 2, 17, 16, 16, 32
    g = I.rng(11)
    X = I.small_ints(g, (N, H, W_, Cin), -2, 2, "f16")
    Wt = I.small_ints(g, (k, k, Cin, Cout), -2, 2, "f16")
    bias = g.integers(-3, 4, size=Cout).astype(np.float32) if has_bias else None
    ref = O.conv2d_nhwc(X, Wt, bias=bias, relu=relu, stride=stride, pad=pad)
    OH, OW = ref.shape[1], ref.shape[2]
    if (N * OH * OW) % 16:
        pytest.skip("M = %d output pixels is not a multiple of the 16-row intrinsic" % (N * OH * OW))
    op = B.conv2d_op(N, H, W_, Cin, Cout, k, k, stride=stride, pad=pad, has_bias=has_bias, relu=relu, out_dtype="f32")
    space = op.space()
    ins = [X, Wt] + ([bias] if has_bias else [])
    for n in range(6):
        t = B.trace_sample_valid(op, space, 12, n)
        print("trace", n, t.decisions(), flush=True)
        got = run_variant(op, space, t, ins, "f32", (N, OH, OW, Cout), instances=2)
        if got is None:
            continue
        assert np.array_equal(got[0], ref) and np.array_equal(got[1], ref), "trace %d" % n


def test_conv_instances_with_distinct_inputs():
    """Three instances, each with its own activations, weights and bias (every input is per instance)."""
    ins = [list(I.c3(seed=s, H=14, W=16, Cin=16, Cout=32)) for s in (1, 2, 3)]
    refs = [O.conv2d_nhwc(x, w, bias=b, relu=True, stride=1, pad=1) for x, w, b in ins]
    op = B.conv2d_op(1, 14, 16, 16, 32, 3, 3, stride=1, pad=1)
    space = op.space()
    for n in range(5):
        t = B.trace_sample_valid(op, space, 13, n)
        print("trace", n, t.decisions(), flush=True)
        got = run_variant_distinct(op, space, t, ins, "f16", (1, 14, 16, 32))
        if got is None:
            continue
        for r in range(3):
            compare.assert_float_close(got[r], refs[r], compare.RTOL_HALF, "instance %d trace %d" % (r, n))


def _traces_with_resident_patch(op, space, seed, count, compute_at=1, max_index=1500):
    """Sampled valid traces with the given compute-location decision: 1 = the input patch of a tile is resident
    in LDS, 2 = also the weights, under persistent workgroups."""
    out = []
    for idx in range(max_index):
        if len(out) == count:
            break
        t = B.trace_sample_valid(op, space, seed, idx)
        if B.trace_validate(op, space, t).compute_at == compute_at:
            out.append(t)
    return out


@pytest.mark.parametrize("compute_at", [1, 2, 3, 4])
def test_c3_conv_resident_patch(compute_at):
    """C3 with the cache-read of X under the workgroup tile loop (sample-compute-location = tile), with the
    weights resident as well (2), with helper wavefronts (3), and with the weights in registers (4): row-aligned tiles and tiles that start in the
    middle of an output row."""
    X, W, bias = I.c3(seed=3)
    ref = O.conv2d_nhwc(X, W, bias=bias, relu=True, stride=1, pad=1)
    op = B.conv2d_op(1, 56, 56, 64, 64, 3, 3, stride=1, pad=1)
    space = op.space()
    traces = _traces_with_resident_patch(op, space, 21, 6, compute_at)
    assert len(traces) == 6
    aligned = [B.trace_validate(op, space, t).block_m % 56 == 0 for t in traces]
    print("row-aligned tiles:", aligned, flush=True)
    for n, t in enumerate(traces):
        print("trace", n, t.decisions(), flush=True)
        got = run_variant(op, space, t, [X, W, bias], "f16", (1, 56, 56, 64))
        if got is None:
            continue
        compare.assert_float_close(got, ref, compare.RTOL_HALF, "C3 compute_at %d, trace %d" % (compute_at, n))


@pytest.mark.parametrize("compute_at", [1, 2, 3, 4])
@pytest.mark.parametrize("stride,pad,k,H,W_", [(1, 1, 3, 16, 16), (2, 1, 3, 16, 32), (1, 0, 1, 8, 16), (2, 3, 7, 32, 16), (1, 2, 5, 12, 16)])
def test_conv_resident_patch_geometries_exact(stride, pad, k, H, W_, compute_at):
    """Resident input patch with other strides, paddings and filter sizes, batch 2, 2 instances with distinct
    data; integer-valued inputs make fp32 accumulation exact: the fp32 output must equal the oracle."""
    N, Cin, Cout = 2, 32, 32
    g = I.rng(17)
    ins, refs = [], []
    for r in range(2):
        X = I.small_ints(g, (N, H, W_, Cin), -2, 2, "f16")
        Wt = I.small_ints(g, (k, k, Cin, Cout), -2, 2, "f16")
        bias = g.integers(-3, 4, size=Cout).astype(np.float32)
        ins.append([X, Wt, bias])
        refs.append(O.conv2d_nhwc(X, Wt, bias=bias, relu=True, stride=stride, pad=pad))
    OH, OW = refs[0].shape[1], refs[0].shape[2]
    assert (OH * OW) % 16 == 0
    op = B.conv2d_op(N, H, W_, Cin, Cout, k, k, stride=stride, pad=pad, out_dtype="f32")
    space = op.space()
    traces = _traces_with_resident_patch(op, space, 5, 4, compute_at)
    assert traces, "no valid trace with compute_at %d" % compute_at
    for n, t in enumerate(traces):
        print("trace", n, t.decisions(), flush=True)
        got = run_variant_distinct(op, space, t, ins, "f32", (N, OH, OW, Cout))
        if got is None:
            continue
        for r in range(2):
            assert np.array_equal(got[r], refs[r]), "instance %d trace %d" % (r, n)


def test_conv_persistent_runs_cross_instances():
    """Resident weights under persistent workgroups, with more tiles than workgroups: every workgroup walks a
    run of consecutive tiles that crosses image and instance boundaries (weights reloaded, patch prefetched).
    600 instances of 5 distinct data sets in rotation; integer-valued inputs, fp32 output: exact equality."""
    N, H, W_, Cin, Cout, R = 2, 16, 16, 32, 32, 600
    g = I.rng(23)
    sets, refs = [], []
    for r in range(5):
        X = I.small_ints(g, (N, H, W_, Cin), -2, 2, "f16")
        Wt = I.small_ints(g, (3, 3, Cin, Cout), -2, 2, "f16")
        bias = g.integers(-3, 4, size=Cout).astype(np.float32)
        sets.append([X, Wt, bias])
        refs.append(O.conv2d_nhwc(X, Wt, bias=bias, relu=True, stride=1, pad=1))
    ins = [sets[r % 5] for r in range(R)]
    op = B.conv2d_op(N, H, W_, Cin, Cout, 3, 3, stride=1, pad=1, out_dtype="f32")
    space = op.space()
    for compute_at, cache_read in ((2, 1), (2, 2), (3, 2), (4, 1), (4, 2)):
        traces = [t for t in _traces_with_resident_patch(op, space, 9, 40, compute_at)
                  if B.trace_validate(op, space, t).cache_read == cache_read][:2]
        assert traces, "no valid trace with compute_at %d and cache_read %d" % (compute_at, cache_read)
        for n, t in enumerate(traces):
            p = B.trace_validate(op, space, t)
            tiles = p.grid[0] * R
            print("compute_at", compute_at, "cache_read", cache_read, "trace", n, t.decisions(), "tiles", tiles, flush=True)
            assert tiles > 4 * 256, "the launch must have several tiles per workgroup"
            got = run_variant_distinct(op, space, t, ins, "f32", (N, H, W_, Cout))
            if got is None:
                continue
            for r in range(R):
                assert np.array_equal(got[r], refs[r % 5]), "instance %d trace %d" % (r, n)


@pytest.mark.parametrize("stride,pad,k,dil,H,W_", [(1, 2, 3, 2, 16, 16), (2, 2, 3, 2, 16, 32), (1, 3, 2, 3, 13, 16), (1, 4, 3, 4, 16, 16)])
def test_dilated_conv_exact_for_every_compute_location(stride, pad, k, dil, H, W_):
    """Dilated conv2d (taps `dil` input elements apart; the paper's DIL workload in small): the im2col loader and
    all resident-patch modes, batch 2, 2 instances with distinct data, integer-valued inputs, fp32 output: exact."""
    N, Cin, Cout = 2, 32, 32
    g = I.rng(29)
    ins, refs = [], []
    for r in range(2):
        X = I.small_ints(g, (N, H, W_, Cin), -2, 2, "f16")
        Wt = I.small_ints(g, (k, k, Cin, Cout), -2, 2, "f16")
        bias = g.integers(-3, 4, size=Cout).astype(np.float32)
        ins.append([X, Wt, bias])
        refs.append(O.conv2d_nhwc(X, Wt, bias=bias, relu=True, stride=stride, pad=pad, dilation=dil))
    OH, OW = refs[0].shape[1], refs[0].shape[2]
    if (N * OH * OW) % 16:
        pytest.skip("M = %d output pixels is not a multiple of the 16-row intrinsic" % (N * OH * OW))
    op = B.conv2d_op(N, H, W_, Cin, Cout, k, k, stride=stride, pad=pad, out_dtype="f32", dilation=dil)
    space = op.space()
    assert op.loops()[0][1] == N * OH * OW
    ran = set()
    for compute_at in (0, 1, 2, 3, 4):
        for n, t in enumerate(_traces_with_resident_patch(op, space, 4, 2, compute_at)):
            print("compute_at", compute_at, "trace", n, t.decisions(), flush=True)
            ran.add(compute_at)
            got = run_variant_distinct(op, space, t, ins, "f32", (N, OH, OW, Cout))
            if got is None:
                continue
            for r in range(2):
                assert np.array_equal(got[r], refs[r]), "compute_at %d instance %d trace %d" % (compute_at, r, n)
    assert {0, 1, 2} <= ran


def test_conv_bf16_every_compute_location():
    """bf16 activations and weights (uint16 bit patterns on the host), fp32 accumulate, bf16 output: the same conv
    kernels with the bf16 intrinsics; 2 instances."""
    X, W, bias = I.c3(seed=5, H=28, W=28, Cin=32, Cout=64, dtype="bf16")
    ref = O.conv2d_nhwc(X, W, bias=bias, relu=True, stride=1, pad=1, bf16=True)
    op = B.conv2d_op(1, 28, 28, 32, 64, 3, 3, stride=1, pad=1, in_dtype="bf16")
    space = op.space()
    ran = set()
    for compute_at in (0, 1, 2, 3, 4):
        for n, t in enumerate(_traces_with_resident_patch(op, space, 6, 2, compute_at)):
            print("compute_at", compute_at, "trace", n, t.decisions(), flush=True)
            ran.add(compute_at)
            got = run_variant(op, space, t, [X, W, bias], "bf16", (1, 28, 28, 64), instances=2)
            if got is None:
                continue
            for r in range(2):
                compare.assert_float_close(got[r], ref, compare.RTOL_HALF, "bf16 conv, compute_at %d trace %d" % (compute_at, n))
    assert {0, 1, 2} <= ran


@pytest.mark.parametrize("Cin,k,stride,pad,H,W_", [(3, 7, 2, 3, 32, 32), (5, 3, 1, 1, 16, 16), (12, 3, 1, 1, 8, 16), (3, 1, 1, 0, 16, 16)])
def test_conv_reduction_extent_not_a_multiple_of_the_intrinsic(Cin, k, stride, pad, H, W_):
    """KH*KW*Cin = 147, 45, 108 and 3: the k split covers the extent rounded up to the intrinsic's k and both loaders
    deliver zeros beyond it (a first layer with 3 input channels is such an operator).  Integer-valued inputs: bit-equal
    to the oracle for every intrinsic that the space offers."""
    N, Cout = 1, 32
    g = I.rng(61)
    X = I.small_ints(g, (N, H, W_, Cin), -2, 2, "f16")
    Wt = I.small_ints(g, (k, k, Cin, Cout), -2, 2, "f16")
    bias = g.integers(-3, 4, size=Cout).astype(np.float32)
    ref = O.conv2d_nhwc(X, Wt, bias=bias, relu=True, stride=stride, pad=pad)
    OH, OW = ref.shape[1], ref.shape[2]
    op = B.conv2d_op(N, H, W_, Cin, Cout, k, k, stride=stride, pad=pad, out_dtype="f32")
    space = op.space()
    cands = [space.slots[0].candidates[i] for i in range(space.slots[0].n_candidates)]
    assert any((k * k * Cin) % (c % 100) for c in cands)
    want = {c: 2 for c in cands}
    idx = 0
    while any(want.values()) and idx < 400:
        t = B.trace_sample_valid(op, space, 62, idx)
        idx += 1
        p = B.trace_validate(op, space, t)
        if want.get(p.mfma, 0) == 0:
            continue
        want[p.mfma] -= 1
        assert p.compute_at == 0 or (k * k * Cin) % p.tile_unit[2] == 0
        print("trace", idx, t.decisions(), flush=True)
        got = run_variant(op, space, t, [X, Wt, bias], "f32", (N, OH, OW, Cout), instances=2)
        if got is None:
            continue
        assert np.array_equal(got[0], ref) and np.array_equal(got[1], ref), "trace %d" % idx
    assert not any(want.values()), want


def test_cbr_first_layer_224x224x3_7x7_stride_2():
    """The paper's CBR shape (Appendix A.2: 224 x 224 x 3 -> 64, 7 x 7, stride 2, padding 3), batch normalisation folded
    into weights and bias: U[0,1] input, N(0, 0.05) weights, fp16 output within the half-precision tolerance."""
    g = I.rng(63)
    X = I.uniform(g, (1, 224, 224, 3), 0.0, 1.0, "f16")
    Wt = I.normal(g, (7, 7, 3, 64), 0.05, "f16")
    bias = I.normal(g, (64,), 0.05, "f32")
    ref = O.conv2d_nhwc(X, Wt, bias=bias, relu=True, stride=2, pad=3)
    op = B.conv2d_op(1, 224, 224, 3, 64, 7, 7, stride=2, pad=3)
    space = op.space()
    for n in range(6):
        t = B.trace_sample_valid(op, space, 64, n)
        print("trace", n, t.decisions(), flush=True)
        got = run_variant(op, space, t, [X, Wt, bias], "f16", ref.shape)
        if got is None:
            continue
        compare.assert_float_close(got, ref, compare.RTOL_HALF, "CBR trace %d" % n)


@pytest.mark.parametrize("stride,pad,k,H,W_", [(2, 1, 4, 8, 8), (1, 0, 3, 6, 6), (2, 0, 2, 8, 4), (3, 2, 5, 6, 6), (1, 1, 3, 8, 16)])
def test_transposed_conv_exact(stride, pad, k, H, W_):
    """Transposed convolution (Appendix A.2: T2D): the kernels gather (output pixel <- the input pixels whose scattered
    filter reaches it), the oracle scatters.  Integer-valued inputs, batch 2, 2 instances: bit-equal fp32 outputs."""
    N, Cin, Cout = 2, 16, 32
    g = I.rng(71)
    X = I.small_ints(g, (N, H, W_, Cin), -2, 2, "f16")
    Wt = I.small_ints(g, (k, k, Cin, Cout), -2, 2, "f16")
    bias = g.integers(-3, 4, size=Cout).astype(np.float32)
    ref = O.conv2d_transposed_nhwc(X, Wt, bias=bias, relu=True, stride=stride, pad=pad)
    OH, OW = ref.shape[1], ref.shape[2]
    assert (OH, OW) == ((H - 1) * stride - 2 * pad + k, (W_ - 1) * stride - 2 * pad + k) and (N * OH * OW) % 16 == 0
    op = B.conv2d_transposed_op(N, H, W_, Cin, Cout, k, k, stride=stride, pad=pad, out_dtype="f32")
    space = op.space()
    for n in range(6):
        t = B.trace_sample_valid(op, space, 72, n)
        print("trace", n, t.decisions(), flush=True)
        got = run_variant(op, space, t, [X, Wt, bias], "f32", (N, OH, OW, Cout), instances=2)
        if got is None:
            continue
        assert np.array_equal(got[0], ref) and np.array_equal(got[1], ref), "trace %d" % n


@pytest.mark.parametrize("stride,pad,k,N,H,W_,flags", [(2, 1, 4, 2, 8, 8, 0xFF), (2, 0, 2, 1, 4, 8, 0x4FF), (4, 0, 4, 2, 8, 4, 0xFF),
                                                         (2, 2, 6, 2, 8, 4, 0x4FF), (3, 0, 3, 1, 8, 6, 0xFF)])
def test_transposed_conv_phases_exact(stride, pad, k, N, H, W_, flags):
    """Traces whose tiles keep to one phase of the output grid and whose k steps keep to one tap: the kernel walks that
    phase's taps only, and traces beside them that do not qualify walk all taps.  Integer-valued inputs, 2 instances:
    bit-equal fp32 outputs in every staging mode drawn."""
    Cin, Cout = 64, 32
    g = I.rng(75)
    X = I.small_ints(g, (N, H, W_, Cin), -2, 2, "f16")
    Wt = I.small_ints(g, (k, k, Cin, Cout), -2, 2, "f16")
    bias = g.integers(-3, 4, size=Cout).astype(np.float32)
    ref = O.conv2d_transposed_nhwc(X, Wt, bias=bias, relu=True, stride=stride, pad=pad)
    assert ref.shape[1:3] == (H * stride, W_ * stride)
    op = B.conv2d_transposed_op(N, H, W_, Cin, Cout, k, k, stride=stride, pad=pad, out_dtype="f32")
    space = op.space(flags)
    modes, plain = {}, 0
    for idx in range(3000):
        t = B.trace_sample_valid(op, space, 76, idx)
        p = B.trace_validate(op, space, t)
        if (N * H * W_) % p.block_m or Cin % p.block_k or p.tk[0] % (stride * stride * p.rfactor) or p.block_m < 32:
            if plain == 2 or p.block_m < 32:
                continue
            plain += 1
            assert "-DCV_PHASES=0" in B.variant_kernel_text(op, p)
            got = run_variant(op, space, t, [X, Wt, bias], "f32", ref.shape, instances=2)
            assert got is None or (np.array_equal(got[0], ref) and np.array_equal(got[1], ref)), "trace %d" % idx
            continue
        assert "-DCV_PHASES=1" in B.variant_kernel_text(op, p)
        mode = (p.cache_read, p.cache_write, p.rfactor > 1)
        if mode in modes:
            continue
        modes[mode] = True
        print("trace", idx, t.decisions(), flush=True)
        got = run_variant(op, space, t, [X, Wt, bias], "f32", ref.shape, instances=2)
        if got is None:
            continue
        assert np.array_equal(got[0], ref) and np.array_equal(got[1], ref), "trace %d" % idx
    assert plain == 2 and len({m[0] for m in modes}) >= 3 and (flags == 0xFF or any(m[2] for m in modes)), modes


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_t2d_config_transposed_conv_4x4x512(dtype):
    """The paper's T2D shape: 4 x 4 x 512 -> 8 x 8 x 256, 4 x 4 filter, stride 2, padding 1 (K = 8192)."""
    g = I.rng(73)
    X = I.normal(g, (1, 4, 4, 512), 1.0, dtype)
    Wt = I.normal(g, (4, 4, 512, 256), 0.05, dtype)
    bias = I.normal(g, (256,), 0.05, "f32")
    ref = O.conv2d_transposed_nhwc(X, Wt, bias=bias, relu=True, stride=2, pad=1, bf16=dtype == "bf16")
    assert ref.shape == (1, 8, 8, 256)
    op = B.conv2d_transposed_op(1, 4, 4, 512, 256, 4, 4, stride=2, pad=1, in_dtype=dtype)
    space = op.space()
    for n in range(6):
        t = B.trace_sample_valid(op, space, 74, n)
        print("trace", n, t.decisions(), flush=True)
        got = run_variant(op, space, t, [X, Wt, bias], dtype, ref.shape)
        if got is None:
            continue
        compare.assert_float_close(got, ref, compare.RTOL_HALF, "T2D %s trace %d" % (dtype, n))


@pytest.mark.parametrize("groups,Cin,Cout,k,stride,pad", [(4, 64, 128, 3, 2, 1), (2, 16, 64, 3, 1, 1), (8, 64, 128, 1, 1, 0), (3, 48, 96, 3, 1, 1)])
def test_grouped_conv_exact(groups, Cin, Cout, k, stride, pad):
    """Grouped convolution (Appendix A.2: GRP): a group is a batch entry of the implicit GEMM, reading its slice of the
    channels of X, its columns of W and the bias, and writing its slice of the channels of Y.  Integer-valued inputs,
    batch 2, 2 instances: bit-equal fp32 outputs."""
    N, H, W_ = 2, 16, 8
    g = I.rng(81)
    X = I.small_ints(g, (N, H, W_, Cin), -2, 2, "f16")
    Wt = I.small_ints(g, (k, k, Cin // groups, Cout), -2, 2, "f16")
    bias = g.integers(-3, 4, size=Cout).astype(np.float32)
    ref = O.conv2d_nhwc(X, Wt, bias=bias, relu=True, stride=stride, pad=pad, groups=groups)
    OH, OW = ref.shape[1], ref.shape[2]
    op = B.conv2d_op(N, H, W_, Cin, Cout, k, k, stride=stride, pad=pad, out_dtype="f32", groups=groups)
    space = op.space()
    seen = set()
    for n in range(16):
        t = B.trace_sample_valid(op, space, 82, n)
        seen.add(B.trace_validate(op, space, t).compute_at)
        print("trace", n, t.decisions(), flush=True)
        got = run_variant(op, space, t, [X, Wt, bias], "f32", (N, OH, OW, Cout), instances=2)
        if got is None:
            continue
        assert np.array_equal(got[0], ref) and np.array_equal(got[1], ref), "trace %d" % n


def test_grouped_conv_persistent_runs_cross_groups_and_instances():
    """Grouped convolution under the persistent compute locations: the tile list runs over instance x group, so a
    workgroup's run of tiles crosses group and instance boundaries (weights and bias slice change, the patch of the
    next group is prefetched).  200 instances of 5 distinct data sets in rotation, integer-valued inputs, fp32
    output: exact equality."""
    N, H, W_, Cin, Cout, G, R = 2, 16, 8, 64, 128, 4, 200
    g = I.rng(85)
    sets, refs = [], []
    for r in range(5):
        X = I.small_ints(g, (N, H, W_, Cin), -2, 2, "f16")
        Wt = I.small_ints(g, (3, 3, Cin // G, Cout), -2, 2, "f16")
        bias = g.integers(-3, 4, size=Cout).astype(np.float32)
        sets.append([X, Wt, bias])
        refs.append(O.conv2d_nhwc(X, Wt, bias=bias, relu=True, stride=1, pad=1, groups=G))
    ins = [sets[r % 5] for r in range(R)]
    op = B.conv2d_op(N, H, W_, Cin, Cout, 3, 3, stride=1, pad=1, out_dtype="f32", groups=G)
    space = op.space()
    for compute_at in (2, 3, 4):
        traces = _traces_with_resident_patch(op, space, 86, 2, compute_at)
        assert traces, "no valid trace with compute_at %d" % compute_at
        for n, t in enumerate(traces):
            p = B.trace_validate(op, space, t)
            tiles = p.grid[0] * p.grid[2] * R
            print("compute_at", compute_at, "trace", n, t.decisions(), "tiles", tiles, flush=True)
            assert p.grid[2] == G and tiles > 1024, "the launch must have more tiles than workgroups"
            got = run_variant_distinct(op, space, t, ins, "f32", (N, H, W_, Cout))
            if got is None:
                continue
            for r in range(R):
                assert np.array_equal(got[r], refs[r % 5]), "instance %d trace %d" % (r, n)


@pytest.mark.parametrize("stride,pad,k,L_", [(1, 1, 3, 32), (2, 2, 5, 64)])
def test_grouped_conv1d_exact(stride, pad, k, L_):
    """Grouped 1-D convolution: the group count of the conv1d descriptor on the conv2d kernels, every compute location
    the space offers.  Reference: the oracle's grouped conv2d on an image of height 1 with a 1 x K filter, whose output
    row that reads the image row (row pad / stride) is the 1-D result.  Integer-valued inputs, batch 2, 2 instances:
    bit-equal fp32 outputs."""
    N, Cin, Cout, G = 2, 64, 64, 4
    g = I.rng(93)
    X = I.small_ints(g, (N, L_, Cin), -2, 2, "f16")
    Wt = I.small_ints(g, (k, Cin // G, Cout), -2, 2, "f16")
    bias = g.integers(-3, 4, size=Cout).astype(np.float32)
    assert pad % stride == 0
    ref = O.conv2d_nhwc(X[:, None], Wt[None], bias=bias, relu=True, stride=stride, pad=pad, groups=G)[:, pad // stride]
    OL = ref.shape[1]
    op = B.conv1d_op(N, L_, Cin, Cout, k, stride=stride, pad=pad, out_dtype="f32", groups=G)
    assert op.loops()[0] == ("g", G, False)
    space = op.space()
    want = {0: 2, 1: 2, 2: 1, 3: 1, 4: 1}
    idx = 0
    while any(want.values()) and idx < 800:
        t = B.trace_sample_valid(op, space, 94, idx)
        idx += 1
        ca = B.trace_validate(op, space, t).compute_at
        if want[ca] == 0:
            continue
        want[ca] -= 1
        print("trace", idx, "compute_at", ca, t.decisions(), flush=True)
        got = run_variant(op, space, t, [X, Wt, bias], "f32", (N, OL, Cout), instances=2)
        if got is None:
            continue
        assert np.array_equal(got[0], ref) and np.array_equal(got[1], ref), "trace %d" % idx
    assert want[0] == 0 and want[1] == 0, want


def test_grp_config_grouped_conv_56x56x64_to_128():
    """The paper's GRP shape: 56 x 56 x 64 -> 28 x 28 x 128, 3 x 3, stride 2, padding 1, 4 groups; fp16."""
    g = I.rng(83)
    X = I.uniform(g, (1, 56, 56, 64), 0.0, 1.0, "f16")
    Wt = I.normal(g, (3, 3, 16, 128), 0.05, "f16")
    bias = I.normal(g, (128,), 0.05, "f32")
    ref = O.conv2d_nhwc(X, Wt, bias=bias, relu=True, stride=2, pad=1, groups=4)
    op = B.conv2d_op(1, 56, 56, 64, 128, 3, 3, stride=2, pad=1, groups=4)
    space = op.space()
    for n in range(8):
        t = B.trace_sample_valid(op, space, 84, n)
        print("trace", n, t.decisions(), flush=True)
        got = run_variant(op, space, t, [X, Wt, bias], "f16", ref.shape)
        if got is None:
            continue
        compare.assert_float_close(got, ref, compare.RTOL_HALF, "GRP trace %d" % n)


@pytest.mark.parametrize("stride,pad,k,dil,L_", [(2, 1, 3, 1, 64), (1, 0, 1, 1, 32), (1, 2, 5, 1, 48), (1, 2, 3, 2, 32), (1, 1, 3, 1, 16)])
def test_conv1d_exact_for_every_compute_location(stride, pad, k, dil, L_):
    """1-D convolution (Appendix A.2: C1D) on the conv2d kernels: an image of height 1, a 1 x K filter, padding at the
    two ends of the row only.  Integer-valued inputs, batch 2, 2 instances: bit-equal fp32 outputs; every cache-read
    location that the space offers is exercised."""
    N, Cin, Cout = 2, 32, 32
    g = I.rng(91)
    X = I.small_ints(g, (N, L_, Cin), -2, 2, "f16")
    Wt = I.small_ints(g, (k, Cin, Cout), -2, 2, "f16")
    bias = g.integers(-3, 4, size=Cout).astype(np.float32)
    ref = O.conv1d_nwc(X, Wt, bias=bias, relu=True, stride=stride, pad=pad, dilation=dil)
    OL = ref.shape[1]
    assert (N * OL) % 16 == 0
    op = B.conv1d_op(N, L_, Cin, Cout, k, stride=stride, pad=pad, out_dtype="f32", dilation=dil)
    space = op.space()
    want = {0: 2, 1: 2, 2: 1, 3: 1, 4: 1}
    idx = 0
    while any(want.values()) and idx < 600:
        t = B.trace_sample_valid(op, space, 92, idx)
        idx += 1
        ca = B.trace_validate(op, space, t).compute_at
        if want[ca] == 0:
            continue
        want[ca] -= 1
        print("trace", idx, "compute_at", ca, t.decisions(), flush=True)
        got = run_variant(op, space, t, [X, Wt, bias], "f32", (N, OL, Cout), instances=2)
        if got is None:
            continue
        assert np.array_equal(got[0], ref) and np.array_equal(got[1], ref), "trace %d" % idx
    assert want[0] == 0 and want[1] == 0, want


def test_c1d_config_conv1d_256x64_to_128():
    """The paper's C1D shape: length 256, 64 -> 128 channels, kernel 3, stride 2, padding 1; fp16."""
    g = I.rng(93)
    X = I.uniform(g, (1, 256, 64), 0.0, 1.0, "f16")
    Wt = I.normal(g, (3, 64, 128), 0.05, "f16")
    bias = I.normal(g, (128,), 0.05, "f32")
    ref = O.conv1d_nwc(X, Wt, bias=bias, relu=True, stride=2, pad=1)
    op = B.conv1d_op(1, 256, 64, 128, 3, stride=2, pad=1)
    space = op.space()
    for n in range(8):
        t = B.trace_sample_valid(op, space, 94, n)
        print("trace", n, t.decisions(), flush=True)
        got = run_variant(op, space, t, [X, Wt, bias], "f16", ref.shape)
        if got is None:
            continue
        compare.assert_float_close(got, ref, compare.RTOL_HALF, "C1D trace %d" % n)


@pytest.mark.parametrize("Cin,k,stride,pad,dil,D,H,W_", [(16, 3, 1, 1, 1, 4, 8, 8), (16, 3, 2, 1, 1, 6, 8, 16), (3, 7, 2, 3, 1, 6, 16, 16),
                                                         (32, 1, 1, 0, 1, 2, 8, 8), (16, 3, 1, 2, 2, 4, 8, 8), (8, 2, 2, 0, 1, 4, 8, 8)])
def test_conv3d_exact(Cin, k, stride, pad, dil, D, H, W_):
    """3-D convolution (Appendix A.2: C3D): the depth is folded into the rows (n, od, oh, ow) and the reduction
    (kd, kh, kw, ci) of the implicit GEMM by the im2col loader.  Integer-valued inputs, batch 2, 2 instances: bit-equal
    fp32 outputs, also where KD*KH*KW*Cin is padded to the intrinsic's k."""
    N, Cout = 2, 32
    g = I.rng(96)
    X = I.small_ints(g, (N, D, H, W_, Cin), -2, 2, "f16")
    Wt = I.small_ints(g, (k, k, k, Cin, Cout), -2, 2, "f16")
    bias = g.integers(-3, 4, size=Cout).astype(np.float32)
    ref = O.conv3d_ndhwc(X, Wt, bias=bias, relu=True, stride=stride, pad=pad, dilation=dil)
    assert ref[0].size // Cout * N % 16 == 0
    op = B.conv3d_op(N, D, H, W_, Cin, Cout, k, stride=stride, pad=pad, out_dtype="f32", dilation=dil)
    space = op.space()
    for n in range(6):
        t = B.trace_sample_valid(op, space, 97, n)
        assert B.trace_validate(op, space, t).compute_at == 0
        print("trace", n, t.decisions(), flush=True)
        got = run_variant(op, space, t, [X, Wt, bias], "f32", ref.shape, instances=2)
        if got is None:
            continue
        assert np.array_equal(got[0], ref) and np.array_equal(got[1], ref), "trace %d" % n

@pytest.mark.parametrize("D,H,W_,Cin,Cout,k,stride,pad,dtype,out", [(6, 16, 16, 3, 64, 7, 2, 3, "f16", "f32"), (4, 9, 24, 1, 32, 3, 2, 1, "bf16", "f32"),
                                                                   (5, 13, 16, 4, 96, 5, 2, 2, "f16", "f16"), (4, 12, 8, 2, 32, 3, 1, 0, "f16", "f32"),
                                                                   (1, 40, 56, 3, 64, 7, 2, 3, "bf16", "f32"), (1, 33, 72, 4, 128, 3, 1, 1, "f16", "f32"),
                                                                   (1, 59, 104, 3, 32, 5, 2, 4, "f16", "f32"),
                                                                   (1, 5, 304, 4, 64, 3, 1, 1, "f16", "f32"), (1, 6, 528, 3, 32, 7, 2, 3, "bf16", "f32"),
                                                                   (2, 3, 272, 2, 96, 3, 1, 2, "f16", "f16"), (1, 4, 264, 4, 32, 3, 1, 1, "f16", "f16")])
def test_first_layer_image_rows_exact(D, H, W_, Cin, Cout, k, stride, pad, dtype, out):
    """Im2col traces of first layers on the image-row kernel: runs with and without a leading element, odd and even chunk
    counts, tiles that end behind the plane, tiles that keep to the columns of a row, every accumulator shape.  Batch 2, 2 instances with their own weights;
    integer-valued inputs -> exact.  An infinite pixel reaches the outputs whose windows hold it and no others."""
    g = I.rng(97)
    shape, wshape = ((2, D, H, W_, Cin), (k, k, k, Cin, Cout)) if D > 1 else ((2, H, W_, Cin), (k, k, Cin, Cout))
    ref_of = O.conv3d_ndhwc if D > 1 else O.conv2d_nhwc
    ins = [[I.small_ints(g, shape, -2, 2, dtype), I.small_ints(g, wshape, 1, 2, dtype), g.integers(-3, 4, size=Cout).astype(np.float32)] for _ in range(2)]
    for x, _, _ in ins:
        x[(1,) + tuple(e // 2 for e in x.shape[1:])] = np.inf if dtype == "f16" else 0x7F80
    kw = {"bf16": True} if dtype == "bf16" else {}
    refs = [ref_of(x, w, bias=b, relu=True, stride=stride, pad=pad, **kw) for x, w, b in ins]
    op = (B.conv3d_op(2, D, H, W_, Cin, Cout, k, stride=stride, pad=pad, in_dtype=dtype, out_dtype=out) if D > 1 else
          B.conv2d_op(2, H, W_, Cin, Cout, k, k, stride=stride, pad=pad, in_dtype=dtype, out_dtype=out))
    space = op.space()
    t = next(t for t in (B.trace_sample_valid(op, space, 98, n) for n in range(200))
             if B.trace_validate(op, space, t).compute_at == 0 and B.trace_validate(op, space, t).family == B.FAM_GEMM_MFMA)
    assert "conv_rows.hip" in B.variant_kernel_text(op, B.trace_validate(op, space, t))
    got = run_variant_distinct(op, space, t, ins, out, refs[0].shape)
    if got is not None:
        for r in range(2):
            assert np.array_equal(got[r], refs[r]), "instance %d" % r


@pytest.mark.parametrize("k,stride,pad,D,H,W_,Cout", [(7, 2, 3, 6, 16, 20, 32), (3, 1, 1, 4, 8, 16, 32), (5, 2, 2, 4, 16, 16, 48)])
def test_conv3d_padded_reduction_beside_the_image_rows(k, stride, pad, D, H, W_, Cout):
    """3-channel 3-D layers that the image-row kernel does not take (rows of broken vectors, odd pixel steps, columns of 48):
    the im2col loop with a reduction that is padded to the intrinsic's k.  Batch 2, integer-valued inputs -> exact."""
    g = I.rng(105)
    X = I.small_ints(g, (2, D, H, W_, 3), -2, 2, "f16")
    Wt = I.small_ints(g, (k, k, k, 3, Cout), -2, 2, "f16")
    bias = g.integers(-3, 4, size=Cout).astype(np.float32)
    ref = O.conv3d_ndhwc(X, Wt, bias=bias, relu=True, stride=stride, pad=pad)
    op = B.conv3d_op(2, D, H, W_, 3, Cout, k, stride=stride, pad=pad, out_dtype="f32")
    space = op.space()
    for n in range(4):
        t = B.trace_sample_valid(op, space, 106, n)
        p = B.trace_validate(op, space, t)
        assert p.body == B.BODY_NEST and (k ** 3 * 3) % p.tile_unit[2]
        got = run_variant(op, space, t, [X, Wt, bias], "f32", ref.shape, instances=2)
        assert got is None or (np.array_equal(got[0], ref) and np.array_equal(got[1], ref)), "trace %d" % n


@pytest.mark.parametrize("Cin,k,stride,pad,H,W_,Cout", [(3, 7, 2, 3, 32, 32, 48), (2, 5, 2, 2, 32, 18, 32), (4, 7, 2, 3, 32, 33, 32)])
def test_filter_rows_beside_the_image_rows(Cin, k, stride, pad, H, W_, Cout):
    """Filter-row layers of 2 to 4 channels that the image-row kernel does not take: im2col staging and the resident patch
    whose weights are staged per step.  Batch 2, integer-valued inputs -> exact."""
    g = I.rng(107)
    X = I.small_ints(g, (2, H, W_, Cin), -2, 2, "f16")
    Wt = I.small_ints(g, (k, k, Cin, Cout), -2, 2, "f16")
    bias = g.integers(-3, 4, size=Cout).astype(np.float32)
    ref = O.conv2d_nhwc(X, Wt, bias=bias, relu=True, stride=stride, pad=pad)
    op = B.conv2d_op(2, H, W_, Cin, Cout, k, k, stride=stride, pad=pad, out_dtype="f32")
    space = op.space(B.SPACE_DEFAULT | B.SPACE_TAP_ROWS)
    want, idx = {0: 2, 1: 3}, 0
    while any(want.values()) and idx < 800:
        t = B.trace_sample_valid(op, space, 108, idx)
        idx += 1
        p = B.trace_validate(op, space, t)
        if not want.get(p.compute_at):
            continue
        want[p.compute_at] -= 1
        assert p.body == B.BODY_NEST and p.tap_rows == 1
        got = run_variant(op, space, t, [X, Wt, bias], "f32", ref.shape, instances=2)
        assert got is None or (np.array_equal(got[0], ref) and np.array_equal(got[1], ref)), "trace %d" % idx
    assert not any(want.values()), want


@pytest.mark.parametrize("H,W_,Cin,Cout,k,stride,R", [(56, 64, 3, 64, 7, 2, 200), (20, 32, 4, 32, 3, 1, 700), (16, 528, 2, 96, 5, 2, 240)])
def test_image_rows_over_many_instances_exact(H, W_, Cin, Cout, k, stride, R):
    """Launches of one instance and of so many that the kernel of the larger tile takes them, three data sets in rotation;
    integer-valued inputs -> exact."""
    g = I.rng(109)
    op = B.conv2d_op(1, H, W_, Cin, Cout, k, k, stride=stride, pad=k // 2, out_dtype="f32")
    sets = [[I.small_ints(g, (1, H, W_, Cin), -2, 2, "f16"), I.small_ints(g, (k, k, Cin, Cout), -2, 2, "f16"),
             g.integers(-3, 4, size=Cout).astype(np.float32)] for _ in range(3)]
    refs = [O.conv2d_nhwc(x, w, bias=b, relu=True, stride=stride, pad=k // 2) for x, w, b in sets]
    space = op.space()
    t = next(t for t in (B.trace_sample_valid(op, space, 110, n) for n in range(100)) if B.trace_validate(op, space, t).body == B.BODY_IMAGE_ROWS)
    v = B.Variant(op, space, t)
    assert v.launch_shape(1)[0] < v.launch_shape(R)[0] == v.params().body_tile_many
    for n in (1, R):
        got = run_variant_distinct(op, space, t, [sets[r % 3] for r in range(n)], "f32", refs[0].shape)
        if got is None:
            continue
        got = got.reshape((n,) + refs[0].shape)
        for r in range(n):
            assert np.array_equal(got[r], refs[r % 3]), "instance %d of %d" % (r, n)


def test_first_layer_tensors_aligned_to_their_elements():
    """Images, weights and outputs that start one element behind a 16-byte boundary: the im2col nest of such a layer reads
    single elements and writes four at a time."""
    g = I.rng(103)
    X, Wt = I.small_ints(g, (1, 16, 24, 3), -2, 2, "f16"), I.small_ints(g, (3, 3, 3, 32), -2, 2, "f16")
    bias = g.integers(-3, 4, size=32).astype(np.float32)
    op = B.conv2d_op(1, 16, 24, 3, 32, 3, 3, stride=2, pad=1)
    space = op.space()
    t = next(t for t in (B.trace_sample_valid(op, space, 104, n) for n in range(50)) if B.trace_validate(op, space, t).body == B.BODY_IMAGE_ROWS)
    got = run_variant_offset(op, space, t, [X, Wt, bias], "f16", (1, 8, 12, 32), [1, 1, 0, 1])
    if got is not None:
        assert np.array_equal(got, O.conv2d_nhwc(X, Wt, bias=bias, relu=True, stride=2, pad=1))


@pytest.mark.parametrize("L_,Cin,Cout,k,stride,pad", [(1056, 4, 64, 7, 1, 3), (4096, 1, 32, 7, 2, 3), (2080, 2, 64, 3, 1, 1)])
def test_conv1d_image_rows_exact(L_, Cin, Cout, k, stride, pad):
    """Rows of several tiles, not a whole number of them: a tile stages the columns that it meets.  Batch 2, integer-valued
    inputs -> exact."""
    g = I.rng(99)
    X = I.small_ints(g, (2, L_, Cin), -2, 2, "f16")
    Wt = I.small_ints(g, (k, Cin, Cout), -2, 2, "f16")
    bias = g.integers(-3, 4, size=Cout).astype(np.float32)
    ref = O.conv1d_nwc(X, Wt, bias=bias, relu=True, stride=stride, pad=pad)
    op = B.conv1d_op(2, L_, Cin, Cout, k, stride=stride, pad=pad, out_dtype="f32")
    space = op.space()
    t = next(t for t in (B.trace_sample_valid(op, space, 100, n) for n in range(200)) if B.trace_validate(op, space, t).body == B.BODY_IMAGE_ROWS)
    assert "-DCR_SPAN=1" in B.variant_kernel_text(op, B.trace_validate(op, space, t))
    got = run_variant(op, space, t, [X, Wt, bias], "f32", ref.shape, instances=2)
    if got is None:
        return
    assert np.array_equal(got[0], ref) and np.array_equal(got[1], ref)


def test_c3d_config_conv3d_16x224x224x3():
    """The paper's C3D shape: 16 x 224 x 224 x 3 -> 8 x 112 x 112 x 64, 7 x 7 x 7, stride 2, padding 3; fp16 (K = 1029)."""
    g = I.rng(98)
    X = I.uniform(g, (1, 16, 224, 224, 3), 0.0, 1.0, "f16")
    Wt = I.normal(g, (7, 7, 7, 3, 64), 0.02, "f16")
    bias = I.normal(g, (64,), 0.05, "f32")
    ref = O.conv3d_ndhwc(X, Wt, bias=bias, relu=True, stride=2, pad=3)
    assert ref.shape == (1, 8, 112, 112, 64)
    op = B.conv3d_op(1, 16, 224, 224, 3, 64, 7, stride=2, pad=3)
    space = op.space()
    for n in range(3):
        t = B.trace_sample_valid(op, space, 99, n)
        print("trace", n, t.decisions(), flush=True)
        got = run_variant(op, space, t, [X, Wt, bias], "f16", ref.shape)
        if got is None:
            continue
        compare.assert_float_close(got, ref, compare.RTOL_HALF, "C3D trace %d" % n)


@pytest.mark.parametrize("Cin,k,stride,pad,H,W_", [(3, 7, 2, 3, 32, 32), (4, 3, 1, 1, 16, 16), (3, 3, 1, 1, 16, 16), (2, 5, 2, 2, 16, 32), (8, 3, 1, 1, 8, 16),
                                                   (4, 7, 2, 3, 32, 16)])
def test_conv_filter_row_layout_exact(Cin, k, stride, pad, H, W_):
    """The opt-in filter-row layout of the reduction (k = filter row, then the KW * Cin contiguous elements of that row,
    rounded up to the intrinsic's k): im2col staging and, where pixels start at multiples of 4 bytes, the resident patch,
    whose fragments are pieces of image rows.  Integer-valued inputs, batch 2, 2 instances: bit-equal fp32 outputs."""
    N, Cout = 2, 32
    g = I.rng(101)
    X = I.small_ints(g, (N, H, W_, Cin), -2, 2, "f16")
    Wt = I.small_ints(g, (k, k, Cin, Cout), -2, 2, "f16")
    bias = g.integers(-3, 4, size=Cout).astype(np.float32)
    ref = O.conv2d_nhwc(X, Wt, bias=bias, relu=True, stride=stride, pad=pad)
    OH, OW = ref.shape[1], ref.shape[2]
    op = B.conv2d_op(N, H, W_, Cin, Cout, k, k, stride=stride, pad=pad, out_dtype="f32")
    space = op.space(B.SPACE_DEFAULT | B.SPACE_TAP_ROWS)
    assert space.flags & B.SPACE_TAP_ROWS
    patch_ok = (stride * Cin * 2) % 4 == 0
    want = {0: 3, 1: 3 if patch_ok else 0, 2: 2 if patch_ok else 0, 3: 1 if patch_ok else 0, 4: 2 if patch_ok else 0}
    idx = 0
    while any(want.values()) and idx < 800:
        t = B.trace_sample_valid(op, space, 102, idx)
        idx += 1
        p = B.trace_validate(op, space, t)
        assert p.tap_rows == 1 and (patch_ok or p.compute_at == 0)
        if want[p.compute_at] == 0:
            continue
        want[p.compute_at] -= 1
        print("trace", idx, "compute_at", p.compute_at, t.decisions(), flush=True)
        got = run_variant(op, space, t, [X, Wt, bias], "f32", (N, OH, OW, Cout), instances=2)
        if got is None:
            continue
        assert np.array_equal(got[0], ref) and np.array_equal(got[1], ref), "trace %d" % idx
    assert want[0] == 0 and want[1] == 0 and want[2] == 0, want


def test_cbr_first_layer_filter_row_layout():
    """The paper's CBR shape in the filter-row layout (K = 7 rows of 21 -> 32 elements), fp16, both cache-read locations."""
    g = I.rng(63)
    X = I.uniform(g, (1, 224, 224, 3), 0.0, 1.0, "f16")
    Wt = I.normal(g, (7, 7, 3, 64), 0.05, "f16")
    bias = I.normal(g, (64,), 0.05, "f32")
    ref = O.conv2d_nhwc(X, Wt, bias=bias, relu=True, stride=2, pad=3)
    op = B.conv2d_op(1, 224, 224, 3, 64, 7, 7, stride=2, pad=3)
    space = op.space(B.SPACE_DEFAULT | B.SPACE_TAP_ROWS)
    want = {0: 2, 1: 2, 2: 2, 3: 1, 4: 1}
    idx = 0
    while any(want.values()) and idx < 400:
        t = B.trace_sample_valid(op, space, 104, idx)
        idx += 1
        ca = B.trace_validate(op, space, t).compute_at
        if want[ca] == 0:
            continue
        want[ca] -= 1
        print("trace", idx, "compute_at", ca, t.decisions(), flush=True)
        got = run_variant(op, space, t, [X, Wt, bias], "f16", ref.shape)
        if got is None:
            continue
        compare.assert_float_close(got, ref, compare.RTOL_HALF, "CBR filter rows trace %d" % idx)
    assert want[0] == 0 and want[1] == 0 and want[2] == 0, want


@pytest.mark.parametrize("N,H,W_,Cin,Cout,k,stride,pad,dil,transposed", [
    (2, 8, 7, 64, 32, 3, 1, 1, 1, False),      # 112 pixels: one tile, its rest masked
    (3, 16, 16, 32, 128, 3, 1, 1, 1, False),   # steps of two taps, the last one half empty
    (2, 15, 11, 96, 256, 3, 2, 1, 1, False),   # steps that straddle taps, stride 2, odd extents
    (4, 14, 14, 128, 96, 3, 1, 2, 2, False),   # dilation, 96 columns
    (4, 7, 4, 72, 128, 1, 1, 0, 1, False),     # 72 channels: a step and an eighth
    (2, 8, 8, 256, 64, 5, 1, 2, 1, False),
    (1, 20, 20, 64, 128, 3, 1, 1, 1, False),
    (2, 6, 4, 64, 64, 3, 1, 1, 1, True),       # one phase
    (2, 4, 6, 128, 64, 4, 2, 1, 1, True),
    (3, 3, 5, 128, 192, 4, 4, 0, 1, True),      # one tap per phase
    (2, 4, 4, 64, 128, 6, 2, 2, 1, True),
])
def test_conv_steps_exact(N, H, W_, Cin, Cout, k, stride, pad, dil, transposed):
    """Convolutions as products on double steps, integer-valued inputs with exact sums: partial tiles, padding, k behind the
    reduction, phases, few and many instances with their own inputs (several tiles per persistent workgroup)."""
    g = I.rng(105)
    pool = [(I.small_ints(g, (N, H, W_, Cin), -2, 2, "f16"), I.small_ints(g, (k, k, Cin, Cout), -1, 1, "f16"),
             g.integers(-3, 4, size=Cout).astype(np.float32)) for _ in range(2)]
    if transposed:
        refs = [O.conv2d_transposed_nhwc(x, w, bias=b, relu=True, stride=stride, pad=pad) for x, w, b in pool]
        op = B.conv2d_transposed_op(N, H, W_, Cin, Cout, k, k, stride=stride, pad=pad, out_dtype="f32")
    else:
        refs = [O.conv2d_nhwc(x, w, bias=b, relu=True, stride=stride, pad=pad, dilation=dil) for x, w, b in pool]
        op = B.conv2d_op(N, H, W_, Cin, Cout, k, k, stride=stride, pad=pad, out_dtype="f32", dilation=dil)
    space = op.space()
    t = next(t for t in (B.trace_sample_valid(op, space, 106, n) for n in range(400)) if B.trace_validate(op, space, t).body == B.BODY_CONV_STEPS)
    p = B.trace_validate(op, space, t)
    for R in (2, 300):
        print("R", R, "tile", p.body_tile, "tiles", p.grid[0], flush=True)
        got = run_variant_distinct(op, space, t, [list(pool[r % 2]) for r in range(R)], "f32", refs[0].shape)
        if got is None:
            continue
        for r in range(R):
            assert np.array_equal(got[r], refs[r % 2]), "instance %d of %d" % (r, R)


@pytest.mark.parametrize("N,H,W_,Cin,Cout,k,stride,pad,transposed,many", [
    (2, 8, 7, 64, 32, 3, 1, 1, False, 700),      # one slot, seven stages, the last of eight wavefronts without a pixel
    (3, 8, 18, 64, 128, 3, 1, 1, False, 120),    # one slot, eight stages of 64 x 64
    (33, 28, 28, 64, 256, 1, 1, 0, False, 6),    # two slots, two stages, one step per tile, 16 pixels in the last tile
    (2, 5, 4, 128, 128, 4, 2, 1, True, 150),     # phases of 40 pixels
])
def test_conv_steps_partial_tiles_without_bias_exact(N, H, W_, Cin, Cout, k, stride, pad, transposed, many):
    """Workgroups that go on after a tile whose last wavefronts have nothing to store: the next tile's operands have to have
    landed all the same.  No bias: nothing else in the epilogue waits for loads."""
    g = I.rng(109)
    pool = [(I.small_ints(g, (N, H, W_, Cin), -2, 2, "f16"), I.small_ints(g, (k, k, Cin, Cout), -1, 1, "f16")) for _ in range(2)]
    ref, mk = (O.conv2d_transposed_nhwc, B.conv2d_transposed_op) if transposed else (O.conv2d_nhwc, B.conv2d_op)
    refs = [ref(x, w, stride=stride, pad=pad) for x, w in pool]
    op = mk(N, H, W_, Cin, Cout, k, k, stride=stride, pad=pad, has_bias=False, relu=False, out_dtype="f32")
    space = op.space()
    t = next(t for t in (B.trace_sample_valid(op, space, 106, n) for n in range(400)) if B.trace_validate(op, space, t).body == B.BODY_CONV_STEPS)
    p = B.trace_validate(op, space, t)
    phases = stride * stride if transposed else 1
    assert N * H * W_ % p.block_m and p.grid[0] * many > 512
    print("R", many, "tile", p.body_tile, "tiles", p.grid[0], "phases", phases, flush=True)
    got = run_variant_distinct(op, space, t, [list(pool[r % 2]) for r in range(many)], "f32", refs[0].shape)
    if got is not None:
        for r in range(many):
            assert np.array_equal(got[r], refs[r % 2]), "instance %d of %d" % (r, many)


@pytest.mark.parametrize("static", [False, True])
def test_conv_steps_operands_off_16_byte_boundaries(static):
    """Loads straight into LDS want aligned groups: operands that are aligned to their elements only run on the trace's nest,
    which the set-up call has ready for the launch that allocates nothing."""
    g = I.rng(107)
    X = I.small_ints(g, (4, 8, 8, 64), -2, 2, "f16")
    Wt = I.small_ints(g, (3, 3, 64, 64), -1, 1, "f16")
    bias = g.integers(-3, 4, size=64).astype(np.float32)
    ref = O.conv2d_nhwc(X, Wt, bias=bias, relu=True, stride=1, pad=1)
    op = B.conv2d_op(4, 8, 8, 64, 64, 3, 3, stride=1, pad=1, out_dtype="f32")
    space = op.space()
    t = next(t for t in (B.trace_sample_valid(op, space, 108, n) for n in range(400)) if B.trace_validate(op, space, t).body == B.BODY_CONV_STEPS)
    for offsets in ([0, 0, 0, 0], [3, 0, 0, 0], [0, 1, 0, 0]):
        got = run_variant_offset(op, space, t, [X, Wt, bias], "f32", ref.shape, offsets, static=static)
        if got is not None:
            assert np.array_equal(got, ref), offsets


@pytest.mark.parametrize("N,H,W_,Cin,Cout,k,pad,dil,transposed,R,dtype", [
    (1, 56, 56, 64, 64, 3, 1, 1, False, 64, "f16"),     # strips of 8 columns, two bands of 7 rows
    (1, 16, 11, 32, 32, 3, 1, 1, False, 400, "f16"),    # one chunk per tile, masked columns, 32 channels per wavefront
    (1, 12, 16, 64, 64, 3, 3, 1, False, 300, "bf16"),   # 4 x 4 blocks, padding wider than the filter's half
    (1, 16, 20, 32, 128, 3, 3, 3, False, 200, "f16"),   # dilation 3, odd row pitch, two column blocks
    (1, 28, 28, 32, 64, 5, 2, 1, False, 200, "bf16"),   # five filter columns
    (1, 40, 40, 96, 32, 3, 2, 2, False, 130, "f16"),    # dilation 2, three chunks
    (40, 12, 28, 64, 256, 3, 2, 2, False, 1, "f16"),    # a batch, wavefronts side by side over channels
    (50, 20, 20, 64, 96, 3, 1, 1, False, 1, "f16"),     # three of 32 channels, rows behind the image
    (237, 8, 8, 64, 64, 3, 1, 1, False, 1, "f16"),
    (96, 5, 10, 32, 64, 2, 0, 1, False, 1, "f16"),      # two filter columns, no padding, rows that no tile fills
    (1602, 2, 7, 32, 64, 2, 1, 1, False, 1, "f16"),    # eight whole images per tile, the last one of two
    (30, 24, 24, 64, 64, 3, 1, 1, True, 1, "f16"),      # transposed: the filter turned round
    (40, 6, 10, 64, 128, 3, 0, 1, True, 1, "bf16"),
])
@pytest.mark.parametrize("epilogue", [True, False])
def test_conv_patch_exact(N, H, W_, Cin, Cout, k, pad, dil, transposed, R, dtype, epilogue):
    """Launches of convolutions that fill the chip run on input patches.  Inputs of two instances in turn, integers whose sums the
    output type holds: equal results."""
    g = I.rng(111)
    kw = {"bf16": True} if dtype == "bf16" else {}
    if transposed:
        ref_of, op = O.conv2d_transposed_nhwc, B.conv2d_transposed_op(N, H, W_, Cin, Cout, k, k, stride=1, pad=pad, in_dtype=dtype, has_bias=epilogue, relu=epilogue)
    else:
        ref_of, op = O.conv2d_nhwc, B.conv2d_op(N, H, W_, Cin, Cout, k, k, stride=1, pad=pad, in_dtype=dtype, dilation=dil, has_bias=epilogue, relu=epilogue)
        kw["dilation"] = dil
    space = op.space()
    t = next(t for t in (B.trace_sample_valid(op, space, 112, n) for n in range(400)) if B.trace_validate(op, space, t).family == B.FAM_GEMM_MFMA)
    v = B.Variant(op, space, t)
    own = v.params().body_tile
    R = R if R == 1 else next(r for r in range(R, 2 * R) if v.launch_shape(r)[0] != own) # instances that make whole rounds of tiles
    tile, groups, _ = v.launch_shape(R)
    assert tile != own
    # one weight in `keep` counts, so that sums of bf16 stay below 256
    keep = 16 if dtype == "bf16" else 2
    pool = []
    for _ in range(min(R, 2)):
        x, w = I.small_ints(g, (N, H, W_, Cin), -2, 2, dtype), I.small_ints(g, (k, k, Cin, Cout), -1, 1, dtype)
        w[g.integers(0, keep, size=w.shape) != 0] = 0
        pool.append([x, w] + ([g.integers(-3, 4, size=Cout).astype(np.float32)] if epilogue else []))
    refs = [ref_of(p[0], p[1], bias=p[2] if epilogue else None, relu=epilogue, stride=1, pad=pad, **kw) for p in pool]
    assert max(np.abs(r).max() for r in refs) <= (256 if dtype == "bf16" else 2048)
    print("tile", tile, "tiles", groups * R, flush=True)
    got = run_variant_distinct(op, space, t, [pool[r % len(pool)] for r in range(R)], dtype, refs[0].shape)
    if got is not None:
        for r in range(R):
            assert np.array_equal(got[r] if R > 1 else got.reshape(refs[0].shape), refs[r % len(pool)]), "instance %d of %d" % (r, R)


@pytest.mark.parametrize("kh,kw", [(1, 3), (3, 2), (2, 5)])
def test_conv_patch_oblong_filters_exact(kh, kw):
    """Filters of one row, and of more columns than rows and fewer, over a batch."""
    g = I.rng(115)
    X, Wt = I.small_ints(g, (112, 16, 17, 64), -2, 2, "f16"), I.small_ints(g, (kh, kw, 64, 64), -1, 1, "f16")
    bias = g.integers(-3, 4, size=64).astype(np.float32)
    ref = O.conv2d_nhwc(X, Wt, bias=bias, relu=True, stride=1, pad=0)
    op = B.conv2d_op(112, 16, 17, 64, 64, kh, kw, stride=1, pad=0)
    space = op.space()
    t = next(t for t in (B.trace_sample_valid(op, space, 116, n) for n in range(400)) if B.trace_validate(op, space, t).family == B.FAM_GEMM_MFMA)
    v = B.Variant(op, space, t)
    assert v.launch_shape(1)[0] != v.params().body_tile
    got = run_variant(op, space, t, [X, Wt, bias], "f16", ref.shape)
    assert got is None or np.array_equal(got.reshape(ref.shape), ref)


def test_conv_patch_operands_off_16_byte_boundaries():
    """Operands that are aligned to their elements only run on the trace's nest also where the launch would fill the chip."""
    g = I.rng(113)
    X, Wt = I.small_ints(g, (64, 16, 16, 32), -2, 2, "f16"), I.small_ints(g, (3, 3, 32, 32), -1, 1, "f16")
    bias = g.integers(-3, 4, size=32).astype(np.float32)
    ref = O.conv2d_nhwc(X, Wt, bias=bias, relu=True, stride=1, pad=1)
    op = B.conv2d_op(64, 16, 16, 32, 32, 3, 3, stride=1, pad=1)
    space = op.space()
    t = next(t for t in (B.trace_sample_valid(op, space, 114, n) for n in range(400)) if B.trace_validate(op, space, t).family == B.FAM_GEMM_MFMA)
    v = B.Variant(op, space, t)
    assert v.launch_shape(1)[0] != v.params().body_tile
    for offsets in ([0, 0, 0, 3], [3, 0, 0, 0], [0, 1, 0, 0]):
        got = run_variant_offset(op, space, t, [X, Wt, bias], "f16", ref.shape, offsets)
        if got is not None:
            assert np.array_equal(got, ref), offsets


def test_conv_patch_static_launch_exact():
    """Input patches through the launch that allocates nothing."""
    g = I.rng(153)
    X, Wt = I.small_ints(g, (64, 16, 16, 32), -2, 2, "f16"), I.small_ints(g, (3, 3, 32, 32), -1, 1, "f16")
    bias = g.integers(-3, 4, size=32).astype(np.float32)
    op = B.conv2d_op(64, 16, 16, 32, 32, 3, 3, stride=1, pad=1)
    space = op.space()
    t = next(t for t in (B.trace_sample_valid(op, space, 114, n) for n in range(400)) if B.trace_validate(op, space, t).family == B.FAM_GEMM_MFMA)
    assert B.Variant(op, space, t).launch_kernel(1)[0].body == B.BODY_CONV_PATCH
    ref = O.conv2d_nhwc(X, Wt, bias=bias, relu=True, stride=1, pad=1)
    got = run_variant_offset(op, space, t, [X, Wt, bias], "f16", ref.shape, [0, 0, 0, 0], static=True)
    assert got is None or np.array_equal(got, ref)


@pytest.mark.parametrize("N,D,H,W_,Cin,Cout,k,stride,pad,dtype,R", [
    (1, 6, 32, 32, 3, 64, 7, 2, 3, "f16", 512),         # planes at the ends of the depth meet fewer filter planes
    (1, 7, 21, 40, 1, 32, 7, 2, 3, "bf16", 512),        # 32 channels, the last tile of a plane in part
    (2, 6, 17, 24, 4, 128, 5, 1, 0, "f16", 256),        # two column blocks, no padding
    (1, 2, 28, 48, 3, 64, 5, 2, 4, "f16", 512),         # output planes that no filter plane meets
    (512, 1, 30, 56, 3, 64, 7, 2, 3, "f16", 1),         # 2-D: one plane per tile, a batch
    (512, 1, 33, 32, 2, 32, 3, 1, 1, "bf16", 1),
    (1, 1, 40, 48, 4, 64, 5, 2, 2, "f16", 512),         # instances with their own weights
])
@pytest.mark.parametrize("epilogue", [True, False])
def test_first_layer_planes_exact(N, D, H, W_, Cin, Cout, k, stride, pad, dtype, R, epilogue):
    """First layers whose tiles make whole rounds (512 images), on persistent workgroups over filter planes.  Inputs of two instances
    in turn, integers whose sums the output type holds; an infinite pixel reaches the outputs whose windows hold it and no others."""
    g = I.rng(117)
    kw = {"bf16": True} if dtype == "bf16" else {}
    shape, wshape = ((N, D, H, W_, Cin), (k, k, k, Cin, Cout)) if D > 1 else ((N, H, W_, Cin), (k, k, Cin, Cout))
    ref_of = O.conv3d_ndhwc if D > 1 else O.conv2d_nhwc
    args = dict(stride=stride, pad=pad, in_dtype=dtype, has_bias=epilogue, relu=epilogue)
    op = B.conv3d_op(N, D, H, W_, Cin, Cout, k, **args) if D > 1 else B.conv2d_op(N, H, W_, Cin, Cout, k, k, **args)
    space = op.space()
    t = next(t for t in (B.trace_sample_valid(op, space, 118, n) for n in range(200))
             if B.trace_validate(op, space, t).compute_at == 0 and B.trace_validate(op, space, t).family == B.FAM_GEMM_MFMA)
    pool = []
    for _ in range(min(R, 2)):
        x, w = I.small_ints(g, shape, -1, 1, dtype), I.small_ints(g, wshape, -1, 1, dtype)
        w[w == 0] = 1 if dtype == "f16" else 0x3F80
        x[tuple(e // 2 for e in x.shape)] = np.inf if dtype == "f16" else 0x7F80
        pool.append([x, w] + ([g.integers(-3, 4, size=Cout).astype(np.float32)] if epilogue else []))
    refs = [ref_of(q[0], q[1], bias=q[2] if epilogue else None, relu=epilogue, stride=stride, pad=pad, **kw) for q in pool]
    assert max(np.abs(r[np.isfinite(r)]).max() for r in refs) <= (256 if dtype == "bf16" else 2048)
    got = run_variant_distinct(op, space, t, [pool[r % len(pool)] for r in range(R)], dtype, refs[0].shape)
    if got is not None:
        for r in range(R):
            assert np.array_equal(got[r] if R > 1 else got.reshape(refs[0].shape), refs[r % len(pool)], equal_nan=True), "instance %d of %d" % (r, R)


@pytest.mark.parametrize("N,H,W_,Cin,Cout,k,R", [(3, 40, 24, 3, 32, 7, 1), (1, 96, 64, 3, 96, 3, 9), (5, 64, 48, 4, 64, 5, 1)])
def test_first_layer_workgroups_no_multiple_of_8_exact(N, H, W_, Cin, Cout, k, R):
    """Image rows whose workgroups are dealt to the XCDs in runs of unequal length, fewer than 8 among them: integers, two inputs in turn."""
    g = I.rng(141)
    op = B.conv2d_op(N, H, W_, Cin, Cout, k, k, stride=2, pad=k // 2)
    space = op.space()
    t = next(t for t in (B.trace_sample_valid(op, space, 142, n) for n in range(200)) if B.trace_validate(op, space, t).body == B.BODY_IMAGE_ROWS)
    assert B.trace_validate(op, space, t).grid[0] * R % 8
    pool = [[I.small_ints(g, (N, H, W_, Cin), -1, 1, "f16"), I.small_ints(g, (k, k, Cin, Cout), -1, 1, "f16"), g.integers(-3, 4, size=Cout).astype(np.float32)]
            for _ in range(2)]
    refs = [O.conv2d_nhwc(q[0], q[1], bias=q[2], relu=True, stride=2, pad=k // 2) for q in pool]
    got = run_variant_distinct(op, space, t, [pool[r % 2] for r in range(R)], "f16", refs[0].shape)
    if got is not None:
        for r in range(R):
            assert np.array_equal(got[r] if R > 1 else got.reshape(refs[0].shape), refs[r % 2]), "instance %d of %d" % (r, R)
