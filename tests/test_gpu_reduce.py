"""GPU parity of the row-reduction kernels (softmax over the last axis, 2-norm per batch entry; Appendix A.2: SFM, NRM)
against the CPU oracle.  fp32 arithmetic on the GPU, float64 in the oracle: fp32 tolerance for fp32 outputs, the
half-precision tolerance where the output is rounded to fp16 / bf16."""
import numpy as np
import pytest

from oracle import compare, oracle as O
from paper_2205_13603_amd import binding as B, inputs as I
from gpu_util import run_variant, run_variant_offset

pytestmark = pytest.mark.gpu


def test_sfm_config_softmax_256x256():
    g = I.rng(50)
    X = I.normal(g, (1, 256, 256), 2.0, "f32")
    ref = O.softmax(X)
    op = B.softmax_op(1, 256, 256)
    space = op.space()
    assert space.family == B.FAM_REDUCE
    seen = set()
    for n in range(24):
        t = B.trace_sample_valid(op, space, 50, n)
        p = B.trace_validate(op, space, t)
        seen.add((p.cache_read, p.tk[2] > 64))
        print("trace", n, t.decisions(), flush=True)
        got = run_variant(op, space, t, [X], "f32", ref.shape, instances=2)
        if got is None:
            continue
        compare.assert_float_close(got[0], ref, compare.RTOL_F32, "softmax trace %d" % n)
        assert np.array_equal(got[0], got[1])
        assert np.max(np.abs(got[0].sum(-1) - 1.0)) < 1e-5
    assert {c for c, _ in seen} == {0, 1}


def test_nrm_config_norm_256x256():
    g = I.rng(51)
    X = I.normal(g, (1, 256, 256), 1.0, "f32")
    ref = O.norm(X)
    op = B.norm_op(1, 256, 256)
    space = op.space()
    for n in range(20):
        t = B.trace_sample_valid(op, space, 51, n)
        print("trace", n, t.decisions(), flush=True)
        got = run_variant(op, space, t, [X], "f32", ref.shape, instances=3)
        if got is None:
            continue
        for r in range(3):
            compare.assert_float_close(got[r], ref, compare.RTOL_F32, "norm trace %d" % n)


def test_groups_wider_than_a_wavefront_and_exact_cases():
    """Rows reduced by 128 and 256 lanes (partial results of the wavefronts meet in LDS), several rows per group in
    flight, both register modes.  Uniform rows of 256 elements give exactly 1/256; sums of squares of small integers
    are exact in fp32."""
    op = B.softmax_op(2, 64, 256)
    space = op.space()
    g = I.rng(52)
    X = I.normal(g, (2, 64, 256), 3.0, "f32")
    X[1, 5, :] = 1.25                  # a uniform row
    X[0, 7, :] = -100.0
    X[0, 7, 100] = 100.0               # one dominant element: no overflow, exp(-200) underflows to 0 in fp32
    ref = O.softmax(X)
    for n, vals in enumerate([[[32, 1, 4, 1], [1, 1, 256, 1], [0]], [[16, 2, 2, 2], [1, 1, 128, 2], [1]],
                              [[8, 4, 4, 1], [1, 2, 128, 1], [1]], [[4, 2, 8, 2], [2, 1, 128, 1], [0]],
                              [[2, 1, 16, 4], [1, 1, 64, 4], [1]], [[1, 2, 64, 1], [4, 4, 16, 1], [0]]]):
        t = B.make_trace(space, vals)
        print("softmax trace", n, vals, flush=True)
        got = run_variant(op, space, t, [X], "f32", ref.shape)
        if got is None:
            continue
        compare.assert_float_close(got, ref, compare.RTOL_F32, "softmax wide trace %d" % n)
        assert np.all(got[1, 5] == 1.0 / 256)
        assert got[0, 7, 100] == 1.0 and np.all(np.delete(got[0, 7], 100) == 0.0)
    op = B.norm_op(4, 96, 128)
    space = op.space()
    Xi = I.small_ints(g, (4, 96, 128), -3, 3, "f32")
    ref = O.norm(Xi)
    for n, vals in enumerate([[[4, 1, 1, 1], [3, 4, 256, 4]], [[2, 1, 2, 1], [6, 4, 128, 4]], [[1, 1, 4, 1], [48, 1, 256, 1]],
                              [[1, 2, 1, 2], [12, 1, 1024, 1]], [[1, 1, 1, 4], [6, 8, 64, 4]]]):
        t = B.make_trace(space, vals)
        print("norm trace", n, vals, flush=True)
        got = run_variant(op, space, t, [Xi], "f32", ref.shape, instances=2)
        if got is None:
            continue
        compare.assert_float_close(got[0], ref, 2e-7, "norm ints trace %d" % n)  # exact sum, one rounding in the root
        assert np.array_equal(got[0], got[1])


@pytest.mark.parametrize("dtype,out", [("f32", "f32"), ("f16", "f16"), ("bf16", "f32")])
@pytest.mark.parametrize("cols", [8, 24, 136, 1000, 1896, 4096])
def test_softmax_whole_vector_rows(cols, dtype, out):
    """Rows of whole 16-byte vectors under narrow lane groups: one lane group of a wavefront holds the row, the last
    vectors masked.  Elements at -inf, a maximum in the last element."""
    g = I.rng(53)
    X = I.normal(g, (1, 24, cols), 2.0, dtype)
    X[0, 3, ::2] = -np.inf if dtype != "bf16" else X[0, 3, 1]
    X[0, 5, cols - 1] = X[0, 4, cols - 1] = X[0].max()
    ref = O.softmax(X) if dtype != "bf16" else O.softmax(X, bf16=True)
    op = B.softmax_op(1, 24, cols, dtype, out)
    space = op.space()
    for vals in ([[3, 1, 8, 1], [cols // 8, 1, 8, 1], [0]], [[1, 3, 8, 1], [1, cols // 8, 8, 1], [1]]):
        if vals[2] == [1] and cols > 8 * 64:
            continue
        t = B.make_trace(space, vals)
        assert "-DROW_VEC=" in B.variant_kernel_text(op, B.trace_validate(op, space, t))
        got = run_variant(op, space, t, [X], out, ref.shape, instances=2)
        if got is None:
            continue
        compare.assert_float_close(got[0], ref, compare.RTOL_F32 if out == dtype == "f32" else compare.RTOL_HALF if out != "f32" else 1e-5, "softmax %d" % cols)
        assert np.array_equal(got[0], got[1])


@pytest.mark.parametrize("rows,i,cols,k", [(27, [27, 1, 1, 1], 1088, [17, 1, 64, 1]), (72, [9, 1, 8, 1], 24, [3, 1, 8, 1])])
def test_softmax_whole_vector_rows_that_no_workgroup_divides(rows, i, cols, k):
    """The last workgroup masks rows (4 rows of 64 lanes, 32 of 8 lanes).  A row of -inf, one with +inf and one with NaN are
    NaN throughout and touch no other row, as in the oracle."""
    X = I.normal(I.rng(57), (1, rows, cols), 2.0, "f32")
    X[0, 1] = -np.inf
    X[0, rows - 2, 3] = np.inf
    X[0, rows - 4, cols - 1] = np.nan
    op = B.softmax_op(1, rows, cols)
    space = op.space()
    t = B.make_trace(space, [i, k, [0]])
    p = B.trace_validate(op, space, t)
    assert p.body == B.BODY_ROW_VECTORS and rows % p.block_m
    got = run_variant(op, space, t, [X], "f32", X.shape, instances=2)
    if got is None:
        return
    bad = [1, rows - 2, rows - 4]
    for r in range(2):
        assert np.all(np.isnan(got[r][0, bad]))
        compare.assert_float_close(np.delete(got[r], bad, 1), O.softmax(np.delete(X, bad, 1)), compare.RTOL_F32, "softmax masked rows")


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("rows,cols,i,k,cache_read", [
    (64, 250, [2, 1, 32, 1], [25, 5, 2, 1], 0), (64, 250, [1, 2, 32, 1], [5, 25, 2, 1], 0),       # not whole vectors
    (16, 6144, [4, 2, 2, 1], [3, 4, 128, 4], 0), (16, 6144, [8, 1, 1, 2], [3, 8, 256, 1], 0),    # rows beyond 4096
    (16, 6144, [4, 1, 4, 1], [6, 4, 64, 4], 0), (8, 6144, [1, 1, 8, 1], [96, 4, 8, 2], 0),
    (16, 4096, [16, 1, 1, 1], [1, 2, 512, 4], 0), (16, 2048, [4, 1, 4, 1], [1, 8, 64, 4], 0),    # few long rows
    (16, 768, [8, 2, 1, 1], [2, 3, 64, 2], 1), (16, 768, [2, 2, 2, 2], [1, 3, 256, 1], 1)])      # staged in registers
def test_softmax_lane_groups_of_the_trace(rows, cols, i, k, cache_read, dtype):
    """Traces that keep their own lane groups: rows read once per pass that are no whole vectors, beyond 4096 elements or
    few and long, rows staged in registers by full lines; groups of 2 to 512 lanes."""
    X = I.normal(I.rng(58), (1, rows, cols), 2.0, dtype)
    X[0, 2, 1::2] = -np.inf
    X[0, 3, cols - 1] = 9.0
    op = B.softmax_op(1, rows, cols, dtype)
    space = op.space()
    t = B.make_trace(space, [i, k, [cache_read]])
    p = B.trace_validate(op, space, t)
    assert p.body == B.BODY_NEST and "-DCACHE_READ=%d" % cache_read in B.variant_kernel_text(op, p)
    got = run_variant(op, space, t, [X], dtype, X.shape, instances=2)
    if got is None:
        return
    compare.assert_float_close(got[0], O.softmax(X), compare.RTOL_F32 if dtype == "f32" else compare.RTOL_HALF, "softmax %d x %d" % (rows, cols))
    assert np.array_equal(got[0], got[1])


@pytest.mark.parametrize("dtype", ["f32", "f16"])
def test_softmax_rows_aligned_to_their_elements(dtype):
    """Whole-vector rows of tensors that start one element behind a 16-byte boundary: the nests that this kernel stands in
    for read single elements."""
    X = I.normal(I.rng(56), (1, 24, 136), 2.0, dtype)
    op = B.softmax_op(1, 24, 136, dtype)
    space = op.space()
    t = B.make_trace(space, [[3, 1, 8, 1], [17, 1, 8, 1], [0]])
    assert B.trace_validate(op, space, t).body == B.BODY_ROW_VECTORS
    got = run_variant_offset(op, space, t, [X], dtype, X.shape, [1, 1])
    if got is not None:
        compare.assert_float_close(got, O.softmax(X), compare.RTOL_F32 if dtype == "f32" else compare.RTOL_HALF, "softmax %s" % dtype)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("rows,cols,lanes", [(4104, 304, 16), (8208, 136, 8), (2056, 552, 32), (2040, 552, 64), (2056, 1064, 32), (2056, 2016, 64)])
def test_softmax_narrow_lane_groups(rows, cols, lanes, dtype):
    """2-byte rows whose lane groups are narrower, with fewer masked vectors, from 4 wavefronts per compute unit on; the last workgroup in
    part.  Lowest values and -infinity take no weight, a row of -infinity is NaN and leaves its neighbours alone."""
    X = I.normal(I.rng(59), (1, rows, cols), 2.0, dtype)
    low, inf = (np.finfo(np.float16).min, -np.inf) if dtype == "f16" else (0xFF7F, 0xFF80)
    X[0, 2, 1::2], X[0, 3, : cols - 1], X[0, rows - 1, 8:] = low, inf, inf
    X[0, 5] = inf
    op = B.softmax_op(1, rows, cols, dtype)
    space = op.space()
    t = B.make_trace(space, [[rows // 8, 1, 8, 1], [cols // 8, 1, 8, 1], [0]])
    p = B.trace_validate(op, space, t)
    assert (p.body, p.tk[2]) == (B.BODY_ROW_VECTORS, lanes)
    got = run_variant(op, space, t, [X], dtype, X.shape)
    if got is not None:
        got = got.reshape(X.shape)
        assert np.all(np.isnan(got[0, 5]))
        ref = O.softmax(np.delete(X, 5, 1), bf16=dtype == "bf16")
        compare.assert_float_close(np.delete(got, 5, 1), ref, compare.RTOL_HALF, "softmax %d x %d" % (rows, cols))


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_softmax_and_norm_half_inputs_odd_shapes(dtype):
    """Extents with factors 3 and 5; the softmax output is rounded once to the input type."""
    g = I.rng(53)
    X = I.normal(g, (3, 20, 96), 2.0, dtype)
    ref = O.softmax(X, bf16=dtype == "bf16")
    op = B.softmax_op(3, 20, 96, dtype)
    space = op.space()
    for n in range(8):
        t = B.trace_sample_valid(op, space, 53, n)
        print("softmax", dtype, "trace", n, t.decisions(), flush=True)
        got = run_variant(op, space, t, [X], dtype, ref.shape)
        if got is None:
            continue
        compare.assert_float_close(got, ref, compare.RTOL_HALF, "softmax %s trace %d" % (dtype, n))
    op = B.softmax_op(3, 20, 96, dtype, "f32")
    space = op.space()
    for n in range(4):
        t = B.trace_sample_valid(op, space, 54, n)
        got = run_variant(op, space, t, [X], "f32", ref.shape)
        if got is None:
            continue
        compare.assert_float_close(got, ref, compare.RTOL_F32, "softmax %s -> f32 trace %d" % (dtype, n))
    ref = O.norm(X, bf16=dtype == "bf16")
    op = B.norm_op(3, 20, 96, dtype)
    space = op.space()
    for n in range(8):
        t = B.trace_sample_valid(op, space, 55, n)
        print("norm", dtype, "trace", n, t.decisions(), flush=True)
        got = run_variant(op, space, t, [X], "f32", ref.shape)
        if got is None:
            continue
        compare.assert_float_close(got, ref, compare.RTOL_F32, "norm %s trace %d" % (dtype, n))
