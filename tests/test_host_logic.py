"""Host logic of libms (no GPU): symbols, op descriptors, space, sampler, mutation, text form,
validator, interpreter coverage."""
import ctypes as C
import collections
import math
import os
import re
import subprocess

import numpy as np
import pytest

from oracle import oracle as O
from paper_2205_13603_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_exports_every_declared_symbol():
    hdr = open(os.path.join(ROOT, "include", "ms.h")).read()
    hdr = re.sub(r"/\*.*?\*/", "", hdr, flags=re.S)
    declared = set(re.findall(r"\b(ms_[a-z0-9_]+)\s*\(", hdr))
    declared -= {n for n in declared if re.search(r"typedef[^;]*\(\s*\*\s*%s\s*\)" % n, hdr)}
    assert declared, "no declarations found"
    L = B.lib()
    for name in sorted(declared):
        assert hasattr(L, name), "libms.so does not export %s" % name
    assert declared == set(B.SYMBOLS), (declared ^ set(B.SYMBOLS))
    assert L.ms_version() == 3


def test_struct_sizes_match_header():
    # computed from the header's field lists (natural alignment)
    assert C.sizeof(B.ms_decision) == 16 + 8 * B.MAX_FACTORS
    assert C.sizeof(B.ms_trace) == 8 + B.MAX_SLOTS * C.sizeof(B.ms_decision)
    assert C.sizeof(B.ms_op_desc) == 8 * 4 + 8 * 8 + 3 * 8 + 3 * 8
    assert C.sizeof(B.ms_slot) == 8 + 16 + 8 + 8 + 8 * B.MAX_CANDS + 4 * B.MAX_CANDS + 8 + 8 * B.MAX_CANDS


def test_op_loops_and_work():
    op = B.gemm_op(128, 128, 128, "f32")
    assert op.loops() == [("i", 128, False), ("j", 128, False), ("k", 128, True)]
    assert op.work() == (4194304.0, 196608.0)
    op = B.gemm_op(1024, 1024, 1024, "f16")
    assert op.work() == (2147483648.0, 6291456.0)
    op = B.conv2d_op(1, 56, 56, 64, 64, 3, 3, stride=1, pad=1)
    assert op.loops() == [("i", 3136, False), ("j", 64, False), ("k", 576, True)]
    f, b = op.work()
    assert f == 231211008.0 and b == 401408 + 73728 + 256 + 401408
    op = B.bmm_op(12, 128, 128, 64, True, "f16")
    assert op.work() == (25165824.0, 786432.0)
    d = op.desc()
    assert list(d.a_strides) == [128 * 64, 64, 1] and list(d.b_strides) == [128 * 64, 1, 64]
    op = B.bmm_op(12, 128, 64, 128, False, "f16")
    assert op.work() == (25165824.0, 786432.0)
    op = B.gemm_op(512, 512, 512, "i8")
    assert op.work() == (268435456.0, 1572864.0)
    op = B.dwconv2d_op(1, 112, 112, 32)
    assert op.work() == (7225344.0, 3212416.0)
    assert [l[0] for l in op.loops()] == ["n", "i", "j", "c", "kh", "kw"]
    op = B.dwconv2d_op(1, 56, 56, 144, stride=2)
    assert op.work() == (2032128.0, 2263104.0)
    assert op.tensor_bytes(-1) == 28 * 28 * 144 * 4


def test_op_errors_do_not_abort():
    with pytest.raises(B.MsError) as e:
        B.gemm_op(0, 4, 4)
    assert e.value.code == B.MS_ERR_BAD_ARG
    with pytest.raises(B.MsError) as e:
        B.gemm_op(4, 4, 4, "i8", "f16")
    assert e.value.code == B.MS_ERR_UNSUPPORTED
    with pytest.raises(B.MsError) as e:
        B.Op(17, "f32", "f32", [1, 1, 1])
    assert e.value.code == B.MS_ERR_BAD_ARG
    assert B.lib().ms_op_create(None, None) == B.MS_ERR_BAD_ARG
    B.lib().ms_op_destroy(None)
    B.lib().ms_variant_destroy(None)
    with pytest.raises(B.MsError) as e:
        B.conv2d_op(1, 8, 8, 4, 4, 3, 3, in_dtype="f32", out_dtype="f32").space()
    assert e.value.code == B.MS_ERR_UNSUPPORTED


def slot_names(sp):
    return [sp.slots[i].name.decode() for i in range(sp.n_slots)]


def test_space_composition_by_flags():
    op = B.gemm_op(128, 128, 128, "f32")
    assert slot_names(op.space(B.SPACE_UNROLL)) == ["i", "j", "k", "unroll"]
    assert op.space(B.SPACE_UNROLL).family == B.FAM_GEMM_ALU
    assert slot_names(op.space(0)) == ["i", "j", "k"]
    sp = op.space()
    assert slot_names(sp) == ["i", "j", "k", "unroll", "cache_read", "vectorize", "vectorize_b", "storage_align", "reorder"]
    un = sp.slots[3]
    assert [un.candidates[i] for i in range(un.n_candidates)] == [0, 16, 64]
    op = B.gemm_op(1024, 1024, 1024, "f16")
    sp = op.space()
    assert sp.family == B.FAM_GEMM_MFMA and slot_names(sp)[0] == "tensorize"
    t = sp.slots[0]
    assert [t.candidates[i] for i in range(t.n_candidates)] == [161616, 323208, 161632, 323216]
    assert sp.slots[1].depends_on == 0 and [sp.slots[1].extent_by_choice[c] for c in range(4)] == [64, 32, 64, 32]
    assert [sp.slots[3].extent_by_choice[c] for c in range(4)] == [64, 128, 32, 64]
    assert op.space(B.SPACE_DEFAULT & ~B.SPACE_TENSORIZE).family == B.FAM_GEMM_ALU
    op = B.dwconv2d_op(1, 112, 112, 32)
    assert slot_names(op.space()) == ["i", "j", "c", "unroll", "cache_read", "reorder"]
    # fp32 on the matrix cores is opt-in; all-ones masks (earlier tuning records) mean the default set
    op = B.gemm_op(128, 128, 128, "f32")
    assert op.space().family == B.FAM_GEMM_ALU and op.space(0xFFFFFFFF).family == B.FAM_GEMM_ALU
    sp = op.space(B.SPACE_DEFAULT | B.SPACE_TENSORIZE_F32)
    assert sp.family == B.FAM_GEMM_MFMA
    assert [sp.slots[0].candidates[i] for i in range(sp.slots[0].n_candidates)] == [161604, 323202]
    assert [sp.slots[1].extent_by_choice[c] for c in range(2)] == [8, 4] and [sp.slots[3].extent_by_choice[c] for c in range(2)] == [32, 64]
    assert B.dwconv2d_op(1, 8, 8, 4).space(B.SPACE_DEFAULT | B.SPACE_TENSORIZE_F32).family == B.FAM_DWCONV
    assert B.gemm_op(64, 64, 64, "f16").space(B.SPACE_DEFAULT | B.SPACE_TENSORIZE_F32).flags == B.SPACE_DEFAULT & ~B.SPACE_COMPUTE_AT


def test_space_size_matches_closed_form():
    op = B.gemm_op(128, 128, 128, "f32")
    assert abs(B.space_log10_size(op.space(B.SPACE_UNROLL)) - math.log10(120 ** 3 * 3)) < 1e-9


@pytest.mark.parametrize("extent", [128, 56, 144, 3136, 12])
def test_sampler_support_and_uniformity(extent):
    """sample-perfect-tile: only members of the brute-force support, all of them reached, uniform."""
    op = B.gemm_op(extent, 4, 4, "f32")
    sp = op.space(0)
    support = {tuple(t) for t in O.perfect_tiles(extent, 4).tolist()}
    n = len(support)
    draws = 60 * n
    cnt = collections.Counter()
    for idx in range(draws):
        t = B.trace_sample(sp, 11, idx)
        f = tuple(t.d[0].v[k] for k in range(4))
        assert f in support
        cnt[f] += 1
    assert set(cnt) == support
    exp = draws / n
    chi2 = sum((c - exp) ** 2 / exp for c in cnt.values())
    # chi-square with n-1 dof: mean n-1, sd sqrt(2(n-1)); 6 sigma
    assert chi2 < (n - 1) + 6 * math.sqrt(2 * (n - 1)), (chi2, n)


def test_sampler_is_deterministic_and_seed_dependent():
    op = B.gemm_op(1024, 1024, 1024, "f16")
    sp = op.space()
    a = [B.trace_sample(sp, 5, i).decisions() for i in range(20)]
    b = [B.trace_sample(sp, 5, i).decisions() for i in range(20)]
    c = [B.trace_sample(sp, 6, i).decisions() for i in range(20)]
    assert a == b and a != c and len({str(x) for x in a}) > 15


def test_categorical_frequencies():
    op = B.gemm_op(128, 128, 128, "f32")
    sp = op.space(B.SPACE_UNROLL)
    cnt = collections.Counter(B.trace_sample(sp, 3, i).d[3].v[0] for i in range(3000))
    assert set(cnt) == {0, 1, 2} and all(abs(c - 1000) < 150 for c in cnt.values())


def test_dependent_tile_extents_follow_the_tensorize_decision():
    op = B.gemm_op(1024, 1024, 1024, "f16")
    sp = op.space()
    seen = set()
    for i in range(200):
        t = B.trace_sample(sp, 9, i)
        code = sp.slots[0].candidates[t.d[0].v[0]]
        m, n, k = code // 10000, code // 100 % 100, code % 100
        seen.add(code)
        assert math.prod(t.d[1].v[q] for q in range(4)) == 1024 // m
        assert math.prod(t.d[2].v[q] for q in range(4)) == 1024 // n
        assert math.prod(t.d[3].v[q] for q in range(4)) == 1024 // k
    assert len(seen) == 4


def test_mutation_changes_one_decision_and_keeps_products():
    op = B.gemm_op(1024, 1024, 1024, "f16")
    sp = op.space()
    t = B.trace_sample(sp, 1, 0)
    changed_slots = collections.Counter()
    for s in range(400):
        m = B.trace_mutate(sp, t, s)
        a, b = t.decisions(), m.decisions()
        diff = [i for i in range(len(a)) if a[i] != b[i]]
        assert diff, "mutation returned the same trace"
        if diff[0] == 0:  # tensorize changed: dependent tiles are redrawn for the new unit
            assert set(diff) <= {0, 1, 2, 3}
        else:
            assert len(diff) == 1
            i = diff[0]
            if sp.slots[i].kind == B.SLOT_PERFECT_TILE:
                assert math.prod(a[i][1]) == math.prod(b[i][1])
                assert sum(1 for x, y in zip(a[i][1], b[i][1]) if x != y) == 2
        changed_slots[diff[0]] += 1
        code = sp.slots[0].candidates[m.d[0].v[0]]
        for l, u in zip((1, 2, 3), (code // 10000, code // 100 % 100, code % 100)):
            assert math.prod(m.d[l].v[q] for q in range(4)) * u == 1024
    assert len(changed_slots) == sp.n_slots


def test_text_round_trip():
    for op in [B.gemm_op(128, 128, 128, "f32"), B.gemm_op(1024, 1024, 1024, "f16"), B.dwconv2d_op(1, 112, 112, 32)]:
        sp = op.space()
        for i in range(10):
            t = B.trace_sample(sp, 2, i)
            text = B.trace_to_text(op, sp, t)
            assert text.count("sample-") == sp.n_slots
            back = B.trace_from_text(sp, text)
            assert back.decisions() == t.decisions()
            assert bytes(back) == bytes(t)


def test_text_worked_example_split():
    """The split of Section 3.1's figure: loop of 1024 into extents 32, 8, 4 (here with a leading 1)."""
    op = B.gemm_op(1024, 4, 4, "f32")
    sp = op.space(0)
    t = B.make_trace(sp, [[1, 32, 8, 4], [1, 1, 4, 1], [1, 1, 4, 1]])
    p = B.trace_validate(op, sp, t)
    assert list(p.ti) == [1, 32, 8, 4] and p.block_m == 1024 and p.threads == 8 * 4
    text = B.trace_to_text(op, sp, t)
    assert "split(loop=i, factors=[1, 32, 8, 4])" in text
    cov = B.variant_coverage(op, p, 1024 * 4)
    assert np.all(cov == 1)


def test_text_errors():
    op = B.gemm_op(128, 128, 128, "f32")
    sp = op.space(B.SPACE_UNROLL)
    t = B.trace_sample(sp, 0, 0)
    text = B.trace_to_text(op, sp, t)
    lines = text.splitlines()
    trunc = "\n".join(l for l in lines if "slot=unroll" not in l)
    with pytest.raises(B.MsError) as e:
        B.trace_from_text(sp, trunc)
    assert e.value.code == B.MS_ERR_INVALID_TRACE and "truncated" in str(e.value)
    swapped = text.replace("slot=i,", "slot=q,")
    with pytest.raises(B.MsError):
        B.trace_from_text(sp, swapped)


def test_validator_rejections():
    op = B.gemm_op(128, 128, 128, "f32")
    sp = op.space()

    def mk(i, j, k, unroll=0, cache=1, vec=1, vec_b=1, pad=0, reorder=0):
        return B.make_trace(sp, [i, j, k, [unroll], [cache], [vec], [vec_b], [pad], [reorder]])

    ok = mk([4, 2, 8, 2], [4, 2, 16, 1], [4, 4, 4, 2])
    p = B.trace_validate(op, sp, ok)
    assert p.threads == 128 and p.block_m == 32 and p.block_n == 32 and p.block_k == 32 and p.grid[0] == 16
    assert p.lds_bytes == 4 * (32 * 32 + 32 * 32) and p.acc_per_thread == 8

    def rejected(t, word):
        with pytest.raises(B.MsError) as e:
            B.trace_validate(op, sp, t)
        assert e.value.code == B.MS_ERR_INVALID_TRACE and word in str(e.value), str(e.value)

    rejected(mk([4, 2, 8, 4], [4, 2, 16, 1], [4, 4, 4, 2]), "multiply to")          # product != extent
    rejected(mk([1, 1, 128, 1], [1, 1, 128, 1], [4, 4, 4, 2]), "threads per workgroup")  # 16384 threads
    rejected(mk([1, 16, 1, 8], [1, 16, 1, 8], [128, 1, 1, 1]), "accumulators per lane")
    rejected(mk([1, 2, 32, 2], [1, 2, 32, 2], [1, 1, 128, 1], cache=2), "LDS tile needs")  # 2*(128*128*2)*4 = 256 KiB
    rejected(mk([4, 2, 8, 2], [4, 2, 16, 1], [4, 4, 4, 2], cache=0, pad=1), "nothing to pad")
    bad = ok.copy()
    bad.d[0].v[0] = 0
    rejected(bad, "factor 0 is 0")
    bad = ok.copy()
    bad.d[3].v[0] = 7
    rejected(bad, "outside")
    bad = ok.copy()
    bad.n = 5
    rejected(bad, "truncated")
    bad = ok.copy()
    bad.d[1].slot_id = 99
    rejected(bad, "slot id")
    # vector width must divide the contiguous tile extent: BK = 2 with 4-wide loads of A; BN = 2 for B
    rejected(mk([4, 2, 8, 2], [4, 2, 16, 1], [64, 1, 1, 2], vec=4), "vector width")
    rejected(mk([4, 2, 8, 2], [64, 1, 2, 1], [4, 4, 4, 2], vec_b=4), "vector width")
    # forced smaller hardware limits reject what passed before, and are restorable
    lim = B.get_limits()
    small = B.ms_limits(64, 4096, 16, 64, 2)
    B.set_limits(small)
    try:
        rejected(ok, "threads per workgroup")
    finally:
        B.set_limits(lim)
    B.trace_validate(op, sp, ok)


def test_validator_mfma_rules():
    op = B.gemm_op(1024, 1024, 1024, "f16")
    sp = op.space()

    def mk(mfma, i, j, k, unroll=0, cache=2, vec=8, vec_b=8, pad=0, reorder=0, cw=0):
        return B.make_trace(sp, [[mfma], i, j, k, [unroll], [cache], [vec], [vec_b], [pad], [reorder], [cw]])

    p = B.trace_validate(op, sp, mk(323216, [4, 2, 2, 2], [4, 2, 2, 2], [16, 1, 2, 2]))
    assert (p.block_m, p.block_n, p.block_k) == (256, 256, 64) and p.waves == 4 and p.threads == 256
    assert p.acc_per_thread == 256 and p.lds_bytes == 2 * (64 // 8) * (256 * 16 + 256 * 16)
    with pytest.raises(B.MsError) as e:
        B.trace_validate(op, sp, mk(323216, [1, 1, 32, 1], [32, 1, 1, 1], [16, 1, 2, 2]))
    assert "wavefronts" in str(e.value)
    with pytest.raises(B.MsError) as e:
        B.trace_validate(op, sp, mk(323216, [2, 4, 1, 4], [2, 4, 1, 4], [16, 1, 2, 2]))
    assert "accumulators" in str(e.value)
    with pytest.raises(B.MsError) as e:  # i tile counted for 16-wide intrinsic but 32-wide chosen
        B.trace_validate(op, sp, mk(323216, [4, 2, 2, 4], [4, 2, 2, 2], [16, 1, 2, 2]))
    assert "multiply to" in str(e.value)


def test_validator_conv_compute_location_rules():
    """sample-compute-location for conv2d: LDS footprints of the resident patch / weights and the constraints
    each location puts on the other decisions (all checked on the host)."""
    op = B.conv2d_op(1, 56, 56, 64, 64, 3, 3, stride=1, pad=1)
    sp = op.space()
    assert slot_names(sp)[-1] == "compute_at"

    def mk(ca, mfma=161632, i=(14, 7, 2, 1), j=(1, 2, 2, 1), k=(9, 1, 2, 1), unroll=64, cache=2, vec=8, vec_b=8, pad=1, reorder=0, cw=1):
        return B.make_trace(sp, [[mfma], list(i), list(j), list(k), [unroll], [cache], [vec], [vec_b], [pad], [reorder], [cw], [ca]])

    planes_b = (64 // 8) * (64 * 16 + 16)             # one k step of the weights: 8 k-group planes of 64 fragments + pad
    patch = 6 * 58 * (64 * 2 + 16)                    # 4 output rows -> 6 input rows x (56 + 2) columns x padded pixel
    ctile = 224 * (64 * 2 + 16)
    p0 = B.trace_validate(op, sp, mk(0))
    assert p0.compute_at == 0 and p0.threads == 256
    p1 = B.trace_validate(op, sp, mk(1))
    assert p1.lds_bytes == 2 * planes_b + patch and p1.grid[0] == 14
    p2 = B.trace_validate(op, sp, mk(2))
    assert p2.lds_bytes == 9 * planes_b + patch + ctile and p2.threads == 256
    p3 = B.trace_validate(op, sp, mk(3))
    assert p3.waves == 8 and p3.threads == 512 and p3.lds_bytes == p2.lds_bytes  # four helper wavefronts
    p4 = B.trace_validate(op, sp, mk(4))
    assert p4.lds_bytes == planes_b + patch + ctile
    assert len({p.key for p in (p0, p1, p2, p3, p4)}) == 5
    for ca, kw, needle in [(1, dict(cache=4), "cache_read"), (2, dict(cache=3), "cache_read"), (2, dict(reorder=2), "reorder"),
                           (3, dict(cw=0), "cache_write"), (3, dict(cache=1), "cache_read"),
                           (4, dict(i=(7, 14, 2, 1), j=(1, 4, 1, 1)), "weights in registers"),
                           (2, dict(i=(7, 14, 2, 1), k=(1, 9, 2, 1)), "LDS")]:
        with pytest.raises(B.MsError) as e:
            B.trace_validate(op, sp, mk(ca, **kw))
        assert needle in str(e.value), (ca, kw, str(e.value))
    # a 16-pixel tile of a 12-wide image starts in the middle of a row: 3 output rows, 5 patch rows; Cin = 24 is not
    # a multiple of the 32-deep intrinsic
    op2 = B.conv2d_op(1, 12, 12, 32, 32, 3, 3, stride=1, pad=1)
    sp2 = op2.space()
    t = B.make_trace(sp2, [[161632], [9, 1, 1, 1], [1, 2, 1, 1], [9, 1, 1, 1], [0], [1], [8], [8], [0], [0], [0], [1]])
    assert B.trace_validate(op2, sp2, t).lds_bytes == 1 * (32 // 8) * (32 * 16) + 5 * 14 * 64
    op3 = B.conv2d_op(1, 12, 12, 16, 32, 3, 3, stride=1, pad=1)
    sp3 = op3.space()
    cands = [sp3.slots[0].candidates[i] for i in range(sp3.slots[0].n_candidates)]
    assert 161616 in cands
    t = B.make_trace(sp3, [[161616], [9, 1, 1, 1], [1, 2, 1, 1], [9, 1, 1, 1], [0], [1], [8], [8], [0], [0], [0], [1]])
    assert B.trace_validate(op3, sp3, t).compute_at == 1
    assert 161632 in cands
    if True:
        # K = 144 is rounded up to 160 for the 32-deep intrinsic (5 k steps, zero padded by the im2col loader only)
        t = B.make_trace(sp3, [[161632], [9, 1, 1, 1], [1, 2, 1, 1], [5, 1, 1, 1], [0], [1], [8], [8], [0], [0], [0], [1]])
        with pytest.raises(B.MsError) as e:
            B.trace_validate(op3, sp3, t)
        assert "Cin" in str(e.value) and "compute_at must be 0" in str(e.value)
        t = B.make_trace(sp3, [[161632], [9, 1, 1, 1], [1, 2, 1, 1], [5, 1, 1, 1], [0], [1], [8], [8], [0], [0], [0], [0]])
        assert B.trace_validate(op3, sp3, t).block_k == 32


CONFIG_OPS = [
    lambda: B.gemm_op(128, 128, 128, "f32"),
    lambda: B.gemm_op(256, 128, 64, "f16"),
    lambda: B.bmm_op(3, 128, 128, 64, True, "f16"),
    lambda: B.gemm_op(128, 64, 128, "i8"),
    lambda: B.conv2d_op(1, 28, 28, 16, 32, 3, 3, stride=1, pad=1),
    lambda: B.dwconv2d_op(1, 28, 28, 12),
    lambda: B.dwconv2d_op(2, 14, 14, 18, stride=2),
]


@pytest.mark.parametrize("mk", CONFIG_OPS)
def test_interpreter_covers_every_output_once(mk):
    """The split/bind structure derived from any valid trace tiles the output exactly once."""
    op = mk()
    sp = op.space()
    elems = op.tensor_bytes(-1) // {B.F32: 4, B.F16: 2, B.BF16: 2, B.I32: 4}[op.desc().out_dtype]
    for idx in range(25):
        t = B.trace_sample_valid(op, sp, 21, idx)
        p = B.trace_validate(op, sp, t)
        cov = B.variant_coverage(op, p, elems)
        assert cov.min() == 1 and cov.max() == 1, t.decisions()


# ---------------------------------------------------------------- softmax / norm (row reductions)

def test_reduce_ops_descriptor_loops_and_work():
    op = B.softmax_op(2, 48, 96, "f16")
    assert op.loops() == [("i", 96, False), ("k", 96, True)]
    assert op.tensor_bytes(0) == 2 * 48 * 96 * 2 and op.tensor_bytes(-1) == 2 * 48 * 96 * 2
    assert op.work()[1] == 2 * 48 * 96 * 4
    op = B.norm_op(3, 16, 20, "bf16")
    assert op.loops() == [("i", 3, False), ("k", 320, True)]
    assert op.tensor_bytes(0) == 3 * 320 * 2 and op.tensor_bytes(-1) == 3 * 4
    assert op.work() == (2.0 * 3 * 320, 3 * 320 * 2 + 12.0)
    with pytest.raises(B.MsError):
        B.Op(B.OP_NORM, "f32", "f16", [1, 4, 4])       # the norm is written in fp32
    with pytest.raises(B.MsError):
        B.Op(B.OP_SOFTMAX, "i8", "i32", [1, 4, 4])
    with pytest.raises(B.MsError):
        B.Op(B.OP_SOFTMAX, "f32", "f32", [1, 4, 4], stride=1)


def test_reduce_space_coverage_and_text_round_trip():
    for op, elems in ((B.softmax_op(1, 256, 256), 65536), (B.softmax_op(3, 20, 96, "f16"), 5760), (B.norm_op(6, 32, 24), 6)):
        sp = op.space()
        assert sp.family == B.FAM_REDUCE
        names = [sp.slots[i].name.decode() for i in range(sp.n_slots)]
        assert names[:2] == ["i", "k"] and (names[2:] == ["cache_read"]) == (elems != 6)
        for idx in range(20):
            t = B.trace_sample_valid(op, sp, 33, idx)
            p = B.trace_validate(op, sp, t)
            assert p.threads == p.ti[2] * p.tk[2] and p.threads % 64 == 0 and p.grid[0] == p.ti[0]
            cov = B.variant_coverage(op, p, elems)
            assert cov.min() == 1 and cov.max() == 1, t.decisions()
            text = B.trace_to_text(op, sp, t)
            assert "cross-thread reduction over %d lanes" % p.tk[2] in text
            assert B.trace_from_text(sp, text).decisions() == t.decisions()
    # without the cache-read module the softmax space has only the two tile slots
    assert B.softmax_op(1, 8, 64).space(0).n_slots == 2


def test_reduce_validator_rejections():
    op = B.softmax_op(1, 64, 256)
    sp = op.space()

    def why(vals):
        with pytest.raises(B.MsError) as e:
            B.trace_validate(op, sp, B.make_trace(sp, vals))
        assert e.value.code == B.MS_ERR_INVALID_TRACE
        return str(e.value)

    assert "at most 16 bytes" in why([[1, 1, 64, 1], [1, 1, 32, 8], [0]])
    assert "power of two" not in why([[1, 1, 64, 1], [1, 1, 32, 8], [0]])
    assert "whole number of wavefronts" in why([[32, 1, 2, 1], [4, 4, 16, 1], [0]])
    assert "threads per workgroup" in why([[1, 1, 64, 1], [2, 1, 32, 4], [0]])
    assert "register budget" in why([[1, 1, 8, 8], [8, 4, 8, 1], [1]])
    op3 = B.softmax_op(1, 64, 96)
    sp3 = op3.space()
    with pytest.raises(B.MsError) as e:
        B.trace_validate(op3, sp3, B.make_trace(sp3, [[1, 1, 64, 1], [1, 8, 12, 1], [0]]))
    assert "power of two" in str(e.value)
    opn = B.norm_op(1, 256, 256)
    spn = opn.space()
    with pytest.raises(B.MsError) as e:
        B.trace_validate(opn, spn, B.make_trace(spn, [[1, 1, 1, 1], [512, 2, 16, 4]]))
    assert "one wavefront per row" in str(e.value)


def test_transposed_conv_descriptor_and_space():
    op = B.conv2d_transposed_op(1, 4, 4, 512, 256, 4, 4, stride=2, pad=1)
    assert op.loops() == [("i", 64, False), ("j", 256, False), ("k", 8192, True)]      # 8 x 8 output pixels
    assert op.tensor_bytes(-1) == 64 * 256 * 2 and op.tensor_bytes(0) == 16 * 512 * 2 and op.tensor_bytes(1) == 8192 * 256 * 2
    assert op.work()[0] == 2.0 * 16 * 8192 * 256
    sp = op.space()
    assert sp.family == B.FAM_GEMM_MFMA
    assert "compute_at" not in [sp.slots[i].name.decode() for i in range(sp.n_slots)]
    t = B.trace_sample_valid(op, sp, 2, 0)
    p = B.trace_validate(op, sp, t)
    assert p.compute_at == 0
    cov = B.variant_coverage(op, p, 64 * 256)
    assert cov.min() == 1 and cov.max() == 1
    assert "op=conv2d_transposed_nhwc" in B.trace_to_text(op, sp, t)
    with pytest.raises(B.MsError):
        B.Op(B.OP_CONV2D_TRANSPOSED_NHWC, "f16", "f16", [1, 4, 4, 8, 8, 3, 3], stride=1, pad=0, dilation=2)
    with pytest.raises(B.MsError):
        B.conv2d_transposed_op(1, 1, 1, 8, 8, 2, 2, stride=1, pad=1)   # empty output


def test_grouped_conv_descriptor_space_and_coverage():
    op = B.conv2d_op(1, 56, 56, 64, 128, 3, 3, stride=2, pad=1, groups=4)
    assert op.loops() == [("g", 4, False), ("i", 784, False), ("j", 32, False), ("k", 144, True)]
    assert op.tensor_bytes(1) == 3 * 3 * 16 * 128 * 2 and op.tensor_bytes(-1) == 784 * 128 * 2 and op.tensor_bytes(2) == 128 * 4
    assert op.work()[0] == 2.0 * 784 * 128 * 144
    sp = op.space()
    ca = [sp.slots[i] for i in range(sp.n_slots) if sp.slots[i].name == b"compute_at"][0]
    assert list(ca.weight)[:5] == [1, 1, 1, 1, 1]      # 16 channels per group: every compute location
    seen = set()
    for idx in range(10):
        t = B.trace_sample_valid(op, sp, 7, idx)
        p = B.trace_validate(op, sp, t)
        assert p.grid[2] == 4
        seen.add(p.compute_at)
        cov = B.variant_coverage(op, p, 784 * 128)
        assert cov.min() == 1 and cov.max() == 1
    with pytest.raises(B.MsError):
        B.conv2d_op(1, 8, 8, 30, 64, 3, 3, groups=4)          # 4 does not divide 30
    with pytest.raises(B.MsError):
        B.Op(B.OP_CONV2D_TRANSPOSED_NHWC, "f16", "f16", [1, 4, 4, 16, 16, 2, 2, 2], stride=1, pad=0)
    # a dense convolution is unchanged by the new field: same kernel key with groups 0 and 1
    d0, d1 = B.conv2d_op(1, 8, 8, 16, 32, 3, 3, pad=1), B.conv2d_op(1, 8, 8, 16, 32, 3, 3, pad=1, groups=1)
    s0 = d0.space()
    t = B.trace_sample_valid(d0, s0, 1, 0)
    assert B.trace_validate(d0, s0, t).key == B.trace_validate(d1, d1.space(), t).key


def test_conv1d_descriptor_runs_on_the_conv2d_space():
    op = B.conv1d_op(1, 256, 64, 128, 3, stride=2, pad=1)
    assert op.loops() == [("i", 128, False), ("j", 128, False), ("k", 192, True)]        # OL = 128
    d = op.desc()
    assert d.kind == B.OP_CONV1D_NWC and list(d.dims)[:5] == [1, 256, 64, 128, 3]        # the descriptor as given
    assert op.tensor_bytes(0) == 256 * 64 * 2 and op.tensor_bytes(1) == 3 * 64 * 128 * 2 and op.tensor_bytes(-1) == 128 * 128 * 2
    sp = op.space()
    assert sp.family == B.FAM_GEMM_MFMA and [sp.slots[i].name for i in range(sp.n_slots)][-1] == b"compute_at"
    t = B.trace_sample_valid(op, sp, 3, 0)
    p = B.trace_validate(op, sp, t)
    assert "op=conv1d_nwc" in B.trace_to_text(op, sp, t)
    # not the same kernel as the 1 x 3 conv2d over an image of height 1, which is also padded vertically (3 output rows)
    op2 = B.conv2d_op(1, 1, 256, 64, 128, 1, 3, stride=2, pad=1)
    assert op2.loops()[0] == ("i", 2 * 128, False)
    with pytest.raises(B.MsError):
        B.conv1d_op(1, 2, 8, 16, 5, stride=1, pad=0)                                      # empty output


def test_conv3d_descriptor_and_space():
    op = B.conv3d_op(1, 16, 224, 224, 3, 64, 7, stride=2, pad=3)
    assert op.loops() == [("i", 8 * 112 * 112, False), ("j", 64, False), ("k", 343 * 3, True)]
    assert op.desc().kind == B.OP_CONV3D_NDHWC and list(op.desc().dims)[:7] == [1, 16, 224, 224, 3, 64, 7]
    assert op.tensor_bytes(0) == 16 * 224 * 224 * 3 * 2 and op.tensor_bytes(1) == 1029 * 64 * 2
    sp = op.space()
    ca = [sp.slots[i] for i in range(sp.n_slots) if sp.slots[i].name == b"compute_at"][0]
    assert list(ca.weight)[:5] == [1, 0, 0, 0, 0]
    op2 = B.conv3d_op(2, 6, 8, 8, 16, 32, 3, stride=1, pad=1)
    sp2 = op2.space()
    t = B.trace_sample_valid(op2, sp2, 5, 0)
    p = B.trace_validate(op2, sp2, t)
    cov = B.variant_coverage(op2, p, 2 * 6 * 8 * 8 * 32)
    assert cov.min() == 1 and cov.max() == 1 and "op=conv3d_ndhwc" in B.trace_to_text(op2, sp2, t)
    # another depth is another kernel
    op3 = B.conv3d_op(2, 5, 8, 8, 16, 32, 3, stride=1, pad=1)
    assert B.trace_validate(op3, op3.space(), B.trace_sample_valid(op3, op3.space(), 5, 0)).key != p.key


def test_filter_row_layout_space_and_rules():
    op = B.conv2d_op(1, 224, 224, 3, 64, 7, 7, stride=2, pad=3)
    sp = op.space(B.SPACE_DEFAULT | B.SPACE_TAP_ROWS)
    assert sp.flags & B.SPACE_TAP_ROWS
    ks = [sp.slots[i] for i in range(sp.n_slots) if sp.slots[i].name == b"k"][0]
    tz = sp.slots[0]
    # 7 runs of 21 elements, each rounded up to the intrinsic's k: 7*32/16, 7*24/8, 7*32/32, 7*32/16
    assert {tz.candidates[c]: ks.extent_by_choice[c] for c in range(tz.n_candidates)} == {161616: 14, 323208: 21, 161632: 7, 323216: 14}
    ca = [sp.slots[i] for i in range(sp.n_slots) if sp.slots[i].name == b"compute_at"][0]
    assert list(ca.weight)[:5] == [1, 1, 1, 1, 1]
    seen = set()
    for idx in range(40):
        t = B.trace_sample_valid(op, sp, 11, idx)
        p = B.trace_validate(op, sp, t)
        assert p.tap_rows == 1 and p.tile_unit[2] * p.tk[0] * p.tk[1] * p.tk[2] * p.tk[3] in (224, 168)
        seen.add(p.compute_at)
        assert "op=conv2d_nhwc" in B.trace_to_text(op, sp, t)
    assert {0, 1, 2} <= seen
    # the same trace in the default space is another kernel (or invalid): the layout is part of the key
    assert not (op.space().flags & B.SPACE_TAP_ROWS)
    # pixels that start at odd multiples of 2 bytes: im2col staging only
    op2 = B.conv2d_op(1, 16, 16, 3, 32, 3, 3, stride=1, pad=1)
    sp2 = op2.space(B.SPACE_DEFAULT | B.SPACE_TAP_ROWS)
    ca2 = [sp2.slots[i] for i in range(sp2.n_slots) if sp2.slots[i].name == b"compute_at"][0]
    assert list(ca2.weight)[:5] == [1, 0, 0, 0, 0]
    # the flag is dropped where the layout does not apply: dilated, grouped, transposed, other operators
    assert not (B.conv2d_op(1, 16, 16, 4, 32, 3, 3, pad=2, dilation=2).space(0x2ff).flags & B.SPACE_TAP_ROWS)
    assert not (B.conv2d_op(1, 16, 16, 8, 32, 3, 3, pad=1, groups=2).space(0x2ff).flags & B.SPACE_TAP_ROWS)
    assert not (B.gemm_op(128, 128, 128, "f16").space(0x2ff).flags & B.SPACE_TAP_ROWS)


# ---------------------------------------------------------------- kernel identity

@pytest.mark.parametrize("mk", CONFIG_OPS + [lambda: B.softmax_op(1, 64, 256)])
def test_equal_kernel_text_means_equal_key(mk):
    """The key names the kernel: traces whose decisions resolve to the same template options (e.g. unroll budgets
    that are clamped alike) share one key, so a search never compiles or measures one kernel twice; different
    options give different keys."""
    op = mk()
    sp = op.space()
    by_text, by_key = {}, {}
    for idx in range(300):
        p = B.trace_validate(op, sp, B.trace_sample_valid(op, sp, 33, idx))
        text = B.variant_kernel_text(op, p)
        assert by_text.setdefault(text, p.key) == p.key, "one kernel, two keys:\n" + text
        assert by_key.setdefault(p.key, text) == text, "one key, two kernels"
    assert len(by_text) > 20


BODY_OPS = [
    (lambda: B.softmax_op(1, 4096, 1000), B.SPACE_DEFAULT, B.BODY_ROW_VECTORS),
    (lambda: B.dwconv2d_op(4, 57, 57, 144, stride=2), B.SPACE_DEFAULT, B.BODY_STRIPS),
    (lambda: B.conv2d_op(1, 224, 224, 3, 64, 7, 7, stride=2, pad=3), B.SPACE_DEFAULT | B.SPACE_TAP_ROWS, B.BODY_IMAGE_ROWS),
    (lambda: B.conv3d_op(1, 16, 64, 64, 3, 64, 7, stride=2, pad=3), B.SPACE_DEFAULT, B.BODY_IMAGE_ROWS),
]


@pytest.mark.parametrize("mk,flags,body", BODY_OPS)
def test_traces_of_one_body_are_one_kernel_with_one_key(mk, flags, body):
    """A body other than the nest reads the operator and its own tile: whatever the decisions, one text and one key, and
    no text with two keys or key with two texts across the bodies of a space."""
    op = mk()
    sp = op.space(flags)
    by_text, by_key, of_body = {}, {}, set()
    for idx in range(300):
        p = B.trace_validate(op, sp, B.trace_sample_valid(op, sp, 34, idx))
        text = B.variant_kernel_text(op, p)
        assert by_text.setdefault(text, p.key) == p.key and by_key.setdefault(p.key, text) == text
        if p.body != B.BODY_NEST:
            assert p.body == body
            of_body.add(p.key)
    assert len(of_body) == 1


@pytest.mark.parametrize("mk,flags,body", [
    (lambda: B.softmax_op(1, 1024, 1000), B.SPACE_DEFAULT, B.BODY_ROW_VECTORS),
    (lambda: B.softmax_op(3, 32, 24, "f16"), B.SPACE_DEFAULT, B.BODY_ROW_VECTORS),
    (lambda: B.dwconv2d_op(2, 57, 23, 7, stride=2), B.SPACE_DEFAULT, B.BODY_STRIPS),
    (lambda: B.dwconv2d_op(1, 4, 38, 1, 2, 2, pad=0), B.SPACE_DEFAULT, B.BODY_STRIPS),
    (lambda: B.conv2d_op(2, 59, 104, 3, 96, 5, 5, stride=2, pad=4), B.SPACE_DEFAULT | B.SPACE_TAP_ROWS, B.BODY_IMAGE_ROWS),
    (lambda: B.conv3d_op(2, 5, 13, 16, 4, 64, 5, stride=2, pad=2), B.SPACE_DEFAULT, B.BODY_IMAGE_ROWS),
    (lambda: B.conv1d_op(2, 528, 3, 32, 7, stride=2, pad=3), B.SPACE_DEFAULT, B.BODY_IMAGE_ROWS),
    (lambda: B.conv1d_op(1, 2080, 2, 64, 3, stride=1, pad=1), B.SPACE_DEFAULT, B.BODY_IMAGE_ROWS),
    (lambda: B.conv2d_op(1, 4, 784, 3, 64, 7, 7, stride=2, pad=3), B.SPACE_DEFAULT, B.BODY_IMAGE_ROWS)])
def test_params_describe_the_body_that_runs(mk, flags, body):
    """Workgroup, grid, LDS, coverage and features of a body other than the nest are those of the kernel it launches, and
    the limits hold for that kernel: under tighter ones the trace keeps its nest."""
    op = mk()
    sp = op.space(flags)
    elems = op.tensor_bytes(-1) // {B.F32: 4, B.F16: 2, B.BF16: 2}[op.desc().out_dtype]
    K = int(np.prod([e for n, e, red in op.loops() if red]))
    traces = [B.trace_sample_valid(op, sp, 35, idx) for idx in range(60)]
    traces = [t for t in traces if B.trace_validate(op, sp, t).body == body]
    assert len(traces) >= 10
    p = B.trace_validate(op, sp, traces[0])
    text = B.variant_kernel_text(op, p)
    d = {k: int(v) for k, v in (line[2:].split("=") for line in text.splitlines()[1:])}
    threads = {B.BODY_ROW_VECTORS: lambda: d["ROW_WAVES"] * 64, B.BODY_STRIPS: lambda: d["STRIP_THREADS"],
               B.BODY_IMAGE_ROWS: lambda: d["CR_WAVES"] * 64}[body]()
    r = B.Variant(op, sp, traces[0]).resources()
    assert p.threads == threads and p.waves == threads // 64 and p.lds_bytes == r.lds_bytes
    cov = B.variant_coverage(op, p, elems)
    assert cov.min() == 1 and cov.max() == 1
    red = B.variant_reduction_coverage(op, p)
    assert len(red) == K and red.min() == 1 and red.max() == 1
    for t in traces[1:]:
        q = B.trace_validate(op, sp, t)
        assert (q.threads, q.waves, list(q.grid), q.lds_bytes, q.acc_per_thread) == (p.threads, p.waves, list(p.grid), p.lds_bytes, p.acc_per_thread)
        assert np.array_equal(B.variant_features(op, q), B.variant_features(op, p))
    assert "body=" in B.trace_to_text(op, sp, traces[0])
    assert "workgroup=%d threads, grid=%d" % (p.threads, p.grid[0] * p.grid[1] * p.grid[2]) in B.trace_to_text(op, sp, traces[0])
    lim = B.get_limits()
    try:
        for field, value in (("max_threads", p.threads - 1), ("max_acc_per_thread", p.acc_per_thread - 1)) + (
                (("max_lds_bytes", p.lds_bytes - 1),) if p.lds_bytes else ()):
            tight = B.get_limits()
            setattr(tight, field, value)
            B.set_limits(tight)
            for t in traces:
                try:
                    q = B.trace_validate(op, sp, t)
                except B.MsError:
                    continue
                assert q.threads <= tight.max_threads and q.lds_bytes <= tight.max_lds_bytes and q.acc_per_thread <= tight.max_acc_per_thread
    finally:
        B.set_limits(lim)


@pytest.mark.parametrize("mk,elements", [(lambda: B.conv1d_op(1, 65536, 1, 64, 7, stride=2, pad=3), 2 * 512 + 16),
                                         (lambda: B.conv1d_op(64, 16384, 4, 64, 7, stride=1, pad=3), 4 * 512 + 32),
                                         (lambda: B.conv2d_op(1, 64, 4096, 4, 64, 3, 3, stride=1, pad=1), 3 * (4 * 512 + 32))])
def test_image_rows_stage_the_columns_of_a_tile_not_whole_rows(mk, elements):
    """Rows of many tiles: the LDS beyond the weights holds at most the columns that a tile of 512 pixels meets."""
    op = mk()
    sp = op.space()
    p = next(p for p in (B.trace_validate(op, sp, B.trace_sample_valid(op, sp, 36, n)) for n in range(50)) if p.body == B.BODY_IMAGE_ROWS)
    weights = p.block_k * (p.block_n * 2 + 32)
    assert p.lds_bytes <= max(weights + 2 * elements, p.waves * 32 * (p.block_n * 2 + 16))


@pytest.mark.parametrize("N,H,W_,Cin,k,stride,pad", [(2, 8, 8, 64, 4, 2, 1), (2, 8, 4, 64, 4, 4, 0), (2, 8, 4, 64, 6, 2, 2), (1, 8, 6, 64, 3, 3, 0)])
def test_phases_cover_the_output_and_the_filter_once(N, H, W_, Cin, k, stride, pad):
    """Transposed convolution: the kernel text says which traces walk the taps of one output phase; the row order of those
    is a permutation of the pixels and their taps of all phases together are the filter."""
    op = B.conv2d_transposed_op(N, H, W_, Cin, 32, k, k, stride=stride, pad=pad)
    sp = op.space(B.SPACE_DEFAULT | B.SPACE_RFACTOR)
    seen = {}
    for idx in range(300):
        t = B.trace_sample_valid(op, sp, 37, idx)
        p = B.trace_validate(op, sp, t)
        qualifies = (N * H * W_) % p.block_m == 0 and Cin % p.block_k == 0 and p.tk[0] % (stride * stride * p.rfactor) == 0 and p.cache_read <= 4
        assert (p.body == B.BODY_PHASES) == qualifies and p.body in (B.BODY_NEST, B.BODY_PHASES)
        assert ("-DCV_PHASES=%d" % qualifies) in B.variant_kernel_text(op, p).splitlines()
        seen[qualifies] = seen.get(qualifies, 0) + 1
        if seen[qualifies] > 12:
            continue
        for cov in (B.variant_coverage(op, p, N * H * W_ * stride * stride * 32), B.variant_reduction_coverage(op, p)):
            assert cov.min() == 1 and cov.max() == 1, t.decisions()
    assert seen.get(True, 0) > 3 and seen.get(False, 0) > 3, seen


def test_double_steps_are_one_kernel_per_wave_tile():
    """Ping-pong rings of whole 128-byte k rows: every ring, k split and unroll budget of one wave tile, in 32-row or 16-row
    intrinsics, is one kernel; its parameters are those of the code object and cover the output and the reduction once.
    Odd reductions and k tiles of 256 bytes keep the nest, and so do stages that a tightened LDS limit does not take."""
    op = B.gemm_op(512, 512, 1024, "f16")
    sp = op.space()

    def params(mfma, i, j, k, cache, cw=1, op=op, sp=sp, unroll=0):
        return B.trace_validate(op, sp, B.make_trace(sp, [[mfma], i, j, k, [unroll], [cache], [8], [8], [0], [3], [cw]]))

    same = [params(323216, [2, 1, 2, 4], [2, 1, 4, 2], [32, 1, 1, 2], 10), params(323216, [2, 1, 2, 4], [2, 1, 4, 2], [32, 1, 2, 1], 9, unroll=16),
            params(161632, [2, 1, 2, 8], [2, 1, 4, 4], [32, 1, 1, 1], 8)]
    assert all(p.body == B.BODY_DOUBLE_STEPS and p.body_tile == 2 for p in same)
    assert len({(p.key, B.variant_kernel_text(op, p)) for p in same}) == 1
    p = params(323216, [4, 1, 2, 2], [4, 1, 4, 1], [16, 1, 2, 2], 8)
    assert p.body_tile == 4 and p.key != same[0].key
    for p in (same[0], p):
        assert p.mfma == 161632 and p.block_k == 32 and p.lds_bytes == p.body_tile * (p.block_m + p.block_n) * 128 + p.waves * 16 * p.tj[3] * 16 * 2
        for cov in (B.variant_coverage(op, p, 512 * 512), B.variant_reduction_coverage(op, p)):
            assert cov.min() == 1 and cov.max() == 1
    t = B.make_trace(sp, [[323216], [4, 1, 2, 2], [4, 1, 4, 1], [16, 1, 2, 2], [0], [8], [8], [8], [0], [3], [1]])
    v = B.Variant(op, sp, t)
    assert v.resources().lds_bytes == v.params().lds_bytes and v.resources().scratch_bytes == 0 and "body=double-steps" in B.trace_to_text(op, sp, t)
    # launches of few tiles take 64 x 64 tiles instead, launches that fill the chip do not, and products that always do have none
    small = v.launch_shape(1)
    assert small[1] == 64 and small[0] >= 3 and v.launch_shape(64) == (4, 16, v.params().lds_bytes)
    big = B.gemm_op(4096, 4096, 1024, "f16")
    bsp = big.space()
    vb = B.Variant(big, bsp, B.make_trace(bsp, [[323216], [16, 1, 2, 4], [16, 1, 4, 2], [32, 1, 1, 2], [0], [10], [8], [8], [0], [3], [1]]))
    assert vb.launch_shape(1) == (2, 256, vb.params().lds_bytes)
    assert params(161632, [4, 1, 2, 4], [4, 1, 4, 2], [8, 1, 2, 2], 8).body == B.BODY_NEST       # 256-byte k tiles
    odd = B.gemm_op(512, 512, 96, "f16")
    assert params(161632, [4, 1, 2, 4], [4, 1, 4, 2], [3, 1, 1, 1], 10, op=odd, sp=odd.space()).body == B.BODY_NEST
    lim = B.get_limits()
    try:
        for lds, stages in ((80 * 1024, 2), (60 * 1024, 0)):
            tight = B.get_limits()
            tight.max_lds_bytes = lds
            B.set_limits(tight)
            p = params(161632, [4, 1, 2, 4], [4, 1, 4, 2], [32, 1, 1, 1], 8)
            assert (p.body_tile, p.body) == (stages, B.BODY_DOUBLE_STEPS if stages else B.BODY_NEST) and p.lds_bytes <= lds
    finally:
        B.set_limits(lim)


def _short_waits(code_object):
    """Loads into LDS of a code object, and those that read a scalar register fewer than five wait states after a vector
    instruction wrote it."""
    text = subprocess.run(["/opt/rocm/llvm/bin/llvm-objdump", "-d", code_object], stdout=subprocess.PIPE, text=True, check=True).stdout
    code = [line.split("//")[0].split(None, 1) for line in text.splitlines() if line.startswith("\t")]
    code = [(c[0], re.split(r"[ ,]+", c[1].strip()) if len(c) > 1 else []) for c in code]

    def scalars(token):
        m = re.fullmatch(r"s(?:(\d+)|\[(\d+):(\d+)\])", token)
        return set() if not m else {int(m[1])} if m[1] else set(range(int(m[2]), int(m[3]) + 1))

    loads, short = 0, []
    for at, (name, args) in enumerate(code):
        if not (name.startswith("global_load_lds") or (name.startswith("buffer_load") and args[-1] == "lds")):
            continue
        loads += 1
        operands, states = set().union(*map(scalars, args)), 0
        for before, what in code[at - 1::-1]:
            if states >= 5:
                break
            if before.startswith("s_mov") and what:
                operands -= scalars(what[0])
            if before.startswith("v_") and what and scalars(what[0]) & operands:
                short.append((before, what, name, args, states))
            states += int(what[0], 0) + 1 if before == "s_nop" else 1
    return loads, short


def test_loads_into_lds_wait_for_their_scalar_operands(tmp_path):
    """The loads are written as assembly, where the compiler does not see the wait states that they need."""
    gemm, conv = B.gemm_op(256, 256, 704, "f16"), B.conv2d_op(8, 12, 14, 64, 128, 3, 3, stride=1, pad=1)
    sp, csp = gemm.space(), conv.space()
    ring = [[323216], [1, 1, 2, 4], [1, 1, 4, 2], [22, 1, 1, 2], [0], [7], [8], [8], [0], [3], [0]]
    gather = next(t for t in (B.trace_sample_valid(conv, csp, 106, n) for n in range(400)) if B.trace_validate(conv, csp, t).body == B.BODY_CONV_STEPS)
    steps = [[161632], [1, 1, 2, 8], [1, 1, 4, 4], [22, 1, 1, 1], [0], [8], [8], [8], [0], [3], [1]]
    try:
        for n, (op, space, t) in enumerate(((gemm, sp, B.make_trace(sp, ring)), (gemm, sp, B.make_trace(sp, steps)), (conv, csp, gather))):
            at = tmp_path / str(n)
            at.mkdir()
            B.set_cache_dir(str(at))
            B.Variant(op, space, t)
            found = [_short_waits(str(f)) for f in at.iterdir() if f.suffix == ".hsaco"]
            assert found and all(loads > 0 and not short for loads, short in found), found
    finally:
        B.set_cache_dir(os.environ.get("MS_CACHE_DIR") or os.path.join(ROOT, "paper_2205_13603_amd", "kcache"))


@pytest.mark.parametrize("M,N,i,j,stages,step", [
    (256, 96, [1, 1, 2, 8], [3, 1, 1, 2], 4, 18), (96, 256, [3, 1, 1, 2], [1, 1, 2, 8], 4, 18), (32, 512, [1, 1, 1, 2], [1, 1, 2, 16], 2, 34),
    (96, 384, [6, 1, 1, 1], [1, 1, 4, 6], 3, 12), (384, 96, [1, 1, 4, 6], [3, 1, 1, 2], 3, 13)])
def test_double_steps_request_every_row_of_a_stage(M, N, i, j, stages, step, tmp_path):
    """Few wavefronts on a long tile: a wavefront's share of a double step, 1 KiB per load, is in the code once per stage filled
    ahead and once in each group's loop, however many loads one part of it holds."""
    op = B.bmm_op(1, M, N, 704, True, "f16")
    sp = op.space()
    t = B.make_trace(sp, [[161632], i, j, [22, 1, 1, 1], [0], [10], [8], [8], [0], [3], [0]])
    p = B.trace_validate(op, sp, t)
    assert (p.body, p.body_tile) == (B.BODY_DOUBLE_STEPS, stages) and (p.block_m + p.block_n) // (8 * p.waves) == step
    try:
        B.set_cache_dir(str(tmp_path))
        B.Variant(op, sp, t)
    finally:
        B.set_cache_dir(os.environ.get("MS_CACHE_DIR") or os.path.join(ROOT, "paper_2205_13603_amd", "kcache"))
    loads, short = max(_short_waits(str(f)) for f in tmp_path.iterdir() if f.suffix == ".hsaco")
    assert loads >= (stages + 1) * step and not short


@pytest.mark.parametrize("mk,elems", [(lambda: B.conv2d_op(2, 15, 11, 96, 256, 3, 3, stride=2, pad=1), 2 * 8 * 6 * 256),
                                      (lambda: B.conv2d_op(4, 14, 14, 128, 96, 3, 3, pad=2, stride=1, dilation=2), 4 * 196 * 96),
                                      (lambda: B.conv2d_transposed_op(2, 4, 6, 128, 64, 4, 4, stride=2, pad=1), 2 * 96 * 64)])
def test_conv_steps_cover_the_output_and_the_filter_once(mk, elems):
    """Convolutions with their cache-read under the k0 loop are one kernel with one key whatever the decisions; its tiles cover
    the output and its steps the filter once, and its resources are those of the code object."""
    op = mk()
    sp = op.space()
    keys, K = set(), int(np.prod([e for n, e, red in op.loops() if red]))
    for idx in range(200):
        t = B.trace_sample_valid(op, sp, 39, idx)
        p = B.trace_validate(op, sp, t)
        assert (p.body == B.BODY_CONV_STEPS) == ("CONV_STEPS=1" in B.variant_kernel_text(op, p))
        if p.body != B.BODY_CONV_STEPS:
            continue
        if not keys:
            for cov in (B.variant_coverage(op, p, elems), B.variant_reduction_coverage(op, p)):
                assert cov.min() == 1 and cov.max() == 1
            assert len(cov) == K and p.body_tile == p.block_m * 1000 + p.block_n
            r = B.Variant(op, sp, t).resources()
            assert r.lds_bytes == p.lds_bytes and r.scratch_bytes == 0 and "body=conv-steps" in B.trace_to_text(op, sp, t)
        keys.add((p.key, B.variant_kernel_text(op, p)))
    assert len(keys) == 1


@pytest.mark.parametrize("mk,image,ahead,step", [
    # bytes of one image, those that an offset starts ahead of the images (padding, or the taps of a phase), images per 16 pixels
    (lambda n: B.conv2d_op(n, 20, 20, 96, 128, 3, 3, stride=1, pad=1), 400 * 96 * 2, 21 * 96 * 2, 1),
    (lambda n: B.conv2d_op(n, 14, 14, 32, 128, 3, 3, stride=1, pad=2, dilation=2), 196 * 32 * 2, 30 * 32 * 2, 4),
    (lambda n: B.conv2d_op(n, 16, 16, 256, 128, 1, 1), 256 * 256 * 2, 0, 1),
    (lambda n: B.conv2d_transposed_op(n, 8, 8, 64, 64, 9, 9, stride=1, pad=4), 64 * 64 * 2, 72 * 64 * 2, 1),
])
def test_conv_steps_end_where_their_offsets_do(mk, image, ahead, step):
    """The gather's 32-bit offsets count from ahead of the image stack: images beyond what they reach keep the nest."""
    most = (0x7ffffff0 - ahead) // image // step * step
    for n, taken in ((most, True), (most + step, False)):
        op = mk(n)
        sp = op.space()
        M, N, K = (e for _, e, _ in op.loops())
        p = B.trace_validate(op, sp, B.make_trace(sp, [[161632], [M // 16, 1, 1, 1], [N // 32, 1, 2, 1], [K // 32, 1, 1, 1], [0], [2], [8], [8], [0], [0], [0], [0]][:sp.n_slots]))
        assert (p.body == B.BODY_CONV_STEPS) == taken, (n, taken, p.body)


@pytest.mark.parametrize("mk", [
    lambda: B.conv2d_op(8, 56, 56, 64, 48, 3, 3, pad=1),                 # 48 output channels: no whole columns of 32
    lambda: B.conv2d_op(1, 20, 20, 32, 16, 3, 3, pad=1, in_dtype="bf16"),
    lambda: B.conv2d_op(1, 256, 256, 64, 64, 3, 3, pad=1),               # a row is 16 strips of 16 columns
    lambda: B.conv1d_op(1, 256, 64, 128, 3, pad=1),
    lambda: B.conv2d_transposed_op(1, 256, 256, 64, 64, 3, 3, pad=1)])
def test_convolutions_without_a_tile_of_input_patches_keep_their_kernel(mk):
    """Stride 1 and whole 32-channel groups of the input, but no tile of input patches fits: a variant builds, and launches of
    any number of instances run what its parameters say."""
    op = mk()
    sp = op.space()
    t = next(t for t in (B.trace_sample_valid(op, sp, 43, n) for n in range(200)) if B.trace_validate(op, sp, t).family == B.FAM_GEMM_MFMA)
    v = B.Variant(op, sp, t)
    p = v.params()
    for instances in (1, 512):
        assert v.launch_shape(instances) == (p.body_tile, p.grid[0] * p.grid[1] * p.grid[2], p.lds_bytes)


def test_first_layers_of_the_planes_tests_run_on_filter_planes():
    """The launches that test_first_layer_planes_exact compares take the kernel it is for: all its shapes, with and without an
    epilogue.  Fewer images than fill the chip stay on image rows."""
    import test_gpu_conv as T
    shapes = next(m for m in T.test_first_layer_planes_exact.pytestmark if m.args[0].startswith("N,D,H"))
    for N, D, H, W_, Cin, Cout, k, stride, pad, dtype, R in shapes.args[1]:
        for epilogue in (True, False):
            args = dict(stride=stride, pad=pad, in_dtype=dtype, has_bias=epilogue, relu=epilogue)
            op = B.conv3d_op(N, D, H, W_, Cin, Cout, k, **args) if D > 1 else B.conv2d_op(N, H, W_, Cin, Cout, k, k, **args)
            sp = op.space()
            t = next(t for t in (B.trace_sample_valid(op, sp, 118, n) for n in range(200))
                     if B.trace_validate(op, sp, t).compute_at == 0 and B.trace_validate(op, sp, t).family == B.FAM_GEMM_MFMA)
            v = B.Variant(op, sp, t)
            assert v.params().body == B.BODY_IMAGE_ROWS
            p, r = v.launch_kernel(R)
            assert p.body == B.BODY_CONV_PLANES and p.lds_bytes == r.lds_bytes
    assert v.launch_kernel(1)[0].body == B.BODY_IMAGE_ROWS
    with pytest.raises(B.MsError):
        v.launch_kernel(0)


def test_no_kernel_is_built_that_no_launch_takes(tmp_path):
    """3-D filters of fewer than four k steps per plane stay on image rows at any number of instances: nothing else is compiled."""
    op = B.conv3d_op(1, 4, 48, 48, 3, 32, 3, stride=2, pad=1)
    sp = op.space()
    before = B.jit_stats()["compiled"]
    B.set_cache_dir(str(tmp_path))
    try:
        v = B.Variant(op, sp, B.trace_sample_valid(op, sp, 44, 0))
    finally:
        B.set_cache_dir(os.environ.get("MS_CACHE_DIR") or os.path.join(ROOT, "paper_2205_13603_amd", "kcache"))
    assert B.jit_stats()["compiled"] - before == 1
    assert all(v.launch_kernel(r)[0].body == B.BODY_IMAGE_ROWS for r in (1, 8, 64, 512, 4096))


def test_order_of_workgroups_is_a_permutation_in_runs(tmp_path):
    """xcd_run() of the kernels, compiled for the host: every workgroup once for any total, and neighbours on one XCD in runs of the
    length asked for."""
    src = open(os.path.join(ROOT, "paper_2205_13603_amd", "csrc", "kernels", "common.h")).read()
    fn = src[src.index("template <unsigned RUN>"):]
    fn = fn[:fn.index("\n}\n") + 3]
    (tmp_path / "t.cpp").write_text("""
#include <cstdio>
#include <vector>
#define __device__
#define __forceinline__
%s
template <unsigned RUN> int check(unsigned total)
{
    std::vector<unsigned> xcd(total, 8);
    for (unsigned f = 0; f < total; ++f) {
        const unsigned g = xcd_run<RUN>(f, total);
        if (g >= total || xcd[g] != 8) return 1;
        xcd[g] = f %% 8;
    }
    unsigned runs = 1;
    for (unsigned g = 1; g < total; ++g) runs += xcd[g] != xcd[g - 1];
    const unsigned pieces = RUN ? (total + RUN * 8 - 1) / (RUN * 8) : 1;
    return runs > pieces * 8;
}
int main()
{
    for (unsigned total = 1; total < 3000; ++total)
        if (check<0>(total) || check<32>(total)) return printf("%%u\\n", total), 1;
    return check<0>(100003) || check<32>(100003);
}
""" % fn)
    subprocess.run(["g++", "-O1", "-o", str(tmp_path / "t"), str(tmp_path / "t.cpp")], check=True)
    subprocess.run([str(tmp_path / "t")], check=True)


@pytest.mark.parametrize("N,size,cout,k,dil,R", [(1, 56, 64, 3, 2, 512), (1, 16, 128, 3, 2, 512), (1, 28, 64, 5, 1, 512), (200, 28, 64, 5, 1, 1),
                                                 (1, 56, 64, 3, 1, 512)])
def test_input_patches_do_not_spill(N, size, cout, k, dil, R):
    """The compiled kernels of residual layers whose tiles are as large as the registers allow: nothing in scratch memory."""
    op = B.conv2d_op(N, size, size, 64, cout, k, k, pad=dil * (k - 1) // 2, dilation=dil)
    sp = op.space()
    t = next(t for t in (B.trace_sample_valid(op, sp, 5, n) for n in range(200)) if B.trace_validate(op, sp, t).family == B.FAM_GEMM_MFMA)
    p, r = B.Variant(op, sp, t).launch_kernel(R)
    assert p.body == B.BODY_CONV_PATCH and r.scratch_bytes == 0 and r.spilled_vgprs == 0


@pytest.mark.parametrize("M,N,K,rf,few", [
    (32, 2048, 4096, 4, False), (32, 2048, 4096, 2, True), (32, 2048, 3072, 4, True), (32, 1024, 4096, 4, True), (16, 3072, 4096, 4, False),
    (48, 1344, 4096, 4, True),
    (16, 1024, 512, 1, True), (16, 1024, 448, 1, False)])  # 1 MiB of weights and less
def test_which_products_of_few_rows_replace_a_nest(M, N, K, rf, few):
    """Long reductions of few tiles that the trace splits over four workgroups and more keep its nest; so do small matrices."""
    op = B.gemm_op(M, N, K, "f16")
    sp = op.space(B.SPACE_DEFAULT | B.SPACE_RFACTOR)
    t = B.make_trace(sp, [[161616], [M // 16, 1, 1, 1], [N // 64, 1, 4, 1], [K // 64, 1, 4, 1], [16], [1], [8], [8], [2], [0], [1 if rf == 1 else 0], [rf]])
    v = B.Variant(op, sp, t)
    assert v.params().rfactor == rf and v.params().body == B.BODY_NEST
    assert v.launch_kernel(1)[0].body == (B.BODY_FEW_ROWS if few else B.BODY_NEST)
    assert v.workspace_bytes() == (rf * M * N * 4 if rf > 1 else 0)


@pytest.mark.parametrize("size,cin,k,batch,planes", [
    (128, 3, 7, 75, False), (192, 3, 7, 36, True), (192, 3, 7, 47, True),   # two rounds: 825 and 864 of 1024 tiles of 3 x 2, 846 of 4 x 2
    (192, 4, 3, 27, False), (224, 3, 5, 18, True),                          # a single round of few steps, of more
    (64, 3, 5, 133, True)])
def test_which_first_layers_fill_their_rounds(size, cin, k, batch, planes):
    op = B.conv2d_op(batch, size, size, cin, 64, k, k, stride=2, pad=k // 2)
    sp = op.space()
    t = next(t for t in (B.trace_sample_valid(op, sp, 45, n) for n in range(200)) if B.trace_validate(op, sp, t).body == B.BODY_IMAGE_ROWS)
    assert B.Variant(op, sp, t).launch_kernel(1)[0].body == (B.BODY_CONV_PLANES if planes else B.BODY_IMAGE_ROWS)


def test_few_long_rows_keep_their_wide_lane_groups():
    """Softmax without staging: a few long rows keep a lane group of a wavefront or more per row; many rows, short rows and
    groups that walk a row or several rows in turn go to the row kernel, as do groups narrower than a line."""
    def body(rows, cols, i, k, cache_read=0):
        op = B.softmax_op(1, rows, cols)
        sp = op.space()
        return B.trace_validate(op, sp, B.make_trace(sp, [i, k, [cache_read]])).body

    assert body(256, 4096, [256, 1, 1, 1], [1, 2, 512, 4]) == B.BODY_NEST
    assert body(1024, 2048, [256, 1, 4, 1], [1, 8, 64, 4]) == B.BODY_NEST
    assert body(2048, 4096, [2048, 1, 1, 1], [1, 2, 512, 4]) == B.BODY_ROW_VECTORS
    assert body(256, 1024, [256, 1, 1, 1], [1, 1, 256, 4]) == B.BODY_ROW_VECTORS
    assert body(256, 4096, [256, 1, 1, 1], [2, 1, 512, 4]) == B.BODY_ROW_VECTORS
    assert body(256, 4096, [128, 2, 1, 1], [1, 2, 512, 4]) == B.BODY_ROW_VECTORS
    assert body(256, 2048, [64, 1, 4, 1], [1, 16, 32, 4]) == B.BODY_ROW_VECTORS
    assert body(256, 4096, [256, 1, 1, 1], [1, 2, 512, 4], 1) == B.BODY_NEST        # staged: one pass, full lines


def test_small_depthwise_launches_keep_a_compact_nest():
    """A small launch keeps a nest of one compact patch per thread; the same decisions on a launch of many strips, and
    nests that are rolled, staged or serial, go to the strips."""
    def body(n, i=(29, 1, 1, 1), j=(29, 1, 1, 1), c=(2, 1, 72, 1), unroll=64, cache_read=0):
        op = B.dwconv2d_op(n, 57, 57, 144, stride=2)
        sp = op.space()
        by = {B.SLOT_TILE_I: list(i), B.SLOT_TILE_J: list(j), B.SLOT_TILE_C: list(c), B.SLOT_UNROLL: [unroll],
              B.SLOT_CACHE_READ: [cache_read], B.SLOT_REORDER: [0]}
        return B.trace_validate(op, sp, B.make_trace(sp, [by[sp.slots[k].slot_id] for k in range(sp.n_slots)])).body

    assert body(1) == B.BODY_NEST                     # 8 x 8 x 144 strips: 144 wavefronts
    assert body(2) == B.BODY_STRIPS                   # 288
    assert body(1, unroll=0) == B.BODY_STRIPS and body(1, cache_read=1) == B.BODY_STRIPS
    assert body(1, c=(1, 2, 72, 1)) == B.BODY_STRIPS  # two channels per thread, one after the other
    assert body(1, j=(1, 1, 1, 29)) == B.BODY_STRIPS  # 3 x 59 input patch against 9 x 9
    assert body(1, c=(9, 1, 16, 1)) == B.BODY_STRIPS  # 16 of 64 lanes


@pytest.mark.parametrize("batch,size,channels,strips", [(65, 8, 256, True), (64, 8, 256, False), (400, 7, 100, False), (29, 56, 12, True)])
def test_large_depthwise_launches_run_on_strips(batch, size, channels, strips):
    """More than four strip wavefronts per compute unit and at least 8 output pixels a side: strips whatever the decisions."""
    op = B.dwconv2d_op(batch, size, size, channels)
    sp = op.space()
    for n in range(20):
        assert B.trace_validate(op, sp, B.trace_sample_valid(op, sp, 16, n)).body == (B.BODY_STRIPS if strips else B.BODY_NEST)


@pytest.mark.parametrize("mk,flags,one,many", [
    (lambda: B.conv2d_op(1, 224, 224, 3, 64, 7, 7, stride=2, pad=3), B.SPACE_DEFAULT | B.SPACE_TAP_ROWS, 1, 4),
    (lambda: B.conv3d_op(1, 16, 224, 224, 3, 64, 7, stride=2, pad=3), B.SPACE_DEFAULT, 2, 4),
    (lambda: B.conv3d_op(1, 16, 224, 224, 4, 64, 7, stride=2, pad=3), B.SPACE_DEFAULT, 2, 0),   # the next plane beside 4 x 2 tiles spills
    (lambda: B.conv3d_op(8, 16, 224, 224, 4, 64, 7, stride=2, pad=3), B.SPACE_DEFAULT, 2, 0),
    (lambda: B.conv2d_op(1, 64, 64, 3, 32, 3, 3, stride=2, pad=1), B.SPACE_DEFAULT, 1, 2),
    (lambda: B.conv2d_op(1, 96, 96, 3, 96, 7, 7, stride=2, pad=3), B.SPACE_DEFAULT, 1, 2),      # 4 x 3 tiles are too many
    (lambda: B.conv2d_op(128, 224, 224, 3, 64, 7, 7, stride=2, pad=3), B.SPACE_DEFAULT, 4, 0)])
def test_image_rows_take_a_larger_tile_where_instances_fill_the_chip(mk, flags, one, many):
    """The tile is chosen for one instance; a second kernel of the same code object serves launches over many.  Coverage of
    both."""
    op = mk()
    sp = op.space(flags)
    t = next(t for t in (B.trace_sample_valid(op, sp, 38, n) for n in range(100)) if B.trace_validate(op, sp, t).body == B.BODY_IMAGE_ROWS)
    v = B.Variant(op, sp, t)
    p = v.params()
    assert (p.body_tile, p.body_tile_many) == (one, many) and v.resources().scratch_bytes == 0
    assert v.launch_shape(1) == (one, p.grid[0], p.lds_bytes)
    tiles = [v.launch_shape(n)[0] for n in (1, 2, 3, 4, 8, 16, 64, 256, 4096)]
    assert set(tiles) <= {one, many or one} and tiles[-1] == (many or one)
    text = B.variant_kernel_text(op, p)
    assert ("-DCR_MANY_TM=%d" % many in text) == bool(many)
    if op.tensor_bytes(-1) < 1 << 24:
        for tile in {one, many or one}:
            p.body_tile = tile
            cov = B.variant_coverage(op, p, op.tensor_bytes(-1) // 2)
            assert cov.min() == 1 and cov.max() == 1
    with pytest.raises(B.MsError):
        v.launch_shape(0)


def test_a_search_measures_a_body_once():
    """Every trace of this operator resolves to the strip kernel: one measurement, the rest are duplicates."""
    op = B.dwconv2d_op(32, 57, 57, 48, stride=2)
    sp = op.space()
    cfg = B.search_cfg_default()
    cfg.seed, cfg.trials = 3, 64
    res = B.search(op, sp, cfg, fake_latency=lambda p: 1.0)
    assert res.n_measured == 1 and res.n_duplicate > 0


@pytest.mark.parametrize("mk,instances,offset,kernels", [
    (lambda: B.conv2d_op(1, 16, 16, 32, 32, 3, 3, pad=1), 512, 0, 2),   # input patches and the nest of the trace that is measured
    (lambda: B.gemm_op(16, 1024, 512, "f16"), 1, 0, 2),                 # few rows
    (lambda: B.gemm_op(16, 1024, 512, "f16"), 1, 4, 40)])               # operands off 16-byte boundaries: nests of their own
def test_a_search_compiles_what_its_launches_run(mk, instances, offset, kernels, tmp_path):
    """Traces whose launches all run one second kernel are one candidate: a search compiles it once, with one nest, and ends.
    Without a GPU every measurement fails, so the search goes through all its proposals."""
    import torch
    if torch.cuda.is_available():
        pytest.skip("the buffers are addresses only")
    op = mk()
    cfg = B.search_cfg_default()
    cfg.seed, cfg.trials, cfg.init_population = 3, 2, 2
    cfg.measure.instances = instances
    if offset:
        cfg.trials = cfg.init_population = 20
    before = B.jit_stats()
    B.set_cache_dir(str(tmp_path))
    try:
        stop = [0]

        def failed(t):
            assert t.status == B.MS_ERR_HIP
            stop[0] += 1
            return stop[0] >= 20

        with pytest.raises(B.MsError) as e:
            B.search(op, op.space(), cfg, [([4096 + offset] * 3, 4096)], on_trial=failed)
        assert e.value.code == B.MS_ERR_HIP
    finally:
        B.set_cache_dir(os.environ.get("MS_CACHE_DIR") or os.path.join(ROOT, "paper_2205_13603_amd", "kcache"))
    built = B.jit_stats()["compiled"] - before["compiled"]
    assert built == kernels if not offset else 15 <= built <= kernels
    assert stop[0] == (1 if not offset else 20)


def test_unroll_budgets_that_resolve_alike_share_a_key():
    op = B.dwconv2d_op(1, 28, 28, 12)
    sp = op.space()
    t = B.trace_sample_valid(op, sp, 1, 0)
    pos = [i for i in range(sp.n_slots) if sp.slots[i].slot_id == B.SLOT_UNROLL][0]
    keys = []
    for choice in range(3):  # budgets 0, 16, 64
        t.d[pos].v[0] = choice
        keys.append(B.trace_validate(op, sp, t).key)
    assert keys[1] == keys[2] and keys[0] != keys[1]  # 16 and 64 both unroll the 9 taps fully


# ---------------------------------------------------------------- rfactor (reduction split across workgroups)

def test_rfactor_is_an_opt_in_module_with_rules():
    op = B.gemm_op(256, 256, 512, "f16")
    assert B.SLOT_RFACTOR not in [op.space().slots[i].slot_id for i in range(op.space().n_slots)]
    sp = op.space(B.SPACE_DEFAULT | B.SPACE_RFACTOR)
    s = sp.slots[sp.n_slots - 1]
    assert s.slot_id == B.SLOT_RFACTOR and [s.candidates[c] for c in range(s.n_candidates)] == [1, 2, 4, 8]
    # the vector-ALU family has no such decision
    sp_alu = B.gemm_op(128, 128, 128, "f32").space(B.SPACE_DEFAULT | B.SPACE_RFACTOR)
    assert B.SLOT_RFACTOR not in [sp_alu.slots[i].slot_id for i in range(sp_alu.n_slots)]

    def mk(k, cache=2, pad=0, reorder=0, cw=0, rf=1):
        return B.make_trace(sp, [[161632], [4, 2, 2, 1], [4, 2, 2, 1], k, [0], [cache], [8], [8], [pad], [reorder], [cw], [rf]])

    base = B.trace_validate(op, sp, mk([8, 1, 1, 2]))
    assert base.rfactor == 1 and base.grid[0] == 16
    p = B.trace_validate(op, sp, mk([8, 1, 1, 2], rf=4))
    assert p.rfactor == 4 and p.grid[0] == 64 and p.key != base.key
    assert "-DRFACTOR=4" in B.variant_kernel_text(op, p)
    assert "rfactor(loop=k0, factor=4)" in B.trace_to_text(op, sp, mk([8, 1, 1, 2], rf=4))
    for bad, why in [(mk([4, 2, 1, 2], rf=8), "does not divide"), (mk([8, 1, 1, 2], rf=2, cw=1), "cache_write"),
                     (mk([8, 1, 1, 2], cache=5, reorder=3, rf=2), "persistent")]:
        with pytest.raises(B.MsError, match=why):
            B.trace_validate(op, sp, bad)
    # launching without the workspace is refused before anything touches a device
    v = B.Variant(op, sp, mk([8, 1, 1, 2], rf=4))
    assert v.workspace_bytes() == 4 * 256 * 256 * 4
    with pytest.raises(B.MsError, match="workspace"):
        v.launch([8, 8], 8)
    with pytest.raises(B.MsError, match="aligned"):
        v.launch([8, 8], 8, workspace=4)


def test_launch_marshals_its_arguments():
    """The binding's native entry hands ms_variant_launch what it was given: the checks that come before any device see it."""
    import ctypes
    op = B.gemm_op(64, 64, 64, "f16")
    sp = op.space()
    v = B.Variant(op, sp, B.trace_sample_valid(op, sp, 0, 0))
    for inputs, output, instances, why in (([8], 8, 1, "NULL tensor"), ([8, None], 8, 1, "NULL tensor"), ([0, 8], 8, 1, "NULL tensor"), ((8, 8), None, 1, "NULL tensor"),
                                           ((p for p in (8, 8)), 0, 1, "NULL tensor"), ([8, 8], 8, 0, "instances = 0"), ([8, 8], 8, -3, "instances = -3")):
        with pytest.raises(B.MsError, match=why):
            v.launch(inputs, output, instances=instances)
    with pytest.raises(B.MsError, match="NULL tensor"):
        v.launch([8], 8, stream=ctypes.c_void_p(None), workspace=ctypes.c_void_p(16))
    for inputs, output in (([8, 8.0], 8), ([8, "8"], 8), ([8, 8], [8]), (8, 8)):
        with pytest.raises(TypeError):
            v.launch(inputs, output)
    with pytest.raises(ValueError):
        v.launch([8] * 5, 8)


@pytest.mark.parametrize("mk", CONFIG_OPS + [lambda: B.softmax_op(1, 64, 256), lambda: B.norm_op(2, 32, 48),
                                             lambda: B.conv2d_op(1, 32, 32, 3, 32, 7, 7, stride=2, pad=3)])
def test_interpreter_visits_every_reduction_position_once(mk):
    """The k split (rfactor run, k0, k1, k2, k3, intrinsic k) of any valid trace visits each position of the
    reduction exactly once: nothing is dropped or counted twice, whatever the decisions."""
    op = mk()
    flags = B.SPACE_DEFAULT | B.SPACE_RFACTOR
    sp = op.space(flags)
    K = [e for n, e, red in op.loops() if red]
    for idx in range(40):
        t = B.trace_sample_valid(op, sp, 22, idx)
        p = B.trace_validate(op, sp, t)
        cov = B.variant_reduction_coverage(op, p)
        assert cov.min() == 1 and cov.max() == 1, t.decisions()
        total = int(np.prod(K))
        assert total <= len(cov) < total + max(1, p.tile_unit[2])  # a convolution may pad K up to the intrinsic's k


# ---------------------------------------------------------------- modules as data, Compose, Stochastic-Compose (Section 3.2)

def test_module_table_and_compose():
    mods = B.modules()
    names = [m["name"] for m in mods]
    assert names[0] == "multi-level-tiling" and mods[0]["flag"] == 0
    assert {"use-mfma", "cache-read", "vectorize", "unroll", "storage-align", "reorder-grid", "cache-write", "compute-location",
            "rfactor"} <= set(names)
    flags = [m["flag"] for m in mods[1:]]
    assert len(set(flags)) == len(flags) and all(f and not (f & (f - 1)) for f in flags)   # one bit each
    by_flag = {m["flag"]: m for m in mods}
    for m in mods:                                                                         # requirements name real modules
        r = m["requires"]
        while r:
            bit = r & -r
            assert bit in by_flag
            r ^= bit
    op = B.gemm_op(256, 256, 256, "f16")
    default = ["multi-level-tiling", "use-mfma", "cache-read", "vectorize", "unroll", "storage-align", "reorder-grid", "cache-write"]
    sp, mask = B.space_compose(op, default)
    assert mask == 0x7F and bytes(sp) == bytes(op.space())          # compute-location does not apply to a matrix product
    # the order of the list does not change the space (slot order is canonical), as long as requirements come first
    sp2, _ = B.space_compose(op, ["multi-level-tiling", "unroll", "use-mfma", "cache-write", "reorder-grid", "storage-align", "vectorize", "cache-read"])
    assert bytes(sp2) == bytes(sp)
    # every prefix of a list is a space of its own: the space grows module by module
    sizes = []
    for n in range(1, len(default) + 1):
        spn, maskn = B.space_compose(op, default[:n])
        sizes.append(B.space_log10_size(spn))
        assert spn.n_slots >= 3
    assert all(b >= a for a, b in zip(sizes[1:], sizes[2:]))        # (the matrix-core module changes the tile units, so [0] -> [1] may shrink)
    with pytest.raises(B.MsError, match="must start with multi-level-tiling"):
        B.space_compose(op, ["use-mfma"])
    with pytest.raises(B.MsError, match="cache-write needs use-mfma"):
        B.space_compose(op, ["multi-level-tiling", "cache-write", "use-mfma"])
    with pytest.raises(B.MsError, match="listed twice"):
        B.space_compose(op, ["multi-level-tiling", "unroll", "unroll"])
    # a module that does not apply to the operator is the identity
    dw = B.dwconv2d_op(1, 28, 28, 16)
    spd, maskd = B.space_compose(dw, default)
    assert bytes(spd) == bytes(dw.space()) and not (maskd & B.SPACE_TENSORIZE)
    conv = B.conv2d_op(1, 28, 28, 16, 32, 3, 3, stride=1, pad=1)
    spc, maskc = B.space_compose(conv, default + ["compute-location"])
    assert maskc == 0xFF and bytes(spc) == bytes(conv.space())


def test_stochastic_compose_is_seeded_and_respects_requirements():
    mods = B.modules()
    req = {m["name"]: m["requires"] for m in mods}
    flag = {m["name"]: m["flag"] for m in mods}
    op = B.conv2d_op(1, 28, 28, 16, 32, 3, 3, stride=1, pad=1)
    every = [m["name"] for m in mods]
    seen_masks, count = set(), {n: 0 for n in every}
    N = 300
    for seed in range(N):
        sp, applied = B.space_stochastic_compose(op, every, seed)
        again_sp, again = B.space_stochastic_compose(op, every, seed)
        assert applied == again and bytes(sp) == bytes(again_sp)
        assert applied[0] == "multi-level-tiling" and len(set(applied)) == len(applied)
        have = 0
        for n in applied:
            assert (req[n] & have) == req[n], (applied, n)          # requirements were applied earlier
            have |= flag[n]
            count[n] += 1
        assert sp.flags == have
        seen_masks.add(sp.flags)
        # the composed space is a working space: a valid trace can be drawn unless the conv has no vector kernel family
        if sp.flags & B.SPACE_TENSORIZE:
            B.trace_sample_valid(op, sp, 1, 0)
    assert len(seen_masks) > 30
    # the first draw at a location with c candidates applies each of them with probability 1 / (c + 1)
    assert count["use-mfma"] == N and count["use-mfma-f32"] == 0 and 0.2 * N < count["compute-location"] < 0.8 * N
    gemm = B.gemm_op(128, 128, 128, "f16")               # has a vector-ALU family: the matrix-core module is one of the draws
    n_mfma = sum("use-mfma" in B.space_stochastic_compose(gemm, every, seed)[1] for seed in range(N))
    assert 0.3 * N < n_mfma < 0.9 * N
    with pytest.raises(B.MsError, match="needs use-mfma"):
        B.space_stochastic_compose(op, ["unroll", "cache-read"], 0)
    # a restricted module set restricts the space
    sp, applied = B.space_stochastic_compose(op, ["use-mfma", "unroll"], 4)
    assert set(applied) <= {"multi-level-tiling", "use-mfma", "unroll"}
    sp, applied = B.space_stochastic_compose(B.gemm_op(128, 128, 128, "f32"), [], 0)
    assert applied == ["multi-level-tiling"] and sp.flags == 0


def test_row_major_b_layout_is_offered_and_validated():
    """storage_align 3 (B row-major in LDS, transposing LDS loads): offered for matrix-core GEMMs whose B is contiguous
    along j; the validator wants 16-byte fragments, 16-byte loads of B and register staging, and counts a dense B tile."""
    def align_candidates(op):
        sp = op.space()
        for i in range(sp.n_slots):
            if sp.slots[i].slot_id == B.SLOT_STORAGE_ALIGN:
                return [sp.slots[i].candidates[c] for c in range(sp.slots[i].n_candidates)]
        return None

    assert align_candidates(B.gemm_op(512, 512, 512, "i8")) == [0, 1, 2, 3, 4]
    assert align_candidates(B.gemm_op(1024, 1024, 1024, "f16")) == [0, 1, 2, 3, 4]
    assert align_candidates(B.bmm_op(4, 64, 64, 64, False, "f16")) == [0, 1, 2, 3, 4]
    assert align_candidates(B.bmm_op(4, 64, 64, 64, True, "f16")) == [0, 1, 2]           # B contiguous along k
    assert align_candidates(B.conv2d_op(1, 56, 56, 64, 64, 3, 3, stride=1, pad=1)) == [0, 1, 2]
    assert align_candidates(B.gemm_op(256, 256, 256, "f8", "f16")) == [0, 1, 2, 3, 4]
    assert align_candidates(B.gemm_op(128, 128, 128, "f32")) == [0, 1]                   # vector-ALU space
    op = B.gemm_op(512, 512, 512, "i8")
    sp = op.space()

    def mk(mfma=161664, k=(4, 1, 2, 1), cache=1, vec_b=16):
        return B.make_trace(sp, [[mfma], [4, 8, 1, 1], [4, 2, 4, 1], list(k), [0], [cache], [16], [vec_b], [3], [2], [0]])

    p = B.trace_validate(op, sp, mk())
    assert p.lds_pad == 3
    # A: 8 planes of 128 fragments of 16 bytes + 16 bytes of padding each; B: 128 k-rows of 128 bytes, dense
    assert p.lds_bytes == 8 * (128 * 16 + 16) + 128 * 128
    assert "transform-layout(buffer=B.lds" in B.trace_to_text(op, sp, mk())
    # 4: no swizzle, every k-row of B padded by 32 bytes
    t4 = B.make_trace(sp, [[161664], [4, 8, 1, 1], [4, 2, 4, 1], [4, 1, 2, 1], [0], [1], [16], [16], [4], [2], [0]])
    p4 = B.trace_validate(op, sp, t4)
    assert p4.lds_pad == 4 and p4.lds_bytes == 8 * (128 * 16 + 16) + 128 * (128 + 32) and p4.key != p.key
    assert "padded by 32 bytes" in B.trace_to_text(op, sp, t4)
    assert B.trace_validate(op, sp, mk(cache=2)).lds_bytes == 2 * p.lds_bytes
    assert B.trace_validate(op, sp, mk(mfma=161632, k=(4, 1, 2, 2))).lds_bytes == 16 * (128 * 8 + 16) + 128 * 128   # 8-byte fragments
    for bad, why in ((mk(vec_b=4), "vectorize_b"), (mk(cache=5), "")):
        with pytest.raises(B.MsError) as e:
            B.trace_validate(op, sp, bad)
        assert why in str(e.value)
    # a different layout is a different kernel
    q = B.trace_validate(op, sp, B.make_trace(sp, [[161664], [4, 8, 1, 1], [4, 2, 4, 1], [4, 1, 2, 1], [0], [1], [16], [16], [2], [2], [0]]))
    assert q.key != p.key and B.variant_kernel_text(op, q) != B.variant_kernel_text(op, p)
