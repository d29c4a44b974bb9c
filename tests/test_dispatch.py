"""The kernels and grids that calls launch, as the library itself decides them
(tests/dispatch.py records them without a GPU, on a device of 256 compute units
of 32 wavefronts), where a wrong decision changes no result but its time."""
from __future__ import annotations

import os

import pytest

import paper_2608_04991_amd as rac
from tests.dispatch import launches

GRP = rac.RAC_FLAG_GROUP_OUTLIERS
BF16 = rac.RAC_FLAG_XHAT_BF16
FIX = rac.RAC_FLAG_FIXED_STEP
STRIDED = rac.RAC_FLAG_LAUNCH_STRIDED
PER_ROW = rac.RAC_FLAG_LAUNCH_PER_ROW
CUS, WAVES = 256, 32  # the recorded device


@pytest.fixture(scope="module")
def record(tmp_path_factory):
    if not os.path.exists(rac.library_path()):
        pytest.fail("librac.so is not built; run __graft_entry__.build()")
    tmp = tmp_path_factory.mktemp("recorder")
    return lambda calls: launches(calls, tmp)


@pytest.mark.parametrize("d", [1024, 3648, 4096, 5120, 7936, 8192])
@pytest.mark.parametrize("k,flags", [(0, 0), (0, BF16), (2, GRP), (8, 0), (4, FIX)])
def test_decode_strides_over_up_to_six_rows_a_resident_workgroup(record, d, k, flags):
    nch = -(-d // 512)
    fits = CUS * (WAVES // nch)
    rows = (256, 257, fits, fits + 1, 6 * fits, 6 * fits + 1)
    got = record([("decode", [T, d, 64, 64, 4, k, flags]) for T in rows])
    # per-token outliers: 16 wavefronts a compute unit, at least two workgroups
    grid = CUS * (max(2, 16 // nch) if k and not flags & GRP else WAVES // nch)
    want = [256, min(257, grid), grid, grid, grid, 6 * fits + 1]
    assert [l.grid for (l,) in got] == want
    assert all(l.threads == 64 * nch and l.kernel.startswith("rac_decode_kernel<4, ") for (l,) in got)


@pytest.mark.parametrize("d,k,flags,form", [
    (512, 0, 0, "chunks"), (4096, 2, GRP, "chunks"), (7168, 0, BF16, "chunks"), (1024, 4, 0, "rows"),
    (4096, 17, 0, "rows"), (4096, 64, 0, "rows"), (5120, 8, 0, "rows"), (8192, 64, 0, "rows")])
def test_strided_hint_takes_the_strided_kernel_at_any_row_count(record, d, k, flags, form):
    # (both kernels with a form that takes one row, or one chunk, have it as
    # their last template argument)
    rows = [1, 256, 257, 300, 1100, 5000, 40000]
    got = record([("encode", [T, d, 64, 64, 4, k, flags | hint]) for hint in (STRIDED, PER_ROW) for T in rows])
    kernel = {"chunks": "rac_encode_kernel<4, 3, 3, ", "rows": "rac_encode_rows_kernel<4, 3, 3, "}[form]
    strided, per_row = got[:len(rows)], got[len(rows):]
    fits = CUS * (WAVES // (4 if form == "rows" else -(-d // 512)))
    for T, (l,) in zip(rows, strided):
        assert l.kernel.startswith(kernel) and l.kernel.endswith(", false>") and l.grid == min(T, fits)
    for T, (l,) in zip(rows, per_row):
        assert l.kernel.startswith(kernel) and l.kernel.endswith(", true>")
        assert l.grid == (T if form == "rows" else -(-T * -(-d // 512) // 4))


@pytest.mark.parametrize("d", [512, 2560, 4096, 8192])
@pytest.mark.parametrize("k,flags", [(0, 0), (2, GRP)])
def test_pooled_encode_strides_up_to_three_rows_a_workgroup(record, d, k, flags):
    # (moments, merge, encode) with pairs given per segment; every other encode
    # of these shapes takes (row, chunk) wavefronts
    nch = -(-d // 512)
    fits = CUS * (WAVES // nch)
    rows = [256, 257, 3 * fits, 3 * fits + 1]
    flat = lambda T: (True, -(-T * nch // 4))
    got = record([("pooled", [T, d, 64, 64, 4, k, flags]) for T in rows])
    assert [len(ls) for ls in got] == [3] * len(rows)
    assert [(ls[2].kernel.endswith(", true>"), ls[2].grid) for ls in got] == \
        [flat(256), (False, min(257, fits)), (False, fits), flat(3 * fits + 1)]
    got = record([("encode", [T, d, 64, 64, 4, k, flags]) for T in rows])
    assert [(l.kernel.endswith(", true>"), l.grid) for (l,) in got] == [flat(T) for T in rows]


@pytest.mark.parametrize("T,d,k,flags,zero_ref,seven", [
    (16385, 3584, 8, 0, False, True), (65536, 3584, 4, 0, False, True), (30000, 4096, 1, 0, False, True),
    (16384, 3584, 8, 0, False, False), (65536, 3520, 4, 0, False, False), (65536, 3584, 9, 0, False, False),
    (65536, 3584, 4, BF16, False, False), (65536, 3584, 4, 0, True, False), (65536, 4160, 4, 0, False, False),
    (8193, 2560, 4, 0, False, False), (32768, 4096, 16, 0, False, False)])
def test_seven_workgroups_a_compute_unit_only_where_they_are_faster(record, T, d, k, flags, zero_ref, seven):
    ((l,),) = record([("encode_zero" if zero_ref else "encode", [T, d, 64, 64, 4, k, flags])])
    assert l.kernel.endswith(", true>") and l.grid == T and (l.lds > 0) == seven


@pytest.mark.parametrize("T,d", [(1, 512), (34, 1280), (1538, 1024), (254, 6400)])
def test_calibration_of_one_candidate_encodes_it(record, T, d):
    # the pass that measures many candidates at once is the slower one for a
    # single candidate; per-token outliers are never measured by it
    one, other, token = [T, d, 64, 64, 4, 0, 0], [T, d, 128, 128, 4, 2, GRP], [T, d, 64, 64, 4, 8, 0]
    got = record([("calibrate", cs) for cs in ([one], [one, token], [one, other], [one, token, other])])
    evals = [sum(l.kernel == "rac_eval_kernel" for l in ls) for ls in got]
    encodes = [sum("rac_encode" in l.kernel for l in ls) for ls in got]
    assert (evals, encodes) == ([0, 0, 1, 1], [1, 2, 0, 1])


def test_every_predictor_kernel_is_run_by_a_gpu_test(record):
    from tests import test_gpu_predictor as G
    shapes = list(G.EVERY_KERNEL)
    for f in (G.test_predictor_product_tiles, G.test_predictor_small_batches_fold_the_norms):
        shapes += next(m for m in f.pytestmark if m.name == "parametrize").args[1]
    shapes += [(4096, 512, 8, 2048, 64, b) for b in (1, 100, 256)] + [(512, 128, 2, 256, w, 8) for w in (300, 1024)]
    every, *got = record([("all", None)] + [("predictor", [*s[:5], 256, s[5]]) for s in shapes])
    kernels = {l.kernel for l in every if l.kernel.startswith("pred_")}
    assert len(kernels) >= 27
    assert kernels - {l.kernel for ls in got for l in ls} == set()


def test_every_form_of_the_rows_kernel_is_run_by_a_gpu_test(record):
    import re
    from tests import test_gpu_launch_shapes as S, test_gpu_pooled as G
    params = lambda f: next(m for m in f.pytestmark if m.name == "parametrize").args[1]
    calls = [(kind, [*c[:6], c[6] | hint]) for kind, f in (("encode", S.test_strided_form_takes_several_rows),
                                                          ("pooled", G.test_pooled_forms_and_launch_shapes))
             for c in params(f) for hint in (0, STRIDED, PER_ROW)]
    fields = lambda c: [c[n] for n in ("tokens", "hidden", "group_align", "group_quant", "bits", "outlier_k")]
    calls += [("encode", [*fields(c), c["flags"] | hint]) for c, _ in S.CASES.values() for hint in (0, STRIDED, PER_ROW)]
    calls += [("pooled", [*fields(c), c["flags"]]) for c, *_ in G.CASES.values()]
    every, *got = record([("all", None)] + calls)
    # (wavefronts, chunks a wavefront, pooled, two-value and large-list
    # thresholds, one row; whatever the bits and group shapes)
    forms = lambda ls: {m.group(1) for l in ls if (m := re.match(r"rac_encode_rows_kernel<\d, -?\d, -?\d, (.*)>", l.kernel))}
    assert len(forms(every)) == 14
    assert forms(every) - {f for ls in got for f in forms(ls)} == set()
