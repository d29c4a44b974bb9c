"""C-ABI checks that need no GPU: the library loads, exports every function
include/rac.h declares, and its host-only logic (layout, header parsing,
argument validation that returns before any launch) behaves as documented.
"""
from __future__ import annotations

import ctypes
import os
import re

import numpy as np
import pytest

import oracle
import paper_2608_04991_amd as rac
from paper_2608_04991_amd import workloads as wl
from tests import wirefmt

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared_functions():
    text = open(os.path.join(ROOT, "include", "rac.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(rac_[a-z_]+)\s*\(", text)))


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(rac.library_path()):
        pytest.fail("librac.so is not built; run __graft_entry__.build()")
    return rac.library()


def test_exports_every_declared_symbol(lib):
    names = _declared_functions()
    assert set(names) == {"rac_wire_layout", "rac_wire_size", "rac_parse_header", "rac_encode",
                          "rac_reconstruct", "rac_decode", "rac_encode_gather", "rac_decode_gather",
                          "rac_status_string", "rac_span_index_create", "rac_span_index_destroy",
                          "rac_span_index_add", "rac_span_select", "rac_encode_pooled",
                          "rac_saturation_summary", "rac_recon_error_workspace", "rac_recon_error",
                          "rac_calibrate_workspace", "rac_calibrate", "rac_recon_error_noalloc",
                          "rac_predictor_layout", "rac_predictor_cache_bytes", "rac_predictor_workspace_bytes",
                          "rac_predictor_step"}
    for n in names:
        assert hasattr(lib, n), n


def test_status_strings(lib):
    for s in range(8):
        assert rac.rac_status_string(s) != "unknown status"
    assert rac.rac_status_string(99) == "unknown status"


CFGS = [
    dict(tokens=4096, hidden=4096, group_align=128, group_quant=128, bits=4, outlier_k=8),
    dict(tokens=65536, hidden=3584, group_align=128, group_quant=128, bits=4, outlier_k=4),
    dict(tokens=256, hidden=4096, group_align=128, group_quant=4096, bits=2),
    dict(tokens=32768, hidden=4096, group_align=64, group_quant=64, bits=3, outlier_k=16),
    dict(tokens=0, hidden=512, group_align=64, group_quant=64, bits=8),
    dict(tokens=7, hidden=520, group_align=8, group_quant=8, bits=3, outlier_k=64,
         flags=rac.RAC_FLAG_FIXED_STEP),
    dict(tokens=4096, hidden=4096, group_align=128, group_quant=128, bits=4, outlier_k=1,
         flags=rac.RAC_FLAG_GROUP_OUTLIERS),
    dict(tokens=9, hidden=4864, group_align=256, group_quant=256, bits=2, outlier_k=16,
         flags=rac.RAC_FLAG_GROUP_OUTLIERS | rac.RAC_FLAG_FIXED_STEP),
    dict(tokens=5, hidden=2888, group_align=8, group_quant=8, bits=3, outlier_k=2,
         flags=rac.RAC_FLAG_GROUP_OUTLIERS),
]


@pytest.mark.parametrize("c", CFGS)
def test_layout_matches_documented_format(lib, c):
    cfg = rac.RacConfig(**c)
    assert rac.rac_wire_layout(cfg) == wirefmt.expected_layout(**c)
    assert rac.rac_wire_size(cfg) == wirefmt.expected_layout(**c)["total"]


def test_payload_ratio_of_the_prefill_uplink_shape(lib):
    cfg = rac.RacConfig(4096, 4096, 128, 128, 4, 8)
    ratio = rac.rac_wire_size(cfg) / (4096 * 4096 * 2)
    assert abs(ratio - 0.2774) < 5e-4   # 4-bit codes + fp16 scale/coef + 8 outliers per row


@pytest.mark.parametrize("bad", [dict(bits=5), dict(group_align=96), dict(group_quant=4),
                                 dict(hidden=100), dict(outlier_k=65), dict(tokens=-1),
                                 dict(tokens=2**31), dict(flags=32), dict(flags=24), dict(group_align=1024)])
def test_invalid_configs_are_rejected(lib, bad):
    c = dict(tokens=4, hidden=512, group_align=64, group_quant=64, bits=4)
    c.update(bad)
    cfg = rac.RacConfig(**c)
    assert rac.rac_wire_size(cfg) == 0
    with pytest.raises(rac.RacError) as e:
        rac.rac_wire_layout(cfg)
    assert e.value.status == 1


@pytest.mark.parametrize("hint", [rac.RAC_FLAG_LAUNCH_STRIDED, rac.RAC_FLAG_LAUNCH_PER_ROW])
def test_launch_hints_leave_the_wire_layout_alone(lib, hint):
    for c in CFGS:
        plain = rac.RacConfig(**c)
        hinted = rac.RacConfig(**dict(c, flags=c.get("flags", 0) | hint))
        assert rac.rac_wire_size(hinted) == rac.rac_wire_size(plain) > 0
        assert rac.rac_wire_layout(hinted) == rac.rac_wire_layout(plain)


def test_parse_header_reads_oracle_headers(lib):
    for c in CFGS[:4] + CFGS[5:]:
        small = dict(c, tokens=3)
        T, d = 3, small["hidden"]
        xb, rb, _ = wl.affine_pair(wl.AffineRecipe(T, d, small["group_align"]), 0)
        steps = np.full(d // small["group_quant"], 0.05, np.float32)
        for ref in (rb, None):
            rc, wire, _ = oracle.encode(xb, ref, steps, want_xhat=False, **small)
            assert rc == 0
            cfg, zero_ref = rac.rac_parse_header(wire[:256].tobytes())
            want = dict(small, flags=small.get("flags", 0) & (rac.RAC_FLAG_FIXED_STEP |
                                                              rac.RAC_FLAG_GROUP_OUTLIERS))
            want.setdefault("outlier_k", 0)
            assert cfg == rac.RacConfig(**want)
            assert zero_ref == (ref is None)


def test_group_outlier_configs_outside_the_domain_are_rejected(lib):
    G = rac.RAC_FLAG_GROUP_OUTLIERS
    base = dict(tokens=4, hidden=512, group_align=64, group_quant=64, bits=4, outlier_k=2, flags=G)
    assert rac.rac_wire_size(rac.RacConfig(**base)) > 0
    for bad in [dict(group_quant=512), dict(outlier_k=0), dict(outlier_k=17), dict(outlier_k=17, group_quant=256),
                dict(group_quant=16, outlier_k=5), dict(group_quant=8, outlier_k=3)]:
        cfg = rac.RacConfig(**dict(base, **bad))
        assert rac.rac_wire_size(cfg) == 0, bad
        assert _encode(cfg) == 1 and _decode(cfg) == 1


def test_group_outlier_payload_of_the_prefill_uplink_shape(lib):
    cfg = rac.RacConfig(4096, 4096, 128, 128, 4, 1, rac.RAC_FLAG_GROUP_OUTLIERS)
    ratio = rac.rac_wire_size(cfg) / (4096 * 4096 * 2)
    # 4-bit codes + fp16 scale/coef + one (u8 offset, fp16 value) per group of 128
    assert abs(ratio - (0.25 + 6 / 256 + 3 / 256)) < 1e-5


def test_parse_header_rejects_corruption_of_group_outlier_headers(lib):
    c = dict(tokens=2, hidden=256, group_align=64, group_quant=64, bits=4, outlier_k=2,
             flags=rac.RAC_FLAG_GROUP_OUTLIERS)
    xb = wl.f32_to_bf16_bits(np.random.default_rng(0).standard_normal((2, 256)))
    rc, wire, _ = oracle.encode(xb, None, want_xhat=False, **c)
    good = wire[:256].tobytes()
    cfg, _ = rac.rac_parse_header(good)
    assert cfg == rac.RacConfig(**c)
    # flags 9 (both outlier kinds), format 1 with flag 8, a moved offset array,
    # k_g above a quarter of the group, bytes past the fields
    for off, val in [(6, 9), (27, 1), (73, 0), (28, 17), (80, 1), (90, 1)]:
        bad = bytearray(good)
        bad[off] = val
        with pytest.raises(rac.RacError) as e:
            rac.rac_parse_header(bytes(bad))
        assert e.value.status == 5, off


def test_parse_header_rejects_corruption(lib):
    c = dict(tokens=2, hidden=64, group_align=64, group_quant=64, bits=4, outlier_k=2)
    xb = wl.f32_to_bf16_bits(np.random.default_rng(0).standard_normal((2, 64)))
    rc, wire, _ = oracle.encode(xb, None, want_xhat=False, **c)
    good = wire[:256].tobytes()
    rac.rac_parse_header(good)
    for off, val in [(0, 0x00), (4, 1), (24, 5), (28, 0), (40, 0x11), (80, 0x13), (100, 1), (6, 0x08), (25, 2)]:
        bad = bytearray(good)
        bad[off] = val
        with pytest.raises(rac.RacError) as e:
            rac.rac_parse_header(bytes(bad))
        assert e.value.status == 5, off
    with pytest.raises(rac.RacError):
        rac.rac_parse_header(good[:200])


# Argument checks happen on the host before anything is enqueued, so they can
# be exercised with fake (never dereferenced) addresses.
FAKE = 1 << 40


def _encode(cfg, x=FAKE, ref=FAKE, steps=None, wire=FAKE, cap=1 << 40, xhat=FAKE):
    return rac.library().rac_encode(ctypes.byref(cfg._c()), x, ref, steps, wire, cap, xhat, 0)


def _decode(cfg, wire=FAKE, ref=FAKE, steps=None, xhat=FAKE):
    return rac.library().rac_decode(ctypes.byref(cfg._c()), wire, ref, steps, xhat, 0)


def test_argument_errors_are_synchronous(lib):
    good = rac.RacConfig(64, 512, 64, 64, 4)
    assert _encode(rac.RacConfig(64, 512, 64, 64, 5)) == 1              # invalid bits
    assert _encode(good, x=None) == 1                                    # x required
    assert _encode(good, x=FAKE + 2) == 2                                # x misaligned
    assert _encode(good, ref=FAKE + 8) == 2                              # ref misaligned
    assert _encode(good, wire=FAKE + 16) == 2                            # wire needs 256 B
    assert _encode(good, xhat=FAKE + 4) == 2                             # xhat misaligned
    assert _encode(good, cap=rac.rac_wire_size(good) - 1) == 3           # capacity
    fixed = rac.RacConfig(64, 512, 64, 64, 4, 0, rac.RAC_FLAG_FIXED_STEP)
    assert _encode(fixed, steps=None) == 1                               # steps required
    big = rac.RacConfig(4, 16384, 128, 128, 4)
    assert _encode(big) == 6                                             # kernels cap d at 8192
    assert _decode(rac.RacConfig(64, 512, 64, 64, 5)) == 1
    assert _decode(good, wire=FAKE + 128) == 2
    assert _decode(good, xhat=None) == 1
    assert rac.library().rac_reconstruct(ctypes.byref(good._c()), FAKE, FAKE, None, FAKE + 1, 0) == 2


def test_gather_argument_errors_are_synchronous(lib):
    good = rac.RacConfig(64, 512, 64, 64, 4)
    L = rac.library()
    enc = lambda store=FAKE, rows=64, idx=FAKE, x=FAKE: L.rac_encode_gather(
        ctypes.byref(good._c()), x, store, rows, idx, None, FAKE, 1 << 40, FAKE, 0)
    dec = lambda store=FAKE, rows=64, idx=FAKE, xhat=FAKE: L.rac_decode_gather(
        ctypes.byref(good._c()), FAKE, store, rows, idx, None, xhat, 0)
    assert enc(idx=None) == 1                   # a store needs its row indices
    assert enc(rows=-1) == 1 and enc(rows=2 ** 31) == 1
    assert enc(idx=FAKE + 2) == 2               # indices are int32
    assert enc(store=FAKE + 8) == 2             # store rows are read 16 bytes at a time
    assert enc(x=None) == 1
    assert dec(idx=None) == 1 and dec(rows=-5) == 1 and dec(idx=FAKE + 1) == 2 and dec(xhat=None) == 1
    big = rac.RacConfig(4, 16384, 128, 128, 4)
    assert L.rac_encode_gather(ctypes.byref(big._c()), FAKE, FAKE, 4, FAKE, None, FAKE, 1 << 40, FAKE, 0) == 6


def test_binding_raises_without_the_library(monkeypatch):
    """No fallback: with librac.so absent every call raises instead of
    computing anything elsewhere."""
    monkeypatch.setattr(rac, "_lib", None)
    monkeypatch.setattr(rac, "library_path", lambda: "/nonexistent/librac.so")
    with pytest.raises(RuntimeError, match="missing"):
        rac.rac_wire_size(rac.RacConfig(4, 512, 64, 64, 4))
    with pytest.raises(RuntimeError, match="missing"):
        rac.rac_encode(rac.RacConfig(4, 512, 64, 64, 4), FAKE, FAKE, None, FAKE, FAKE, stream=0, wire_cap=1)
    with pytest.raises(RuntimeError, match="missing"):
        rac.SpanIndex(8)


def test_pooled_argument_errors_are_synchronous(lib):
    L = rac.library()
    enc = lambda cfg, segs=4, starts=FAKE, x=FAKE: L.rac_encode_pooled(
        ctypes.byref(cfg._c()), x, FAKE, segs, starts, None, FAKE, 1 << 40, FAKE, 0)
    good = rac.RacConfig(64, 512, 64, 64, 4)
    assert enc(good, starts=None) == 1 and enc(good, segs=0) == 1 and enc(good, segs=65) == 1
    assert enc(good, x=None) == 1 and enc(good, starts=FAKE + 2) == 2
    assert enc(rac.RacConfig(64, 2048, 1024, 64, 4)) == 6        # groups wider than a chunk
    assert enc(rac.RacConfig(64, 512, 32, 64, 2)) == 6           # moments do not fit the code section
    assert enc(rac.RacConfig(0, 512, 64, 64, 4), segs=1) == 1    # no rows to pool


def test_rejected_pooled_call_leaves_the_wire_untouched(lib):
    """Every argument check of rac_encode_pooled, the UNSUPPORTED one for
    segments * (d / g_a) >= 2^31 included, comes before its first launch: a
    rejected call writes nothing.  The wire here is host memory the call
    would fault on if it launched anything."""
    T = 1 << 25
    cfg = rac.RacConfig(T, 4096, 32, 128, 4)          # 128 groups per row, T segments
    buf = np.full(4096, 0x5A, dtype=np.uint8)
    base = (buf.ctypes.data + 255) & ~255
    st = rac.library().rac_encode_pooled(ctypes.byref(cfg._c()), FAKE, FAKE, T, FAKE, None, base,
                                         1 << 62, FAKE, 0)
    assert st == 6
    assert (buf == 0x5A).all()


class _FakeTensor:
    """Stands in for a torch tensor in the binding's argument checks."""

    def __init__(self, numel, esize, cuda=True, contiguous=True):
        self._n, self._e, self.is_cuda, self._c = numel, esize, cuda, contiguous

    def numel(self):
        return self._n

    def element_size(self):
        return self._e

    def is_contiguous(self):
        return self._c

    def data_ptr(self):
        return FAKE


def test_binding_checks_tensor_arguments_before_the_call(lib, monkeypatch):
    """Host-side checks of the binding: a CPU tensor, a non-contiguous one, a
    wrong element size or too few elements raise ValueError before the
    library is called."""
    called = []
    monkeypatch.setattr(rac, "library", lambda: type("L", (), {
        "rac_encode": lambda *a: called.append(a) or 0,
        "rac_decode": lambda *a: called.append(a) or 0,
        "rac_wire_size": lib.rac_wire_size})())
    cfg = rac.RacConfig(4, 512, 64, 64, 4)
    n = 4 * 512
    ok = dict(x=_FakeTensor(n, 2), ref=_FakeTensor(n, 2), wire=_FakeTensor(1 << 20, 1),
              xhat=_FakeTensor(n, 4))
    rac.rac_encode(cfg, ok["x"], ok["ref"], None, ok["wire"], ok["xhat"], stream=0)
    assert len(called) == 1
    bad = [dict(x=_FakeTensor(n, 2, cuda=False)), dict(x=_FakeTensor(n, 2, contiguous=False)),
           dict(x=_FakeTensor(n, 4)), dict(ref=_FakeTensor(n - 1, 2)), dict(xhat=_FakeTensor(n, 2)),
           dict(xhat=_FakeTensor(n - 8, 4))]
    for b in bad:
        a = dict(ok, **b)
        with pytest.raises(ValueError):
            rac.rac_encode(cfg, a["x"], a["ref"], None, a["wire"], a["xhat"], stream=0)
    with pytest.raises(ValueError):
        rac.rac_decode(cfg, _FakeTensor(100, 1), ok["ref"], None, ok["xhat"], stream=0)
    assert len(called) == 1


def test_calibration_argument_errors_are_synchronous(lib):
    L = rac.library()
    # error reduction: hidden not a multiple of 8, bad flags, misalignment, small workspace
    err = lambda T=16, d=512, flags=0, x=FAKE, xh=FAKE, st=FAKE, ws=FAKE, cap=1 << 20: L.rac_recon_error(
        T, d, flags, x, xh, st, ws, cap, 0)
    assert err(d=516) == 1 and err(flags=rac.RAC_FLAG_FIXED_STEP) == 1 and err(st=None) == 1
    assert err(x=FAKE + 2) == 2 and err(xh=FAKE + 8) == 2 and err(st=FAKE + 4) == 2
    assert err(cap=rac.rac_recon_error_workspace(16) - 1) == 3
    assert rac.rac_recon_error_workspace(16) == 48 and rac.rac_recon_error_workspace(17) == 72
    # calibration: candidates must share the sample's shape and use no step table
    good = [rac.RacConfig(64, 512, 64, 64, 4), rac.RacConfig(64, 512, 128, 128, 2, 1, rac.RAC_FLAG_GROUP_OUTLIERS)]
    assert rac.rac_calibrate_workspace(good) > 64 * 512 * 4
    assert rac.rac_calibrate_workspace(good + [rac.RacConfig(32, 512, 64, 64, 4)]) == 0
    assert rac.rac_calibrate_workspace(good + [rac.RacConfig(64, 512, 64, 64, 4, 0, rac.RAC_FLAG_FIXED_STEP)]) == 0
    arr = rac._candidates(good)
    ch = ctypes.c_int32(-7)
    need = rac.rac_calibrate_workspace(good)
    cal = lambda x=FAKE, tgt=0.01, ws=FAKE, cap=need, chosen=ctypes.byref(ch): L.rac_calibrate(
        x, FAKE, arr, 2, tgt, ws, cap, chosen, 0)
    assert cal(tgt=-1.0) == 1 and cal(tgt=float("nan")) == 1 and cal(x=None) == 1 and cal(chosen=None) == 1
    assert cal(cap=need - 1) == 3 and cal(ws=FAKE + 16) == 2 and cal(x=FAKE + 2) == 2
    assert ch.value == -7


def test_saturation_summary_reads_the_infinity_marks_of_oracle_wires(lib):
    """rac_saturation_summary on wires the oracle wrote, against the
    test-side reader of the format: per-token and per-group outliers, fixed
    steps (no scale section), and a short buffer."""
    x = np.zeros((4, 1024), np.float32)
    x[0, 0:128] = np.tile([2.0 ** 20, -2.0 ** 20], 64)          # row 0: scale past the range (+ outliers)
    x[2, 600], x[2, 601] = 131072.0, -131072.0                  # row 2: outlier values past the range
    x[3, 512:576] = 65536.0                                      # row 3: beta past the range
    xb = wl.f32_to_bf16_bits(x)
    for flags, k in ((0, 2), (rac.RAC_FLAG_GROUP_OUTLIERS, 1), (0, 0)):
        c = dict(tokens=4, hidden=1024, group_align=64, group_quant=128, bits=4, outlier_k=k, flags=flags)
        rc, wire, _ = oracle.encode(xb, None, want_xhat=False, **c)
        assert rc == 0
        marks = wirefmt.saturation_marks(wire)
        rows, bits = rac.rac_saturation_summary(rac.RacConfig(**c), wire)
        # (without outliers row 2's large values are dense and covered by a finite scale)
        assert rows == int((marks != 0).sum()) == (3 if k else 2) and bits == int(np.bitwise_or.reduce(marks))
        assert marks[3] == 1 and marks[1] == 0
        with pytest.raises(rac.RacError):
            rac.rac_saturation_summary(rac.RacConfig(**c), wire[:-1])
    c = dict(tokens=4, hidden=1024, group_align=64, group_quant=128, bits=4, outlier_k=2,
             flags=rac.RAC_FLAG_FIXED_STEP)
    rc, wire, _ = oracle.encode(xb, None, np.full(8, 1.0, np.float32), want_xhat=False, **c)
    # rows 0 and 2: outlier values past the range; row 3: beta; no scale section
    assert rac.rac_saturation_summary(rac.RacConfig(**c), wire) == (3, 5)


def test_predictor_layout_is_the_documented_one_and_errors_are_synchronous(lib):
    up = lambda v: (v + 255) // 256 * 256
    cfg = rac.PredictorConfig(4096, 512, 8, 2048, 64, 256)
    lay = rac.rac_predictor_layout(cfg)
    d, m, f = 4096, 512, 2048
    o, want = 0, {}
    for name, n in (("w_in", m * d), ("g1", m), ("w_qkv", 3 * m * m), ("w_o", m * m), ("g2", m),
                    ("w_gu", 2 * f * m), ("w_down", m * f), ("g3", m), ("w_out", d * m)):
        want[name] = o
        o = up(o + 2 * n)
    want["total"] = o
    assert lay == want
    assert rac.rac_predictor_cache_bytes(cfg) == 256 * 64 * 2 * 512 * 2
    assert rac.rac_predictor_workspace_bytes(cfg) > 0
    for bad in (rac.PredictorConfig(4000, 512, 8, 2048, 64, 8), rac.PredictorConfig(4096, 512, 4, 2048, 64, 8),
                rac.PredictorConfig(4096, 512, 8, 2000, 64, 8), rac.PredictorConfig(4096, 512, 8, 2048, 0, 8),
                rac.PredictorConfig(4096, 512, 8, 2048, 64, 257), rac.PredictorConfig(4096, 192, 3, 2048, 64, 8)):
        assert rac.rac_predictor_workspace_bytes(bad) == 0
        with pytest.raises(rac.RacError):
            rac.rac_predictor_layout(bad)
    L = rac.library()
    step = lambda B=4, w=FAKE, c=FAKE, p=FAKE, x=FAKE, r=FAKE, ws=FAKE, cap=1 << 40: L.rac_predictor_step(
        ctypes.byref(cfg._c()), w, c, p, B, x, r, ws, cap, 0)
    assert step(B=257) == 1 and step(B=-1) == 1 and step(w=None) == 1 and step(p=None) == 1
    assert step(w=FAKE + 16) == 2 and step(x=FAKE + 8) == 2 and step(p=FAKE + 2) == 2 and step(ws=FAKE + 64) == 2
    assert step(cap=rac.rac_predictor_workspace_bytes(cfg) - 1) == 3
    assert step(B=0, w=None, p=None) == 0      # an empty batch enqueues nothing


@pytest.mark.parametrize("missing", [(), ("_cuda_getCurrentRawStream",), ("_cuda_getDevice",)])
@pytest.mark.parametrize("initialized", [True, False])
def test_current_stream_with_and_without_the_raw_handle(missing, initialized):
    # the raw handle is read by names of torch that are not public: without
    # them, and before the device is initialized, the Stream object's is taken
    import types
    C = types.SimpleNamespace(_cuda_getCurrentRawStream=lambda dev: 100 + dev, _cuda_getDevice=lambda: 3)
    for name in missing:
        delattr(C, name)
    cuda = types.SimpleNamespace(is_initialized=lambda: initialized,
                                 current_stream=lambda: types.SimpleNamespace(cuda_stream=7))
    read = rac._stream_reader(types.SimpleNamespace(_C=C, cuda=cuda))
    assert read() == (103 if initialized and not missing else 7)
