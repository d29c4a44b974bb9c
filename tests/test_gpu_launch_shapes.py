"""GPU: the launch hints change how rows are spread over workgroups, never a
byte of the output.  Above 256 rows a launch runs either on the strided grid
(the workgroups the device holds at once, each taking rows in strides with
its next row prefetched) or on one workgroup per row; the default picks by
rows per workgroup.  Each case runs the default, RAC_FLAG_LAUNCH_STRIDED and
RAC_FLAG_LAUNCH_PER_ROW and requires identical wires and reconstructions; the
default is also held to the oracle.  The cases cover the outlier modes, the
bf16 reconstruction and a step table.
"""
from __future__ import annotations

import numpy as np
import pytest

import paper_2608_04991_amd as rac
from paper_2608_04991_amd import workloads as wl
from tests.gpu_util import assert_parity, cfgd, gpu_run, oracle_run, say, to_dev

pytestmark = pytest.mark.gpu
GRP = rac.RAC_FLAG_GROUP_OUTLIERS
HINTS = (0, rac.RAC_FLAG_LAUNCH_STRIDED, rac.RAC_FLAG_LAUNCH_PER_ROW)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rac.library()


def _bytes(a):
    return np.ascontiguousarray(a).view(np.uint8)


CASES = {
    # per-token outliers (the rows kernel and the per-token decode)
    "per_token_3000x1024_g128_b4_k8": (cfgd(3000, 1024, 128, 128, 4, 8), 0),
    # per-group outliers (one wavefront per chunk)
    "per_group_2999x1024_ga64_gq128_b3_kg2": (cfgd(2999, 1024, 64, 128, 3, 2, GRP), 1),
    # no outliers, bf16 reconstruction, a ragged chunk (1536 = 3 chunks)
    "none_bf16_2600x1536_g128_b8": (cfgd(2600, 1536, 128, 128, 8, 0, rac.RAC_FLAG_XHAT_BF16), 2),
    "per_token_1000x4096_g64_b2_k16": (cfgd(1000, 4096, 64, 64, 2, 16), 3),
    # 16 < k <= 48: the two-value threshold variant of the rows kernel
    "per_token_1500x2048_g128_b4_k32": (cfgd(1500, 2048, 128, 128, 4, 32), 5),
    # k > 48: the four-value threshold and the list of 128 candidates
    "per_token_2100x4096_g128_b4_k64": (cfgd(2100, 4096, 128, 128, 4, 64), 6),
    # bf16 reconstruction from the rows kernel (one and two threshold values)
    "per_token_bf16_2000x2048_g128_b4_k8": (cfgd(2000, 2048, 128, 128, 4, 8, rac.RAC_FLAG_XHAT_BF16), 7),
    "per_token_bf16_1100x4096_g128_b3_k32": (cfgd(1100, 4096, 128, 128, 3, 32, rac.RAC_FLAG_XHAT_BF16), 8),
    # a step table (the chunk kernel's per-token and per-group selections;
    # codes clip by design)
    "fixed_step_per_token_1800x2048_g128_b4_k4": (cfgd(1800, 2048, 128, 128, 4, 4, rac.RAC_FLAG_FIXED_STEP), 9),
    "fixed_step_per_group_1500x1024_g64_b4_kg2": (cfgd(1500, 1024, 64, 64, 4, 2, rac.RAC_FLAG_FIXED_STEP | GRP), 10),
}


def _steps(c, seed):
    """A step per quantization group for the step-table cases (None otherwise)."""
    if not c["flags"] & rac.RAC_FLAG_FIXED_STEP:
        return None
    return np.random.default_rng(seed).uniform(0.01, 0.2, c["hidden"] // c["group_quant"]).astype(np.float32)


@pytest.mark.parametrize("name", list(CASES))
def test_launch_shapes_give_identical_bytes(name):
    c, seed = CASES[name]
    T, d = c["tokens"], c["hidden"]
    xb, rb, _ = wl.prefill_uplink(seed, tokens=T, hidden=d)
    steps = _steps(c, seed)
    outs = []
    for hint in HINTS:
        say(f"[gpu] launch shapes {name}: hint {hint}")
        outs.append(gpu_run(dict(c, flags=c["flags"] | hint), xb, rb, steps))
    for o in outs[1:]:
        for a, b in zip(outs[0], o):
            assert np.array_equal(_bytes(a), _bytes(b))
    ow, ox = oracle_run(c, xb, rb, steps)
    assert_parity(c, outs[0][0], outs[0][1], ow, ox)


def test_launch_shapes_gathered_and_pooled():
    """The gathered reference (at most 64 rows per workgroup on the strided
    grid) and the pooled fit's encode launch under every hint."""
    import torch
    T, d = 3000, 1024
    c = cfgd(T, d, 128, 128, 4, 4)
    xb, rb, _ = wl.prefill_uplink(4, tokens=T, hidden=d)
    rng = np.random.default_rng(8)
    S = T + 500
    store = wl.f32_to_bf16_bits(rng.standard_normal((S, d)).astype(np.float32))
    pos = rng.permutation(S)[:T]
    store[pos] = rb
    idx = pos.astype(np.int32)
    idx[rng.random(T) < 0.2] = -1
    cuts = np.unique(np.concatenate([[0, T], np.cumsum(rng.integers(1, 300, 20))]))
    seg = cuts[cuts <= T].astype(np.int32)
    x, st, ref = to_dev(xb), to_dev(store), to_dev(rb)
    ix, sg = torch.from_numpy(idx).cuda(), torch.from_numpy(seg).cuda()
    res = []
    for hint in HINTS:
        say(f"[gpu] launch shapes gathered/pooled {T}x{d}: hint {hint}")
        cfg = rac.RacConfig(**dict(c, flags=hint))
        wb = rac.rac_wire_size(cfg)
        w1, w2 = (torch.full((wb,), 0xAB, dtype=torch.uint8, device="cuda") for _ in range(2))
        h1, h2, d1 = (torch.full((T, d), -1.0, dtype=torch.float32, device="cuda") for _ in range(3))
        rac.rac_encode_gather(cfg, x, st, ix, None, w1, h1, store_rows=S)
        rac.rac_decode_gather(cfg, w1, st, ix, None, d1, store_rows=S)
        rac.rac_encode_pooled(cfg, x, ref, sg, None, w2, h2)
        torch.cuda.synchronize()
        res.append([t.cpu().numpy() for t in (w1, h1, d1, w2, h2)])
    for r in res[1:]:
        for a, b in zip(res[0], r):
            assert np.array_equal(_bytes(a), _bytes(b))
    assert np.array_equal(_bytes(res[0][1]), _bytes(res[0][2]))
    gref = np.zeros_like(rb)
    ok = idx >= 0
    gref[ok] = store[idx[ok]]
    ow, ox = oracle_run(c, xb, gref)
    assert_parity(c, res[0][0], res[0][1], ow, ox)


def test_more_rows_than_one_dispatch_holds():
    """17,000,000 rows of 8 channels: one workgroup per row would exceed the
    2^32 work-items of a dispatch for the 256-thread outlier encode, so its
    grid stops at 16,777,215 workgroups and some take a second row.  Sampled
    rows (the ends of the grid and past it) must equal the oracle's, decode
    and reconstruct the sender's on every row, and a gathered call with a
    fifth of its rows missing the same bytes as the materialized call."""
    import torch
    from tests.gpu_util import gpu_run_rows
    T, d = 17_000_000, 8
    c = cfgd(T, d, 8, 8, 4, 2)
    say(f"[gpu] {T}x{d} k2: generating")
    # the tiny recipe's distribution, drawn in bulk: x = a ref + b + noise with
    # (a, b) per row, a fifth of the rows against a zero reference
    rng = np.random.default_rng(11)
    ref = rng.standard_normal((T, d), dtype=np.float32)
    x = (rng.uniform(0.8, 1.2, (T, 1)).astype(np.float32) * ref
         + (0.1 * rng.standard_normal((T, 1))).astype(np.float32)
         + np.float32(0.05) * rng.standard_normal((T, d), dtype=np.float32))
    ref[rng.random(T) < 0.2] = 0.0
    xb, rb = wl.f32_to_bf16_bits(x), wl.f32_to_bf16_bits(ref)
    del x, ref
    cap = 0xFFFFFFFF // 256
    rows = np.unique(np.concatenate([[0, 1, cap - 1, cap, cap + 1, T - 2, T - 1],
                                     rng.choice(T, 40, replace=False)]))
    say(f"[gpu] {T}x{d} k2: encode, decode, reconstruct")
    gw, gx = gpu_run_rows(c, xb, rb, rows)
    ow, ox = oracle_run(dict(c, tokens=rows.size), xb[rows], rb[rows])
    assert_parity(c, gw, gx, ow, ox, g_rows=rows, o_rows=slice(None), g_xhat_sampled=True)
    # gathered: the store is the reference itself, and a fifth of the rows
    # name no row (their reference is zero in the materialized call)
    miss = rng.random(T) < 0.2
    idx = np.arange(T, dtype=np.int32)
    idx[miss] = -1
    rz = rb.copy()
    rz[miss] = 0
    say(f"[gpu] {T}x{d} k2: gathered against materialized")
    cfg = rac.RacConfig(**c)
    x, st, ix = to_dev(xb), to_dev(rb), torch.from_numpy(idx).cuda()
    wg = torch.empty(rac.rac_wire_size(cfg), dtype=torch.uint8, device="cuda")
    rac.rac_encode_gather(cfg, x, st, ix, None, wg, None, store_rows=T)
    torch.cuda.synchronize()
    del st
    wm = torch.empty_like(wg)
    rac.rac_encode(cfg, x, to_dev(rz), None, wm, None)
    torch.cuda.synchronize()
    assert torch.equal(wg, wm)
    del x, ix, wg, wm
    torch.cuda.empty_cache()


@pytest.mark.parametrize("d,g,k,bits", [(520, 8, 1, 4), (2048, 128, 16, 2), (4096, 128, 17, 3), (4096, 64, 48, 8),
                                        (4096, 128, 49, 4), (5120, 128, 16, 4), (8192, 64, 64, 3)])
def test_one_row_and_strided_forms_on_ties_and_plain_rows(d, g, k, bits):
    # the per-token kernel's two forms (one workgroup per row, which keeps R~;
    # strided, which forms it again) on rows of equal |E| (the candidate list
    # overflows and the exact search runs), rows with a zero residual and
    # ordinary ones; at the edges of the threshold's variants (k = 16, 17, 48,
    # 49), of two and four chunks a wavefront, and of a ragged last chunk
    T = 300
    rng = np.random.default_rng([d, k])
    xb, rb, _ = wl.prefill_uplink(11, tokens=T, hidden=d) if d % 128 == 0 else \
        wl.affine_pair(wl.AffineRecipe(T, d, 8), 11)
    xb, rb = xb.copy(), rb.copy()
    xb[0::3] = wl.f32_to_bf16_bits(rng.choice([-1.5, 1.5], size=xb[0::3].shape).astype(np.float32))
    rb[0::3] = 0
    xb[1::30] = rb[1::30]
    c = cfgd(T, d, g, g, bits, k)
    outs = []
    for hint in HINTS:
        say(f"[gpu] one row and strided forms {T}x{d} g={g} k={k} b={bits}: hint {hint}")
        outs.append(gpu_run(dict(c, flags=c["flags"] | hint), xb, rb, None))
    for o in outs[1:]:
        for a, b in zip(outs[0], o):
            assert np.array_equal(_bytes(a), _bytes(b))
    ow, ox = oracle_run(c, xb, rb, None)
    assert_parity(c, outs[0][0], outs[0][1], ow, ox)


@pytest.mark.parametrize("T,d,ga,gq,bits,k", [(1, 512, 64, 64, 4, 0), (257, 520, 8, 8, 3, 2), (333, 1536, 512, 256, 2, 16),
                                              (301, 7168, 128, 64, 8, 1), (259, 8192, 64, 128, 4, 4),
                                              (263, 4608, 256, 512, 3, 0)])
def test_flat_and_strided_forms_of_the_chunk_kernel(T, d, ga, gq, bits, k):
    # a (row, chunk) per wavefront against strided rows, plain, gathered (with
    # rows that name no store row) and with a bf16 reconstruction: rows of 1 to
    # 16 chunks, so that workgroups of four wavefronts straddle rows and the
    # last one is partly empty
    rng = np.random.default_rng([d, T])
    xb, rb, _ = wl.prefill_uplink(12, tokens=T, hidden=d) if d % 128 == 0 else \
        wl.affine_pair(wl.AffineRecipe(T, d, 8), 12)
    idx = rng.permutation(T).astype(np.int32)
    idx[rng.random(T) < 0.2] = -1
    gathered = np.where(idx[:, None] >= 0, rb[np.maximum(idx, 0)], 0).astype(np.uint16)
    import torch
    for bf16 in (0, rac.RAC_FLAG_XHAT_BF16):
        c = cfgd(T, d, ga, gq, bits, k, (GRP if k else 0) | bf16)
        ow, ox = oracle_run(c, xb, rb, None)
        gw, gx = oracle_run(c, xb, gathered, None)
        for hint in HINTS:
            say(f"[gpu] flat and strided {T}x{d} g={ga}/{gq} b={bits} k_g={k} bf16={bf16}: hint {hint}")
            out = gpu_run(dict(c, flags=c["flags"] | hint), xb, rb, None)
            assert_parity(c, out[0], out[1], ow, ox)
            cfg = rac.RacConfig(**dict(c, flags=c["flags"] | hint))
            wire = torch.empty(rac.rac_wire_size(cfg), dtype=torch.uint8, device="cuda")
            xh = torch.empty((T, d), dtype=torch.int16 if bf16 else torch.float32, device="cuda")
            rac.rac_encode_gather(cfg, to_dev(xb), to_dev(rb), torch.from_numpy(idx).cuda(), None, wire, xh)
            torch.cuda.synchronize()
            assert np.array_equal(wire.cpu().numpy(), _bytes(gw).ravel())
            assert np.array_equal(_bytes(xh.cpu().numpy()), _bytes(gx))


@pytest.mark.parametrize("T,d,ga,gq,bits,k,flags", [
    (2900, 4608, 128, 128, 4, 8, 0), (2700, 8192, 64, 64, 3, 16, 0), (2700, 8192, 128, 64, 8, 48, 0),  # four chunks a
    (2700, 7680, 64, 128, 2, 64, 0), (2700, 8192, 256, 256, 4, 17, 0),                                # wavefront
    (3900, 1024, 128, 128, 4, 48, 0), (3900, 2048, 32, 32, 2, 17, 0), (4100, 520, 8, 8, 3, 64, 0),     # two
    (4700, 2048, 128, 128, 4, 2, GRP), (4700, 2560, 64, 64, 8, 0, rac.RAC_FLAG_XHAT_BF16)])            # (row, chunk) forms
def test_strided_form_takes_several_rows(T, d, ga, gq, bits, k, flags):
    # more rows than two rounds of resident workgroups, so that the strided
    # kernels work on prefetched rows; tied, zero-residual and ordinary rows
    # side by side.  Rows are coded independently, so the oracle codes a sample
    # of them: the ends, every multiple of 256 and its neighbours
    rng = np.random.default_rng([d, k, T])
    xb, rb, _ = wl.prefill_uplink(13, tokens=T, hidden=d) if d % 128 == 0 else \
        wl.affine_pair(wl.AffineRecipe(T, d, 8), 13)
    xb, rb = xb.copy(), rb.copy()
    xb[0::3] = wl.f32_to_bf16_bits(rng.choice([-1.5, 1.5], size=xb[0::3].shape).astype(np.float32))
    rb[0::3] = 0
    xb[1::30] = rb[1::30]
    c = cfgd(T, d, ga, gq, bits, k, flags)
    rows = np.unique(np.clip(np.concatenate([np.arange(0, T, 256) + o for o in (-1, 0, 1)] + [[T - 1]]), 0, T - 1))
    outs = []
    for hint in HINTS:
        say(f"[gpu] strided over several rows {T}x{d} g={ga}/{gq} b={bits} k={k} flags={flags}: hint {hint}")
        outs.append(gpu_run(dict(c, flags=flags | hint), xb, rb, None))
    for o in outs[1:]:
        for a, b in zip(outs[0], o):
            assert np.array_equal(_bytes(a), _bytes(b))
    ow, ox = oracle_run(dict(c, tokens=rows.size), xb[rows], rb[rows], None)
    assert_parity(c, outs[1][0], outs[1][1], ow, ox, g_rows=rows, o_rows=slice(None))
