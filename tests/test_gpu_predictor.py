"""GPU parity of the decode-phase reference predictor against its binary64
oracle, through the C ABI.

The bar, per output element: |R_gpu - r| <= 2^-8 |r| + 2^-6 rms(y), with r
the oracle's unrounded x + y and y its predicted update, and on average
mean|R_gpu - r| <= 2^-9 mean|r| + 2^-10 rms(y).  Where it comes from: R is
bf16 (at most half an ulp, 2^-9 |r|, a quarter ulp on average);
the GPU accumulates in binary32 in another order than the binary64 oracle,
so the bf16 rounding of an intermediate activation (the normalized inputs,
the attention output, the SwiGLU output, the cached keys and values) lands on
the other neighbour where the exact value sits next to a rounding boundary,
which moves that activation by one bf16 ulp and the outputs it feeds by a
small fraction of rms(y).  A wrong lane layout, weight section, rotation or
window would be off by about rms(y).  The cached keys and values are checked
the same way against the oracle's cache.
"""
from __future__ import annotations

import numpy as np
import pytest

import paper_2608_04991_amd as rac
from oracle import predictor as P
from paper_2608_04991_amd import workloads as wl
from tests.gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rac.library()


def _run(cfg, batch, steps, pos_of, seed=0, check_every=1):
    import torch
    weights = wl.predictor_weights(cfg.hidden, cfg.model, cfg.ffn, seed)
    blob = torch.from_numpy(rac.predictor_pack(cfg, weights)).cuda()
    cache = torch.zeros(rac.rac_predictor_cache_bytes(cfg) // 2, dtype=torch.int16, device="cuda")
    ws = torch.empty(rac.rac_predictor_workspace_bytes(cfg), dtype=torch.uint8, device="cuda")
    ref = P.Predictor(weights, cfg.hidden, cfg.model, cfg.heads, cfg.ffn, cfg.window, cfg.max_batch)
    xs = wl.decode_sequence(batch, steps, seed, hidden=cfg.hidden)
    out = torch.empty(batch, cfg.hidden, dtype=torch.int16, device="cuda")
    worst = 0.0
    for s in range(steps):
        pos = np.asarray([pos_of(s, b) for b in range(batch)], np.int32)
        x = torch.from_numpy(xs[s].view(np.int16)).cuda()
        rac.rac_predictor_step(cfg, blob, cache, torch.from_numpy(pos).cuda(), x, out, ws, batch)
        _, inter = ref.step(xs[s], pos)
        if s % check_every and s != steps - 1:
            continue
        torch.cuda.synchronize()
        g = P.bf16_to_f64(out.cpu().numpy().view(np.uint16))
        r, y = inter["r"], inter["y"]
        ry = np.sqrt(np.mean(y * y))
        err = np.abs(g - r)
        assert np.all(err <= 2.0 ** -8 * np.abs(r) + 2.0 ** -6 * ry), \
            f"step {s}: worst {np.max(err / (2.0 ** -8 * np.abs(r) + 2.0 ** -6 * ry)):.3f} of the bar"
        assert err.mean() <= 2.0 ** -9 * np.abs(r).mean() + 2.0 ** -10 * ry, (s, err.mean() / ry)
        worst = max(worst, float((err / ry).max()))
        # (for the record: elements whose bf16 differs from the oracle's rounding of r)
        off = float(np.mean(g != P.to_bf16(r)))
        say(f"[gpu]   step {s}: max |R - r| {err.max() / ry:.2e} rms(y), mean {err.mean() / ry:.2e}, "
            f"{off:.2%} of elements off the oracle's bf16")
    torch.cuda.synchronize()
    gc = P.bf16_to_f64(cache.cpu().numpy().view(np.uint16)).reshape(ref.cache.shape)
    used = np.zeros(ref.cache.shape[:2], dtype=bool)
    for b in range(batch):
        for s in range(steps):
            used[b, pos_of(s, b) % cfg.window] = True
    oc = ref.cache[used]
    rc = np.sqrt(np.mean(oc * oc))
    assert np.all(np.abs(gc[used] - oc) <= 2.0 ** -7 * np.abs(oc) + 2.0 ** -7 * rc)
    return worst


def test_predictor_glm_shape_70_steps_window_wraps():
    cfg = rac.PredictorConfig(4096, 512, 8, 2048, 64, 64)
    say("[gpu] predictor 4096/512/8/2048, window 64, batch 16, 70 steps")
    worst = _run(cfg, 16, 70, lambda s, b: s, check_every=7)
    say(f"[gpu] predictor: worst |R - r| = {worst:.2e} rms(y)")


def test_predictor_ragged_batch_with_staggered_and_restarted_positions():
    cfg = rac.PredictorConfig(512, 128, 2, 256, 5, 40)
    # sequence b starts at position 7 (b % 3); every fifth restarts at step 6
    pos = lambda s, b: (s - 6 if (b % 5 == 0 and s >= 6) else s + 7 * (b % 3))
    say("[gpu] predictor 512/128/2/256, window 5, batch 37, 12 steps")
    _run(cfg, 37, 12, pos)


@pytest.mark.parametrize("batch", [1, 100, 256])
def test_predictor_single_and_full_batches(batch):
    # (100: ragged row tiles, 6 x 16 + 4 and 3 x 32 + 4)
    cfg = rac.PredictorConfig(4096, 512, 8, 2048, 64, 256)
    say(f"[gpu] predictor batch {batch}, 3 steps")
    _run(cfg, batch, 3, lambda s, b: s + 100 * (b % 2), seed=1)


@pytest.mark.parametrize("window,start", [(300, 400), (1024, 1500)])
def test_predictor_windows_longer_than_one_pass_of_64_positions(window, start):
    # sequences start deep into their positions, so the window reaches back
    # over slots never written (zero on both sides) and spans several passes
    # of 64 positions in the score loop
    cfg = rac.PredictorConfig(512, 128, 2, 256, window, 8)
    say(f"[gpu] predictor 512/128/2/256, window {window}, batch 8, 4 steps from position {start}")
    _run(cfg, 8, 4, lambda s, b: start + s + 37 * b, seed=2)



@pytest.mark.parametrize("hidden,model,heads,ffn,window,batch", [
    (4096, 512, 8, 2048, 64, 2), (4096, 512, 8, 2048, 64, 4),
    (1024, 2048, 32, 512, 16, 3), (512, 128, 2, 256, 5, 4)])
def test_predictor_small_batches_fold_the_norms(hidden, model, heads, ffn, window, batch):
    # a few rows in the smallest tiles, whose products form the norm of what
    # they read; model widths 128 to 2048, and down projections of 4, 8 and 32
    # units of 64 channels over eight wavefronts
    cfg = rac.PredictorConfig(hidden, model, heads, ffn, window, 4)
    say(f"[gpu] predictor {hidden}/{model}/{heads}/{ffn}, window {window}, batch {batch}, 6 steps")
    _run(cfg, batch, 6, lambda s, b: s + 3 * b, seed=4)


@pytest.mark.parametrize("hidden,model,heads,ffn,window,batch", [
    (512, 2048, 32, 256, 3, 33), (8192, 128, 2, 8192, 5, 1), (512, 2048, 32, 128, 2, 130),
    (8192, 1536, 24, 8192, 3, 75), (2048, 2048, 32, 4096, 2, 60)])
def test_predictor_product_tiles(hidden, model, heads, ffn, window, batch):
    # tiles of the products with a ragged last row tile (33 = 2 x 16 + 1
    # and 32 + 1; 130 = 4 x 32 + 2; 1), and K shares from none at all (two
    # units of 64 channels over eight wavefronts) to sixteen units; the last
    # three also take products whose rows are normalized ahead of them
    cfg = rac.PredictorConfig(hidden, model, heads, ffn, window, batch)
    say(f"[gpu] predictor {hidden}/{model}/{heads}/{ffn}, window {window}, batch {batch}, 3 steps")
    _run(cfg, batch, 3, lambda s, b: s + b % 4, seed=5)


# With the shapes above every kernel of the predictor (tests/test_dispatch.py
# holds the library to that): each tile of each product, rows normalized on the
# way and ahead, and the attention's one, two and four wavefronts, the two at
# both ends of their windows (66 and 129)
EVERY_KERNEL = [
    (8192, 1024, 16, 4096, 66, 16), (8192, 1024, 16, 4096, 100, 250), (512, 2048, 32, 128, 129, 32),
    (8192, 128, 2, 128, 3, 32), (512, 1536, 24, 128, 2, 130)]


@pytest.mark.parametrize("hidden,model,heads,ffn,window,batch", EVERY_KERNEL)
def test_predictor_every_kernel(hidden, model, heads, ffn, window, batch):
    # positions from inside the first window to past its second turn
    cfg = rac.PredictorConfig(hidden, model, heads, ffn, window, batch)
    say(f"[gpu] predictor {hidden}/{model}/{heads}/{ffn}, window {window}, batch {batch}, 3 steps")
    _run(cfg, batch, 3, lambda s, b: s + (2 * window * b) // max(1, batch - 1) if batch > 1 else s, seed=6)


@pytest.mark.parametrize("hidden,model,batch", [
    (2048, 128, 64), (8192, 128, 64), (8192, 512, 80), (8192, 1024, 100), (8192, 1024, 250), (4096, 2048, 160)])
def test_predictor_products_onto_the_model_width_keep_their_accuracy(hidden, model, batch):
    """The fp32 error of h0 = x W_in^T, made visible: the channels come in pairs
    with x equal and W_in opposite, at random places, so a sum cancels to the
    one signal of 2^-18 and what else is left of it is rounding error.  W_o and
    W_down are zero, the gains one and W_out passes the model width through to
    channels where x is zero, so R there is RMSNorm(h0): a signal common to the
    row with the errors around it, about 2^-6 of it, well over bf16's 2^-9.

    The bar is a simulation of fp32 sums in chains of 128 channels, each 32 of
    them added exactly, four chains and then the ranges of 512 in order, times
    1.35: the matrix core rounds inside its 32 channels as well, with which such
    chains measured 1.0 to 1.3 of the simulation for these shapes.  One
    accumulator over the channels of a wavefront measures 1.5 to 2.6."""
    import torch
    say(f"[gpu] predictor accuracy {hidden}/{model}, batch {batch}")
    signal = 2.0 ** -18
    rng = np.random.default_rng([hidden, model, batch])
    half = (hidden - model) // 2
    to_bf = lambda a: wl.f32_to_bf16_bits(np.asarray(a, np.float32))
    rounded = lambda a: wl.bf16_bits_to_f32(to_bf(a))
    x, w = np.zeros((batch, hidden), np.float32), np.zeros((model, hidden), np.float32)
    place = model + rng.permutation(2 * half)
    a, b = place[:half], place[half:]
    x[:, a] = x[:, b] = rounded(rng.standard_normal((batch, half)))
    w[:, a] = rounded(rng.standard_normal((model, half)) / np.sqrt(2 * half))
    w[:, b] = -w[:, a]
    x[:, a[0]], w[:, a[0]], w[:, b[0]] = 1.0, signal, 0.0
    through = np.zeros((hidden, model), np.float32)
    through[np.arange(model), np.arange(model)] = 1.0
    zero, one = (lambda *s: np.zeros(s, np.uint16)), to_bf(np.ones(model))
    weights = dict(w_in=to_bf(w), g1=one, w_qkv=zero(3 * model, model), w_o=zero(model, model), g2=one,
                   w_gu=zero(256, model), w_down=zero(model, 128), g3=one, w_out=to_bf(through))
    cfg = rac.PredictorConfig(hidden, model, model // 64, 128, 4, batch)
    blob = torch.from_numpy(rac.predictor_pack(cfg, weights)).cuda()
    cache = torch.zeros(rac.rac_predictor_cache_bytes(cfg) // 2, dtype=torch.int16, device="cuda")
    ws = torch.empty(rac.rac_predictor_workspace_bytes(cfg), dtype=torch.uint8, device="cuda")
    out = torch.empty(batch, hidden, dtype=torch.int16, device="cuda")
    rac.rac_predictor_step(cfg, blob, cache, torch.zeros(batch, dtype=torch.int32, device="cuda"),
                           torch.from_numpy(to_bf(x).view(np.int16)).cuda(), out, ws, batch)
    torch.cuda.synchronize()
    r = P.bf16_to_f64(out.cpu().numpy().view(np.uint16))[:, :model]
    err = np.sqrt(np.mean((signal * (r / r.mean(1, keepdims=True) - 1.0)) ** 2))
    rows = x[:max(2, 4096 // model)].astype(np.float64).reshape(-1, 1, hidden // 32, 32)
    dots = np.stack([(r * w.astype(np.float64).reshape(model, hidden // 32, 32)).sum(-1) for r in rows])
    add = lambda s, v: (s + v).astype(np.float32).astype(np.float64)
    total = 0.0
    for k in range(0, hidden // 32, 16):
        chains = []
        for q in range(k, k + 16, 4):
            c = add(0.0, dots[..., q])
            for i in range(q + 1, q + 4):
                c = add(c, dots[..., i])
            chains.append(c)
        total = add(total, add(add(add(chains[0], chains[1]), chains[2]), chains[3]))
    bar = np.sqrt(np.mean((total - signal) ** 2))
    say(f"[gpu]   error {err:.3e}, chains of 128 {bar:.3e} ({err / bar:.2f})")
    assert err <= 1.35 * bar
