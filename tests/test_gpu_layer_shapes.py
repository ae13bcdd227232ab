"""One DiT layer against the float64 oracle at the sizes where the projection
and attention kernels change form: tile edges, remainders and the branches of
their dispatch, every row of the layer's update h_1 - h_0."""
import numpy as np
import pytest

from oracle import dit as OD
from synth import get_workload, make_weights, make_initial_noise, make_observations
from gpu_common import device, to_dev, f32_sigmas, BF16_UPDATE_TOL

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return device()


def _update_error(dev, spec, k=3, weight_std=0.05, rows=None):
    """max |update error| over max |update|, and the float32 spacing of h over
    max |update| (the rounding of the stored h); over the given rows of B T, or
    all."""
    from paper_2609_34608_amd import runtime as R
    W = make_weights(spec, bias_std=0.02, gain_std=0.1, weight_std=weight_std)
    m = R.WamModel(R.config_of(spec), W, device=dev)
    sig = f32_sigmas(spec.K)
    m.set_schedule(sig)
    x, cond = to_dev(make_initial_noise(spec), dev), to_dev(make_observations(spec, 0)[0], dev)
    h0 = m.hidden(k, x, cond, 0).cpu().numpy()
    h1 = m.hidden(k, x, cond, 1).cpu().numpy()
    m.close()
    c = OD.cond_vector(W, sig[k])
    if rows is None:
        ref = OD.dit_layer(W, spec, 0, h0, c) - h0
    else:
        ref = OD.dit_layer_rows(W, spec, 0, h0, c, rows)
        h0, h1 = (h.reshape(-1, spec.D)[rows] for h in (h0, h1))
        ref -= h0
    upd = np.max(np.abs(ref))
    return float(np.max(np.abs((h1 - h0) - ref)) / upd), float(2.0 ** -24 * np.max(np.abs(h1)) / upd)


def _spec(dtype, B, T, D, dh, F, qk_norm=True):
    na, no = min(7, T // 3), min(5, T // 4)
    return get_workload("tiny").replace(L=1, B=B, D=D, H=D // dh, F=F, Nv=T - na - no, Na=na, No=no, dtype=dtype,
                                        qk_norm=qk_norm)


# (B, T, D, head size, F, QK-norm).  Lengths around the 16-query tiles and the
# 64-key tiles (one to five key tiles over four waves, so some waves get none);
# head sizes 32 and 64; each of the three attention forms at both (2112 and more
# query tiles: no key split; 8320 and more: two tiles per wave) and each
# projection tile in each epilogue that the planner gives it, with rows and
# columns left over.  tests/test_plan_coverage.py checks that none is missing.
FP32_LAYERS = [
    (1, 3, 64, 32, 64, True), (1, 16, 64, 64, 192, True), (2, 17, 128, 32, 320, False), (1, 63, 192, 64, 768, True),
    (3, 64, 128, 64, 512, True), (1, 65, 320, 32, 1280, True), (1, 129, 192, 32, 448, False),
    (2, 321, 256, 64, 1024, True), (1, 2100, 512, 32, 512, True), (16, 1030, 256, 32, 256, True),
    (8, 43, 64, 64, 2240, True), (16, 34, 64, 64, 3008, False), (16, 74, 64, 64, 2752, True),
    (16, 119, 192, 64, 128, True), (16, 125, 192, 32, 512, True), (8, 139, 704, 32, 128, False),
    (16, 139, 320, 64, 128, True), (16, 268, 576, 64, 576, True), (16, 210, 320, 32, 320, True),
    (16, 319, 320, 64, 192, False), (16, 474, 448, 32, 128, True), (16, 709, 768, 64, 128, True),
    (1, 864, 768, 64, 3072, True),
]


@pytest.mark.parametrize("B,T,D,dh,F,qk_norm", FP32_LAYERS)
def test_float32_layer(dev, B, T, D, dh, F, qk_norm):
    err, ulp = _update_error(dev, _spec("fp32", B, T, D, dh, F, qk_norm))
    print(f"fp32 B={B} T={T} D={D} dh={dh} F={F}: update rel err {err:.2e}, h rounding {ulp:.2e}")
    # rounding of the stored h0 and h1 (two roundings each), and the first-order
    # bound of the float32 sums (one 2^-24 per term)
    assert err <= 4 * ulp + (F + 3 * D) * 2.0 ** -24, (err, ulp)


# (B, T, D, F).  Row counts off every tile height, widths 3 D, D and F that end
# inside a 128- or 64-column tile (odd head counts among them), from one block of
# rows to several rounds of the chip.
BF16_LAYERS = [
    (1, 3, 64, 128), (1, 70, 192, 512), (2, 137, 320, 1280), (1, 505, 640, 2560), (3, 400, 448, 1152),
    (2, 1100, 832, 2176), (2, 901, 1216, 4864), (4, 577, 1088, 2944), (1, 2650, 1600, 3200),
]


@pytest.mark.parametrize("B,T,D,F", BF16_LAYERS)
def test_bf16_layer(dev, B, T, D, F):
    err, _ = _update_error(dev, _spec("bf16", B, T, D, 64, F), weight_std=0.02)
    print(f"bf16 B={B} T={T} D={D} F={F}: update rel err {err:.2e}")
    assert err <= BF16_UPDATE_TOL, err


# (B, T, D, F).  With the sizes above, each projection tile in each epilogue that
# the planner gives it (tests/test_plan_coverage.py), rows left over in every one
# and columns too in the 256-column tiles: the last wave columns then lie past N
# and leave before the epilogue.
BF16_TILES = [
    (2, 5513, 128, 512), (2, 4946, 320, 896), (1, 3, 256, 640), (2, 3126, 64, 256), (1, 2691, 192, 768),
    (1, 5391, 192, 768), (2, 5514, 448, 1152), (3, 542, 640, 1664), (4, 605, 640, 2560), (2, 5541, 704, 1408),
    (3, 3279, 1088, 2944), (2, 5426, 1344, 3584),
]


@pytest.mark.parametrize("B,T,D,F", BF16_TILES)
def test_bf16_tiles(dev, B, T, D, F):
    """Every column of sampled rows: the ends of the samples, the last row tile
    (up to 320 rows), and rows of the others."""
    M = B * T
    rows = np.unique(np.r_[0, T - 1, M - 1 - T % 7, range(max(0, M - 320), M, 9), M - 1,
                           np.random.default_rng(5).integers(0, M, 40)])
    err, _ = _update_error(dev, _spec("bf16", B, T, D, 64, F), weight_std=0.02, rows=rows)
    print(f"bf16 B={B} T={T} D={D} F={F}: {len(rows)} rows' update rel err {err:.2e}")
    assert err <= BF16_UPDATE_TOL, err


# Attention forms of the automatic choice, bounded (QK-norm) and running max
# (without): (B, T, D).  Short sequences of few heads (key split, 16 queries per
# wave; one key tile, so that the second key group gets none) to grids of several
# blocks per CU (32, 48 and 64 queries per wave, 48 over eight waves), lengths off
# every block of queries and short enough in the last block that whole waves lie
# past T; every form of both tables is among them
# (tests/test_plan_coverage.py).  The scores of the unnormalised model spread over
# tens of log2 units, so the running max moves.
BF16_ATTENTION = [
    (1, 37, 64), (1, 449, 320), (4, 333, 1024), (16, 150, 512), (1, 2211, 512), (2, 1130, 1088),
    (16, 40, 1088), (1, 450, 64), (16, 513, 128), (16, 646, 192), (16, 769, 448), (16, 782, 320), (8, 1544, 256),
]


@pytest.mark.parametrize("qk_norm", [True, False])
@pytest.mark.parametrize("B,T,D", BF16_ATTENTION)
def test_bf16_attention_forms(dev, B, T, D, qk_norm):
    err, _ = _update_error(dev, _spec("bf16", B, T, D, 64, 2 * D, qk_norm), weight_std=0.02 if qk_norm else 0.045)
    print(f"bf16 attention B={B} T={T} D={D} qk_norm={qk_norm}: update rel err {err:.2e}")
    assert err <= BF16_UPDATE_TOL, err


@pytest.mark.parametrize("dtype,n_layers", [("bf16", 0), ("bf16", 1), ("bf16", 2), ("fp32", 2)])
def test_hidden_into_unaligned_output(dev, dtype, n_layers):
    """The last layer stores into a 16-byte aligned output itself; any other
    output receives a copy.  Same bits either way, no write past the end, and
    repeated calls start from the same embedding."""
    import torch
    from paper_2609_34608_amd import runtime as R
    spec = _spec(dtype, 2, 77, 128, 64, 512).replace(L=2)
    m = R.WamModel(R.config_of(spec), make_weights(spec, bias_std=0.02), device=dev)
    m.set_schedule(f32_sigmas(spec.K))
    x, cond = to_dev(make_initial_noise(spec), dev), to_dev(make_observations(spec, 0)[0], dev)
    n = spec.B * spec.T * spec.D
    ref = m.hidden(1, x, cond, n_layers)
    buf = torch.full((n + 2,), -7.0, device=dev)
    got = m.hidden(1, x, cond, n_layers, buf[1:n + 1].view(spec.B, spec.T, spec.D))
    assert torch.equal(ref, got) and float(buf[0]) == -7.0 and float(buf[-1]) == -7.0
    assert torch.equal(ref, m.hidden(1, x, cond, n_layers))
    m.close()


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
def test_overflowing_rows(dev, dtype, monkeypatch):
    """Rows whose sum of squares overflows float32 have scale zero: LayerNorm
    leaves the shift of its modulation, and q and k of such a head are zero
    (its softmax uniform), in the layer and in the final layer.  The trajectory
    rows here are of order 1e20 (their update is lost in h's rounding), the
    observation rows ordinary, and one head has a q bias of 1e21."""
    from paper_2609_34608_amd import runtime as R
    spec = _spec(dtype, 2, 77, 128, 64, 256)
    W = make_weights(spec, bias_std=0.02, gain_std=0.1, weight_std=0.05)
    W["l0.qkv_b"][:64] = 1e21
    m = R.WamModel(R.config_of(spec), W, device=dev)
    sig = f32_sigmas(spec.K)
    m.set_schedule(sig)
    x, cond = to_dev(make_initial_noise(spec) * 1e21, dev), to_dev(make_observations(spec, 0)[0], dev)
    h0 = m.hidden(3, x, cond, 0).cpu().numpy()
    h1 = m.hidden(3, x, cond, 1).cpu().numpy()
    v = m.velocity(3, x, cond)[0].cpu().numpy()
    m.close()
    obs = spec.Nv + spec.Na
    lim = float(np.finfo(np.float32).max)
    ln, rms = OD.layer_norm, OD.rms_norm
    over = lambda s: s.sum(-1, keepdims=True) > lim  # noqa: E731
    monkeypatch.setattr(OD, "layer_norm", lambda a, e: np.where(over((a - a.mean(-1, keepdims=True)) ** 2), 0, ln(a, e)))
    monkeypatch.setattr(OD, "rms_norm", lambda a, e: np.where(over(a * a), 0, rms(a, e)))
    c = OD.cond_vector(W, sig[3])
    ref = OD.dit_layer(W, spec, 0, h0, c)
    assert np.min(np.max(np.abs(h0[:, :obs]), -1)) > 1e19
    np.testing.assert_array_equal(h1[:, :obs], h0[:, :obs])
    upd = (ref - h0)[:, obs:]
    err = float(np.max(np.abs((h1 - h0)[:, obs:] - upd)) / np.max(np.abs(upd)))
    vref = OD.final_layer(W, spec, h1, c)
    verr = float(np.max(np.abs(v - vref)) / np.max(np.abs(vref)))
    print(f"{dtype}: observation rows' update rel err {err:.2e}, velocity {verr:.2e}")
    # float32: rounding of the stored h0 and h1 (two each) and the first-order
    # bound of the sums (one 2^-24 per term); the velocity is a D-term sum
    ulp = 2.0 ** -24 * float(np.max(np.abs(h1[:, obs:])) / np.max(np.abs(upd)))
    tol = BF16_UPDATE_TOL if dtype == "bf16" else 4 * ulp + (spec.F + 3 * spec.D) * 2.0 ** -24
    assert err <= tol and verr <= (2 * spec.D + 16) * 2.0 ** -24, (err, verr)
