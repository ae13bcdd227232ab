"""GPU parity: the HIP path through the C ABI against the float64 oracle.

Tolerances (max |got - ref| / max |ref| per compared tensor): 1e-4 in fp32
mode; 2e-2 on the final action chunk in bf16 mode.  Residual-Rescaling
decisions follow the decision-trace protocol: the oracle is forced to the
device's accept/refresh trace and the per-step statistics are compared.
"""
from collections import deque

import numpy as np
import pytest
import torch

from oracle import dit as OD, method as OM
from synth import get_workload, make_weights, make_initial_noise, make_observations, make_remap_noise
from gpu_common import (device, to_dev, rel_err, rr_of, f32_sigmas, model_for, layer_update_errors,
                        BF16_UPDATE_TOL)

pytestmark = pytest.mark.gpu

FP32_TOL = 1e-4
BF16_TOL = 2e-2


@pytest.fixture(scope="module")
def dev():
    return device()


def _tiny(dev, name="tiny", B=1, own_stream=False):
    spec, W, m = model_for(name, dev, own_stream=own_stream, B=B, bias_std=0.02, gain_std=0.1)
    sig = f32_sigmas(spec.K)
    m.set_schedule(sig)
    return spec, W, m, sig


# ------------------------------------------------------------------ fp32, layer level
def test_tiny_hidden_states_per_layer(dev):
    spec, W, m, sig = _tiny(dev, B=2)
    x0 = make_initial_noise(spec)
    cond = make_observations(spec, 0)[0]
    for k in (0, 2):
        for n in range(spec.L + 1):
            got = m.hidden(k, to_dev(x0, dev), to_dev(cond, dev), n).cpu().numpy()
            ref = OD.hidden_after(W, spec, x0, cond, sig[k], n)
            err = rel_err(got, ref)
            assert err <= 1e-5, (k, n, err)


def test_tiny_velocity_each_step(dev):
    spec, W, m, sig = _tiny(dev)
    x0 = make_initial_noise(spec)
    cond = make_observations(spec, 0)[0]
    for k in range(spec.K):
        v, _ = m.velocity(k, to_dev(x0, dev), to_dev(cond, dev))
        ref = OD.velocity(W, spec, x0, cond, sig[k])
        assert rel_err(v.cpu().numpy(), ref) <= FP32_TOL, k


# (D, H, B, Nv): every instantiation of the final-layer kernel (registers for up
# to 4, 8, 12, 16, 24 or 32 chunks of 64 columns; the modulation and the head's
# weights requested ahead of the reductions up to 12), on the tiny token layout
# with L = 1, with one block of 16 rows to a few hundred.
_FINAL_FORMS = [
    (192, 3, 1, 64), (1088, 17, 1, 64), (2048, 32, 1, 64),   # 3, 17 and 32 chunks
    (768, 12, 1, 64), (256, 4, 4, 1024),                     # 12 and 4, each the most its form holds
    (1024, 16, 1, 64), (1024, 16, 4, 1024),                  # 16
    (1536, 24, 1, 64), (1536, 24, 4, 1024),                  # 24
    (384, 6, 1, 64), (384, 6, 4, 1024), (1152, 18, 1, 64),   # 6 and 18
    (320, 5, 4, 1024),                                       # 5
]


@pytest.mark.parametrize("D,H,B,Nv", _FINAL_FORMS)
def test_hidden_sizes_velocity(dev, D, H, B, Nv):
    """Velocity within 1e-4 at hidden sizes that select each form of the
    final-layer kernel, few and many rows."""
    from paper_2609_34608_amd import runtime as R
    spec = get_workload("tiny").replace(D=D, H=H, L=1, B=B, Nv=Nv)
    W = make_weights(spec, bias_std=0.02)
    m = R.WamModel(R.config_of(spec), W, device=dev)
    sig = f32_sigmas(spec.K)
    m.set_schedule(sig)
    x0 = make_initial_noise(spec)
    cond = make_observations(spec, 0)[0]
    v, _ = m.velocity(1, to_dev(x0, dev), to_dev(cond, dev))
    ref = OD.velocity(W, spec, x0, cond, sig[1])
    assert rel_err(v.cpu().numpy(), ref) <= FP32_TOL
    m.close()


def test_tiny_native_chunk_and_capture(dev):
    spec, W, m, sig = _tiny(dev)
    x0 = make_initial_noise(spec)
    cond = make_observations(spec, 0)[0]
    x = to_dev(x0, dev)
    cap = torch.zeros_like(x)
    m.continue_(0, spec.K, x, to_dev(cond, dev), capture_stage=2, x_capture=cap)
    ref, ref_cap, _ = OM.denoise(W, spec, x0, cond, sig, 0, spec.K, None, OM.LayerState(), capture_stage=2)
    assert rel_err(x.cpu().numpy(), ref) <= FP32_TOL
    assert rel_err(cap.cpu().numpy(), ref_cap) <= FP32_TOL
    # the action chunk specifically
    a_got = OM.action_chunk(spec, x.cpu().numpy())
    assert rel_err(a_got, OM.action_chunk(spec, ref)) <= FP32_TOL


def test_determinism(dev):
    spec, W, m, sig = _tiny(dev)
    x0 = to_dev(make_initial_noise(spec), dev)
    c = to_dev(make_observations(spec, 0)[0], dev)
    outs = []
    for _ in range(2):
        x = x0.clone()
        m.continue_(0, spec.K, x, c)
        outs.append(x.cpu().numpy())
    np.testing.assert_array_equal(outs[0], outs[1])


# ------------------------------------------------------------------ Residual Rescaling
# hidden 128 takes the per-row gate kernels, hidden 256 (a multiple of 256)
# the per-block partial gate kernels
_RR_MODELS = ["tiny_rr", "tiny_rr256"]


@pytest.mark.parametrize("model,B", [(m, 2) for m in _RR_MODELS] + [("tiny_rr256", 16)])
@pytest.mark.parametrize("mode_name", ["AUTO", "FORCE_SKIP", "FORCE_FULL", "NEVER"])
def test_rr_modes_match_oracle(dev, mode_name, model, B):
    """Every RR mode against the oracle forced to the device's decision trace,
    with alpha / cos / fit per (sample, branch); B = 16 fills the per-sample
    statistics the ABI reports (WAM_MAX_BATCH)."""
    from paper_2609_34608_amd import _lib as L
    spec, W, m, sig = _tiny(dev, model, B=B)
    modes = {"AUTO": (L.WAM_RR_AUTO, {}), "FORCE_SKIP": (L.WAM_RR_FORCE_SKIP, {}),
             "FORCE_FULL": (L.WAM_RR_FORCE_FULL, {}), "NEVER": (L.WAM_RR_AUTO, {"gamma_cos": 1.5})}
    mode, kw = modes[mode_name]
    rr_g, rr_o = rr_of(spec, mode, **kw)
    x0 = make_initial_noise(spec)
    cond = make_observations(spec, 0)[0]
    m.reset_layer_state()
    x = to_dev(x0, dev)
    infos = m.continue_(0, spec.K, x, to_dev(cond, dev), rr=rr_g)
    trace = deque(i.accepted for i in infos if i.attempted)
    st = OM.LayerState()
    ref, _, oinfos = OM.denoise(W, spec, x0, cond, sig, 0, spec.K, rr_o, st, forced=trace)
    assert rel_err(x.cpu().numpy(), ref) <= FP32_TOL
    for gi, oi in zip(infos, oinfos):
        assert gi.attempted == oi.attempted and gi.accepted == oi.accepted
        assert gi.layers_evaluated == oi.layers_evaluated
        if gi.attempted:
            np.testing.assert_allclose(gi.alpha, oi.alpha, atol=1e-4)
            np.testing.assert_allclose(gi.cos, oi.cos, atol=1e-4)
            np.testing.assert_allclose(gi.fit, oi.fit, atol=1e-3)
    if mode_name in ("FORCE_FULL", "NEVER"):
        assert not any(i.accepted for i in infos)
    if mode_name == "FORCE_SKIP":
        assert all(i.accepted for i in infos[1:])


@pytest.mark.parametrize("model", _RR_MODELS)
def test_rr_identity_adaptation(dev, model):
    """The same step twice: the second reuses with alpha = 1, cos = 1, fit ~ 0."""
    from paper_2609_34608_amd import _lib as L
    spec, W, m, sig = _tiny(dev, model, B=2)
    rr_g, _ = rr_of(spec, L.WAM_RR_AUTO)
    x0 = to_dev(make_initial_noise(spec), dev)
    c = to_dev(make_observations(spec, 0)[0], dev)
    m.reset_layer_state()
    v1, i1 = m.velocity(1, x0, c, rr=rr_g)
    v1 = v1.clone()
    v2, i2 = m.velocity(1, x0, c, rr=rr_g)
    assert not i1.attempted and i2.attempted and i2.accepted
    np.testing.assert_allclose(i2.alpha, 1.0, atol=1e-6)
    np.testing.assert_allclose(i2.cos, 1.0, atol=1e-6)
    assert np.all(i2.fit < 1e-3)
    assert rel_err(v2.cpu().numpy(), v1.cpu().numpy()) <= 1e-5


@pytest.mark.parametrize("model", _RR_MODELS)
@pytest.mark.parametrize("mode_name", ["AUTO", "FORCE_SKIP", "FORCE_FULL", "NEVER", "MIXED"])
def test_device_decision_matches_host_decision(dev, mode_name, model):
    """The device-resident decision runs the same kernels in the same order:
    bit-identical trajectories and identical step reports."""
    from paper_2609_34608_amd import _lib as L
    spec, W, m, sig = _tiny(dev, model, B=2)
    modes = {"AUTO": (L.WAM_RR_AUTO, {}), "FORCE_SKIP": (L.WAM_RR_FORCE_SKIP, {}),
             "FORCE_FULL": (L.WAM_RR_FORCE_FULL, {}), "NEVER": (L.WAM_RR_AUTO, {"gamma_cos": 1.5}),
             "MIXED": (L.WAM_RR_AUTO, {"gamma_cos": 0.0, "gamma_fit": 1.02})}
    mode, kw = modes[mode_name]
    rr_g, rr_o = rr_of(spec, mode, **kw)
    x0 = make_initial_noise(spec)
    cond = to_dev(make_observations(spec, 0)[0], dev)
    outs, infos = [], []
    for devdec in (0, 1):
        m.set_option(L.WAM_OPT_DEVICE_DECISION, devdec)
        m.reset_layer_state()
        x = to_dev(x0, dev)
        infos.append(m.continue_(0, spec.K, x, cond, rr=rr_g))
        outs.append(x.cpu().numpy())
    m.set_option(L.WAM_OPT_DEVICE_DECISION, 0)
    np.testing.assert_array_equal(outs[0], outs[1])
    for a, b in zip(*infos):
        assert (a.attempted, a.accepted, a.layers_evaluated) == (b.attempted, b.accepted, b.layers_evaluated)
        np.testing.assert_array_equal(a.alpha, b.alpha)
        np.testing.assert_array_equal(a.fit, b.fit)
    # and the forced oracle agrees with the device-decision run
    trace = deque(i.accepted for i in infos[1] if i.attempted)
    ref, _, _ = OM.denoise(W, spec, x0, make_observations(spec, 0)[0], sig, 0, spec.K, rr_o, OM.LayerState(),
                           forced=trace)
    assert rel_err(outs[1], ref) <= FP32_TOL


# ------------------------------------------------------------------ TR and OR
@pytest.mark.parametrize("shift_a,shift_v", [(0, 0), (3, 0), (5, 7), (16, 0), (20, 64)])
def test_remap_matches_oracle(dev, shift_a, shift_v):
    spec, W, m, sig = _tiny(dev, B=2)
    rng = np.random.default_rng(11)
    xb, xr, eps = (rng.standard_normal((spec.B, spec.traj)).astype(np.float32) for _ in range(3))
    sr, sb = np.float32(0.6), np.float32(0.75)
    got = m.remap(to_dev(xb, dev), to_dev(xr, dev), float(sr), float(sb), shift_a, shift_v, to_dev(eps, dev))
    d = OM.tr_direction(spec, xr, xb, float(sr))
    ref = OM.tr_remap(spec, xb, d, float(sb), shift_a, shift_v, eps)
    assert rel_err(got.cpu().numpy(), ref) <= 1e-6


def test_consistency_score_matches_oracle(dev):
    spec, W, m, sig = _tiny(dev)
    rng = np.random.default_rng(12)
    comps = [(rng.standard_normal(n).astype(np.float32), rng.standard_normal(n).astype(np.float32))
             for n in (100, 7, 4096)]
    delta, weight = [255.0, 2.0, 0.5], [0.5, 0.3, 0.2]
    S = m.consistency_score([to_dev(a, dev) for a, _ in comps], [to_dev(b, dev) for _, b in comps], delta, weight)
    errs = [OM.or_component_error(a, b, dl) for (a, b), dl in zip(comps, delta)]
    assert S == pytest.approx(OM.or_score(errs, weight), rel=1e-12)


# ------------------------------------------------------------------ joint runtime
def _replan_args(spec):
    q = spec
    return dict(b0=q.tr_b0, r=q.tr_r, shift_action=q.shift_action, shift_video=q.shift_video, k1=q.or_k1,
                tau=q.or_tau, kappa_max=q.or_kappa_max)


@pytest.mark.parametrize("tau,graphs", [(0.5, False), (0.3, False), (0.5, True)])
def test_closed_loop_replans_match_oracle(dev, tau, graphs):
    """Teacher-forced per replan: the oracle starts from the device's retained
    state and follows its RR decision trace.  With graphs, every step is
    replayed from a captured graph with the decision kept on the device."""
    from paper_2609_34608_amd import _lib as L
    spec, W, m, sig = _tiny(dev, "tiny_replay", own_stream=graphs)
    m.set_option(L.WAM_OPT_DEVICE_DECISION, int(graphs))
    m.set_option(L.WAM_OPT_GRAPHS, int(graphs))
    spec = spec.replace(or_tau=tau)
    rr_g, rr_o = rr_of(spec, L.WAM_RR_AUTO)
    ra = _replan_args(spec)
    rho = spec.ar_rho
    delta = 1.0 / np.sqrt(1 - rho * rho)
    obs = make_observations(spec, spec.control_steps)
    m.reset_all()
    prof = OM.RuntimeProfile(**ra)
    rt = OM.ReplanRuntime(W, spec, sig, rr_o, prof)
    x_out = m.new_traj()
    paths = []
    for t in range(spec.control_steps):
        c_real = obs[t]
        c_pred = (rho * obs[t - 1]).astype(np.float32) if t > 0 else obs[t]
        if t > 0:
            xb, xr, kappa = m.get_replan_state()
            rt.set_state(xb.cpu().numpy(), xr.cpu().numpy(), kappa)
        cr, cp = to_dev(c_real, dev), to_dev(c_pred, dev)
        info = m.replan(cr, x_out, to_dev(make_remap_noise(spec, t), dev), cond_pred=cp, u_hat=[cp], u=[cr],
                        delta=[delta], weight=[1.0], noise_first=to_dev(make_initial_noise(spec), dev),
                        rr=rr_g, **ra)
        trace = deque(int(d) for d in info.decision[:info.steps] if d >= 0)
        ref, rinfo = rt.replan(c_real, c_pred, [c_pred], [c_real], [delta], [1.0],
                               noise_first=make_initial_noise(spec), noise_remap=make_remap_noise(spec, t),
                               forced=trace)
        assert info.path == rinfo.path, t
        assert info.steps == rinfo.steps and info.kappa == rinfo.kappa
        if rinfo.S is not None:
            assert info.S == pytest.approx(rinfo.S, rel=1e-9)
        assert rel_err(x_out.cpu().numpy(), ref) <= FP32_TOL, t
        paths.append(info.path)
    if tau == 0.5:  # S ~ 0.44 < 0.5: accepted until kappa reaches kappa_max
        assert paths == [L.WAM_PATH_FIRST, L.WAM_PATH_ACCEPT, L.WAM_PATH_ACCEPT, L.WAM_PATH_ACCEPT,
                         L.WAM_PATH_FORCED, L.WAM_PATH_ACCEPT][:len(paths)]
    else:
        assert all(p == L.WAM_PATH_REJECT for p in paths[1:])


def test_small_replay_replans_match_oracle(dev):
    """The closed-loop replay workload itself (small bf16 model, action shift
    8, AR(1) observations, TR + OR + RR): three replans, teacher-forced per
    replan as above, each action chunk within 2e-2 of the oracle.  The first
    replan runs all 10 steps; the next two are accepted rebindings (S < tau),
    2 prefix steps under the predicted observation and 3 under the real one."""
    from paper_2609_34608_amd import _lib as L
    spec, W, m = model_for("replay", dev)
    sig = f32_sigmas(spec.K)
    m.set_schedule(sig)
    rr_g, rr_o = rr_of(spec, L.WAM_RR_AUTO)
    ra = _replan_args(spec)
    rho = spec.ar_rho
    delta = 1.0 / np.sqrt(1 - rho * rho)
    n_ctrl = 3
    obs = make_observations(spec, n_ctrl)
    m.reset_all()
    rt = OM.ReplanRuntime(W, spec, sig, rr_o, OM.RuntimeProfile(**ra))
    x_out = m.new_traj()
    paths = []
    for t in range(n_ctrl):
        c_real = obs[t]
        c_pred = (rho * obs[t - 1]).astype(np.float32) if t > 0 else obs[t]
        if t > 0:
            xb, xr, kappa = m.get_replan_state()
            rt.set_state(xb.cpu().numpy(), xr.cpu().numpy(), kappa)
        cr, cp = to_dev(c_real, dev), to_dev(c_pred, dev)
        info = m.replan(cr, x_out, to_dev(make_remap_noise(spec, t), dev), cond_pred=cp, u_hat=[cp], u=[cr],
                        delta=[delta], weight=[1.0], noise_first=to_dev(make_initial_noise(spec), dev),
                        rr=rr_g, **ra)
        trace = deque(int(d) for d in info.decision[:info.steps] if d >= 0)
        ref, rinfo = rt.replan(c_real, c_pred, [c_pred], [c_real], [delta], [1.0],
                               noise_first=make_initial_noise(spec), noise_remap=make_remap_noise(spec, t),
                               forced=trace)
        assert info.path == rinfo.path, t
        assert info.steps == rinfo.steps and info.kappa == rinfo.kappa
        if rinfo.S is not None:
            assert info.S == pytest.approx(rinfo.S, rel=1e-6)
        got = x_out.cpu().numpy()
        e = rel_err(OM.action_chunk(spec, got), OM.action_chunk(spec, ref))
        print(f"replay replan {t}: path {info.path}, {info.steps} steps, action chunk rel err {e:.3e}")
        assert e <= BF16_TOL, (t, e)
        paths.append(info.path)
    assert paths == [L.WAM_PATH_FIRST, L.WAM_PATH_ACCEPT, L.WAM_PATH_ACCEPT]


def test_replay_100_control_steps(dev):
    """The closed-loop replay over 100 control steps (the replay workload's
    length): every chunk finite, the rebinding pattern the thresholds imply
    (first replan native; afterwards kappa_max accepted rebindings, then one
    forced refresh, repeating), and the 100th replan, teacher-forced from the
    device's retained state after 99, within 2e-2 of the oracle."""
    from paper_2609_34608_amd import _lib as L
    spec, W, m = model_for("replay", dev)
    sig = f32_sigmas(spec.K)
    m.set_schedule(sig)
    rr_g, rr_o = rr_of(spec, L.WAM_RR_AUTO)
    ra = _replan_args(spec)
    rho = spec.ar_rho
    delta = 1.0 / np.sqrt(1 - rho * rho)
    n_ctrl = 100
    obs = make_observations(spec, n_ctrl)
    obs_d = torch.from_numpy(obs).to(dev)
    pred = [obs[0]] + [(rho * obs[t - 1]).astype(np.float32) for t in range(1, n_ctrl)]
    pred_d = torch.from_numpy(np.stack(pred)).to(dev)
    noise_first = to_dev(make_initial_noise(spec), dev)
    m.reset_all()
    x_out = m.new_traj()
    paths = []
    for t in range(n_ctrl):
        if t == n_ctrl - 1:
            xb, xr, kappa = m.get_replan_state()
        info = m.replan(obs_d[t], x_out, to_dev(make_remap_noise(spec, t), dev), cond_pred=pred_d[t],
                        u_hat=[pred_d[t]], u=[obs_d[t]], delta=[delta], weight=[1.0], noise_first=noise_first,
                        rr=rr_g, **ra)
        paths.append(info.path)
        assert torch.isfinite(x_out).all(), t
    # with always-passing rebinding scores, kappa_max accepts then one forced refresh
    period = [L.WAM_PATH_ACCEPT] * spec.or_kappa_max + [L.WAM_PATH_FORCED]
    expect = [L.WAM_PATH_FIRST] + [period[(t - 1) % len(period)] for t in range(1, n_ctrl)]
    if paths != expect:  # a rejected score restarts the cycle: check the rules instead
        kap = 0
        for t, pth in enumerate(paths[1:], 1):
            assert pth in (L.WAM_PATH_ACCEPT, L.WAM_PATH_REJECT, L.WAM_PATH_FORCED), (t, pth)
            assert (pth == L.WAM_PATH_FORCED) == (kap >= spec.or_kappa_max), (t, pth, kap)
            kap = kap + 1 if pth == L.WAM_PATH_ACCEPT else 0
    # the last replan against the oracle from the same retained state
    rt = OM.ReplanRuntime(W, spec, sig, rr_o, OM.RuntimeProfile(**ra))
    rt.set_state(xb.cpu().numpy(), xr.cpu().numpy(), kappa)
    t = n_ctrl - 1
    trace = deque(int(d) for d in info.decision[:info.steps] if d >= 0)
    ref, rinfo = rt.replan(obs[t], pred[t], [pred[t]], [obs[t]], [delta], [1.0],
                           noise_first=make_initial_noise(spec), noise_remap=make_remap_noise(spec, t),
                           forced=trace)
    assert info.path == rinfo.path and info.steps == rinfo.steps
    e = rel_err(OM.action_chunk(spec, x_out.cpu().numpy()), OM.action_chunk(spec, ref))
    print(f"replay control step {t}: path {info.path}, action chunk rel err {e:.3e}")
    assert e <= BF16_TOL, e


# ------------------------------------------------------------------ bf16 workloads
def test_small_bf16_native_chunk(dev):
    spec, W, m = model_for("small", dev)
    sig = f32_sigmas(spec.K)
    m.set_schedule(sig)
    x0 = make_initial_noise(spec)
    cond = make_observations(spec, 0)[0]
    v, _ = m.velocity(0, to_dev(x0, dev), to_dev(cond, dev))
    vref = OD.velocity(W, spec, x0, cond, sig[0])
    ev = rel_err(v.cpu().numpy(), vref)
    print(f"small bf16 velocity(step 0) rel err {ev:.3e}")
    assert ev <= BF16_TOL
    x = to_dev(x0, dev)
    m.continue_(0, spec.K, x, to_dev(cond, dev))
    ref, _, _ = OM.denoise(W, spec, x0, cond, sig, 0, spec.K, None, OM.LayerState())
    ea = rel_err(OM.action_chunk(spec, x.cpu().numpy()), OM.action_chunk(spec, ref))
    print(f"small bf16 action chunk rel err {ea:.3e}")
    assert ea <= BF16_TOL


@pytest.mark.parametrize("k", [0, 7])
def test_small_bf16_layer_updates_every_layer(dev, k):
    """Every layer of the small model (the replay workload's kernels: the
    M = 864 GEMM tiles, the key-split attention) checked on its own: the
    device's update of each layer against the oracle's on the same input,
    every row.  Removing attention or the MLP moves this quantity by at least
    ten times the tolerance (tests/test_oracle_sensitivity.py)."""
    spec, W, m = model_for("small", dev)
    sig = f32_sigmas(spec.K)
    m.set_schedule(sig)
    x0 = make_initial_noise(spec)
    cond = make_observations(spec, 0)[0]
    errs = layer_update_errors(m, W, spec, k, x0, cond, sig[k], list(range(spec.L)), dev)
    print(f"small bf16 step {k} layer-update rel err: " + " ".join(f"{e:.2e}" for _, e in errs))
    for l, e in errs:
        assert e <= BF16_UPDATE_TOL, (l, e)


@pytest.mark.parametrize("name,layers,every_row", [("mid", (0, 11), True), ("large", (0,), True),
                                                   ("large", (17,), False)])
def test_full_size_layer_updates(dev, name, layers, every_row):
    """Single DiT layers at full size (bf16 GEMMs and attention at their real
    shapes: B = 4 x T = 2306, and T = 10176 with 24 heads): the device's
    update h_{l+1} - h_l against the oracle's on the device's own h_l, on
    every row (mid layers 0 and 11, large layer 0) or on sampled rows that the
    oracle computes one by one (large layer 17)."""
    spec, W, m = model_for(name, dev)
    sig = f32_sigmas(spec.K)
    m.set_schedule(sig)
    x0 = make_initial_noise(spec)
    cond = make_observations(spec, 0)[0]
    k = 3
    if every_row:
        OD.ATTENTION_THREADS = 8
        try:
            errs = layer_update_errors(m, W, spec, k, x0, cond, sig[k], list(layers), dev)
        finally:
            OD.ATTENTION_THREADS = 1
        for l, e in errs:
            print(f"{name} layer {l} every-row update rel err {e:.3e}")
            assert e <= BF16_UPDATE_TOL, (l, e)
        return
    c = OD.cond_vector(W, sig[k])
    rng = np.random.default_rng(5)
    rows = np.unique(np.r_[0, spec.M - 1, spec.T - 1, spec.Nv, spec.Nv + spec.Na,
                           rng.integers(0, spec.M, 12)])
    for l in layers:
        h_in = m.hidden(k, to_dev(x0, dev), to_dev(cond, dev), l).cpu().numpy()
        h_out = m.hidden(k, to_dev(x0, dev), to_dev(cond, dev), l + 1).cpu().numpy().reshape(-1, spec.D)
        ref = OD.dit_layer_rows(W, spec, l, h_in, c, rows)
        upd_got = h_out[rows] - h_in.reshape(-1, spec.D)[rows]
        upd_ref = ref - h_in.reshape(-1, spec.D)[rows]
        e = rel_err(upd_got, upd_ref)
        print(f"{name} layer {l} sampled-row update rel err {e:.3e}")
        assert e <= BF16_UPDATE_TOL, (l, e)


def test_split_replan_matches_one_call(dev):
    """wam_replan_begin (remap + prefix enqueued without waiting) followed by
    wam_replan_end equals wam_replan, replan by replan, bit for bit."""
    from paper_2609_34608_amd import _lib as L
    spec, W, m, sig = _tiny(dev, "tiny_replay", own_stream=True)
    m.set_option(L.WAM_OPT_GRAPHS, 0)
    m.set_option(L.WAM_OPT_DEVICE_DECISION, 1)
    rr_g, _ = rr_of(spec, L.WAM_RR_AUTO, gamma_cos=0.0, gamma_fit=1.02)
    ra = _replan_args(spec)
    rho = spec.ar_rho
    delta = 1.0 / np.sqrt(1 - rho * rho)
    obs = make_observations(spec, spec.control_steps)
    runs = []
    for split in (False, True):
        m.reset_all()
        x_out = m.new_traj()
        outs, paths = [], []
        for t in range(spec.control_steps):
            cr = to_dev(obs[t], dev)
            cp = to_dev((rho * obs[t - 1]).astype(np.float32) if t > 0 else obs[t], dev)
            kw = dict(cond_pred=cp, u_hat=[cp], u=[cr], delta=[delta], weight=[1.0],
                      noise_first=to_dev(make_initial_noise(spec), dev), rr=rr_g, **ra)
            noise = to_dev(make_remap_noise(spec, t), dev)
            if split:
                a = m.replan_args(cr, x_out, noise, **kw)
                m.replan_begin(a)
                info = m.replan_end(a)
            else:
                info = m.replan(cr, x_out, noise, **kw)
            outs.append(x_out.cpu().numpy())
            paths.append((info.path, info.steps, info.kappa, list(info.decision[:info.steps])))
        runs.append((outs, paths))
    m.set_option(L.WAM_OPT_DEVICE_DECISION, 0)
    assert runs[0][1] == runs[1][1]
    for a, b in zip(runs[0][0], runs[1][0]):
        np.testing.assert_array_equal(a, b)


# ------------------------------------------------------------------ edge cases
@pytest.mark.parametrize("shape", [dict(Nv=0), dict(No=0), dict(Na=1, A=1), dict(B=16, Nv=24, No=3),
                                   dict(Nv=63, No=1)])
def test_degenerate_shapes_chunk_matches_oracle(dev, shape):
    """No video tokens, no observation tokens, a one-slot one-dim action
    chunk, the maximum batch, and ragged T: native chunk within 1e-4."""
    from paper_2609_34608_amd import runtime as R
    spec = get_workload("tiny").replace(**shape)
    W = make_weights(spec, bias_std=0.02)
    m = R.WamModel(R.config_of(spec), W, device=dev)
    sig = f32_sigmas(spec.K)
    m.set_schedule(sig)
    x0 = make_initial_noise(spec)
    cond = make_observations(spec, 0)[0]
    x = to_dev(x0, dev)
    m.continue_(0, spec.K, x, to_dev(cond, dev))
    ref, _, _ = OM.denoise(W, spec, x0, cond, sig, 0, spec.K, None, OM.LayerState())
    assert rel_err(x.cpu().numpy(), ref) <= FP32_TOL
    m.close()


def test_kappa_max_zero_always_refreshes(dev):
    """kappa_max = 0: no prefix is ever started; every replan refreshes from
    the remapped initialisation (FORCED path), K - b0 steps."""
    from paper_2609_34608_amd import _lib as L
    spec, W, m, sig = _tiny(dev, "tiny_replay")
    m.set_option(L.WAM_OPT_GRAPHS, 0)
    m.set_option(L.WAM_OPT_DEVICE_DECISION, 0)
    ra = dict(_replan_args(spec), kappa_max=0)
    obs = make_observations(spec, 3)
    m.reset_all()
    x_out = m.new_traj()
    for t in range(4):
        c = to_dev(obs[t], dev)
        info = m.replan(c, x_out, to_dev(make_remap_noise(spec, t), dev), cond_pred=c, u_hat=[c], u=[c],
                        delta=[1.0], weight=[1.0], noise_first=to_dev(make_initial_noise(spec), dev), **ra)
        if t > 0:
            assert info.path == L.WAM_PATH_FORCED and info.n_start == 0 and info.steps == spec.K - spec.tr_b0
            assert info.S == -1.0


def test_error_returns(dev):
    """Invalid arguments return an error status and leave the handle usable."""
    from paper_2609_34608_amd import _lib as L
    from paper_2609_34608_amd.runtime import WamError, rr_profile
    spec, W, m, sig = _tiny(dev, "tiny_rr")
    x = to_dev(make_initial_noise(spec), dev)
    c = to_dev(make_observations(spec, 0)[0], dev)
    with pytest.raises(WamError, match="sigma_r"):
        m.remap(x, x.clone(), 0.0, 0.5, 0, 0, x.clone())
    with pytest.raises(WamError, match="shifts"):
        m.remap(x, x.clone(), 0.5, 0.5, -1, 0, x.clone())
    with pytest.raises(WamError, match="0 < q < s < e < L"):
        m.velocity(0, x, c, rr=rr_profile(2, 2, 3, L.WAM_RR_AUTO))
    with pytest.raises(WamError, match="step index"):
        m.velocity(spec.K, x, c)
    with pytest.raises(WamError, match="strictly"):
        m.set_schedule(np.array([1.0, 0.5, 0.5, 0.0]))
    with pytest.raises(WamError, match="unknown attention kernel"):
        m.set_option(L.WAM_OPT_ATTENTION, L.WAM_ATTN_PLAIN + 1)
    m.set_schedule(sig)
    v, _ = m.velocity(0, x, c)  # still usable
    assert torch.isfinite(v).all()
