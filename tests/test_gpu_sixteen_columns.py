"""The sixteen-column matrix-core kernels (binary32 and bf16, obs <= 64) and the LDS kernel on the shapes that are theirs.

Up to one pass of four copies per compute unit a policy runs on the four-copy kernels, so these populations make more than 256
passes; a few steps each, and eight individuals from both ends against the CPU checker.  The LDS kernel serves what no register
kernel holds: more than four narrow layers, wide observations or actions beside narrow layers."""
import math
from dataclasses import replace

import numpy as np
import pytest
import torch

import oracle
from paper_2501_15129_amd.workloads import CONFIGS, Workload, make_inputs
from gpu_util import compare_rollout, dev, noise_to_device, probe_rollout, run_rollout

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def es():
    import paper_2501_15129_amd as pkg
    assert torch.cuda.is_available(), "these tests need the GPU"
    return pkg


def _run(es, w, kernel, norm=False, ends=4):
    """The whole population on the GPU, twice (a rerun is bit-identical); the first and the last `ends` individuals against the checker."""
    ws = replace(w, noise_dtype=w.noise_dtype & 1)
    a_mat, b_mat, theta = make_inputs(w)
    rng = np.random.default_rng(w.seed)
    theta = (theta + rng.standard_normal(theta.size) * 0.02).astype(np.float32)     # non-zero biases
    stats = ((rng.standard_normal(w.obs) * 0.05).astype(np.float32), (1.0 / (0.33 + rng.random(w.obs) * 0.67)).astype(np.float32)) if norm else None
    ctx = es.EsContext(w)
    assert ctx.rollout_kernel == kernel
    if norm:
        held = (dev(stats[0]), dev(stats[1]))
        ctx.set_obs_norm(*held)
    if ctx.noise_table:
        noise = ctx.alloc_noise()
        ctx.build_noise_table(noise)
        ctx.sample_population(2, noise)
        eps = oracle.table_rows(w, 2, w.noise_table_len, ctx.noise_ld, w.noise_dtype == 5)
    else:
        eps = oracle.sample_population(ws, 2)
        noise = None if ctx.noise_regenerated else noise_to_device(ctx, eps)
    got = run_rollout(ctx, w, 2, theta, noise, a_mat, b_mat)
    again = run_rollout(ctx, w, 2, theta, noise, a_mat, b_mat)
    for x, y in zip(got, again):
        assert np.array_equal(x.view(np.uint32), y.view(np.uint32)), f"{w.name}: a rerun differs"
    assert np.all(np.isfinite(got[0])) and np.all(got[1] >= 1) and np.all(got[1] <= w.horizon)
    for ind in {(0, min(w.pop, ends)), (max(0, w.pop - ends), w.pop)}:
        ref = oracle.rollout(ws, 2, theta, eps, a_mat, b_mat, individuals=ind, obs_norm=stats)
        probe = probe_rollout(ws, 2, theta, eps, a_mat, b_mat, ref=ref, individuals=ind, obs_norm=stats)
        flips, worst, sens, chaotic = compare_rollout(ws, tuple(x[ind[0]:ind[1]] for x in got), ref, w.name, probe)
        print(f"[{w.name}] individuals {ind} kernel={ctx.rollout_kernel} worst {worst:.2e} flips {flips} sensitive {sens}")
        assert not chaotic
    return got


F = Workload("f32c16", pop=68, envs=16, horizon=30, obs=27, hid=256, act=8, dtype=0, noise_dtype=0, seed=701)


@pytest.mark.parametrize("norm", [False, True], ids=["plain", "norm"])
@pytest.mark.parametrize("w", [
    F, replace(F, name="f32c16-32-129-16-relu", obs=32, hid=129, act=16, hidden_act=1), replace(F, name="f32c16-1-200-1-E9", obs=1, hid=200, act=1, envs=9, pop=88),
    replace(F, name="f32c16-33-255-5-E21", obs=33, hid=255, act=5, envs=21, pop=44, horizon=15), replace(F, name="f32c16-64-256-16-relu", obs=64, act=16, hidden_act=1),
    replace(F, name="f32c16-linear-noanti", out_tanh=0, antithetic=0, pop=67), replace(F, name="f32c16-N300", pop=300, horizon=5),
    replace(F, name="f32c16-len1", done_thresh=1e-6), replace(F, name="f32c16-T1", horizon=1), replace(F, name="f32c16-ends", done_thresh=0.5),
    replace(F, name="f32c16-k3", envs=4, episodes=3, pop=90)], ids=lambda w: w.name)
def test_binary32(es, w, norm):
    _run(es, w, "rollout_mfma_reg_f32<obs%d,hid256,act16>" % (32 if w.obs <= 32 else 64), norm)


@pytest.mark.parametrize("kw", [dict(noise_dtype=1), dict(noise_dtype=2), dict(noise_dtype=3, obs=50), dict(noise_dtype=4, noise_table_len=1 << 18),
                                dict(noise_dtype=5, noise_table_len=1 << 18, obs=50)], ids=lambda kw: f"noise{kw['noise_dtype']}")
def test_binary32_noise_modes(es, kw):
    w = replace(F, name=f"f32c16-noise{kw['noise_dtype']}", horizon=15, **kw)
    _run(es, w, "rollout_mfma_reg_f32<obs%d,hid256,act16>" % (32 if w.obs <= 32 else 64))


def test_binary32_sigma_zero(es):
    got = _run(es, replace(F, name="f32c16-sigma0", sigma=0.0), "rollout_mfma_reg_f32<obs32,hid256,act16>")
    assert np.all(got[2].view(np.uint32) == got[2].view(np.uint32)[0])


B = Workload("bf16c16", pop=68, envs=16, horizon=30, obs=27, hid=256, act=8, dtype=1, noise_dtype=1, seed=731)


def _bf16_name(w):
    return "rollout_mfma_reg_bf16<obs%d,hid256,act16>" % (32 if w.obs <= 32 else 64) + (f",depth{w.num_hidden}" if w.num_hidden != 2 else "")


@pytest.mark.parametrize("layers", [1, 2, 3, 4])
@pytest.mark.parametrize("kw,norm", [
    (dict(), False), (dict(hidden_act=1), True), (dict(obs=60), False), (dict(obs=64, act=16, hidden_act=1), True), (dict(obs=33, act=1, hid=200, envs=21, pop=44, horizon=15), False),
    (dict(obs=1, act=16, hid=129, envs=9, pop=88), True), (dict(noise_dtype=3), False), (dict(obs=40, noise_dtype=2), True), (dict(noise_dtype=5, noise_table_len=1 << 19), False),
    (dict(obs=40, noise_dtype=4, noise_table_len=1 << 19), False), (dict(out_tanh=0, antithetic=0, pop=67, obs=32), False), (dict(pop=516, horizon=4), True),
    (dict(pop=300, horizon=4, obs=50), False), (dict(done_thresh=1e-6), False), (dict(horizon=1, obs=50), False), (dict(done_thresh=0.5, obs=50, envs=4, episodes=4), True)],
    ids=lambda v: "-".join(f"{k}{x}" for k, x in v.items()) if isinstance(v, dict) else "norm" if v else "plain")
def test_bf16(es, layers, kw, norm):
    w = replace(B, name=f"bf16c16-m{layers}-" + "-".join(f"{k}{x}" for k, x in kw.items()), num_hidden=layers, seed=731 + layers)
    _run(es, replace(w, **kw), _bf16_name(replace(w, **kw)), norm)


@pytest.mark.parametrize("layers,norm", [(1, False), (2, True)])
def test_bf16_128_units(es, layers, norm):
    w = replace(B, name=f"bf16c16-m{layers}-hid128", hid=128, pop=512, envs=15, horizon=8, num_hidden=layers)
    _run(es, w, _bf16_name(w), norm)


@pytest.mark.parametrize("layers", [3, 4])
@pytest.mark.parametrize("hid,obs,norm", [(65, 27, False), (96, 64, True), (127, 20, False)])
def test_bf16_three_and_four_middle_layers(es, layers, hid, obs, norm):
    w = replace(B, name=f"bf16c16-m{layers}-hid{hid}", hid=hid, obs=obs, num_hidden=layers, hidden_act=int(norm))
    _run(es, w, _bf16_name(w), norm)


@pytest.mark.parametrize("layers,obs", [(1, 27), (3, 27), (4, 27), (1, 50), (2, 50), (3, 50), (4, 50)])
def test_bf16_contractive_twins_full_horizon(es, layers, obs):
    """One to four hidden layers of 256 on sixteen copies, T = 1000, on the contractive twin: every compared episode strictly within 2e-2."""
    w = replace(CONFIGS[3].contractive(), name=f"contractive-m{layers}-obs{obs}-n68", pop=68, num_hidden=layers, obs=obs)
    got = _run(es, w, _bf16_name(w), ends=2)
    assert np.all(got[1] == w.horizon) and compare_rollout.last_excused == 0


def test_binary32_contractive_twin_full_horizon(es):
    """The same in binary32, two layers: strictly within 1e-4."""
    w = replace(CONFIGS[3].contractive(), name="contractive-f32-n68", pop=68, dtype=0, noise_dtype=0)
    got = _run(es, w, "rollout_mfma_reg_f32<obs32,hid256,act16>", ends=2)
    assert np.all(got[1] == w.horizon) and compare_rollout.last_excused == 0


def test_shape_sweep(es):
    rng = np.random.default_rng(741)
    for n in range(24):
        dt = int(rng.integers(0, 4) > 0)
        m = int(rng.integers(1, 5)) if dt else 2
        obs, envs = int(rng.integers(1, 65)), int(rng.integers(9, 22))
        w = Workload(f"sweep16-{n}", pop=2 * int(-(-260 // ((envs + 3) // 4)) // 2 + 1), envs=envs, horizon=int(rng.integers(1, 17)), obs=obs,
                     hid=int(rng.integers(129, 257)), act=int(rng.integers(1, 17)), dtype=dt, noise_dtype=int(rng.choice([dt, 2 + dt])), seed=7400 + n,
                     hidden_act=int(rng.integers(0, 2)), out_tanh=int(rng.integers(0, 2)), done_thresh=float(rng.choice([0.95, 0.5, math.inf])), num_hidden=m)
        name = _bf16_name(w) if dt else "rollout_mfma_reg_f32<obs%d,hid256,act16>" % (32 if obs <= 32 else 64)
        _run(es, w, name, norm=bool(rng.integers(0, 2)), ends=2)


L = Workload("lds", pop=6, envs=3, horizon=30, obs=70, hid=40, act=9, dtype=0, noise_dtype=0, seed=761)


@pytest.mark.parametrize("norm", [False, True], ids=["plain", "norm"])
@pytest.mark.parametrize("w", [
    L, replace(L, name="lds-m1", num_hidden=1), replace(L, name="lds-m3-relu", num_hidden=3, hidden_act=1), replace(L, name="lds-m5", num_hidden=5, obs=13, hid=24),
    replace(L, name="lds-m6-act17-linear", num_hidden=6, obs=20, hid=20, act=17, out_tanh=0), replace(L, name="lds-regen", noise_dtype=2), replace(L, name="lds-regen-rounded-m3", noise_dtype=3, num_hidden=3),
    replace(L, name="lds-table", noise_dtype=4, noise_table_len=1 << 16), replace(L, name="lds-noanti-ends", antithetic=0, pop=5, done_thresh=0.5), replace(L, name="lds-k2", episodes=2),
    replace(L, name="lds-bf16", dtype=1, noise_dtype=1), replace(L, name="lds-bf16-m1-relu", dtype=1, noise_dtype=1, num_hidden=1, hidden_act=1),
    replace(L, name="lds-bf16-m5", dtype=1, noise_dtype=1, num_hidden=5, obs=13, hid=24), replace(L, name="lds-bf16-regen", dtype=1, noise_dtype=3),
    replace(L, name="lds-bf16-table", dtype=1, noise_dtype=5, noise_table_len=1 << 16), replace(L, name="lds-bf16-env-f32", dtype=1, noise_dtype=1, env_dtype=1),
    replace(L, name="lds-bf16-act33", dtype=1, noise_dtype=1, obs=30, hid=100, act=33)], ids=lambda w: w.name)
def test_lds_kernel(es, w, norm):
    _run(es, w, "rollout_wave_lds_bf16" if w.dtype == 1 else "rollout_wave_lds_f32", norm, ends=3)
