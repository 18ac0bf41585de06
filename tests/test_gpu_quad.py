"""The four-copy rollout kernels (4x4 matrix-core shapes) at the edges of their classes - hidden widths around multiples
of 64, observation widths around 32, 64 and 128, ragged passes, one copy, several passes per individual, depths, state rows
spread over the wavefronts, narrow binary32 policies in numbers - and one, three and four narrow layers in one wavefront, against
the CPU checker."""
import math
from dataclasses import replace

import numpy as np
import pytest
import torch

import oracle
from paper_2501_15129_amd.workloads import Workload, make_inputs
from gpu_util import compare_rollout, dev, noise_to_device, probe_rollout, run_rollout

pytestmark = pytest.mark.gpu

B = Workload("quad", pop=4, envs=4, horizon=30, obs=27, hid=256, act=8, dtype=1, noise_dtype=1, seed=401)


@pytest.fixture(scope="module")
def es():
    import paper_2501_15129_amd as pkg
    assert torch.cuda.is_available(), "these tests need the GPU"
    return pkg


def _case(es, w, norm=False):
    ws = replace(w, noise_dtype=w.noise_dtype & 1)
    a_mat, b_mat, theta = make_inputs(w)
    rng = np.random.default_rng(w.seed)
    theta = (theta + rng.standard_normal(theta.size) * 0.02).astype(np.float32)     # non-zero biases
    stats = ((rng.standard_normal(w.obs) * 0.05).astype(np.float32), (1.0 / (0.33 + rng.random(w.obs) * 0.67)).astype(np.float32)) if norm else None
    ctx = es.EsContext(w)
    if norm:
        held = (dev(stats[0]), dev(stats[1]))
        ctx.set_obs_norm(*held)
    eps = oracle.sample_population(ws, 2)
    noise = None if ctx.noise_regenerated else noise_to_device(ctx, eps)
    got = run_rollout(ctx, w, 2, theta, noise, a_mat, b_mat)
    again = run_rollout(ctx, w, 2, theta, noise, a_mat, b_mat)
    for x, y in zip(got, again):
        assert np.array_equal(x.view(np.uint32), y.view(np.uint32)), f"{w.name}: a rerun differs"
    n = min(w.pop, 8)
    few = tuple(x[:n] for x in got)
    ref = oracle.rollout(ws, 2, theta, eps, a_mat, b_mat, individuals=(0, n), obs_norm=stats)
    probe = probe_rollout(ws, 2, theta, eps, a_mat, b_mat, ref=ref, individuals=(0, n), obs_norm=stats)
    flips, worst, sens, chaotic = compare_rollout(ws, few, ref, w.name, probe)
    print(f"[{w.name}] kernel={ctx.rollout_kernel} worst {worst:.2e} flips {flips} sensitive {sens}")
    assert not chaotic
    return ctx


@pytest.mark.parametrize("obs,hid,act,envs,layers,kw", [
    (1, 65, 1, 1, 2, {}), (32, 128, 16, 4, 2, {}), (33, 127, 16, 3, 1, {}), (64, 100, 15, 5, 2, dict(hidden_act=1)),
    (65, 128, 1, 4, 2, {}), (128, 66, 32, 2, 1, {}), (20, 128, 17, 7, 2, {}), (97, 99, 20, 16, 2, dict(done_thresh=math.inf)),
    (32, 129, 16, 1, 2, dict(hidden_act=1)), (33, 192, 3, 4, 2, {}), (64, 193, 16, 2, 1, {}), (8, 255, 5, 1, 1, dict(out_tanh=0)),
    (32, 256, 1, 8, 2, {}), (27, 256, 8, 6, 3, {}), (64, 256, 16, 1, 3, dict(hidden_act=1)), (64, 256, 16, 1, 4, {}), (31, 200, 9, 1, 4, {}),
    (17, 256, 6, 3, 4, dict(noise_dtype=3)), (40, 256, 7, 4, 2, dict(noise_dtype=0, antithetic=0, pop=3)), (27, 256, 8, 4, 2, dict(done_thresh=1e-6)),
    (27, 256, 8, 1, 2, dict(horizon=1)), (13, 130, 4, 2, 2, dict(envs=3, episodes=3)), (75, 90, 11, 4, 2, dict(done_thresh=0.5))],
    ids=lambda v: str(v) if not isinstance(v, dict) else "-".join(f"{k}{x}" for k, x in v.items()))
def test_bf16_edges(es, obs, hid, act, envs, layers, kw):
    w = replace(B, name=f"quad-{obs}-{hid}x{layers}-{act}-E{envs}", obs=obs, hid=hid, act=act, envs=envs, num_hidden=layers, seed=401 + obs + hid)
    ctx = _case(es, replace(w, **kw))
    assert "quad_bf16" in ctx.rollout_kernel


@pytest.mark.parametrize("w", [B, replace(B, name="quad-norm-60-E1-relu", obs=60, envs=1, hidden_act=1), replace(B, name="quad-norm-mid-spread", obs=90, hid=100, act=12),
                               replace(B, name="quad-norm-deep4", num_hidden=4, envs=3)], ids=lambda w: w.name)
def test_bf16_observation_statistics(es, w):
    _case(es, w, norm=True)


def test_more_individuals_than_the_chip_holds_at_once(es):
    for w in (replace(B, name="quad-N700-E1", pop=700, envs=1, horizon=5), replace(B, name="quad-N300-E4-m3", pop=300, num_hidden=3, horizon=4),
              replace(B, name="quad-N40-E21", pop=40, envs=21, horizon=6), replace(B, name="quad-mid-N1100-E6", pop=1100, hid=80, envs=6, horizon=4)):
        _case(es, w)


F = Workload("quadf", pop=4, envs=4, horizon=30, obs=27, hid=256, act=8, dtype=0, noise_dtype=0, seed=501)


@pytest.mark.parametrize("obs,hid,act,envs,layers,kw", [
    (16, 65, 16, 4, 2, {}), (17, 128, 1, 1, 2, {}), (33, 100, 5, 9, 2, dict(hidden_act=1)), (64, 128, 16, 3, 3, {}), (5, 70, 2, 1, 3, {}), (32, 127, 3, 2, 1, {}),
    (16, 129, 4, 1, 2, dict(out_tanh=0)), (32, 256, 16, 8, 2, {}), (64, 200, 7, 12, 2, {}), (64, 256, 16, 1, 2, {}), (33, 256, 9, 5, 1, dict(done_thresh=0.5))],
    ids=lambda v: str(v) if not isinstance(v, dict) else "-".join(f"{k}{x}" for k, x in v.items()))
def test_f32_edges(es, obs, hid, act, envs, layers, kw):
    w = replace(F, name=f"quadf-{obs}-{hid}x{layers}-{act}-E{envs}", obs=obs, hid=hid, act=act, envs=envs, num_hidden=layers, seed=501 + obs + hid)
    ctx = _case(es, replace(w, **kw))      # (small populations: one copy per workgroup up to 128 units, and up to 32 observations)
    assert ("single_f32" if hid <= 128 or obs <= 32 else "quad_f32") in ctx.rollout_kernel


@pytest.mark.parametrize("w", [
    replace(F, name="quadn-16-64", pop=800, envs=13, horizon=12, obs=16, hid=64, act=16), replace(F, name="quadn-32-49-relu", pop=1100, envs=11, horizon=12, obs=32, hid=49, act=3, hidden_act=1),
    replace(F, name="quadn-64-33-linear", pop=1026, envs=11, horizon=12, obs=64, hid=33, act=7, out_tanh=0, done_thresh=0.5),
    replace(B, name="quadn-bf16-32-64", pop=1100, envs=8, horizon=12, obs=32, hid=64, act=16), replace(B, name="quadn-bf16-33-16", pop=900, envs=11, horizon=12, obs=33, hid=16, act=1)],
    ids=lambda w: w.name)
def test_narrow_policies_in_numbers(es, w):
    """passes of sixteen copies, one of them of four (the latter's own: test_gpu_larger_populations.py)"""
    assert ("rollout_mfma_quad_f32<obs32,hid64,act16>" if w.hid == 49 else "rollout_mfma_cols_") in _case(es, w).rollout_kernel
    _case(es, w, norm=True)


# one wavefront per episode at the other depths: edges of the width classes, horizons around the four steps of a turn, early ends
@pytest.mark.parametrize("w", [
    replace(F, name=f"narrow-depth{m}-{o}-{h}-{a}-{t}", num_hidden=m, pop=4, envs=3, obs=o, hid=h, act=a, horizon=t, **kw) for m, o, h, a, t, kw in [
        (1, 16, 64, 8, 1, {}), (1, 17, 33, 9, 2, dict(hidden_act=1)), (1, 64, 1, 16, 3, dict(noise_dtype=2)), (3, 1, 16, 1, 4, dict(done_thresh=1e-6)),
        (3, 33, 64, 16, 5, dict(out_tanh=0)), (3, 32, 17, 8, 30, dict(done_thresh=0.5)), (4, 64, 64, 16, 7, dict(noise_dtype=1)), (4, 16, 32, 4, 30, dict(dtype=1, noise_dtype=1)),
        (1, 40, 48, 5, 6, dict(dtype=1, noise_dtype=3)), (2, 17, 64, 6, 6, dict(noise_dtype=2, done_thresh=0.5)), (2, 11, 32, 3, 3, {})]],
    ids=lambda w: w.name)
def test_narrow_depths(es, w):
    assert "wave_reg" in _case(es, w).rollout_kernel


# bf16 policies of fewer than 128 units (and narrow ones of one, three and four layers): small activations have bf16 neighbours a
# few 1e-5 apart, so a tanh that is off by 1.2e-7 rounds one operand in a thousand the other way and moves most returns visibly
@pytest.mark.parametrize("kw", [dict(), dict(obs=90, act=12), dict(hid=70, num_hidden=1), dict(hid=96, num_hidden=3), dict(hid=96, num_hidden=4),
                                dict(hid=96, num_hidden=3, pop=68, envs=16), dict(hid=96, num_hidden=4, pop=68, envs=16),
                                dict(hid=40, num_hidden=1), dict(hid=40, num_hidden=3), dict(hid=40, num_hidden=4)],
                         ids=lambda kw: "-".join(f"{k}{x}" for k, x in kw.items()) or "two-layers")
def test_operands_near_zero_round_as_they_should(es, kw):
    w = replace(Workload("near", pop=64, envs=4, horizon=4, obs=27, hid=100, act=8, dtype=1, noise_dtype=1, seed=801, done_thresh=math.inf), **kw)
    a_mat, b_mat, theta = make_inputs(w)
    eps = oracle.sample_population(w, 0)
    ctx = es.EsContext(w)
    got = run_rollout(ctx, w, 0, theta, noise_to_device(ctx, eps), a_mat, b_mat)
    ref = oracle.rollout(w, 0, theta, eps, a_mat, b_mat)
    moved = float(np.mean(np.abs(got[0] - ref[0]) > 2e-6 * np.abs(ref[0])))
    # episodes with an operand rounded the other way, over these ten workloads: tanh to 1.2e-7 2-29 % (12 % on average), to
    # 4e-8 0-4.7 % (2.5 %); half as much again is allowed
    print(f"[{w.name} {kw}] kernel={ctx.rollout_kernel} episodes moved {moved:.3f}")
    assert moved <= 0.07
