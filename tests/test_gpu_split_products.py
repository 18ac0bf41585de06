"""Binary32 policies in passes of sixteen copies, whose products run on three-piece values: every way the pairs of a lane are grouped (one, two, three padded to four, four, six
and eight pairs), both activations - against the CPU checker, to binary32's own precision over a few steps; the populations at which the smallest class changes its form, with
statistics; and actions, parameters and statistics beyond the pieces' range."""
from dataclasses import replace

import numpy as np
import pytest
import torch

import oracle
from gpu_util import dev, noise_to_device, run_rollout
from paper_2501_15129_amd.workloads import Workload, make_inputs
from test_gpu_quad import es  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

F = Workload("split", pop=1200, envs=16, horizon=3, obs=17, hid=48, act=5, dtype=0, noise_dtype=0, seed=901)


@pytest.mark.parametrize("relu", [0, 1])
@pytest.mark.parametrize("obs,hid,act", [(3, 16, 2), (16, 17, 9), (17, 48, 8), (20, 33, 16), (32, 64, 5), (33, 16, 3), (48, 60, 16), (64, 32, 12), (64, 48, 4), (48, 64, 16)])
def test_binary32_precision(es, obs, hid, act, relu):  # noqa: F811
    """Three steps: each product is good to 2^-24, each sum of up to 64 of them to some 2^-24 of its terms, each tanh to 1.2e-7, so a step moves a reward (1 less means of squares) by
    1e-7 or so; 2e-6 is some twenty times that.  (A missing piece averages out over the elements and stays within it: those are test_gpu_piece_terms.py.)"""
    w = replace(F, name=f"split-{obs}-{hid}-{act}", obs=obs, hid=hid, act=act, hidden_act=relu, seed=901 + obs + hid)
    ctx = es.EsContext(w)
    assert "rollout_mfma_cols_f32" in ctx.rollout_kernel
    a_mat, b_mat, theta = make_inputs(w)
    eps = oracle.sample_population(w, 0)
    ret, _, _ = run_rollout(ctx, w, 0, theta, noise_to_device(ctx, eps), a_mat, b_mat)
    ref = oracle.rollout(w, 0, theta, eps, a_mat, b_mat, individuals=(590, 610))[0]
    assert np.abs(ret[590:610] - ref).max() <= 2e-6 * np.abs(ref).max()


def _precise(es, w, norm):
    ctx = es.EsContext(w)
    stats = None
    if norm:
        rng = np.random.default_rng(w.seed)
        stats = (rng.standard_normal(w.obs) * 0.05).astype(np.float32), (1.0 / (0.33 + rng.random(w.obs) * 0.67)).astype(np.float32)
        held = tuple(dev(v) for v in stats)
        ctx.set_obs_norm(*held)
    assert "rollout_mfma_cols_f32" in ctx.rollout_kernel
    a_mat, b_mat, theta = make_inputs(w)
    eps = oracle.sample_population(w, 0)
    ret, _, _ = run_rollout(ctx, w, 0, theta, noise_to_device(ctx, eps), a_mat, b_mat)
    few = (590, 610)
    ref = oracle.rollout(w, 0, theta, eps, a_mat, b_mat, individuals=few, obs_norm=stats)[0]
    assert np.abs(ret[slice(*few)] - ref).max() <= 2e-6 * np.abs(ref).max()


@pytest.mark.parametrize("norm,act", [(True, 4), (False, 16)])
@pytest.mark.parametrize("wavefronts,extra", [(3, 0), (3, 2), (4, 0), (4, 2)])
def test_smallest_class_around_a_full_chip(es, wavefronts, extra, norm, act):  # noqa: F811
    """Up to 16 observations and units: pieces, but for four wavefronts a compute unit (16x16x4) - the same precision on both sides of both lines."""
    pop = wavefronts * torch.cuda.get_device_properties(0).multi_processor_count + extra
    _precise(es, replace(F, name=f"split-smallest-{pop}", obs=16, hid=16, act=act, pop=pop, seed=951), norm)


def test_actions_beyond_the_pieces_range(es):  # noqa: F811
    """A linear output that overflows (one action, so that no infinities meet): the copy ends where it ends on one wavefront an episode, binary32 throughout, and
    its return is infinite there as here."""
    few, many = (replace(F, name="split-overflow", obs=16, hid=32, act=1, out_tanh=0, done_thresh=0.95, horizon=6, pop=n, envs=e) for n, e in ((4, 2), (2000, 16)))
    a_mat, b_mat, theta = make_inputs(few)
    o, h, a = few.obs, few.hid, few.act
    w3 = (o + 1) * h + (h + 1) * h
    theta[w3:w3 + a * h] = np.float32(2.9e38) * np.sign(theta[w3:w3 + a * h])
    got = []
    for w in (few, many):
        ctx = es.EsContext(w)
        got.append(run_rollout(ctx, w, 0, theta, noise_to_device(ctx, oracle.sample_population(w, 0)), a_mat, b_mat))
    assert "cols_f32" in ctx.rollout_kernel
    assert np.isinf(got[0][0]).any() and (got[0][1] < few.horizon).all()
    assert np.array_equal(got[0][1], got[1][1][:4, :2])
    assert np.array_equal(got[0][0], got[1][0][:4, :2])


def _infinite_weight(w, theta):
    theta[0] = np.inf


def _not_a_number(w, theta):
    theta[w.obs * w.hid] = np.nan      # b1[0]


def _overflowing_products(w, theta):
    """Units that overflow by one product, whose pieces' products are infinities of both signs."""
    o, h, a = w.obs, w.hid, w.act
    w2, w3 = (o + 1) * h, (o + 1) * h + (h + 1) * h
    theta[:o * h] *= np.float32(1e20)
    theta[w2:w2 + h * h] = (np.float32(1e20) * np.eye(h, dtype=np.float32)).ravel()
    theta[w3:w3 + a * h] = np.abs(theta[w3:w3 + a * h]) + np.float32(0.1)


@pytest.mark.parametrize("relu,change,mean,inv,finite", [
    (0, None, 1e9, 1e-9, True), (1, None, -3e8, 1e-8, True), (1, None, 0.0, 1e14, True), (0, None, 0.0, 3e30, True), (0, None, 0.0, np.inf, False), (1, None, np.nan, 1.0, True),
    (1, _infinite_weight, None, None, False), (1, _overflowing_products, None, None, True), (0, _not_a_number, None, None, False)],
    ids=lambda v: v.__name__.strip("_") if callable(v) else str(v))
def test_values_beyond_the_pieces_range(es, relu, change, mean, inv, finite):  # noqa: F811
    """Statistics and parameters that three bf16 pieces do not carry: the individual runs on the binary32 shape, and its returns are the CPU checker's, infinities and NaN
    included.  (Widths without padding, where an infinity would meet a zero.)"""
    w = replace(F, name="split-range", obs=16, hid=32, act=16, hidden_act=relu, horizon=4, pop=2000)
    a_mat, b_mat, theta = make_inputs(w)
    if change:
        change(w, theta)
    ctx = es.EsContext(w)
    assert "cols_f32" in ctx.rollout_kernel
    stats = None if mean is None else tuple(np.full(w.obs, v, np.float32) for v in (mean, inv))
    if stats:
        held = tuple(dev(v) for v in stats)
        ctx.set_obs_norm(*held)
    eps = oracle.sample_population(w, 0)
    ret, length, _ = run_rollout(ctx, w, 0, theta, noise_to_device(ctx, eps), a_mat, b_mat)
    want, ref_len, _, _ = oracle.rollout(w, 0, theta, eps, a_mat, b_mat, individuals=(0, 6), obs_norm=stats)
    have = ret[:6]
    assert np.array_equal(length[:6], ref_len)
    assert np.isfinite(want).all() == finite
    assert np.array_equal(np.isnan(want), np.isnan(have)) and np.array_equal(np.isinf(want), np.isinf(have))
    ok = np.isfinite(want)
    assert np.all(np.abs(want - have)[ok] <= 2e-6 * np.abs(want[ok]))      # (test_binary32_precision)
