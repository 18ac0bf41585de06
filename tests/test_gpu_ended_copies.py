"""Copies that share a pass of a matrix-core rollout kernel run on together after one of them has ended.  What an ended copy does from then on - here its
linear action grows until its square is beyond binary32 - must not reach its return, which counts the steps up to its end: against the CPU checker."""
from dataclasses import replace

import numpy as np
import pytest
import torch

import oracle
from paper_2501_15129_amd.workloads import Workload
from gpu_util import dev, noise_to_device, run_rollout

pytestmark = pytest.mark.gpu

F = Workload("ended", pop=4, envs=4, horizon=14, obs=20, hid=100, act=5, dtype=0, noise_dtype=0, seed=77, sigma=0.0, done_thresh=0.5, hidden_act=1, out_tanh=0)
BF = dict(dtype=1, noise_dtype=1)


def policy(w):
    """The first unit of every layer passes max(s_0 - 0.55, 0) on, times 1e22 in the action: zero while a copy runs."""
    theta, at, width = [], 0, w.obs
    for layer in range(w.num_hidden + 1):
        rows = w.hid if layer < w.num_hidden else w.act
        m, b = np.zeros((rows, width), np.float32), np.zeros(rows, np.float32)
        m[0, 0] = 1e11 if layer in (0, w.num_hidden) else 1.0
        if layer == 0:
            b[0] = -0.55e11
        theta += [m.ravel(), b]
        width = rows
    return np.concatenate(theta)


@pytest.mark.parametrize("kw", [
    # sixteen copies in one wavefront
    dict(pop=1000, envs=16, hid=48), dict(pop=1000, envs=13, hid=64, obs=40, act=12), dict(BF, pop=1000, envs=16, hid=64),
    # passes of four and of two copies: one, two and four wavefronts, one row of the action per lane or one copy's, deep, state rows spread
    dict(pop=1100, envs=8, hid=49, obs=32), dict(BF, pop=512, envs=4, hid=64), dict(pop=200, envs=7), dict(hid=256, pop=100, envs=8),
    dict(BF, pop=100, envs=7), dict(BF, pop=200, envs=8), dict(BF, pop=200, envs=4, obs=100, act=20), dict(BF, hid=256, pop=70, envs=8), dict(BF, hid=256, pop=200, envs=8, num_hidden=1),
    dict(BF, hid=256, pop=300, num_hidden=3), dict(BF, hid=256, pop=300, num_hidden=4), dict(BF, hid=256, pop=300, envs=2, obs=244, act=17), dict(BF, hid=256, pop=300, obs=244, act=17),
    # sixteen copies of a workgroup, and one a wavefront or workgroup
    dict(BF, hid=256, pop=512, envs=16), dict(hid=256, pop=300, envs=16), dict(hid=256), dict(hid=64), dict(hid=32)], ids=str)
def test_an_ended_copy_keeps_its_return(kw):
    import paper_2501_15129_amd as es
    w = replace(F, **kw)
    a_mat, b_mat, theta = np.zeros((w.obs, w.obs), np.float32), np.zeros((w.obs, w.act), np.float32), policy(w)
    a_mat[0, 0] = 2.0
    ctx = es.EsContext(w)
    assert theta.size == ctx.param_count
    eps = oracle.sample_population(w, 3)
    ret, length, fit = run_rollout(ctx, w, 3, theta, noise_to_device(ctx, eps), a_mat, b_mat)
    r_ret, r_len, r_fit, margin = oracle.rollout(w, 3, theta, eps, a_mat, b_mat, individuals=(0, 2))
    assert len(set(r_len[0])) > 1 and margin.min() > 1e-3 and np.isfinite(r_ret).all(), "copies that end one after the other"
    tol = 1e-4 if w.dtype == 0 else 2e-2
    print(f"kernel={ctx.rollout_kernel} lengths {sorted(set(r_len[0].tolist()))} not finite {int(np.sum(~np.isfinite(ret)))} of {ret.size}", flush=True)
    assert np.array_equal(length, np.broadcast_to(r_len[0], length.shape))
    assert np.all(np.abs(ret - r_ret[0]) <= tol * np.abs(r_ret[0]))
    assert np.all(np.abs(fit - r_fit[0]) <= tol * np.abs(r_fit[0]))
