"""Layers that run as paired products, held so closely that one input less would show: parameters and environment of small whole numbers, whose sums are exact in any order, ReLU and a
linear output, two steps.  Without the last input of a single matrix the CPU checker's own returns are beyond the tolerance (shown here on the CPU)."""
from dataclasses import replace

import numpy as np
import pytest
import torch

import oracle
from gpu_util import noise_to_device, run_rollout
from paper_2501_15129_amd.workloads import Workload, layer_shapes

# (sigma: the perturbation vanishes beside every parameter)
W = Workload("inputs", pop=4, envs=1, horizon=2, obs=27, hid=128, act=8, dtype=1, noise_dtype=1, seed=961, sigma=1e-30, out_tanh=0, act_cost=1024.0, hidden_act=1, done_thresh=float("inf"))
# A few operands whose sums end within a rounding error of a boundary of bf16 go the other way, by 2^-9 of one input of 65 or more
RTOL = 5e-4
SHAPES = [(9, 65, 2), (33, 127, 2), (27, 128, 2), (8, 129, 2), (64, 191, 2), (5, 193, 3), (40, 255, 3), (12, 66, 4), (20, 100, 3), (32, 256, 4), (65, 128, 2), (128, 129, 2), (129, 192, 2),
          (192, 256, 2), (193, 200, 2), (256, 256, 2), (66, 100, 1), (100, 65, 2), (250, 128, 2), (110, 127, 1)]


def _workload(obs, hid, layers, pop=4, envs=1):
    return replace(W, name=f"inputs-{obs}-{hid}x{layers}-{envs}", obs=obs, hid=hid, act=1 + obs % 16, num_hidden=layers, pop=pop, envs=envs, seed=961 + obs + hid + layers)


def _inputs(w):
    rng = np.random.default_rng([w.seed, 3])
    whole = lambda shape, size: (rng.integers(1, size + 1, shape) * rng.choice([-1, 1], shape)).astype(np.float32)      # noqa: E731
    parts, n = [], len(layer_shapes(w))
    for k, shape in enumerate(layer_shapes(w)):
        last = k >= n - 2
        if len(shape) == 1:
            parts.append(np.abs(whole(shape, 4)) / (16 if last else 1))
        else:      # (a layer's outputs about as large as its inputs)
            parts.append(whole(shape, 3) / np.float32(2.0 ** round(np.log2(2 * np.sqrt(shape[1])) if k else 0)) / (16 if last else 1))
    a_mat = whole((w.obs, w.obs), 3) / 4
    b_mat = whole((w.obs, w.act), 3) / 16
    return a_mat, b_mat, np.concatenate([p.ravel() for p in parts]).astype(np.float32), parts


def _expected(w, a_mat, b_mat, theta):
    return oracle.rollout(w, 0, theta, np.zeros((w.noise_rows, theta.size), np.float32), a_mat, b_mat, individuals=(0, 2))[0]


@pytest.mark.parametrize("obs,hid,layers", SHAPES)
def test_an_input_less_shows(obs, hid, layers):
    w = _workload(obs, hid, layers, envs=4)
    a_mat, b_mat, theta, parts = _inputs(w)
    want = _expected(w, a_mat, b_mat, theta)
    for k in range(0, len(parts) - 2, 2):      # the last input of each hidden layer
        less = [p.copy() for p in parts]
        less[k][:, -1] = 0.0
        got = _expected(w, a_mat, b_mat, np.concatenate([p.ravel() for p in less]))
        assert np.abs(got - want).max() > 2 * RTOL * np.abs(want).max(), f"layer {k // 2}"
    less = a_mat.copy()
    less[:, -1] = 0.0
    assert np.abs(_expected(w, less, b_mat, theta) - want).max() > 2 * RTOL * np.abs(want).max()


@pytest.mark.gpu
@pytest.mark.parametrize("copies", [1, 2, 4])
@pytest.mark.parametrize("obs,hid,layers", SHAPES)
def test_every_input_counts(obs, hid, layers, copies):
    from paper_2501_15129_amd import EsContext
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    # one copy a pass; too many for one, for two
    w = _workload(obs, hid, layers, 6 if copies == 1 else cus // 2 + 2 if copies == 2 else cus + 2, copies)
    a_mat, b_mat, theta, _ = _inputs(w)
    ctx = EsContext(w)
    assert "quad_bf16" in ctx.rollout_kernel
    ret, _, _ = run_rollout(ctx, w, 0, theta, noise_to_device(ctx, oracle.sample_population(w, 0)), a_mat, b_mat)
    want = _expected(w, a_mat, b_mat, theta)
    assert np.abs(ret[:2] - want).max() <= RTOL * np.abs(want).max()
