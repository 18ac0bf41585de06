"""Wavefront priorities of the sixteen-column bf16 kernel are a matter of speed only: populations on both sides of the rule evaluate the
same individuals bit for bit (full rounds and more than half a round: with priorities; up to half a round left over: without)."""
from dataclasses import replace

import numpy as np
import pytest
import torch

from paper_2501_15129_amd.workloads import Workload, make_inputs
from gpu_util import run_rollout

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw", [dict(), dict(hidden_act=1), dict(num_hidden=1), dict(envs=20), dict(env_dtype=1)], ids=str)
def test_both_sides_of_the_rule(kw):
    import paper_2501_15129_amd as es
    slots = 2 * torch.cuda.get_device_properties(0).multi_processor_count
    base = replace(Workload("order", pop=slots, envs=16, horizon=6, obs=27, hid=256, act=8, dtype=1, noise_dtype=1, seed=901), **kw).contractive()
    a_mat, b_mat, theta = make_inputs(base)
    got = {}
    for pop in (slots, slots + 8, slots + slots // 2, slots + slots // 2 + 2, 2 * slots):
        w = replace(base, pop=pop)
        ctx = es.EsContext(w)
        assert "rollout_mfma_reg_bf16<obs32" in ctx.rollout_kernel
        noise = ctx.alloc_noise()
        ctx.sample_population(1, noise)
        got[pop] = run_rollout(ctx, w, 1, theta, noise, a_mat, b_mat)
    for pop, r in got.items():
        assert np.isfinite(r[0]).all()
        for x, y in zip(r, got[2 * slots]):
            assert np.array_equal(x.view(np.uint32), y[:pop].view(np.uint32)), pop
