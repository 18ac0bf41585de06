"""Binary32 policies of 65 to 256 units with one copy per workgroup on the vector ALU (up to one episode per compute unit, and what single_pays adds): the
edges of the width classes, depths, every noise mode and activation, the four steps of a turn, early ends, observation statistics - against the CPU
checker; and both sides of the rule."""
from dataclasses import replace

import numpy as np
import pytest
import torch

from paper_2501_15129_amd.workloads import Workload, make_inputs
from gpu_util import run_rollout
from test_gpu_quad import _case, es  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

F = Workload("single", pop=4, envs=1, horizon=30, obs=17, hid=128, act=6, dtype=0, noise_dtype=0, seed=951)


@pytest.mark.parametrize("m,obs,hid,act,T,kw", [
    (1, 1, 65, 1, 1, {}), (1, 64, 128, 16, 2, dict(hidden_act=1)), (2, 20, 96, 4, 3, {}), (2, 21, 97, 5, 4, dict(out_tanh=0)), (2, 33, 127, 8, 5, dict(noise_dtype=2)),
    (2, 64, 128, 9, 30, dict(done_thresh=0.5)), (3, 32, 66, 16, 6, dict(hidden_act=1)), (3, 64, 128, 7, 7, dict(noise_dtype=1)), (3, 5, 100, 2, 30, dict(done_thresh=0.5, envs=5)),
    (1, 12, 129, 3, 5, {}), (1, 32, 256, 16, 30, dict(done_thresh=0.5)), (2, 8, 256, 2, 30, {}), (2, 13, 255, 8, 6, dict(hidden_act=1, envs=3)), (2, 20, 160, 1, 7, dict(noise_dtype=3)),
    (2, 21, 161, 12, 9, dict(antithetic=0, pop=3)), (2, 32, 256, 16, 30, dict(done_thresh=1e-6)), (2, 27, 193, 4, 8, dict(out_tanh=0, noise_dtype=1))],
    ids=lambda v: str(v) if not isinstance(v, dict) else "-".join(f"{k}{x}" for k, x in v.items()))
def test_edges(es, m, obs, hid, act, T, kw):  # noqa: F811
    w = replace(F, name=f"single-{obs}-{hid}x{m}-{act}-T{T}", num_hidden=m, obs=obs, hid=hid, act=act, horizon=T, seed=951 + obs + hid)
    assert "rollout_single_f32" in _case(es, replace(w, **kw)).rollout_kernel


@pytest.mark.parametrize("kw", [dict(), dict(num_hidden=3, obs=50), dict(hid=256, obs=30), dict(hid=200, num_hidden=1, hidden_act=1)], ids=str)
def test_observation_statistics(es, kw):  # noqa: F811
    assert "rollout_single_f32" in _case(es, replace(F, name="single-norm", **kw), norm=True).rollout_kernel


# (the number of individuals up to which the rule takes them, in quarters of the compute units)
@pytest.mark.parametrize("kw,quarters", [(dict(), 4), (dict(envs=2), 4), (dict(envs=4, num_hidden=3), 2), (dict(hid=256, envs=4), 1), (dict(hid=200, num_hidden=1), 4)], ids=str)
def test_both_sides_of_the_rule(es, kw, quarters):  # noqa: F811
    """The two kernels add the same products in another order, which forty contracting steps turn into less than 1e-5 of a return."""
    got = []
    most = torch.cuda.get_device_properties(0).multi_processor_count * quarters // 8 * 2
    pops = (most, most + 2)
    base = replace(F, name="single-rule", horizon=40, **kw)
    a_mat, b_mat, theta = make_inputs(replace(base, pop=pops[0]).contractive())
    for pop, kernel in zip(pops, ("rollout_single_f32", "rollout_mfma_quad_f32")):
        w = replace(base, pop=pop).contractive()
        ctx = es.EsContext(w)
        assert kernel in ctx.rollout_kernel
        noise = ctx.alloc_noise()
        ctx.sample_population(3, noise)
        got.append(run_rollout(ctx, w, 3, theta, noise, a_mat, b_mat))
    n = pops[0]
    assert np.isfinite(got[0][0]).all() and np.array_equal(got[0][1], got[1][1][:n])
    assert np.all(np.abs(got[0][0] - got[1][0][:n]) <= 1e-5 * np.abs(got[0][0]))
    assert np.all(np.abs(got[0][2] - got[0][0].mean(axis=1)) <= 1e-6 * np.abs(got[0][2]))
