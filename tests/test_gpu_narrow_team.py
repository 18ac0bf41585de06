"""Narrow policies in four wavefronts per episode (33 to 64 hidden units, up to one episode per compute unit): the edges of the width
classes and of the four steps of a turn, odd and even depths, both precisions, every noise mode and activation, early ends - against
the CPU checker; and the largest population it takes against the next one, which has one wavefront per episode."""
from dataclasses import replace

import numpy as np
import pytest
import torch

from paper_2501_15129_amd.workloads import Workload
from test_gpu_quad import _case, es  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

F = Workload("team", pop=4, envs=3, horizon=30, obs=17, hid=64, act=6, dtype=0, noise_dtype=0, seed=701)


@pytest.mark.parametrize("m,obs,hid,act,T,kw", [
    (2, 1, 33, 1, 1, {}), (2, 20, 64, 4, 2, {}), (2, 21, 48, 5, 3, dict(hidden_act=1)), (2, 32, 49, 6, 4, {}), (2, 33, 64, 7, 5, dict(out_tanh=0)),
    (2, 48, 63, 8, 6, dict(noise_dtype=2)), (2, 49, 64, 9, 7, {}), (2, 64, 64, 16, 30, dict(done_thresh=0.5)), (2, 17, 64, 6, 30, dict(done_thresh=1e-6)),
    (3, 17, 64, 6, 5, {}), (3, 20, 33, 16, 6, dict(hidden_act=1)), (3, 33, 50, 8, 7, dict(noise_dtype=1)), (3, 64, 64, 16, 30, dict(done_thresh=0.5)),
    (4, 5, 40, 3, 3, {}), (4, 48, 64, 9, 6, dict(out_tanh=0)), (4, 64, 64, 16, 9, dict(antithetic=0, pop=3)), (4, 32, 34, 2, 30, dict(done_thresh=0.5, hidden_act=1)),
    (2, 17, 64, 6, 30, dict(dtype=1, noise_dtype=1)), (2, 64, 33, 16, 9, dict(dtype=1, noise_dtype=3, hidden_act=1)), (3, 40, 48, 8, 30, dict(dtype=1, noise_dtype=1)),
    (4, 20, 64, 1, 7, dict(dtype=1, noise_dtype=1)), (2, 27, 48, 8, 30, dict(dtype=1, noise_dtype=1, env_dtype=1))],
    ids=lambda v: str(v) if not isinstance(v, dict) else "-".join(f"{k}{x}" for k, x in v.items()))
def test_edges(es, m, obs, hid, act, T, kw):  # noqa: F811
    w = replace(F, name=f"team-{obs}-{hid}x{m}-{act}-T{T}", num_hidden=m, obs=obs, hid=hid, act=act, horizon=T, seed=701 + obs + hid)
    assert "wave_reg_team_" in _case(es, replace(w, **kw)).rollout_kernel


@pytest.mark.parametrize("m,dtype", [(2, 0), (3, 0), (4, 0), (2, 1), (3, 1)])
def test_observation_statistics(es, m, dtype):  # noqa: F811
    w = replace(F, name=f"team-norm-x{m}-{dtype}", num_hidden=m, obs=40, dtype=dtype, noise_dtype=dtype, seed=733 + m)
    assert "wave_reg_team_" in _case(es, w, norm=True).rollout_kernel


@pytest.mark.parametrize("m", [2, 3, 4])
def test_four_wavefronts_and_one_evaluate_the_same(es, m):  # noqa: F811
    """The first individuals of a population that fills the compute units, and of one that does not fit them: the two kernels add the
    same products in another order, which forty contracting steps turn into less than 1e-5 of a return."""
    from paper_2501_15129_amd import make_inputs
    from gpu_util import run_rollout
    most = torch.cuda.get_device_properties(0).multi_processor_count * (2 if m == 4 else 1)      # episodes that four wavefronts each are used for
    few = replace(F, name="team-few", num_hidden=m, pop=most - most % 2, envs=1, horizon=40, seed=750 + m).contractive()
    many = replace(few, pop=few.pop + 2)
    a_mat, b_mat, theta = make_inputs(few)
    got = []
    for w, kernel in ((few, "rollout_wave_reg_team_f32"), (many, "rollout_wave_reg_f32")):
        ctx = es.EsContext(w)
        assert kernel in ctx.rollout_kernel
        noise = ctx.alloc_noise()
        ctx.sample_population(3, noise)
        got.append(run_rollout(ctx, w, 3, theta, noise, a_mat, b_mat))
    n = few.pop
    assert np.array_equal(got[0][1], got[1][1][:n]) and np.isfinite(got[0][0]).all()
    assert np.all(np.abs(got[0][0] - got[1][0][:n]) <= 1e-5 * np.abs(got[0][0]))
    assert np.array_equal(got[0][2], got[0][0][:, 0])
