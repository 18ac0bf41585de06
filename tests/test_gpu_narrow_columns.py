"""Narrow policies in passes of sixteen copies, one wavefront each (populations whose episodes outnumber the wavefronts of the chip): the edges
of the width classes, ragged and several passes, both precisions, every noise mode and activation, early ends, observation statistics - against
the CPU checker."""
from dataclasses import replace

import pytest

from paper_2501_15129_amd.workloads import Workload
from test_gpu_quad import _case, es  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

F = Workload("columns", pop=1000, envs=16, horizon=7, obs=17, hid=48, act=5, dtype=0, noise_dtype=0, seed=801)
BF = dict(dtype=1, noise_dtype=1)


@pytest.mark.parametrize("obs,hid,act,kw", [
    (1, 17, 1, {}), (16, 16, 4, dict(horizon=30)), (17, 33, 8, dict(hidden_act=1)), (20, 32, 9, {}), (21, 48, 16, dict(out_tanh=0)), (32, 49, 8, dict(done_thresh=0.5)),
    (33, 64, 5, dict(envs=13)), (48, 50, 16, dict(noise_dtype=2)), (49, 64, 8, dict(hidden_act=1, horizon=30)), (64, 64, 16, dict(done_thresh=0.3)), (3, 64, 2, dict(noise_dtype=3)),
    (19, 48, 5, dict(pop=500, envs=36, hidden_act=1)), (11, 25, 3, dict(pop=900, envs=5, episodes=4)), (17, 64, 6, dict(done_thresh=1e-6)), (27, 41, 7, dict(horizon=1, pop=999, antithetic=0)),
    (16, 16, 4, BF), (17, 64, 6, dict(BF, horizon=30)), (32, 33, 16, dict(BF, hidden_act=1)), (33, 48, 1, dict(BF, noise_dtype=3)), (64, 64, 16, dict(BF, done_thresh=0.5)),
    (5, 20, 9, dict(BF, pop=500, envs=36, out_tanh=0)), (48, 49, 8, dict(BF, envs=13))],
    ids=lambda v: str(v) if not isinstance(v, dict) else "-".join(f"{k}{x}" for k, x in v.items()))
def test_edges(es, obs, hid, act, kw):  # noqa: F811
    w = replace(F, name=f"columns-{obs}-{hid}-{act}", obs=obs, hid=hid, act=act, seed=801 + obs + hid)
    assert "rollout_mfma_cols_" in _case(es, replace(w, **kw)).rollout_kernel


@pytest.mark.parametrize("kw", [dict(), dict(obs=64, hid=64, act=16, hidden_act=1), dict(BF, obs=40), dict(BF, obs=20, hid=64, hidden_act=1)], ids=str)
def test_observation_statistics(es, kw):  # noqa: F811
    assert "rollout_mfma_cols_" in _case(es, replace(F, name="columns-norm", seed=833, **kw), norm=True).rollout_kernel
