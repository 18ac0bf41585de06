"""Kernels that small populations do not reach: one wavefront per episode at 33 to 64 units (beyond one episode per compute unit, two with four
layers), the four-copy kernel for narrow policies (populations between one and sixteen copies a wavefront) and for binary32 policies of 65 to 256 units
(beyond one episode per compute unit) - edges of the width classes, depths, both activations, every noise mode, statistics, early ends, and the full
horizon - against the CPU checker, each with the exact name of the kernel."""
from dataclasses import replace

import numpy as np
import pytest

import oracle
from paper_2501_15129_amd.workloads import make_inputs
from gpu_util import compare_rollout, noise_to_device, probe_rollout, run_rollout
from test_gpu_quad import F, _case, es  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

BF = dict(dtype=1, noise_dtype=1)
ONE = replace(F, name="one", pop=260, envs=1, horizon=10)


@pytest.mark.parametrize("m,obs,hid,act,kw,kernel", [
    (2, 17, 64, 6, dict(hidden_act=1), "f32<17,64,6>"), (2, 17, 64, 6, dict(out_tanh=0, noise_dtype=2), "f32<17,64,6>"), (2, 16, 33, 4, dict(), "f32<obs<=16,hid<=64,act<=4>"),
    (2, 1, 64, 16, dict(hidden_act=1, done_thresh=0.5), "f32<obs<=16,hid<=64,act<=16>"), (2, 32, 50, 8, dict(noise_dtype=3), "f32<obs<=32,hid<=64,act<=8>"),
    (2, 17, 64, 9, dict(done_thresh=1e-6), "f32<obs<=32,hid<=64,act<=16>"), (2, 33, 64, 4, dict(out_tanh=0), "f32<obs<=64,hid<=64,act<=4>"),
    (2, 64, 64, 16, dict(hidden_act=1, horizon=30), "f32<obs<=64,hid<=64,act<=16>"), (2, 64, 49, 5, dict(noise_dtype=1, pop=130, envs=2), "f32<obs<=64,hid<=64,act<=8>"),
    (3, 16, 64, 8, dict(horizon=3), "f32<obs<=16,hid<=64,act<=8>,depth3"), (3, 40, 33, 4, dict(hidden_act=1), "f32<obs<=64,hid<=64,act<=4>,depth3"),
    (3, 64, 64, 16, dict(done_thresh=0.5, out_tanh=0), "f32<obs<=64,hid<=64,act<=16>,depth3"), (4, 20, 48, 3, dict(pop=516), "f32<obs<=32,hid<=64,act<=4>,depth4"),
    (4, 64, 64, 16, dict(pop=514, hidden_act=1, noise_dtype=2), "f32<obs<=64,hid<=64,act<=16>,depth4"), (4, 5, 40, 7, dict(pop=258, envs=2, done_thresh=0.5), "f32<obs<=16,hid<=64,act<=8>,depth4"),
    (2, 16, 64, 8, dict(BF, horizon=30), "bf16<obs<=16,hid<=64,act<=8>"), (2, 32, 33, 4, dict(BF, hidden_act=1), "bf16<obs<=32,hid<=64,act<=4>"), (2, 17, 64, 16, dict(BF, noise_dtype=3, out_tanh=0), "bf16<obs<=32,hid<=64,act<=16>"),
    (2, 40, 48, 8, dict(BF, env_dtype=1), "bf16<obs<=64,hid<=64,act<=8>"), (3, 33, 64, 6, dict(BF, done_thresh=0.5), "bf16<obs<=64,hid<=64,act<=8>,depth3"),
    (3, 20, 40, 9, dict(BF, hidden_act=1), "bf16<obs<=32,hid<=64,act<=16>,depth3"), (4, 16, 64, 4, dict(BF, pop=514), "bf16<obs<=16,hid<=64,act<=4>,depth4"), (4, 64, 34, 16, dict(BF, pop=514, noise_dtype=3), "bf16<obs<=64,hid<=64,act<=16>,depth4")],
    ids=lambda v: str(v) if not isinstance(v, dict) else "-".join(f"{k}{x}" for k, x in v.items()))
def test_one_wavefront_at_33_to_64_units(es, m, obs, hid, act, kw, kernel):  # noqa: F811
    w = replace(ONE, name=f"one-{obs}-{hid}x{m}-{act}", num_hidden=m, obs=obs, hid=hid, act=act, seed=601 + obs + hid)
    assert _case(es, replace(w, **kw)).rollout_kernel == "rollout_wave_reg_" + kernel


@pytest.mark.parametrize("kw", [dict(), dict(obs=40, act=12, hidden_act=1), dict(num_hidden=3), dict(num_hidden=4, pop=514, obs=50), dict(BF), dict(BF, num_hidden=3, obs=40), dict(BF, num_hidden=4, pop=514)], ids=str)
def test_one_wavefront_observation_statistics(es, kw):  # noqa: F811
    name = _case(es, replace(ONE, name="one-norm", **{"obs": 17, "hid": 64, "act": 6, **kw}), norm=True).rollout_kernel
    assert "rollout_wave_reg_" in name and "team" not in name


@pytest.mark.parametrize("obs,hid,act,pop,envs,kw,kernel", [
    (1, 33, 1, 600, 4, dict(), "f32<obs16"), (16, 64, 16, 512, 8, dict(hidden_act=1), "f32<obs16"), (17, 48, 8, 512, 8, dict(out_tanh=0), "f32<obs32"), (32, 64, 16, 700, 7, dict(done_thresh=0.5), "f32<obs32"),
    (33, 33, 4, 600, 4, dict(noise_dtype=2), "f32<obs64"), (64, 64, 16, 512, 7, dict(hidden_act=1, done_thresh=0.5), "f32<obs64"), (48, 64, 9, 1000, 3, dict(noise_dtype=1), "f32<obs64"),
    (5, 64, 3, 300, 5, dict(BF), "bf16<obs32"), (32, 64, 16, 512, 4, dict(BF, hidden_act=1), "bf16<obs32"), (17, 60, 6, 400, 3, dict(BF, noise_dtype=3, out_tanh=0), "bf16<obs32"),
    (33, 33, 1, 260, 1, dict(BF), "bf16<obs64"), (64, 64, 16, 300, 5, dict(BF, done_thresh=0.5), "bf16<obs64"), (48, 40, 8, 300, 3, dict(BF, hidden_act=1, antithetic=0), "bf16<obs64")],
    ids=lambda v: str(v) if not isinstance(v, dict) else "-".join(f"{k}{x}" for k, x in v.items()))
def test_narrow_policies_in_passes_of_four(es, obs, hid, act, pop, envs, kw, kernel):  # noqa: F811
    w = replace(replace(F, name=f"four-{obs}-{hid}-{act}", horizon=10, obs=obs, hid=hid, act=act, pop=pop, envs=envs, seed=621 + obs + hid), **kw)
    name = f"rollout_mfma_quad_{kernel},hid64,act16>"
    assert _case(es, w).rollout_kernel == name
    assert _case(es, w, norm=True).rollout_kernel == name


@pytest.mark.parametrize("m,obs,hid,act,pop,envs,kw,kernel", [
    (2, 8, 256, 2, 128, 4, dict(), "obs16,hid256"), (2, 16, 129, 16, 300, 2, dict(hidden_act=1), "obs16,hid256"), (1, 12, 200, 5, 90, 3, dict(out_tanh=0), "obs16,hid256"),
    (2, 17, 256, 8, 66, 4, dict(noise_dtype=2), "obs32,hid256"), (2, 32, 200, 3, 130, 8, dict(done_thresh=0.5), "obs32,hid256"), (1, 32, 256, 16, 300, 5, dict(hidden_act=1), "obs32,hid256"),
    (2, 16, 65, 4, 130, 6, dict(), "obs16,hid128"), (1, 5, 128, 1, 300, 2, dict(noise_dtype=3), "obs16,hid128"), (3, 16, 100, 16, 70, 9, dict(hidden_act=1), "obs16,hid128"),
    (2, 17, 128, 6, 514, 1, dict(done_thresh=0.5), "obs32,hid128"), (3, 32, 96, 9, 200, 3, dict(out_tanh=0), "obs32,hid128"), (2, 64, 128, 16, 130, 5, dict(hidden_act=1), "obs64,hid128"),
    (3, 64, 100, 8, 600, 1, dict(done_thresh=0.5), "obs64,hid128")],
    ids=lambda v: str(v) if not isinstance(v, dict) else "-".join(f"{k}{x}" for k, x in v.items()))
def test_wide_binary32_policies_in_passes_of_up_to_four(es, m, obs, hid, act, pop, envs, kw, kernel):  # noqa: F811
    w = replace(replace(F, name=f"wide-{obs}-{hid}x{m}-{act}", horizon=10, num_hidden=m, obs=obs, hid=hid, act=act, pop=pop, envs=envs, seed=641 + obs + hid), **kw)
    name = f"rollout_mfma_quad_f32<{kernel},act16>" + ("" if m == 2 else f",depth{m}")
    assert _case(es, w).rollout_kernel == name
    # (statistics: the widest observation class whatever the width)
    assert _case(es, w, norm=True).rollout_kernel == name


def test_paper_base_shape_on_four_copies_at_the_full_horizon(es):  # noqa: F811
    """Two hidden layers of 256 at 8 observations and 2 actions, 128 individuals on four copies, a thousand steps in binary32: within 1e-4 on the contractive twin."""
    w = replace(F, name="paper-base-four-copies", pop=128, envs=4, horizon=1000, obs=8, hid=256, act=2, seed=5).contractive()
    a_mat, b_mat, theta = make_inputs(w)
    ctx = es.EsContext(w)
    assert ctx.rollout_kernel == "rollout_mfma_quad_f32<obs16,hid256,act16>"
    eps = oracle.sample_population(w, 0)
    got = run_rollout(ctx, w, 0, theta, noise_to_device(ctx, eps), a_mat, b_mat)
    n = (0, 16)
    ref = oracle.rollout(w, 0, theta, eps, a_mat, b_mat, individuals=n)
    probe = probe_rollout(w, 0, theta, eps, a_mat, b_mat, ref=ref, probes=1, individuals=n)
    flips, worst, sens, chaotic = compare_rollout(w, tuple(x[:n[1]] for x in got), ref, w.name, probe)
    print(f"[{w.name}] worst {worst:.2e} sensitive {sens}")
    assert not chaotic and compare_rollout.last_excused == 0 and np.all(got[1] == w.horizon)
