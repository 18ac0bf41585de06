"""Where the selection and update kernels change form: a generation whose last launch does fitness, ranks and update; narrow
matrices of many rows, split into chunks; the one-workgroup selections at the edges of their groups of 64."""
from dataclasses import replace

import numpy as np
import pytest
import torch

import oracle
from paper_2501_15129_amd.workloads import Workload, make_inputs, random_fitness
from gpu_util import assert_params_close, dev, noise_to_device
from test_gpu_generation import GpuChain, es  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu

NARROW = Workload("edge", pop=2, envs=1, horizon=6, obs=5, hid=9, act=2, dtype=0, noise_dtype=0, seed=3)
ONE_CALL = [
    NARROW,
    replace(NARROW, pop=1, antithetic=0),
    replace(NARROW, pop=62, envs=3),
    replace(NARROW, pop=66, envs=9, noise_dtype=1),
    replace(NARROW, pop=512, envs=8),                       # the largest population and number of returns of one launch
    replace(NARROW, pop=512, envs=9),                       # one return too many per individual
    replace(NARROW, pop=514),
    replace(NARROW, pop=511, antithetic=0, envs=2),
    replace(NARROW, pop=130, envs=17, noise_dtype=4, noise_table_len=1 << 14),
    replace(NARROW, pop=130, obs=27, hid=100, envs=5, dtype=1, noise_dtype=1),      # four-copy rollout
    replace(NARROW, pop=10, obs=20, hid=65, act=20, envs=2),                        # rollout from the LDS
    replace(NARROW, pop=20, obs=100, hid=200, act=17, envs=2, dtype=1, noise_dtype=5, noise_table_len=1 << 18),
]


@pytest.mark.parametrize("w", ONE_CALL, ids=lambda w: f"N{w.pop}-E{w.envs}-{w.obs}-{w.hid}-{w.act}-nz{w.noise_dtype}")
def test_one_call_equals_four_calls(es, w):  # noqa: F811
    a_mat, b_mat, theta = make_inputs(w)
    four, one = GpuChain(es, w, theta, a_mat, b_mat), GpuChain(es, w, theta, a_mat, b_mat)
    for c in (four, one):
        if c.ctx.noise_table:
            c.ctx.build_noise_table(c.noise)
    for g in range(2):
        four.generation(g)
        one.generation_one_call(g)
    torch.cuda.synchronize()
    for name in ("theta", "m", "v", "ret", "len", "fit", "rank", "shaped"):
        x, y = getattr(four, name).cpu().numpy(), getattr(one, name).cpu().numpy()
        assert np.array_equal(x.view(np.uint32), y.view(np.uint32)), name
    want, shaped = oracle.rank(one.fit.cpu().numpy())
    assert np.array_equal(one.rank.cpu().numpy(), want)
    assert np.array_equal(one.shaped.cpu().numpy().view(np.uint32), shaped.view(np.uint32))


MANY_ROWS = [
    replace(NARROW, pop=1300, antithetic=0),
    replace(NARROW, pop=2602, obs=13, hid=29, act=7, noise_dtype=1),
    replace(NARROW, pop=1026, noise_dtype=2),
    replace(NARROW, pop=768),
    replace(NARROW, pop=770, noise_dtype=1),
    replace(NARROW, pop=385, antithetic=0, envs=11, noise_dtype=1),
    replace(NARROW, pop=1300, antithetic=0, obs=13, hid=29, act=7, noise_dtype=3),
]


@pytest.mark.parametrize("w", MANY_ROWS, ids=lambda w: f"N{w.pop}-nz{w.noise_dtype}")
def test_update_of_narrow_matrices_of_many_rows(es, w):  # noqa: F811
    ws = replace(w, noise_dtype=w.noise_dtype & 1)
    ctx, d, rng = es.EsContext(w), w.n_params, np.random.default_rng(w.pop)
    assert ctx.update_kernel.startswith("grad_")
    theta = (rng.standard_normal(d) * 0.1).astype(np.float32)
    m, v = np.zeros(d, dtype=np.float32), np.zeros(d, dtype=np.float32)
    th_d, m_d, v_d, g_d = dev(theta), dev(m), dev(v), torch.empty(d, device="cuda")
    wsp = ctx.alloc_workspace()
    for k in (1, 2):
        eps = oracle.sample_population(ws, k)
        _, shaped = oracle.rank(random_fitness(w.pop, seed=k, ties=True))
        theta, m, v, g = oracle.update(ws, k, eps, shaped, theta, m, v)
        if ctx.noise_regenerated:
            ctx.sample_population(k, None)
        ctx.update(k, None if ctx.noise_regenerated else noise_to_device(ctx, eps), dev(shaped), th_d, m_d, v_d, g_d, wsp)
        torch.cuda.synchronize()
        for got, ref, name in ((g_d, g, "grad"), (th_d, theta, "theta"), (m_d, m, "m"), (v_d, v, "v")):
            assert_params_close(got.cpu().numpy(), ref, f"step {k} {name}")


@pytest.mark.parametrize("n,b", [(2, 1), (126, 63), (128, 1), (130, 65), (510, 200), (512, 256), (514, 3)])
def test_ars_selection_edges(es, n, b):  # noqa: F811
    f = random_fitness(n, seed=n, ties=True)
    ctx = es.EsContext(replace(NARROW, pop=n, algorithm=1, num_elites=b))
    r, u = torch.empty(n, dtype=torch.int32, device="cuda"), torch.empty(n, device="cuda")
    ctx.rank(dev(f), r, u)
    torch.cuda.synchronize()
    want_r, want_u = oracle.rank_ars(f, b)
    assert np.array_equal(r.cpu().numpy(), want_r)
    assert np.allclose(u.cpu().numpy(), want_u, rtol=2e-6, atol=0)


@pytest.mark.parametrize("n,mu", [(1, 1), (63, 63), (64, 1), (65, 64), (511, 65), (512, 512), (513, 4)])
def test_vanilla_selection_edges(es, n, mu):  # noqa: F811
    f = random_fitness(n, seed=n, ties=n > 1)
    ctx = es.EsContext(replace(NARROW, pop=n, antithetic=0, algorithm=2, num_elites=mu))
    r, u = torch.empty(n, dtype=torch.int32, device="cuda"), torch.empty(n, device="cuda")
    ctx.rank(dev(f), r, u)
    torch.cuda.synchronize()
    want_r, want_u = oracle.rank_vanilla(f, mu)
    assert np.array_equal(r.cpu().numpy(), want_r)
    assert np.allclose(u.cpu().numpy(), want_u, rtol=2e-6, atol=0)
