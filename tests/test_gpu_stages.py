"""GPU parity of es_sample_population, es_rank and es_update against the CPU checker,
called through the C boundary.  Integer / bit-defined outputs must match bit for bit."""
from dataclasses import replace

import numpy as np
import pytest
import torch

import oracle
from paper_2501_15129_amd.workloads import CONFIGS, Workload, random_fitness
from gpu_util import assert_params_close, dev, noise_from_device, noise_to_device

pytestmark = pytest.mark.gpu

SMALL = Workload("small", pop=8, envs=2, horizon=5, obs=3, hid=4, act=2, dtype=0, noise_dtype=0, seed=11)
# D = 1153 (ragged: 1153 = 4*288 + 1), several 256-thread blocks per row, bf16 noise
RAGGED = Workload("ragged", pop=12, envs=1, horizon=1, obs=13, hid=29, act=7, dtype=1, noise_dtype=1,
                  seed=(5 << 32) | 77)
MID = Workload("mid", pop=96, envs=1, horizon=1, obs=40, hid=96, act=9, dtype=0, noise_dtype=0, seed=3)


@pytest.fixture(scope="module")
def es():
    import paper_2501_15129_amd as pkg
    assert torch.cuda.is_available(), "these tests need the GPU"
    return pkg


def _sample(es, w, gen):
    ctx = es.EsContext(w)
    noise = ctx.alloc_noise()
    noise.fill_(7.0)
    ctx.sample_population(gen, noise)
    torch.cuda.synchronize()
    return ctx, noise


@pytest.mark.parametrize("w", [SMALL, RAGGED, MID, CONFIGS[0], CONFIGS[1],
                               replace(RAGGED, antithetic=0, noise_dtype=0),
                               replace(SMALL, pop=2)], ids=lambda w: w.name)
@pytest.mark.parametrize("gen", [0, 3, 2 ** 32 - 1])
def test_sample_population_bit_exact(es, w, gen):
    ctx, noise = _sample(es, w, gen)
    got = noise_from_device(ctx, noise)
    want = oracle.sample_population(w, gen)
    d = w.n_params
    assert got.shape == (w.noise_rows, ctx.noise_ld)
    assert np.array_equal(got[:, :d].view(np.uint32), want.view(np.uint32))
    assert np.all(got[:, d:] == 0.0)


def test_sample_population_more_rows_than_a_grid_dimension(es):
    """70 000 noise rows (more than the 65 535 workgroups one grid dimension holds): first, last and the rows
    around the limit against the checker."""
    w = Workload("many-rows", pop=140000, envs=1, horizon=1, obs=2, hid=3, act=1, dtype=0, noise_dtype=1, seed=31)
    ctx, noise = _sample(es, w, gen=4)
    for j in (0, 65534, 65535, 65536, 69999):
        want = oracle.sample_population(w, 4, rows=(j, j + 1))[0]
        got = noise[j].float().cpu().numpy()
        assert np.array_equal(got[: w.n_params].view(np.uint32), want.view(np.uint32)), j
        assert np.all(got[w.n_params:] == 0.0)
    del noise
    torch.cuda.empty_cache()


@pytest.mark.parametrize("idx", [3, 4])
def test_sample_population_full_size_sampled_rows(es, idx):
    """cfg3 (512 x 75264 bf16) and cfg4 (2048 x 133120 bf16) at full size: rows against the checker
    bit for bit, all rows finite."""
    w = CONFIGS[idx]
    ctx, noise = _sample(es, w, gen=1)
    for j in (0, 1, 2, 3, w.noise_rows // 3, w.noise_rows // 2, w.noise_rows - 2, w.noise_rows - 1):
        want = oracle.sample_population(w, 1, rows=(j, j + 1))[0]
        got = noise[j].float().cpu().numpy()
        assert np.array_equal(got[: w.n_params].view(np.uint32), want.view(np.uint32))
        assert np.all(got[w.n_params:] == 0.0)
    assert bool(torch.isfinite(noise.float().abs().max()))
    # column moments over the whole matrix: a property that holds at any size
    col_mean = noise[:, : w.n_params].float().mean(dim=0)
    assert float(col_mean.abs().max()) < 6.0 / np.sqrt(w.noise_rows)
    del noise
    torch.cuda.empty_cache()


@pytest.mark.parametrize("n,ties", [(2, False), (8, True), (16, False), (254, True), (4096, True), (5000, False), (9001, True)])
def test_rank_bit_exact(es, n, ties):
    w = replace(SMALL, pop=n, antithetic=0)
    ctx = es.EsContext(w)
    f = random_fitness(n, seed=n, ties=ties)
    if n >= 16:
        f[3], f[5], f[7], f[9] = np.inf, -np.inf, 0.0, -0.0
    r = torch.full((n,), -1, dtype=torch.int32, device="cuda")
    u = torch.full((n,), float("nan"), dtype=torch.float32, device="cuda")
    ctx.rank(dev(f), r, u)
    torch.cuda.synchronize()
    want_r, want_u = oracle.rank(f)
    assert np.array_equal(r.cpu().numpy(), want_r)
    assert np.array_equal(u.cpu().numpy().view(np.uint32), want_u.view(np.uint32))


def test_rank_nan_and_constant(es):
    for f in (np.array([1.0, np.nan, -3.0, np.nan, 2.0, -np.inf], dtype=np.float32), np.full(10, 2.5, dtype=np.float32)):
        w = replace(SMALL, pop=f.size)
        ctx = es.EsContext(w)
        r = torch.empty(f.size, dtype=torch.int32, device="cuda")
        u = torch.empty(f.size, dtype=torch.float32, device="cuda")
        ctx.rank(dev(f), r, u)
        torch.cuda.synchronize()
        want_r, want_u = oracle.rank(f)
        assert np.array_equal(r.cpu().numpy(), want_r) and np.array_equal(u.cpu().numpy(), want_u)


def _update_case(es, w, steps, seed):
    rng = np.random.default_rng(seed)
    ctx = es.EsContext(w)
    d = w.n_params
    theta = (rng.standard_normal(d) * 0.1).astype(np.float32)
    theta[rng.integers(0, d, size=max(1, d // 10))] = 0.0          # biases start at zero in the workloads
    m = np.zeros(d, dtype=np.float32)
    v = np.zeros(d, dtype=np.float32)
    th_d, m_d, v_d = dev(theta), dev(m), dev(v)
    g_d = torch.empty(d, dtype=torch.float32, device="cuda")
    ws = ctx.alloc_workspace()
    for k in range(1, steps + 1):
        eps = oracle.sample_population(w, gen=k)
        _, shaped = oracle.rank(random_fitness(w.pop, seed=seed + k, ties=True))
        theta, m, v, g = oracle.update(w, k, eps, shaped, theta, m, v)
        ctx.update(k, noise_to_device(ctx, eps), dev(shaped), th_d, m_d, v_d, g_d, ws)
        torch.cuda.synchronize()
        assert_params_close(g_d.cpu().numpy(), g, f"{w.name} step {k} grad")
        assert_params_close(th_d.cpu().numpy(), theta, f"{w.name} step {k} theta")
        assert_params_close(m_d.cpu().numpy(), m, f"{w.name} step {k} m")
        assert_params_close(v_d.cpu().numpy(), v, f"{w.name} step {k} v")
        # the moments and parameters are binary64 results rounded once: expect (near) bit equality
        assert np.mean(th_d.cpu().numpy() == theta) > 0.999


@pytest.mark.parametrize("w", [SMALL, RAGGED, MID, CONFIGS[0], CONFIGS[1], CONFIGS[2],
                               replace(MID, antithetic=0, weight_decay=0.0),
                               replace(RAGGED, pop=2), replace(MID, pop=1024, noise_dtype=1)],
                         ids=lambda w: f"{w.name}-N{w.pop}-a{w.antithetic}")
def test_update_matches_checker(es, w):
    _update_case(es, w, steps=3, seed=w.pop)


def test_update_grad_pointer_optional_and_rerun_identical(es):
    w = MID
    ctx = es.EsContext(w)
    d = w.n_params
    eps = oracle.sample_population(w, 0)
    _, shaped = oracle.rank(random_fitness(w.pop, 1))
    outs = []
    for _ in range(2):
        th, m, v = (torch.zeros(d, device="cuda") for _ in range(3))
        th += 0.25
        ctx.update(1, noise_to_device(ctx, eps), dev(shaped), th, m, v, None, ctx.alloc_workspace())
        torch.cuda.synchronize()
        outs.append((th.cpu().numpy(), m.cpu().numpy(), v.cpu().numpy()))
    for a, b in zip(*outs):
        assert np.array_equal(a.view(np.uint32), b.view(np.uint32))


@pytest.mark.parametrize("idx", [3, 4])
def test_update_full_size(es, idx):
    """cfg3 (one-launch kernel, 512 rows x 75 016 parameters) and cfg4 (chunked stream, 2048 rows x
    132 881 parameters) at full size: GPU-sampled noise (bit-equal to the checker's, see the sampling test),
    checker-side update over every parameter from the checker's own matrix."""
    w = CONFIGS[idx]
    assert ("single_pass" in es.EsContext(w).update_kernel) == (idx == 3)
    ctx, noise = _sample(es, w, gen=2)
    d = w.n_params
    rng = np.random.default_rng(4)
    theta = (rng.standard_normal(d) * 0.05).astype(np.float32)
    m = (rng.standard_normal(d) * 0.01).astype(np.float32)
    v = (rng.random(d) * 1e-3).astype(np.float32)
    _, shaped = oracle.rank(random_fitness(w.pop, 9, ties=True))
    eps = oracle.sample_population(w, 2)                       # independent of the GPU matrix
    want = oracle.update(w, 5, eps, shaped, theta, m, v)
    th_d, m_d, v_d = dev(theta), dev(m), dev(v)
    g_d = torch.empty(d, dtype=torch.float32, device="cuda")
    ctx.update(5, noise, dev(shaped), th_d, m_d, v_d, g_d, ctx.alloc_workspace())
    torch.cuda.synchronize()
    for got, ref, name in ((th_d, want[0], "theta"), (m_d, want[1], "m"), (v_d, want[2], "v"), (g_d, want[3], "grad")):
        assert_params_close(got.cpu().numpy(), ref, f"{w.name} {name}")
    del noise
    torch.cuda.empty_cache()
