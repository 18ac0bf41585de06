"""Binary32 products of three-piece values, held so closely that one of the six partial products less would show: weights whose pieces are as large as they get and of one sign, units
that are all alike (their errors add up instead of averaging out), a linear output whose cost is nearly the whole return.  The kernel's arithmetic, emulated on the CPU, is within the tolerance,
and without any one term of any one matrix beyond it."""
from dataclasses import replace

import numpy as np
import pytest

import oracle
from gpu_util import dev, noise_to_device, run_rollout
from paper_2501_15129_amd.workloads import Workload, layer_shapes

W = Workload("terms", pop=1200, envs=16, horizon=5, obs=17, hid=48, act=5, dtype=0, noise_dtype=0, seed=901, sigma=0.01, out_tanh=0, act_cost=64.0, done_thresh=float("inf"))
SHOWN = 8      # individuals compared
# Relative root mean square over their episodes.  Emulated (below): 2.1e-7 to 5e-7, the short tanh of hundreds of equal units above all; with a term less 8e-7 at least.
RMS = 6.5e-7
# all the groupings of a lane's pairs and all tile counts; the last two do not fit the registers beside statistics
SHAPES = [(3, 16, 2), (16, 17, 9), (17, 48, 8), (20, 33, 16), (32, 64, 5), (33, 16, 3), (48, 48, 16), (64, 32, 12), (48, 60, 16), (64, 48, 4)]
CASES = [(*s, relu, norm) for s in SHAPES for relu in (0, 1) for norm in (0, 1) if not (norm and s in SHAPES[-2:])]


def _piecewise(x):
    """The nearest value below whose second and third piece are positive and nearly as large as they can be."""
    return ((np.float32(x).view(np.uint32) & np.uint32(0xFFFF0000)) | np.uint32(0x7EBF)).view(np.float32)


def _inputs(obs, hid, act, relu, norm):
    w = replace(W, name=f"terms-{obs}-{hid}-{act}", obs=obs, hid=hid, act=act, hidden_act=relu)
    full = lambda rows, cols, gain: np.full((rows, cols), _piecewise(gain / cols), np.float32)      # noqa: E731
    rng = np.random.default_rng(w.seed)
    theta, eps = [], []
    for k, shape in enumerate(layer_shapes(w)):
        theta.append((full(*shape, 1.0) if len(shape) == 2 else np.full(shape, 0.25 if k == 5 else 0.0, np.float32)).ravel())
        # individuals differ by their biases
        eps.append(np.repeat(rng.standard_normal((w.noise_rows, 1)) if len(shape) == 1 else np.zeros((w.noise_rows, 1)), theta[-1].size, axis=1))
    stats = (np.full(obs, 0.03, np.float32), np.full(obs, 1.25, np.float32)) if norm else None
    return w, full(obs, obs, 0.75), full(obs, act, 0.35), np.concatenate(theta), np.concatenate(eps, axis=1).astype(np.float32), stats


def _pieces(x):
    out, rest = [], np.asarray(x, np.float32)
    for _ in range(3):
        bits = rest.view(np.uint32)
        out.append(((bits + 0x7FFF + ((bits >> 16) & 1)) & np.uint32(0xFFFF0000)).view(np.float32))
        rest = rest - out[-1]
    return [p.astype(np.float64) for p in out]


def _tanh(z):
    f = np.float32
    u = np.exp2((z * f(2.88539008)).astype(np.float64)).astype(f) + f(1)
    return (1.0 - 2.0 * (1.0 / u.astype(np.float64)).astype(f).astype(np.float64)).astype(f)


def _emulate(w, a_mat, b_mat, theta, stats, without=(None, None)):
    parts, at = [], 0
    for shape in layer_shapes(w):
        parts.append(theta[at:at + int(np.prod(shape))].reshape(shape))
        at += parts[-1].size
    mats = dict(zip(("W1", "W2", "W3", "A", "B"), map(_pieces, (parts[0], parts[2], parts[4], a_mat, b_mat))))

    def product(name, x):
        q = _pieces(x)
        return sum(mats[name][i] @ q[j] for i, j in ((0, 0), (0, 1), (1, 0), (0, 2), (1, 1), (2, 0)) if without != (name, (i, j)))

    hidden = (lambda z: np.maximum(z, 0)) if w.hidden_act else _tanh
    s = np.stack([oracle.reset(w, 0, e) for e in range(w.envs)], axis=1)
    total = np.zeros(w.envs)
    for _ in range(w.horizon):
        h = s if stats is None else (s - stats[0][:, None]) * stats[1][:, None]
        for k, name in ((1, "W1"), (3, "W2")):
            h = hidden((product(name, h) + parts[k][:, None]).astype(np.float32))
        act = (product("W3", h) + parts[5][:, None]).astype(np.float32)
        total += 1 - (s.astype(np.float64) ** 2).mean(0) - w.act_cost * (act.astype(np.float64) ** 2).sum(0)
        s = _tanh((product("A", s) + product("B", act)).astype(np.float32))
    return total


def _rms(got, want):
    return float(np.sqrt(np.mean(((np.asarray(got, np.float64) - want) / want) ** 2)))


@pytest.mark.parametrize("obs,hid,act,relu,norm", CASES)
def test_a_term_less_shows(obs, hid, act, relu, norm):
    w, a_mat, b_mat, theta, eps, stats = _inputs(obs, hid, act, relu, norm)
    want = oracle.rollout(w, 0, theta, eps, a_mat, b_mat, individuals=(0, SHOWN), obs_norm=stats)[0].astype(np.float64)
    each = [oracle.perturb(w, theta, eps, i) for i in range(SHOWN)]
    off = lambda without: _rms([_emulate(w, a_mat, b_mat, t, stats, without) for t in each], want)      # noqa: E731
    assert off((None, None)) < 0.85 * RMS
    for name in ("W1", "W2", "W3", "A", "B"):
        for term in ((0, 2), (1, 1), (2, 0)):
            assert off((name, term)) > 1.15 * RMS, (name, term)


@pytest.mark.gpu
@pytest.mark.parametrize("obs,hid,act,relu,norm", CASES)
def test_every_term_counts(obs, hid, act, relu, norm):
    from paper_2501_15129_amd import EsContext
    w, a_mat, b_mat, theta, eps, stats = _inputs(obs, hid, act, relu, norm)
    ctx = EsContext(w)
    if norm:
        held = tuple(dev(v) for v in stats)
        ctx.set_obs_norm(*held)
    assert "rollout_mfma_cols_f32" in ctx.rollout_kernel
    ret, _, _ = run_rollout(ctx, w, 0, theta, noise_to_device(ctx, eps), a_mat, b_mat)
    want = oracle.rollout(w, 0, theta, eps, a_mat, b_mat, individuals=(0, SHOWN), obs_norm=stats)[0].astype(np.float64)
    assert _rms(ret[:SHOWN], want) <= RMS
