"""The four-copy rollout kernels in passes of two and four copies, which populations that do not fit the chip one copy a pass run in, and the placement
of two-wavefront workgroups where two share a compute unit: ragged passes, both activations, state rows spread over the wavefronts, statistics, early
ends - against the CPU checker."""
from dataclasses import replace

import pytest

from test_gpu_quad import B, F, _case, es  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pop,envs,kw", [
    # 65 to 128 units: 257 to 512 workgroups of two copies, 260 and 600 of four
    (100, 7, dict(hid=100)), (260, 2, dict(hid=128, hidden_act=1, obs=60)), (60, 9, dict(hid=65, num_hidden=1, done_thresh=0.5)), (100, 6, dict(hid=100, noise_dtype=3, out_tanh=0)),
    (130, 8, dict(hid=100)), (130, 7, dict(hid=127, hidden_act=1, done_thresh=0.5)), (130, 5, dict(hid=90, num_hidden=1, obs=64)), (300, 8, dict(hid=70)), (66, 13, dict(hid=100, obs=100, act=20)),
    (130, 3, dict(hid=100, obs=70, act=17, done_thresh=0.5)), (514, 1, dict(hid=100)), (270, 1, dict(hid=80, num_hidden=1)), (256, 2, dict(hid=128, episodes=2)),
    # ... state rows spread over the wavefronts: one copy, two, four
    (20, 4, dict(hid=100, obs=128, act=32)), (300, 1, dict(hid=65, obs=65, act=3, done_thresh=0.5)), (100, 6, dict(hid=128, obs=90, act=17, hidden_act=1)), (200, 3, dict(hid=100, obs=127, num_hidden=1, done_thresh=0.5)),
    (300, 4, dict(hid=100, obs=128, act=32)), (300, 3, dict(hid=128, obs=65, act=5, num_hidden=1, done_thresh=0.5)), (514, 1, dict(hid=90, obs=100)),
    # 129 to 256 units: two copies, four
    (40, 7, dict()), (40, 8, dict(obs=50, hidden_act=1, done_thresh=0.5)), (300, 2, dict(num_hidden=1, hid=200)), (70, 4, dict()), (70, 3, dict(hid=150, obs=40, done_thresh=0.5)),
    (100, 3, dict(num_hidden=3, hid=100, obs=50, done_thresh=0.5)), (300, 4, dict(num_hidden=3)), (300, 3, dict(num_hidden=3, hid=90, hidden_act=1)),
    (70, 4, dict(num_hidden=3)), (70, 4, dict(num_hidden=4, hidden_act=1)), (70, 4, dict(num_hidden=3, hid=90, done_thresh=0.5)), (70, 3, dict(num_hidden=4, hid=90))], ids=str)
def test_bf16(es, pop, envs, kw):  # noqa: F811
    w = replace(B, name=f"copies-{pop}x{envs}", horizon=14, **{"pop": pop, "envs": envs, "seed": 411 + pop + envs, **kw})
    assert "quad_bf16" in _case(es, w).rollout_kernel


@pytest.mark.parametrize("pop,envs,kw", [(100, 7, dict(hid=100)), (10, 4, dict(hid=100, obs=70, act=17)), (90, 6, dict(hid=80, obs=128, act=30, num_hidden=1)), (300, 4, dict(hid=90, obs=100, act=20)), (40, 8, dict(hidden_act=1, obs=40)), (130, 8, dict(hid=100, obs=40)), (66, 13, dict(hid=120, obs=100, act=20)), (70, 4, dict(num_hidden=3))], ids=str)
def test_bf16_statistics(es, pop, envs, kw):  # noqa: F811
    _case(es, replace(B, name=f"copies-norm-{pop}x{envs}", horizon=10, pop=pop, envs=envs, **kw), norm=True)


@pytest.mark.parametrize("pop,envs,kw", [(100, 7, dict(hid=100)), (130, 8, dict(hid=128, hidden_act=1, obs=50)), (300, 2, dict(hid=80, num_hidden=3)), (70, 4, dict(obs=50)), (70, 8, dict(num_hidden=1, hid=200, done_thresh=0.5)),
                                         (600, 1, dict(hid=100, num_hidden=1)), (130, 4, dict(obs=20, done_thresh=0.5))], ids=str)
def test_f32(es, pop, envs, kw):  # noqa: F811
    w = replace(F, name=f"copies-f32-{pop}x{envs}", horizon=14, pop=pop, envs=envs, seed=511 + pop + envs, **kw)
    assert "quad_f32" in _case(es, w).rollout_kernel
