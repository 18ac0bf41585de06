"""The four-copy rollout kernel with 65 to 256 observations and up to 32 actions, the state rows spread over four wavefronts: edges of the width classes,
one, two and four copies a pass, passes side by side, both activations, statistics, early ends, more individuals than the chip holds - against the
CPU checker."""
from dataclasses import replace

import pytest
import torch

from test_gpu_quad import B, _case, es  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


def kernel(family, obs, classes):
    return f"rollout_mfma_{family}_bf16<obs{next(c for c in classes if obs <= c)},hid256,act32>"



CASES = [(65, 17, 8, 1, dict()), (128, 32, 300, 3, dict(done_thresh=0.5)), (129, 1, 300, 4, dict(hidden_act=1)), (130, 20, 16, 7, dict(hid=128)), (192, 32, 130, 2, dict(hid=200, out_tanh=0)),
         (193, 18, 300, 2, dict(done_thresh=0.5)), (244, 17, 300, 4, dict()), (255, 31, 70, 4, dict(hid=129, done_thresh=0.5)), (256, 32, 40, 8, dict(hidden_act=1)), (256, 3, 258, 1, dict(noise_dtype=3)),
         (250, 9, 6, 13, dict(done_thresh=0.5)), (100, 5, 66, 3, dict(episodes=2, hid=256)), (64, 17, 70, 4, dict()), (16, 32, 12, 4, dict(done_thresh=0.5))]


@pytest.mark.parametrize("obs,act,pop,envs,kw", CASES, ids=str)
def test_wide_observations(es, obs, act, pop, envs, kw):  # noqa: F811
    w = replace(B, name=f"wideobs-{obs}-{act}-{pop}x{envs}", horizon=12, **{"obs": obs, "act": act, "pop": pop, "envs": envs, "hid": 256, "seed": 611 + obs + envs, **kw})
    assert _case(es, w).rollout_kernel == kernel("quad", obs, (128, 192, 256))


@pytest.mark.parametrize("obs,act,pop,envs,kw", [(65, 17, 300, 4, dict()), (160, 32, 40, 3, dict(hidden_act=1)), (244, 17, 130, 2, dict(done_thresh=0.5)), (256, 8, 10, 1, dict())], ids=str)
def test_statistics(es, obs, act, pop, envs, kw):  # noqa: F811
    w = replace(B, name=f"wideobs-norm-{obs}-{pop}x{envs}", horizon=10, obs=obs, act=act, pop=pop, envs=envs, hid=256, **kw)
    assert _case(es, w, norm=True).rollout_kernel == kernel("quad", obs, (128, 192, 256))


@pytest.mark.parametrize("obs,act,pop,envs,kw,norm", [(100, 17, 130, 9, dict(), False), (128, 32, 90, 16, dict(hidden_act=1), False), (65, 3, 130, 5, dict(done_thresh=0.5), True),
                                                      (244, 17, 130, 9, dict(), False), (200, 32, 70, 18, dict(done_thresh=0.5), False), (256, 20, 130, 6, dict(hidden_act=1), True)], ids=str)
def test_sixteen_columns(es, obs, act, pop, envs, kw, norm):  # noqa: F811
    """more than four copies, and more passes of four than compute units: the 16-column kernel of the same widths"""
    assert pop * ((envs + 3) // 4) > torch.cuda.get_device_properties(0).multi_processor_count
    w = replace(B, name=f"wideobs-16-{obs}-{pop}x{envs}", horizon=8, obs=obs, act=act, pop=pop, envs=envs, hid=256, seed=711 + obs, **kw)
    assert _case(es, w, norm=norm).rollout_kernel == kernel("reg", obs, (128, 256))
