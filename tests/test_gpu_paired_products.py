"""Layers that run as paired products (two rows of the matrix instruction a copy, bf16, more than one wavefront): hidden widths and observation widths on both sides
of every multiple of 64, where a K slice or a wavefront's tile is nearly empty or full, with one, two and four copies a pass - against the CPU checker."""
from dataclasses import replace

import pytest
import torch

from test_gpu_quad import B, _case, es  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("copies", [1, 2, 4])
@pytest.mark.parametrize("obs,hid,layers", [(9, 65, 2), (33, 127, 2), (27, 128, 2), (8, 129, 2), (64, 191, 2), (5, 193, 3), (40, 255, 3), (12, 66, 4), (65, 128, 2), (128, 129, 2), (129, 192, 2), (192, 256, 2), (193, 200, 2), (256, 256, 2),
                                            (66, 100, 1)])
def test_edges_of_the_widths(es, obs, hid, layers, copies):  # noqa: F811
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    # one copy a pass; too many for one, for two
    pop = 6 if copies == 1 else cus // 2 + 2 if copies == 2 else cus + 2
    w = replace(B, name=f"pairs-{obs}-{hid}x{layers}-{copies}", horizon=9, obs=obs, hid=hid, act=3 + obs % 5, num_hidden=layers, pop=pop, envs=copies, seed=811 + obs + hid)
    assert "quad_bf16" in _case(es, w).rollout_kernel
