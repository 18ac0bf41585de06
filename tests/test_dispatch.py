"""Which rollout kernel a configuration is given (es_create decides on the host, so no GPU is needed)."""
from dataclasses import replace

import pytest

from paper_2501_15129_amd.workloads import Workload

F32 = Workload("dispatch-f32", pop=128, envs=1, horizon=10, obs=27, hid=256, act=8, dtype=0, noise_dtype=0, seed=1)


@pytest.fixture(scope="module")
def kernel():
    from paper_2501_15129_amd.binding import EsContext

    def name(w):
        ctx = EsContext(w)
        try:
            return ctx.rollout_kernel
        finally:
            ctx.close()
    return name


@pytest.mark.parametrize("obs,hid,act,envs,layers,pop", [
    (27, 256, 8, 1, 1, 128), (27, 256, 8, 16, 1, 512), (8, 256, 2, 4, 2, 128), (64, 200, 16, 8, 2, 128), (27, 256, 8, 16, 2, 512),
    (20, 100, 5, 3, 3, 64), (17, 64, 6, 16, 2, 1000), (17, 64, 6, 1, 2, 16), (70, 40, 9, 2, 2, 16)])
def test_env_dtype_counts_with_bf16_operands_only(kernel, obs, hid, act, envs, layers, pop):
    """A binary32 context is binary32 throughout whatever env_dtype says, so the field must not move it to another kernel."""
    w = replace(F32, obs=obs, hid=hid, act=act, envs=envs, num_hidden=layers, pop=pop)
    assert kernel(replace(w, env_dtype=1)) == kernel(w)
