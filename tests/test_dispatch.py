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


@pytest.mark.parametrize("kw,name", [
    (dict(), "rollout_single_f32<obs32,hid256,act16>"),
    (dict(obs=16, envs=16, pop=16), "rollout_single_f32<obs20,hid256,act16>"),
    (dict(obs=12, pop=512), "rollout_single_f32<obs12,hid256,act16>"),
    (dict(obs=33, hid=128, num_hidden=3), "rollout_single_f32<obs64,hid128,act16>,depth3"),
    (dict(envs=4), "rollout_mfma_quad_f32<obs32,hid256,act16>"),
    (dict(obs=16, pop=128, envs=3), "rollout_mfma_quad_f32<obs16,hid256,act16>"),
    (dict(obs=33), "rollout_mfma_quad_f32<obs64,hid256,act16>"),
    (dict(envs=16), "rollout_mfma_reg_f32<obs32,hid256,act16>"),
    (dict(envs=16, hid=128), "rollout_mfma_quad_f32<obs32,hid128,act16>"),
    (dict(hid=64, obs=17, act=6), "rollout_wave_reg_team_f32<obs<=20,hid<=64,act<=6>"),
    (dict(hid=64, obs=17, act=6, pop=258), "rollout_wave_reg_f32<17,64,6>"),
    (dict(hid=64, obs=17, act=6, envs=8, pop=512), "rollout_mfma_quad_f32<obs32,hid64,act16>"),
    (dict(hid=64, obs=17, act=6, envs=16, pop=1000), "rollout_mfma_cols_f32<obs20,hid64,act8>"),
    (dict(hid=30, obs=40, act=9, envs=16, pop=1000), "rollout_mfma_cols_f32<obs48,hid32,act16>"),
    (dict(hid=20, envs=16, pop=1000, dtype=1, noise_dtype=1), "rollout_mfma_cols_bf16<obs32,hid32,act16>"),
    (dict(hid=64, obs=17, act=6, num_hidden=3), "rollout_wave_reg_team_f32<obs<=20,hid<=64,act<=6>,depth3"),
    (dict(hid=64, obs=17, act=6, num_hidden=3, pop=258), "rollout_wave_reg_f32<obs<=32,hid<=64,act<=8>,depth3"),
    (dict(hid=40, obs=50, num_hidden=4, pop=512, dtype=1, noise_dtype=1), "rollout_wave_reg_team_bf16<obs<=64,hid<=64,act<=8>,depth4"),
    (dict(hid=24, num_hidden=5), "rollout_wave_lds_f32"),
    (dict(obs=70, hid=100), "rollout_wave_lds_f32"),
    (dict(dtype=1, noise_dtype=1, hid=48, num_hidden=1), "rollout_wave_reg_bf16<obs<=32,hid<=64,act<=8>,depth1"),
    (dict(dtype=1, noise_dtype=1, hid=100, obs=70), "rollout_mfma_quad_bf16<obs128,hid128,act32>"),
    (dict(dtype=1, noise_dtype=1, num_hidden=3), "rollout_mfma_quad_bf16<obs32,hid256,act16>,depth3"),
    (dict(dtype=1, noise_dtype=1, envs=16, pop=512, num_hidden=3), "rollout_mfma_reg_bf16<obs32,hid256,act16>,depth3"),
    (dict(dtype=1, noise_dtype=1, envs=4, obs=244, act=17), "rollout_mfma_quad_bf16<obs256,hid256,act32>"),
    (dict(dtype=1, noise_dtype=1, envs=4, obs=129), "rollout_mfma_quad_bf16<obs192,hid256,act32>"),
    (dict(dtype=1, noise_dtype=1, envs=16, obs=40, act=17, pop=64), "rollout_mfma_quad_bf16<obs128,hid256,act32>"),
    (dict(dtype=1, noise_dtype=1, envs=16, obs=244, act=17), "rollout_mfma_reg_bf16<obs256,hid256,act32>"),
    (dict(dtype=1, noise_dtype=1, env_dtype=1), "rollout_mfma_reg_bf16<obs32,hid256,act16>,env_f32"),
    (dict(dtype=1, noise_dtype=1, obs=70, hid=40), "rollout_wave_lds_bf16"),
], ids=lambda v: v if isinstance(v, str) else "")
def test_the_name_is_that_of_the_kernel(kernel, kw, name):
    assert kernel(replace(F32, **kw)) == name


@pytest.mark.parametrize("layers", [3, 4])
@pytest.mark.parametrize("hid", [65, 96, 127])
@pytest.mark.parametrize("pop,envs", [(200, 5), (512, 16), (256, 20), (128, 4), (64, 16), (2, 21)])
def test_three_and_four_middle_layers_stay_on_the_matrix_cores(kernel, layers, hid, pop, envs):
    """bf16 policies of 65..127 units with three or four hidden layers: a matrix-core kernel holds them whatever the number of passes."""
    assert "mfma" in kernel(replace(F32, dtype=1, noise_dtype=1, hid=hid, num_hidden=layers, pop=pop, envs=envs))


@pytest.mark.parametrize("hid", [100, 200, 256])
@pytest.mark.parametrize("obs,envs,name", [(32, 4, "quad"), (33, 4, "reg"), (64, 16, "reg"), (33, 2, "reg"), (64, 1, "quad")])
def test_four_layers_of_several_copies_and_wide_observations_run_in_sixteen_columns(kernel, hid, obs, envs, name):
    """The four-copy kernel spills there; the 16-column kernel is 10 to 17 % faster."""
    assert f"rollout_mfma_{name}_bf16" in kernel(replace(F32, dtype=1, noise_dtype=1, num_hidden=4, pop=32, hid=hid, obs=obs, envs=envs))


@pytest.mark.parametrize("kw,name", [(dict(), "reg"), (dict(envs=13), "reg"), (dict(envs=12), "quad"), (dict(envs=32), "reg"), (dict(pop=510), "quad"), (dict(obs=33), "quad"), (dict(hid=127), "quad"),
                                     (dict(act=17), "quad"), (dict(envs=8, episodes=2), "reg")], ids=str)
@pytest.mark.parametrize("layers", [1, 2])
def test_128_units_on_full_columns(kernel, layers, kw, name):
    w = replace(F32, dtype=1, noise_dtype=1, num_hidden=layers, pop=512, hid=128, envs=16)
    assert f"rollout_mfma_{name}_bf16" in kernel(replace(w, **kw))


@pytest.mark.parametrize("kw,split", [
    (dict(pop=766), False), (dict(pop=768), True), (dict(pop=512, antithetic=0), False), (dict(pop=514, antithetic=0), True), (dict(pop=384, antithetic=0, envs=10), False),
    (dict(pop=384, antithetic=0, envs=11), True), (dict(pop=512, antithetic=0, algorithm=2, num_elites=5), True), (dict(pop=768, obs=120, hid=128, act=17), False),
    (dict(pop=2048, obs=64, hid=128, act=17), True), (dict(pop=8, obs=64, hid=128), False)], ids=str)
def test_rows_of_the_update_are_split_where_it_pays(kw, split):
    """From 384 rows on and below 120 column tiles, unless fitness, ranks and update are one launch."""
    from paper_2501_15129_amd.binding import EsContext
    ctx = EsContext(replace(replace(F32, obs=17, hid=64, act=6), **kw))
    assert ctx.update_kernel == ("grad_partial_kernel+adam_kernel" if split else "update_single_pass_kernel")


@pytest.mark.parametrize("kw,without,with_stats", [
    (dict(obs=45, hid=52, act=4, pop=614, envs=5), "mfma_cols_f32<obs48,hid64,act8>", "wave_reg_f32<obs<=64,hid<=64,act<=4>"),
    (dict(obs=63, hid=48, act=4, pop=1064, envs=5), "mfma_cols_f32<obs64,hid48,act8>", "wave_reg_f32<obs<=64,hid<=64,act<=4>"),
    (dict(obs=38, hid=56, act=12, pop=578, envs=10), "mfma_cols_f32<obs48,hid64,act16>", "mfma_cols_f32<obs48,hid64,act16>"),
    (dict(obs=48, hid=48, act=4, pop=614, envs=5), "mfma_cols_f32<obs48,hid48,act8>", "mfma_cols_f32<obs48,hid48,act8>")], ids=str)
def test_statistics_have_a_choice_of_their_own(kw, without, with_stats):
    """Where the three-piece products do not fit beside statistics, sixteen columns are counted as what runs there then, the binary32 shape; back without statistics the first choice holds again."""
    from paper_2501_15129_amd.binding import EsContext, _lib
    ctx = EsContext(replace(F32, **kw))
    name = lambda: _lib.es_rollout_kernel(ctx._h).decode().replace("rollout_", "")      # noqa: E731
    assert name() == without
    for ptr, expected in ((1 << 20, with_stats), (None, without)):      # (the call is host-side: the pointers are not followed)
        assert _lib.es_set_obs_norm(ctx._h, ptr, ptr) == 0
        assert name() == expected


@pytest.mark.parametrize("kw,name", [
    (dict(obs=26, hid=19, act=5, pop=1456, envs=4), "wave_reg_f32<obs<=32,hid<=32,act<=8>"), (dict(obs=24, hid=8, act=16, pop=1922, envs=2), "wave_reg_f32<obs<=32,hid<=16,act<=16>"),
    (dict(obs=26, hid=19, act=5, pop=1456, envs=8), "mfma_cols_f32<obs32,hid32,act8>"), (dict(obs=26, hid=19, act=5, pop=1456, envs=4, hidden_act=1), "mfma_cols_f32<obs32,hid32,act8>")], ids=str)
def test_several_column_wavefronts_on_a_simd(kernel, kw, name):
    """Two or three wavefronts of sixteen copies on a SIMD take 0.88 (tanh) of two or three times one's time: a few copies each stay in one wavefront an episode."""
    assert kernel(replace(F32, **kw)) == "rollout_" + name
