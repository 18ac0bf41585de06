"""Build the HIP library for gfx950 in-tree (hipcc cross-compiles without a GPU)."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor
from pathlib import Path

HERE = Path(__file__).resolve().parent
CSRC = HERE / "csrc"
LIB = HERE / "libes_hip.so"
MICRO_LIB = HERE / "libes_microbench.so"
# (the longest compilations first)
SOURCES = ["rollout_quad_f32_mid.hip", "rollout_mfma.hip", "rollout_quad_bf16_mid4.hip", "rollout_quad_bf16_deep4.hip", "rollout_quad_f32_wide.hip",
           "rollout_quad_bf16_mid3.hip", "rollout_quad_bf16_deep3.hip", "rollout_quad_bf16_wide.hip", "rollout_quad_bf16_mid.hip",
           "rollout_wave_reg_deep.hip", "rollout_wave_team_f32.hip", "rollout_wave_team_bf16.hip", "rollout_quad_obs256.hip", "rollout_quad_obs192.hip", "rollout_quad_obs128.hip",
           "rollout_single_mid.hip", "rollout_single_wide.hip", "rollout_cols_f32_64.hip", "rollout_cols_f32_48.hip", "rollout_cols_f32_small.hip", "rollout_cols_bf16.hip",
           "rollout_quad_narrow.hip", "rollout_wave_reg_bf16.hip", "rollout_wave_reg_f32.hip",
           "rollout_mfma_f32.hip", "rollout_wave_reg.hip", "api.hip", "sample.hip", "rank.hip", "update.hip", "rollout_wave.hip",
           "rollout_quad.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
    "-fhip-fp32-correctly-rounded-divide-sqrt",
    # packed-FP32 instructions are kept out of the generated code on purpose
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # MFMA accumulators in architectural VGPRs: the accumulation-register half of the file is
    # reserved for the register-resident policy weights of the rollout kernel
    "-mllvm", "-amdgpu-mfma-vgpr-form",
    "-Wall", "-Wno-unused-command-line-argument",
]


def _compile(src: str) -> Path:
    obj = CSRC / (Path(src).stem + ".o")
    extra = os.environ.get("ES_EXTRA_HIPCC_FLAGS", "").split()      # tuning experiments only
    cmd = [HIPCC, *FLAGS, *extra, "-c", str(CSRC / src), "-o", str(obj)]
    subprocess.check_call(cmd, cwd=str(CSRC))
    return obj


def build(verbose: bool = True) -> Path:
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB.with_suffix(f".tmp{os.getpid()}.so")
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", str(tmp), *map(str, objs)])
    os.replace(tmp, LIB)
    # rate micro-benchmarks (bench.py --peaks) and the Gaussian transform on given words: a library of their own, not part of the boundary
    tmp = MICRO_LIB.with_suffix(f".tmp{os.getpid()}.so")
    micro = [CSRC / "microbench.o", _compile("gauss_words.hip")]      # (the transform is compiled with the product's flags)
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Xclang", "-target-feature", "-Xclang",
                           "-packed-fp32-ops", "-Wall", "-Wno-unused-command-line-argument", "-c", str(CSRC / "microbench.hip"), "-o", str(micro[0])])
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", str(tmp), *map(str, micro)])
    os.replace(tmp, MICRO_LIB)
    if verbose:
        print(f"built {LIB} and {MICRO_LIB}", file=sys.stderr)
    return LIB


if __name__ == "__main__":
    build()
