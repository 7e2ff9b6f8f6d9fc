"""Which neighbours of the schedule go out in one launch, without a GPU (merge_host.cpp)."""
import os
import subprocess

import pytest

from paper_2506_06472_amd import binding, build
from test_gpu_train import MERGED

HERE = os.path.dirname(os.path.abspath(__file__))
ROCM = "/opt/rocm"


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    binding.lib()
    out = str(tmp_path_factory.mktemp("merge") / "host")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-D__HIP_PLATFORM_AMD__", f"-I{ROCM}/include", os.path.join(HERE, "merge_host.cpp"),
                    build.LIB, "-o", out, f"-Wl,-rpath,{os.path.dirname(build.LIB)}", "-Wl,--unresolved-symbols=ignore-in-shared-libs"], check=True)
    return out


def test_updates_of_one_launch_share_no_memory(program):
    r = subprocess.run([program, "independent"], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr)


OP_GEMM_DX, OP_ATTN_BWD_PRE, OP_ADAMW = 9, 16, 21


def _merged(program, cfg):
    """[(op of the first kernel, kernels, rows of the two output tiles)] of the launches of more than one kernel."""
    c = binding.model_cfg(cfg)
    args = [c.arch, c.n_layers, c.d_model, c.n_heads, c.d_ff, c.vocab, c.seq_len, c.batch, c.precision, c.micro_batches]
    r = subprocess.run([program, "launches", *map(str, args)], capture_output=True, text=True, timeout=60, check=True)
    return [(v[0], v[1], tuple(v[2:])) for v in (list(map(int, line.split())) for line in r.stdout.splitlines())]


def test_the_configurations_of_the_gpu_test_merge_what_they_are_there_for(program):
    tiles = set()
    for cfg in MERGED:
        out = _merged(program, cfg)
        ops = {op for op, _, _ in out}
        assert OP_ATTN_BWD_PRE in ops, cfg
        if cfg["arch"] == "gpt":                 # weights and norms with a bias beside them
            assert OP_ADAMW in ops, cfg
        if cfg["precision"] == "fp32":
            assert OP_GEMM_DX in ops, cfg
        tiles |= {t for op, _, t in out if op == OP_GEMM_DX}
    assert tiles == {(16, 16), (16, 32), (32, 16), (32, 32)}
