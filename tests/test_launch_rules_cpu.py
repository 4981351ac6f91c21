"""Host arithmetic of launches (csrc/launch_rules.h), compiled alone by the C++ compiler."""
import ctypes
import os
import subprocess

import pytest

SHIM = """
#include "launch_rules.h"
extern "C" int tokens_per_block(int bf16, int T) { return moe::route_tokens_per_block(bf16 != 0, T); }
extern "C" int launch_fits(int64_t blocks, int threads) { return moe::launch_fits(blocks, threads); }
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory, repo_root):
    folder = tmp_path_factory.mktemp("rules")
    (folder / "shim.cpp").write_text(SHIM)
    csrc = os.path.join(repo_root, "paper_2603_06350_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I", csrc, "shim.cpp", "-o", "shim.so"],
                   cwd=folder, check=True)
    lib = ctypes.CDLL(str(folder / "shim.so"))
    lib.launch_fits.argtypes = [ctypes.c_int64, ctypes.c_int]
    return lib


def sizes():
    near = sorted({max(1, 2 ** b + o) for b in range(28) for o in (-16, -15, -1, 0, 1)})
    return [t for t in near if t <= 2 ** 27 - 16]


@pytest.mark.parametrize("bf16", [0, 1])
def test_every_batch_of_the_per_tile_routing_kernel_fits_one_launch(rules, bf16):
    # HIP: gridDim.x * blockDim.x < 2^32, and the kernel has 512 threads and 16 token rows
    for T in sizes():
        tpb = rules.tokens_per_block(bf16, T)
        assert tpb in (1, 2, 4, 8, 16)
        blocks = -(-T // tpb)
        assert blocks * 512 < 2 ** 32 and rules.launch_fits(blocks, 512), (T, tpb)
    assert not rules.launch_fits(2 ** 23, 512) and rules.launch_fits(2 ** 23 - 1, 512)
