"""Host arithmetic of launches (csrc/launch_rules.h), compiled alone by the C++ compiler."""
import ctypes
import os
import subprocess

import pytest

SHIM = """
#include "launch_rules.h"
extern "C" int tokens_per_block(int bf16, int T, int E, int d, int cus) {
  return moe::route_tokens_per_block(bf16 != 0, T, E, d, cus);
}
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
    for E, d in ((1, 4), (8, 4096), (64, 128), (64, 1024), (64, 4096), (128, 1024), (256, 8), (256, 2 ** 20)):
        for T in sizes():
            tpb = rules.tokens_per_block(bf16, T, E, d, 256)
            assert tpb in (1, 2, 4, 8, 16)
            blocks = -(-T // tpb)
            assert blocks * 512 < 2 ** 32 and rules.launch_fits(blocks, 512), (T, tpb)
    assert not rules.launch_fits(2 ** 23, 512) and rules.launch_fits(2 ** 23 - 1, 512)


def test_tokens_per_block_of_the_per_tile_routing_kernel(rules):
    def tpb(bf16, T, E, d, cus=256):
        return rules.tokens_per_block(bf16, T, E, d, cus)

    # bf16: the fewest tokens per block that leave one block per compute unit; a full tile above
    for i in range(4):
        assert tpb(1, 256 << i, 8, 4096) == 1 << i and tpb(1, (256 << i) + 1, 8, 4096) == 2 << i
    assert tpb(1, 4096, 8, 4096) == tpb(1, 4097, 8, 4096) == 16
    assert tpb(1, 257, 8, 4096, 304) == 1
    # fp32: never more tokens on a compute unit than with one token per block
    for E, d in ((8, 128), (16, 1024), (24, 1024), (64, 128), (64, 1024), (64, 4096), (128, 1024), (256, 128)):
        for T in list(range(1, 4200, 7)) + [8192, 16384, 65536]:
            t = tpb(0, T, E, d)
            assert -(-(-(-T // t)) // 256) * t <= -(-T // 256), (E, d, T, t)
    # ... and more than one only where that was measured faster
    assert [tpb(0, T, 16, 128) for T in (512, 700, 1000, 1024, 2000, 2048, 3000, 6000, 8192)] == [1, 1, 2, 2, 4, 4, 2, 4, 16]
    assert [tpb(0, T, 16, 1024) for T in (512, 700, 1000, 2048, 3000, 8192)] == [1, 1, 2, 2, 2, 2]
    assert all(tpb(0, T, 24, 1024) == tpb(0, T, 64, 1024) == 1 for T in (512, 1000, 2048, 8192))
    assert [tpb(0, T, 128, 1024) for T in (300, 512, 1000, 2048, 4096, 8192)] == [2, 2, 4, 8, 16, 1]
    assert all(tpb(0, T, 128, 512) == 1 for T in (512, 1000, 2048, 8192))
    assert [tpb(0, T, 256, 128) for T in (256, 512, 1024, 8192)] == [1, 2, 4, 16]
