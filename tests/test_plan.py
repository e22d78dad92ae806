"""The launch choices of csrc/plan.h, which are pure functions of sizes and compute units: compiled here with the host
compiler and called at sizes on both sides of where one shape was measured faster than the other. No choice changes a
result, so the parity tests cannot see a wrong one."""

import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2605_14220_amd", "csrc")
CUS = 256  # an MI355X

SHIM = """
#include "plan.h"
extern "C" int response_blocks(int term, int64_t T, int64_t n_seq, int64_t cus) {
  return tim::response_blocks((tim::ResponseTerm)term, T, n_seq, cus);
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "shim.cpp").write_text(SHIM)
    so = str(d / "plan.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, "-o", so,
                    str(d / "shim.cpp")], check=True)
    lib = ctypes.CDLL(so)
    lib.response_blocks.argtypes = [ctypes.c_int] + [ctypes.c_int64] * 3
    return lib


K1, K3, PPO = 0, 1, 2


@pytest.mark.parametrize("term", [K1, K3, PPO])
@pytest.mark.parametrize("n", [513, 1024, 8192, 20000, 1 << 22])
@pytest.mark.parametrize("mean", [100, 550, 1100, 6000, 16384])
def test_many_responses_take_one_block(plan, term, n, mean):
    """More than two responses per CU: four blocks of threads each were 1.3 to 4 times slower at every length."""
    assert plan.response_blocks(term, n * mean, n, CUS) == 1


@pytest.mark.parametrize("term,n,mean,want", [
    (K3, 64, 512, 1), (K3, 256, 1300, 1), (K3, 256, 1600, 4), (K3, 1, 16384, 4),
    (K3, 257, 4096, 1), (K3, 512, 6000, 4),
    (K1, 256, 2048, 1), (K1, 256, 3072, 4), (K1, 512, 6000, 1), (K1, 512, 8192, 4),
    (PPO, 256, 1024, 1), (PPO, 200, 1300, 4), (PPO, 64, 1600, 4), (PPO, 512, 6000, 1), (PPO, 257, 8192, 4),
])
def test_long_responses_take_four_blocks_where_they_pay(plan, term, n, mean, want):
    assert plan.response_blocks(term, n * mean, n, CUS) == want
