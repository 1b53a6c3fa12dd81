"""The consistency guard of the one-wavefront kernels (rkc_guard.h), compiled for the host: an eviction loop
whose pass takes nothing still ends, and the pool's blocks then no longer add up, which the kernels report as
RKC_PS_INTERNAL."""
import ctypes
import os
import re
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_24259_amd", "csrc")
SOURCE = r"""
#include "rkc_guard.h"
// an active request of `need` blocks in a pool of U blocks, F free, PR protected and E evictable, served by an
// eviction loop whose passes take at most take[i] blocks (1 each from there on): {passes, adds up}
extern "C" void serve(uint32_t U, uint32_t F, uint32_t E, uint32_t PR, uint32_t need, const uint32_t* take, int n, uint32_t* out) {
  uint32_t K = need > F ? need - F : 0u, A = U - F - E - PR;
  F = need > F ? 0u : F - need;
  int i = 0;
  for (; K > 0; i++) {
    const uint32_t run = i < n ? take[i] : 1u, m = K < run ? K : run;
    E -= m;
    K = rkc_left(K, m);
  }
  A += need;
  out[0] = (uint32_t)i;
  out[1] = rkc_adds_up(U, F, A, E + PR);
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("guard")
    src, so = d / "guard.cpp", d / "libguard.so"
    src.write_text(SOURCE)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(so)])
    return ctypes.CDLL(str(so))


@pytest.mark.parametrize("need,take,passes,adds_up", [
    (5, [], 0, 1), (10, [1], 0, 1), (17, [3, 4], 2, 1), (17, [3, 9], 2, 1), (30, [20], 1, 1), (30, [], 20, 1),
    (17, [3, 0, 4], 3, 0), (11, [0], 1, 0), (30, [0, 0, 20], 3, 0), (30, [19, 0], 2, 0)])
def test_pass_that_takes_nothing_shows(lib, need, take, passes, adds_up):
    out = (ctypes.c_uint32 * 2)()
    u = ctypes.c_uint32
    lib.serve(u(100), u(10), u(20), u(30), u(need), (u * max(len(take), 1))(*take), len(take), out)
    assert list(out) == [passes, adds_up]


@pytest.mark.parametrize("source", ["rkc_lean.hip", "rkc_big.hip"])
def test_kernels_test_that_the_pool_adds_up(source):
    text = open(os.path.join(CSRC, source)).read()
    assert text.count("K = rkc_left(K, m);") == 2 and "K -=" not in text
    assert re.search(r"rkc_adds_up\(U, P\.F, P\.A, (cached|P\.E \+ P\.PR)\) \? 0u : 0x80000000u", text)
    assert text.count("P.E + P.PR") == 1
