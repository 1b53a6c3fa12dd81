"""The build refuses static LDS in the kernels that address their dynamic LDS from 0."""
import os
import subprocess

import pytest

SOURCE = r"""
#include <hip/hip_runtime.h>
namespace {
template <int N> __global__ void rkc_lean(int* p) { %s *p = N; }
__global__ void rkc_lean_order(int* p) { __shared__ int v[8]; v[threadIdx.x & 7] = *p; __syncthreads(); *p = v[0]; }
}
void launch(int* p) { rkc_lean<1><<<1, 64>>>(p); rkc_lean_order<<<1, 64>>>(p); }
"""
PLANTED = "__shared__ int v[16]; v[threadIdx.x & 15] = *p; __syncthreads(); p[1] = v[3];"


@pytest.mark.parametrize("body", ["", PLANTED], ids=["dynamic only", "planted"])
def test_static_lds_is_refused(tmp_path, body):
    from paper_2605_24259_amd import build
    if not os.path.exists(build.hipcc()):
        pytest.skip("no hipcc")
    src, obj = tmp_path / "k.hip", tmp_path / "k.o"
    src.write_text(SOURCE % body)
    flags = [build.hipcc(), "-O3", "-std=c++17", f"--offload-arch={build.ARCH}"]
    if body:
        with pytest.raises(RuntimeError, match="rkc_lean"):
            build.compile_source(str(src), str(obj), flags)
        assert not obj.exists()
    else:
        build.compile_source(str(src), str(obj), flags)
        assert obj.exists()


def test_compiler_errors_are_raised(tmp_path):
    from paper_2605_24259_amd import build
    if not os.path.exists(build.hipcc()):
        pytest.skip("no hipcc")
    src = tmp_path / "k.hip"
    src.write_text("int f() { return")
    with pytest.raises(subprocess.CalledProcessError):
        build.compile_source(str(src), str(tmp_path / "k.o"), [build.hipcc(), f"--offload-arch={build.ARCH}"])


def test_the_kernels_are_known_by_name():
    """The mangled names of the kernels concerned, and of the launch-order kernels, which have static LDS."""
    from paper_2605_24259_amd.build import LDS_FROM_ZERO
    for name in ("_ZN12_GLOBAL__N_18rkc_leanILi4ELi1ELb0EEEv13rkc_lean_argsPK9rkc_event",
                 "_ZN12_GLOBAL__N_17rkc_bigE12rkc_big_args"):
        assert LDS_FROM_ZERO.search(name)
    assert not LDS_FROM_ZERO.search("_ZN12_GLOBAL__N_120rkc_lean_order_countEPK13rkc_pool_desciPhPj")
