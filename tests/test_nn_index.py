"""Address arithmetic of the convolution kernels' staged tensors on boxes of more
than 2^31 and 2^32 voxels (no card holds a test of that size in reasonable time):
the kernels' own index function, built for the host."""
import ctypes as ct
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2302_04659_amd", "csrc")


@pytest.fixture(scope="module")
def index(tmp_path_factory):
    d = tmp_path_factory.mktemp("nn_index")
    src, lib = str(d / "index.cpp"), str(d / "index.so")
    with open(src, "w") as f:
        f.write('#include "%s"\n' % os.path.join(CSRC, "nn_kernels.hpp"))
        f.write('extern "C" unsigned long long voxel(int d, int h, int w, int c, int z, int y, int x)\n'
                "{ return nn::VoxelIndex(h, w, c, nn::VoxelIndex::needs_wide(d, h, w))(z, y, x); }\n")
    subprocess.run(["g++", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-O1", "-std=c++17", "-fPIC", "-shared",
                    "-o", lib, src], check=True, capture_output=True)
    fn = ct.CDLL(lib).voxel
    fn.restype = ct.c_ulonglong
    return fn


@pytest.mark.parametrize("d,h,w,c", [(40, 24, 40, 32), (2048, 1024, 1024, 8), (2100, 1031, 1999, 16), (70000, 70000, 1, 8),
                                     (3, 1, 2000000000, 64)])
def test_voxel_offsets(index, d, h, w, c):
    for z, y, x in ((0, 0, 0), (d - 1, h - 1, w - 1), (d // 2, h - 1, w // 3), (d - 1, 0, w - 1)):
        assert index(d, h, w, c, z, y, x) == ((z * h + y) * w + x) * c
