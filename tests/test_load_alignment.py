"""The alignment that the compiler is promised for the parameters which a gradient's kernel averages on the way: a network's layers
and rows start on any 4-byte boundary, so a load of several floats may promise no more."""
import os
import re
import subprocess

import pytest

from paper_2102_06280_amd import build

# the vector types that the kernels average: a lane's two or four gradients
SOURCE = """
#include "average.h"
#include "fc_head.h"
typedef float pair __attribute__((ext_vector_type(2)));
#define KERNEL(NAME, V)                                                                                \\
    extern "C" __global__ void NAME(average::Args a, const uint32_t *at, V *out)                       \\
    {                                                                                                  \\
        const average::Row r = average::row(a, blockIdx.x);                                            \\
        const uint32_t off[1] = {at[threadIdx.x]};                                                     \\
        V acc[1];                                                                                      \\
        average::gather<V, 1, true>(a, r, blockIdx.x, 4, off, acc);                                    \\
        out[threadIdx.x] = acc[0];                                                                     \\
    }
KERNEL(two, pair)
KERNEL(four, fchead::f32x4)
"""


@pytest.fixture(scope="module")
def code(tmp_path_factory):
    """The device code as the compiler's optimiser leaves it, a text per kernel."""
    path = tmp_path_factory.mktemp("loads") / "loads.hip"
    path.write_text(SOURCE)
    r = subprocess.run([build.HIPCC, *build.FLAGS, "--cuda-device-only", "-S", "-emit-llvm", str(path), "-o", "-"],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return {m[1]: m[2] for m in re.finditer(r"^define [^\n]*@(two|four)\((.*?)^}", r.stdout, re.S | re.M)}


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="needs hipcc")
@pytest.mark.parametrize("kernel,floats", [("two", 2), ("four", 4)])
def test_neighbours_rows_are_read_on_any_boundary(code, kernel, floats):
    loads = [int(a) for a in re.findall(rf"= load (?:<{floats} x float>|i{32 * floats}), ptr addrspace\(1\)[^\n]*align (\d+)", code[kernel])]
    assert len(loads) >= 5                             # the own row, four neighbours at a time, the rest of a long list
    assert set(loads) == {4}, loads
