"""Which short-batch forward products are formed in parts: the shapes that the GPU tests of the parts use, and shapes on both sides of the
rule.  The timing names don't tell parts from whole products."""
import os
import subprocess

import pytest

import test_gpu_thin
import test_gpu_wide_head
from paper_2102_06280_amd import build

SOURCE = """
#include <stdio.h>
#include <stdlib.h>
#include "mlp_thin_plan.h"
int main(int, char **v)
{
    const mlpthin::ThinPlan p = mlpthin::thin_plan(atoi(v[1]), atoi(v[2]), atoi(v[3]), atoi(v[4]), atoi(v[5]) != 0);
    printf("%d %d\\n", p.splits, p.kper);
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    path = tmp_path_factory.mktemp("plan")
    (path / "plan.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(build.HERE, "csrc"), str(path / "plan.cpp"), "-o", str(path / "plan")], check=True)
    return lambda *sizes: tuple(map(int, subprocess.run([str(path / "plan"), *map(str, sizes)], check=True, capture_output=True, text=True).stdout.split()))


PARTS = [s[:3] for s in test_gpu_thin.SHAPES + test_gpu_wide_head.GRADIENTS if s[0][0] > 1600]


@pytest.mark.parametrize("dims,batch,n", PARTS, ids=["-".join(map(str, s[0])) for s in PARTS])
def test_shapes_of_the_gpu_tests_are_in_parts(plan, dims, batch, n):
    """Three layers, a hidden width that divides by four, a head: the product below it may be left in parts.  None of them is empty."""
    assert len(dims) == 3 and dims[1] % 4 == 0 and dims[2] <= 32
    splits, kper = plan(batch, dims[0], dims[1], n, 1)
    chunks = (dims[0] + 15) // 16
    assert splits > 1 and (splits - 1) * kper < chunks <= splits * kper
    assert plan(batch, dims[0], dims[1], n, 0) == (1, chunks)


@pytest.mark.parametrize("batch,k,n,workers,splits", [(64, 784, 200, 32, 1), (64, 784, 200, 8, 2), (17, 256, 128, 5, 2), (17, 224, 128, 5, 1), (30, 1605, 36, 64, 1)])
def test_parts_fill_the_chip(plan, batch, k, n, workers, splits):
    assert plan(batch, k, n, workers, 1)[0] == splits
