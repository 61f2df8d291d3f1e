"""The number of K steps of a chunk, which the kernels and the schedule share: chunks
go up to 2^31 - 1 elements, where rounding up to whole steps passes the largest
signed value (a negative count of steps left the products out)."""
import os
import subprocess

import numpy as np

import paper_2512_22142_amd as cleave
from paper_2512_22142_amd import build

SOURCE = r"""
#include "plan_internal.h"
using cleave::chunk_steps;
constexpr uint32_t kMost = 2147483647u;
%s
static_assert(chunk_steps(8, cleave::kDirectKStep) == 1 && chunk_steps(72, cleave::kDirectKStep) == 2, "");
"""


def test_steps_of_chunks_up_to_the_largest(tmp_path):
    checks = ["static_assert(chunk_steps(%s, %d) == %d, \"\");" % (text, step, -(-value // step))
              for step in (32, 64)
              for text, value in [("1", 1), ("kMost", 2**31 - 1)] +
              [("%du" % (x + d), x + d) for x in (step, 1000 * step, 2**31 - step) for d in (-1, 0, 1) if x + d < 2**31]]
    src = tmp_path / "steps.cpp"
    src.write_text(SOURCE % "\n".join(checks))
    rocm = os.path.dirname(os.path.dirname(build.HIPCC))
    res = subprocess.run(["g++", "-std=c++17", "-fsyntax-only", "-D__HIP_PLATFORM_AMD__", "-isystem", os.path.join(rocm, "include"),
                          "-I" + os.path.join(build.ROOT, "include"), "-I" + build.CSRC, str(src)],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr


def test_cost_of_the_longest_chunk():
    plan = cleave.plan_uniform(8, 8, 2**31 - 1, 8, 8, 1)
    for which in (1, 2):
        assert np.array_equal(cleave.schedule_loads(plan, which, 1), [2**25 + 4.5])
