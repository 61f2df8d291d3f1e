"""Patches in which the work items of an XCD's region are listed (host logic)."""
import os
import subprocess

import pytest

from paper_2512_22142_amd import build

SOURCE = r"""
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include "plan_internal.h"

// M N K tile splits members list: rows and columns of sub-tiles that the first items of XCD 0 span
int main(int, char** a) {
  const auto arg = [&](int i) { return std::atoll(a[i]); };
  cleave_plan* plan = nullptr;
  const int rc = arg(6) ? cleave_plan_batched(arg(1), arg(2), arg(3), arg(4), arg(4), arg(5), arg(6), &plan)
                        : cleave_plan_uniform(arg(1), arg(2), arg(3), arg(4), arg(4), arg(5), 0, &plan);
  if (rc != CLEAVE_OK) return 1;
  const bool large = arg(7) == 1;
  const std::vector<cleave::WorkItem>& items = large ? plan->items[cleave::kTileLarge] : plan->items_fine;
  const uint32_t edge = large ? 256 : 128;
  for (int first : {32, 64}) {
    uint32_t rows = 0, cols = 0;
    for (int i = 0; i < first; ++i) {   // list position i belongs to XCD i % 8
      rows = std::max(rows, items[8 * i].m_base / edge + 1);
      cols = std::max(cols, items[8 * i].n_base / edge + 1);
    }
    std::printf("%ux%u ", rows, cols);
  }
  std::printf("%zu", items.size());
  return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("patches")
    src, exe = tmp / "patches.cpp", tmp / "patches"
    src.write_text(SOURCE)
    rocm = os.path.dirname(os.path.dirname(build.HIPCC))
    res = subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-isystem", os.path.join(rocm, "include"),
                          "-I" + os.path.join(build.ROOT, "include"), "-I" + build.CSRC, str(src),
                          os.path.join(build.CSRC, "plan.cpp"), "-o", str(exe)], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    return str(exe)


def listed(program, M, N, K, tile, S, members, large):
    res = subprocess.run([program] + [str(x) for x in (M, N, K, tile, S, members, int(large))], capture_output=True, text=True)
    assert res.returncode == 0
    return res.stdout.split()


@pytest.mark.parametrize("M,N,items", [(16384, 8192, 2048), (16384, 16384, 4096)])
def test_large_items_are_listed_in_patches_of_four_rows(program, M, N, items):
    """32 items and 64: one patch and the next one beside it."""
    assert listed(program, M, N, 64, 512, 1, 0, True) == ["4x8", "4x16", str(items)]


@pytest.mark.parametrize("M,N,rows", [(4096, 8192, 4), (8192, 8192, 8)])
def test_more_than_2048_small_items_are_listed_in_patches_of_eight_rows(program, M, N, rows):
    first = {4: ["4x8", "4x16", "2048"], 8: ["4x8", "8x8", "4096"]}[rows]
    assert listed(program, M, N, 64, 128, 1, 0, False) == first


@pytest.mark.parametrize("M,N,members,then", [(1024, 2048, 24, "4x16"), (4096, 4096, 3, "4x8")])
def test_small_items_of_several_members_are_listed_in_patches_of_four_rows(program, M, N, members, then):
    """More than 2048 items: members on an XCD each, the patch beside it next; members spread over
    the XCDs, the same patch of the next member next."""
    assert listed(program, M, N, 64, 128, 1, members, False) == ["4x8", then, str(members * M * N // 16384)]
