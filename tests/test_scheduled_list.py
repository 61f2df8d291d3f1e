"""The work-item list of a heterogeneous plan as it is uploaded (host logic): a list
that the general kernel runs too keeps the order it was laid out in, XCD by XCD,
and the order of the persistent kernel's runs stands behind it."""
import os
import subprocess

import pytest

from paper_2512_22142_amd import build

SOURCE = r"""
#include <cstdio>
#include <cstring>
#include "plan_internal.h"

#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)

int main() {
  // 12 x 8 tiles of 512 x 512 with 1, 2, 4 and 8 splits; K is no multiple of a K step
  const int64_t K = KVALUE;
  std::vector<int64_t> heights(8, 512), widths(96, 512);
  std::vector<int32_t> columns(8, 12), splits;
  for (int i = 0; i < 8; ++i)
    for (int j = 0; j < 12; ++j) splits.push_back(1 << ((3 * i + j) % 4));
  cleave_plan* plan = nullptr;
  CHECK(cleave_plan_explicit(4096, 6144, K, 8, heights.data(), columns.data(), widths.data(), splits.data(), 0, &plan) == CLEAVE_OK);
  const std::vector<cleave::WorkItem>& items = plan->items_fine;
  const size_t n = items.size();
  const int grid = 512;
  CHECK(n > 2 * static_cast<size_t>(grid) && cleave::needs_balance(items, grid));
  std::vector<uint32_t> ranges, again;
  const std::vector<cleave::WorkItem> both = cleave::scheduled_list(items, grid, true, &ranges);
  CHECK(both.size() == 2 * n && ranges.size() == static_cast<size_t>(grid) + 1);
  CHECK(std::memcmp(both.data(), items.data(), n * sizeof(cleave::WorkItem)) == 0);      // as laid out
  const std::vector<cleave::WorkItem> alone = cleave::scheduled_list(items, grid, false, &again);
  CHECK(alone.size() == n && again == ranges && ranges.front() == 0 && ranges.back() == n);
  CHECK(std::memcmp(both.data() + n, alone.data(), n * sizeof(cleave::WorkItem)) == 0);
  CHECK(std::memcmp(alone.data(), items.data(), n * sizeof(cleave::WorkItem)) != 0);     // the runs' order is another
  std::vector<int> seen(plan->tasks.size() * 64, 0);
  for (const cleave::WorkItem& w : alone) CHECK(++seen[w.task * 64 + w.sub] == 1);
  // nothing to balance: no list, no ranges
  CHECK(cleave::scheduled_list(items, static_cast<int>(n), true, &ranges).empty() && ranges.empty());
  return 0;
}
"""


@pytest.mark.parametrize("K", [4104, 4096])
def test_the_order_laid_out_is_kept_for_the_general_kernel(tmp_path, K):
    src, exe = tmp_path / "order.cpp", tmp_path / "order"
    src.write_text(SOURCE.replace("KVALUE", str(K)))
    rocm = os.path.dirname(os.path.dirname(build.HIPCC))
    res = subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-isystem", os.path.join(rocm, "include"),
                          "-I" + os.path.join(build.ROOT, "include"), "-I" + build.CSRC, str(src),
                          os.path.join(build.CSRC, "plan.cpp"), "-o", str(exe)], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    res = subprocess.run([str(exe)], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout
