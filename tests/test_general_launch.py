"""How a launch of the general kernel is laid out (host logic): between one round of the
chip and two, the resident workgroups take the second tiles only where the chunks are of
equal length, and an item is cut into the tiles that its list's blocks fill."""
import os
import subprocess

import pytest

from paper_2512_22142_amd import build

SOURCE = r"""
#include <cstdio>
#include "kernels.h"

#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)

using cleave::general_workgroups;
using cleave::parts_along;
using cleave::second_tiles_taken_up_to;

// a band of 12 tiles of 128 x 128, tile j with splits[j % n]
cleave_plan* band(int64_t K, const std::vector<int32_t>& splits) {
  const int64_t height = 128;
  const int32_t columns = 12;
  const std::vector<int64_t> widths(12, 128);
  std::vector<int32_t> all;
  for (int j = 0; j < 12; ++j) all.push_back(splits[j % splits.size()]);
  cleave_plan* plan = nullptr;
  return cleave_plan_explicit(128, 1536, K, 1, &height, &columns, widths.data(), all.data(), 0, &plan) == CLEAVE_OK ? plan : nullptr;
}

int main() {
BODY
  return 0;
}
"""

CASES = {
    "unequal_chunks_are_left_to_the_dispatcher": """
  CHECK(!band(1024, {1, 2, 4})->shape.equal() && !band(128, {1, 2})->shape.equal());
  CHECK(second_tiles_taken_up_to(512, 128, band(1024, {1, 2, 4})->shape) == 0 && second_tiles_taken_up_to(1024, 64, band(128, {1, 2})->shape) == 0);
  CHECK(general_workgroups(600, 512, 0) == 600 && general_workgroups(1024, 512, 0) == 1024);
""",
    "equal_ones_and_a_shorter_last_chunk_are_not": """
  CHECK(band(1024, {1})->shape.equal() && band(1024, {4})->shape.equal() && band(3001, {4})->shape.equal());
  CHECK(band(1501, {2})->shape.equal() && !band(10, {4})->shape.equal());
  CHECK(general_workgroups(513, 512, 768) == 512 && general_workgroups(768, 512, 768) == 512 && general_workgroups(1024, 512, 1024) == 512);
""",
    "one_round_and_more_than_two": """
  CHECK(general_workgroups(512, 512, 1024) == 512 && general_workgroups(8, 512, 1024) == 8 && general_workgroups(769, 512, 768) == 769);
  CHECK(general_workgroups(1025, 512, 1024) == 1025 && general_workgroups(int64_t{1} << 40, 512, 1024) == 1 << 20);
""",
    "the_large_tile_to_half_of_the_second_round": """
  CHECK(second_tiles_taken_up_to(512, 128, band(257, {1})->shape) == 768 && second_tiles_taken_up_to(512, 128, band(4096, {1})->shape) == 768);
  CHECK(second_tiles_taken_up_to(512, 128, band(256, {1})->shape) == 1024 && second_tiles_taken_up_to(512, 128, band(1024, {4})->shape) == 1024);
  CHECK(second_tiles_taken_up_to(1024, 64, band(4096, {1})->shape) == 2048);
""",
    "no_tiles_that_hold_nothing": """
  cleave_plan* plan = nullptr;
  CHECK(cleave_plan_uniform(1000, 700, 64, 64, 100, 1, 0, &plan) == CLEAVE_OK);
  CHECK(plan->shape.rows == 64 && plan->shape.cols == 100);
  CHECK(parts_along(64, 128, 64) == 1 && parts_along(65, 128, 64) == 2 && parts_along(100, 128, 128) == 1);
  CHECK(parts_along(1, 128, 32) == 1 && parts_along(33, 128, 32) == 2 && parts_along(128, 128, 32) == 4);
  CHECK(parts_along(129, 128, 64) == 2 && parts_along(2147483647u, 256, 128) == 2 && parts_along(4294967295u, 256, 256) == 1);
  CHECK(parts_along(129, 256, 128) == 2 && parts_along(129, 256, 64) == 3 && parts_along(256, 256, 64) == 4);
""",
    "waves_of_the_large_tile": """
  cleave::ListShape l;
  cleave_task t{};
  t.m_len = t.n_len = t.k_len = 128;
  l.add(t);
  const auto four = [&](int dtype, int ta, int tb, int64_t items) { return cleave::four_waves(dtype, ta, tb, items, l, 256); };
  CHECK(four(CLEAVE_BF16, 0, 1, 769) && !four(CLEAVE_BF16, 0, 1, 768));
  CHECK(!four(CLEAVE_BF16, 0, 0, 4096) && !four(CLEAVE_BF16, 1, 0, 4096) && !four(CLEAVE_BF16, 1, 1, 4096));
  CHECK(four(CLEAVE_F32, 0, 1, 1025) && four(CLEAVE_F32, 1, 0, 1025) && four(CLEAVE_F32, 1, 1, 1025));
  CHECK(!four(CLEAVE_F32, 0, 0, 4096) && !four(CLEAVE_F32, 0, 1, 1024));
  t.k_len = 129;
  l.add(t);
  CHECK(!four(CLEAVE_F32, 0, 1, 4096) && four(CLEAVE_BF16, 0, 1, 4096));
  t.k_len = 257;
  l.add(t);
  CHECK(four(CLEAVE_BF16, 1, 0, 1793) && !four(CLEAVE_BF16, 1, 0, 1792) && four(CLEAVE_BF16, 0, 1, 4096));
  CHECK(!four(CLEAVE_BF16, 0, 0, 4096) && !four(CLEAVE_BF16, 1, 1, 4096));
""",
    "one_workgroup_of_64_per_cu_reads_ahead": """
  cleave::ListShape l;
  cleave_task t{};
  t.m_len = t.n_len = 128;
  t.k_len = 224;
  l.add(t);
  const auto lone = [&](int dtype, int cls, int64_t items) { return cleave::runs_lone(dtype, cls, items, l, 256); };
  CHECK(!lone(CLEAVE_F32, cleave::kTileSmall, 8));
  t.k_len = 225;
  l.add(t);
  CHECK(lone(CLEAVE_F32, cleave::kTileSmall, 64) && lone(CLEAVE_F32, cleave::kTileSmall, 57) && !lone(CLEAVE_F32, cleave::kTileSmall, 65) && !lone(CLEAVE_BF16, cleave::kTileSmall, 64));
  t.k_len = 448;
  l.add(t);
  CHECK(!lone(CLEAVE_BF16, cleave::kTileSmall, 64));
  t.k_len = 449;
  l.add(t);
  CHECK(lone(CLEAVE_BF16, cleave::kTileSmall, 64) && !lone(CLEAVE_BF16, cleave::kTileSmall, 65));
  t.m_len = t.n_len = 256;
  l.add(t);
  CHECK(lone(CLEAVE_F32, cleave::kTileLarge, 16) && !lone(CLEAVE_F32, cleave::kTileLarge, 17));
  cleave::ListShape small;
  t.m_len = t.n_len = 64;
  small.add(t);
  CHECK(cleave::runs_lone(CLEAVE_F32, cleave::kTileSmall, 256, small, 256) && !cleave::runs_lone(CLEAVE_F32, cleave::kTileSmall, 257, small, 256));
""",
    "the_longest_chunks": """
  cleave::ListShape l;
  cleave_task t{};
  t.m_len = t.n_len = 2147483647u;
  t.k_len = 2147483647u;
  l.add(t);
  t.k_len = 2013265920u;
  l.add(t);
  CHECK(l.equal());
  t.k_len = 2013265919u;
  l.add(t);
  CHECK(!l.equal() && l.rows == 2147483647u && l.parts64 == 3 * (int64_t{1} << 50));
""",
}


@pytest.mark.parametrize("case", list(CASES))
def test_grid_of_the_general_kernel(tmp_path, case):
    src, exe = tmp_path / "launch.cpp", tmp_path / "launch"
    src.write_text(SOURCE.replace("BODY", CASES[case]))
    rocm = os.path.dirname(os.path.dirname(build.HIPCC))
    res = subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-isystem", os.path.join(rocm, "include"),
                          "-I" + os.path.join(build.ROOT, "include"), "-I" + build.CSRC, str(src),
                          os.path.join(build.CSRC, "plan.cpp"), "-o", str(exe)], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    res = subprocess.run([str(exe)], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout
