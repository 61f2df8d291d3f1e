"""Which checked sums and assembled outputs leave through non-temporal stores (host
logic): those that lose nothing, whether or not the next launch reads them."""
import os
import subprocess

import pytest

from paper_2512_22142_amd import build

SOURCE = r"""
#include <cstdio>
#include <cstdlib>
#include "kernels.h"
int main(int, char** v) {
  const int64_t outputs = std::atoll(v[2]) * std::atoll(v[3]), x = std::atoll(v[4]);
  if (v[1][0] == 's') std::printf("%d", cleave::streamed_sum(outputs, outputs * x));
  else std::printf("%d", cleave::streamed_output(outputs * x, v[1][0] == 'b'));
  return 0;
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    folder = tmp_path_factory.mktemp("rule")
    src, exe = folder / "rule.cpp", folder / "rule"
    src.write_text(SOURCE)
    rocm = os.path.dirname(os.path.dirname(build.HIPCC))
    res = subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-isystem", os.path.join(rocm, "include"),
                          "-I" + os.path.join(build.ROOT, "include"), "-I" + build.CSRC, str(src), "-o", str(exe)],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    return lambda *size: subprocess.run([str(exe)] + [str(x) for x in size], capture_output=True, text=True).stdout == "1"


@pytest.mark.parametrize("M,N,S,streams", [
    (4096, 4096, 4, False), (4096, 8192, 4, False),                          # 67 and 134 MB: read from the cache
    (4096, 10240, 4, True), (4096, 11008, 4, True), (4096, 11008, 8, False),   # 168 and 180 MB
    (4096, 12288, 4, False), (8192, 8192, 2, False), (8192, 8192, 8, False),   # 201 and 268 MB
    (8192, 9216, 1, True), (8192, 10240, 4, True), (8192, 10240, 6, False), (16384, 16384, 4, True),
    (2**29, 2**30, 1, True)])
def test_sums_that_a_reader_would_miss_stay_in_the_cache(rule, M, N, S, streams):
    assert rule("sum", M, N, S) == streams


@pytest.mark.parametrize("M,N,element,single,batch", [
    (16384, 4096, 2, False, False), (16384, 8184, 2, False, False), (16384, 8192, 2, False, True), (8192, 8192, 4, False, True),
    (8192, 9208, 4, False, True), (8192, 9216, 4, True, True), (16384, 16384, 2, True, True)])
def test_a_single_output_is_streamed_later_than_a_batch(rule, M, N, element, single, batch):
    assert rule("output", M, N, element) == single and rule("batch", M, N, element) == batch
