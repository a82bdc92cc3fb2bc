"""How strips mark a published value with the use of its place, on the host: the functions are the kernels' own,
compiled from their header (csrc/sinkhorn_strip.hpp)."""
import os
import subprocess

import numpy as np
import pytest

from paper_2605_00392_amd import build

SOURCE = r"""
#include "rtprune.h"
#include "common.hpp"
#include "sinkhorn_strip.hpp"
#include <cstdio>
#include <cstring>
using namespace rtp;
// per value on the input: what a reader gets from its place, and of which use the place is seen to be (bit 0: the one it was
// marked with, bit 1: the other), for both uses
int main() {
  double v;
  while (fread(&v, 8, 1, stdin) == 1)
    for (uint32_t use : {0u, kExOdd}) {
      uint32_t w[2];
      memcpy(w, &v, 8);
      w[1] = ex_mark(w[1], use);
      const double seen = ex_is_of(w[1], use) + 2 * ex_is_of(w[1], use ^ kExOdd);
      double marked;
      memcpy(&marked, w, 8);
      const double out[2] = {ex_value(marked), seen};
      fwrite(out, 8, 2, stdout);
    }
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    path = tmp_path_factory.mktemp("host")
    (path / "exchange.hip").write_text(SOURCE)
    includes = [f for f in build.FLAGS if f.startswith("-I")]
    subprocess.run([build.HIPCC, "--offload-host-only", "-std=c++17", "-O1", *includes, "-o", str(path / "exchange"),
                    str(path / "exchange.hip")], check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    return os.fspath(path / "exchange")


def test_a_place_holds_all_bits_of_its_value_and_the_use(program):
    """Sums and reciprocals of positive numbers, zero, the smallest and the largest, infinity: what arrives is what was
    published, to the bit, and its place is of the one use and not of the other; a NaN of either sign arrives as one."""
    rng = np.random.default_rng(3)
    tiny = np.array([0.0, 5e-324, 1e-310, 2.2250738585072014e-308, 1.7976931348623157e308, np.inf])
    v = np.concatenate([np.exp(rng.uniform(-700, 700, 5000)), 1.0 + rng.integers(0, 4, 100) * 2.0 ** -52, tiny, [np.nan, -np.nan]])
    out = subprocess.run([program], input=v.tobytes(), stdout=subprocess.PIPE, check=True).stdout
    got = np.frombuffer(out).reshape(len(v), 2, 2)
    assert (got[:, :, 1] == 1).all()
    for use in range(2):
        np.testing.assert_array_equal(got[:-2, use, 0].view(np.int64), v[:-2].view(np.int64))
        assert np.isnan(got[-2:, use, 0]).all()
