"""Which form of the strips' exchange the images of the GPU tests take, and over how many workgroups: asked of the kernels'
own rules (csrc/sinkhorn_team.hpp), compiled for the host."""
import os
import subprocess

import numpy as np
import pytest

from paper_2605_00392_amd import build
from paper_2605_00392_amd import rtprune as rt
from tests.test_gpu_parity import STRIP_BATCHES, STRIP_EDGES
from tests.test_routes_cpu import kept_count

SOURCE = r"""
#include "rtprune.h"
#include "common.hpp"
#include "sinkhorn_team.hpp"
#include <cstdio>
using namespace rtp;
// per line "shape thin kept pruned": compute units, workgroups, one trip
int main() {
  int shape, thin, m, r;
  while (scanf("%d %d %d %d", &shape, &thin, &m, &r) == 4) {
    const int mode = thin ? kModeStripThin : 0, teams = strip_teams(shape, m, mode);
    printf("%d %d %d\n", strip_groups(shape, m, mode), teams, strip_direct(shape, r, teams) ? 1 : 0);
  }
}
"""
A, B, C, D = 1, 2, 3, 4                                # strip shapes: 144 x 576, 80 x 960, 64 x 1408, 48 x 1792


@pytest.fixture(scope="module")
def forms(tmp_path_factory):
    path = tmp_path_factory.mktemp("host")
    (path / "forms.hip").write_text(SOURCE)
    includes = [f for f in build.FLAGS if f.startswith("-I")]
    subprocess.run([build.HIPCC, "--offload-host-only", "-std=c++17", "-O1", *includes, "-o", str(path / "forms"),
                    str(path / "forms.hip")], check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)

    def ask(shape, thin, images):
        lines = "".join(f"{shape} {int(thin)} {m} {r}\n" for m, r in images)
        out = subprocess.run([os.fspath(path / "forms")], input=lines, stdout=subprocess.PIPE, check=True, text=True).stdout
        return [tuple(int(v) for v in line.split()) for line in out.splitlines()]
    return ask


def are_strips(batch, max_tokens, images, own, **params):
    m, r = (np.array(v) for v in zip(*images))
    rc, to = rt.rtprune_sinkhorn_routes(batch, max_tokens, rt.make_params(**params), own, m, r)
    return rc == rt.RTP_OK and (to & 15 == rt.RTP_ROUTE_STRIPS).all()


@pytest.mark.parametrize("name,shape", [("72 x 576", A), ("40 x 960", B)])
def test_the_edges_are_edges(forms, name, shape):
    top, want = STRIP_EDGES[name]
    n = sum(top)
    assert are_strips(2 * len(want), n, list(want), 1, ratio=top[0] / n)
    got = forms(shape, False, list(want))
    assert {image: form[1:] for image, form in zip(want, got)} == {i: (t, int(d)) for i, (t, d) in want.items()}


@pytest.mark.parametrize("name,shape,thin,units", [("3 units, one trip", A, False, 3), ("4 units", A, False, 4), ("16 units", B, False, 16),
                                                   ("24 units", C, False, 24), ("one page", A, True, 14),
                                                   ("one page, one trip", A, True, 7)])
def test_the_batches_take_the_exchange_they_say(forms, name, shape, thin, units):
    counts, ratio, _, one_trip = STRIP_BATCHES[name]
    n = np.array(counts)
    m = kept_count(ratio, n)
    images = list(zip(m.tolist(), (n - m).tolist()))
    assert are_strips(len(counts), max(counts), images, 0, ratio=ratio)
    got = forms(shape, thin, images)
    assert max(g[0] for g in got) == units and all(g[2] == int(one_trip) and g[1] > 1 for g in got), got


def test_thin_strips_give_a_wave_one_reductions_rows(forms):
    """Four waves of at most eight rows to a workgroup, whatever the number of rows, and two of them to a compute unit."""
    rows = list(range(1, 1025)) + [1500, 4096]
    for m, (units, teams, _) in zip(rows, forms(A, True, [(m, 300) for m in rows])):
        assert -(-m // teams) <= 32 and teams <= 2 * units, (m, units, teams)
