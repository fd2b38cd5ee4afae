"""The split kernel's assignment of sequences to workgroups (csrc/attn_grid.h), on the CPU:
every split index takes each sequence once, and a sequence's splits do not gather in one of
the 32 classes (XCD, shader engine) that workgroups are dealt to in turn."""
import os
import subprocess

import numpy as np
import pytest

from paper_2609_11133_amd import build

PROG = r"""
#include <cstdio>
#include "attn_grid.h"
int main()
{
    unsigned heads, batch, splits;
    while (scanf("%u %u %u", &heads, &batch, &splits) == 3) {
        const attn::RowRotation r(heads, batch);
        for (unsigned c = 0; c < splits; ++c)
            for (unsigned y = 0; y < batch; ++y) printf("%u ", r.sequence(y, c));
        printf("\n");
    }
}
"""
# (key/value heads, batch, splits), split counts up to the second kernel's 4096; 16 heads:
# every batch is rotated
SPREAD = [(4, 24, 7), (2, 48, 7), (2, 32, 12), (1, 96, 12), (8, 12, 7), (4, 40, 10), (4, 64, 8), (8, 48, 4)]
CASES = SPREAD + [(16, b, 33) for b in range(1, 70)] + [(3, 7, 5), (4, 35, 12), (16, 127, 33), (16, 1000, 33),
                                                        (16, 4095, 33), (1, 4096, 33), (2, 8, 4096), (16, 37, 4096),
                                                        (1, 4096, 130)]


@pytest.fixture(scope="module")
def tables(tmp_path_factory):
    d = tmp_path_factory.mktemp("grid")
    src, exe = d / "grid.hip", d / "grid"
    src.write_text(PROG)
    subprocess.run([build.HIPCC, "-O1", "-std=c++17", f"--offload-arch={build.ARCH}", "-I", build.CSRC, str(src), "-o", str(exe)],
                   check=True, capture_output=True)
    env = {k: v for k, v in os.environ.items() if not k.startswith("ROCPROF")}
    out = subprocess.run([str(exe)], input="".join("%d %d %d\n" % c for c in CASES), text=True, check=True,
                         capture_output=True, env=env).stdout.splitlines()
    return {c: np.array(line.split(), np.int64).reshape(c[2], c[1]) for c, line in zip(CASES, out)}


def test_each_split_takes_every_sequence(tables):
    for (h, b, s), t in tables.items():
        assert np.array_equal(np.sort(t, axis=1), np.broadcast_to(np.arange(b), (s, b))), (h, b, s)


@pytest.mark.parametrize("heads,batch,splits", SPREAD)
def test_splits_of_a_row_spread_over_the_chip(tables, heads, batch, splits):
    """Without the rotation every split of a row falls into one class here (heads * batch is
    a multiple of 32); with it as many classes as the heads leave."""
    t, rows = tables[(heads, batch, splits)], heads * batch
    assert rows % 32 == 0
    for b in range(batch):
        y = [int(np.flatnonzero(t[c] == b)[0]) for c in range(splits)]
        classes = {(heads * y[c] + rows * c) % 32 for c in range(splits)}
        assert len(classes) >= min(splits, 32 // heads) - 1, (b, classes)
