"""Committed counter records carry the digest of the sources that they were taken
on, which must cover every source of the kernels that they describe."""
import os
import re

import bench

CSRC = os.path.join(bench.ROOT, bench.KERNEL_SOURCE_DIR)


def includes(path, seen):
    """The files under csrc/ that `path` includes, itself among them."""
    path = os.path.normpath(path)
    if path in seen or not os.path.exists(path):
        return seen
    seen.add(path)
    with open(path) as f:
        for name in re.findall(r'#include "([^"]+)"', f.read()):
            includes(os.path.join(os.path.dirname(path), name), seen)
    return seen


def test_the_convolution_digest_covers_its_headers(monkeypatch):
    read = set()
    real = open

    def spy(path, *a, **k):
        read.add(os.path.normpath(str(path)))
        return real(path, *a, **k)

    monkeypatch.setattr("builtins.open", spy)
    bench.kernel_source_digest(conv=True)
    monkeypatch.undo()
    used = includes(os.path.join(CSRC, "conv", "conv_f32.hip"), set())
    assert {os.path.join(CSRC, n) for n in ("tiles_split.h", "rows_f32.h")} <= used
    assert used <= read, sorted(used - read)
