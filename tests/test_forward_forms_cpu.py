"""Choice of the strict forward's form (host only)."""
import random

import pytest

from forms import FWD_ROWS, few_rows, fwd_form


def shapes(n):
    rng = random.Random(5)
    for _ in range(n):
        H = int(2 ** rng.uniform(0, 11))
        Lq = int(2 ** rng.uniform(0, 11))
        Lk = Lq if rng.random() < 0.5 else int(2 ** rng.uniform(0, 12))
        yield 1, H, Lq, Lk, rng.choice((32, 64, 128)), rng.choice(("causal", "full", "padded"))


def test_a_tile_is_not_mostly_padding():
    """A head's last tile may be cut, but no form of 128 or 256 rows is taken
    that a head fills less than half (with far more keys than rows the waves
    without rows help to stage them)."""
    for s in shapes(5000):
        rows = FWD_ROWS[fwd_form(*s)]
        assert rows <= 64 or s[2] > rows // 2 or s[3] > 4 * s[2], s


def test_every_instance_exists():
    for s in shapes(5000):
        d, form = s[4], fwd_form(*s)
        assert form not in (("rows32", "rows32_quad") if d == 128 else ("rows256",)), s


@pytest.mark.parametrize("shape,form", [
    ((1, 1351, 55, 55, 128, "causal"), "rows64"), ((32, 51, 32, 32, 32, "full"), "few_wave"),
    ((8, 8, 1024, 1024, 64, "causal"), "rows128"), ((2, 6, 1500, 1500, 64, "full"), "rows64_pair"),
    ((2, 8, 1024, 1024, 128, "causal"), "rows64_pair"), ((4, 4, 256, 256, 64, "causal"), "few"),
    ((8, 16, 1, 4096, 128, "padded"), "few_long"), ((1, 1, 64, 64, 32, "causal"), "few"),
    # both sides fill their tiles; and where they do not, or lengths cut them
    ((8, 32, 128, 128, 32, "full"), "rows128"), ((8, 32, 256, 256, 64, "full"), "rows128"),
    ((8, 32, 110, 128, 32, "full"), "rows64"), ((64, 16, 128, 128, 64, "padded"), "rows64"),
    ((8, 8, 128, 128, 64, "full"), "rows32"), ((8, 8, 112, 112, 64, "full"), "few"),
    ((8, 8, 256, 256, 32, "causal"), "rows32"), ((8, 8, 200, 200, 32, "causal"), "few"),
    # K and V read again by every 16 rows
    ((1, 384, 17, 2048, 64, "full"), "rows32"), ((64, 16, 7, 2048, 64, "padded"), "few_long"),
])
def test_forms_of_named_shapes(shape, form):
    assert fwd_form(*shape) == form


@pytest.mark.parametrize("shape,few", [
    ((8, 16, 1, 4096, 128, "full"), True), ((2, 4, 1024, 1024, 64, "causal"), True),
    ((8, 8, 128, 128, 128, "full"), True), ((1, 55, 70, 70, 128, "full"), True), ((1, 200, 17, 4096, 32, "full"), True),
    # a head's K and V would be read once per block from memory
    ((1, 256, 32, 2048, 128, "full"), False), ((1, 73, 100, 1000, 128, "causal"), False),
    ((1, 43, 128, 4000, 64, "full"), False),
])
def test_bf16_few_rows(shape, few):
    assert few_rows("fast_bf16", *shape) == few


def test_accelerated_few_rows():
    assert few_rows("accelerated", 4, 4, 256, 256, 64, "causal")
    assert not few_rows("accelerated", 1, 4, 2048, 2048, 128, "full")
