"""March lengths of the x pass in the automatic plan (ch_plan.h on the CPU)."""
import pytest

from tests.test_plan_report import reported


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("shape", [(64, 64, 64), (128, 64, 64), (100, 40, 33), (96, 96, 8)])
def test_narrow_groups_march_no_less_than_for_2048_groups(shape, prec):
    """One row of at most 64 cells per task: work-groups of one wave, of which
    2048 hold fewer threads than the count the longer marches come down to."""
    nz, ny, _ = shape
    got = reported([shape], 2e-4, prec, x_rows=1)
    assert got["z_chunk"] >= min(16, max(1, ny * nz // 2048))


@pytest.mark.parametrize("shapes,longer", [
    ([(40, 80, 160)] * 2, True),                          # one launch, 3 planes by the 2048
    ([(29, 119, 65)] * 4, True),                          # several rows per task
    ([(49, 37, 192), (79, 32, 161)], True),
    ([(65, 97, 145)] * 2, False),                         # 6 planes by the 2048
    ([(157, 57, 95)] * 4, False),
    ([(44, 184, 75), (101, 37, 176)], False),             # one launch per row mode
    ([(49, 35, 146), (66, 124, 48), (43, 44, 69)], False)])
def test_batches_march_further_only_where_it_was_measured(shapes, longer):
    for prec in (0, 1):
        nx = max(s[2] for s in shapes)
        R = max(1, min(256 // nx, max(s[1] for s in shapes), 16))
        base = max(1, sum(s[0] * s[1] * s[2] for s in shapes) // nx // R // 2048)
        got = reported(shapes, 1e-4, prec)["z_chunk"]
        assert got > base if longer else got == base


@pytest.mark.parametrize("shape", [(92, 266, 302), (154, 148, 234), (81, 320, 247)])
def test_long_marches_stay(shape):
    """Eleven planes and more by the 2048: one plane more or a better fit of the
    last work-groups was measured to gain nothing."""
    nz, ny, nx = shape
    base = ny * nz // max(1, 256 // nx) // 2048
    assert base >= 11
    for prec in (0, 1):
        assert reported([shape], 1e-4, prec)["z_chunk"] == min(16, base)
