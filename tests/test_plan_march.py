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
