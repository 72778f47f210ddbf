"""Host checks of dense ROI tables (no GPU): the extents read from a table's
memory agree with the descriptors, tables that do not fit a base are refused
with the first bad ROI, and the uncovered ranges are those of a count per
element."""
import numpy as np
import pytest

from paper_2510_02894_amd import shape3d as S


def table(rows):
    return S.roi_table([r[0] for r in rows], [r[1] for r in rows], [(1.0, 0.5, 2.0)] * len(rows))


@pytest.mark.parametrize("rows", [[(0, (2, 3, 4))], [(0, (2, 3, 4)), (24, (1, 1, 1))], [(6, (1, 1, 1)), (0, (1, 2, 3))]])
def test_tables_that_fit(rows):
    S._check_extents(table(rows), 25)


@pytest.mark.parametrize("rows,bad", [
    ([(0, (2, 3, 4)), (2, (2, 3, 4))], 1), ([(-1, (1, 1, 1))], 0), ([(0, (0, 3, 4))], 0), ([(0, (1, -3, 4))], 0),
    ([(0, (1, 1, 1)), (25, (1, 1, 1))], 1), ([(0, (2 ** 31, 2 ** 31, 2 ** 31))], 0), ([(2 ** 62, (5, 5, 1))], 0),
    ([(0, (2 ** 32, 2 ** 32, 1))], 0), ([(0, (-2, -3, 4))], 0)])
def test_tables_that_do_not_fit(rows, bad):
    with pytest.raises(ValueError, match="ROI %d " % bad):
        S._check_extents(table(rows), 25)


def test_uncovered_ranges():
    g = np.random.default_rng(3)
    for _ in range(200):
        numel = int(g.integers(1, 60))
        rows = [(int(g.integers(0, 50)), tuple(int(v) for v in g.integers(1, 4, size=3)))
                for _ in range(int(g.integers(0, 6)))]
        covered = np.zeros(200, dtype=bool)
        for off, d in rows:
            covered[off:off + int(np.prod(d))] = True
        want = ~covered[:numel]
        got = np.zeros(numel, dtype=bool)
        ranges = S._uncovered(table(rows), numel)
        for a, b in ranges:
            assert 0 <= a < b <= numel and not got[a:b].any()
            got[a:b] = True
        np.testing.assert_array_equal(got, want)
