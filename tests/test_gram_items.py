"""X^T X, host logic: the (split, pair) items of four classes of tiles are merged
into one launch list by where in the rows they start.  Every place of the list has
exactly one item, each class's come in order, and an item stands where its start
(i + 1/2) / n does among the others'."""
import numpy as np
import pytest

from paper_1608_04329_amd import hsp

RNG = np.random.default_rng(7)
CASES = [(0, 0, 0, 1), (0, 0, 0, 342), (0, 1, 1, 1), (1, 2, 2, 1), (21 * 46, 7 * 30, 7 * 40, 26), (65341, 361, 361, 1),
         (0, 53, 27, 14), (4096, 1, 1, 4096), (1, 100_000, 1, 3), (7, 7, 7, 7), (0, 0, 5, 0), (3, 0, 0, 100_000)]
CASES += [tuple(int(v) for v in np.exp(RNG.uniform(0, 9, 4)).astype(int) * (RNG.random(4) < 0.8)) for _ in range(40)]


@pytest.mark.parametrize("n", [c for c in CASES if sum(c)])
def test_merging_is_a_bijection_in_order(n):
    total = sum(n)
    cls, item = hsp.hsp_gram_items(n, 0, total)
    for c in range(4):
        assert np.array_equal(item[cls == c], np.arange(n[c]))
    # whole numbers: (2 i + 1) / n_c does not fall along the list, ties to the lower class
    num, den = 2 * item + 1, np.array(n, np.int64)[cls]
    lhs, rhs = num[:-1] * den[1:], num[1:] * den[:-1]
    assert np.all((lhs < rhs) | ((lhs == rhs) & (cls[:-1] <= cls[1:])))


def test_places_of_a_long_list():
    """The far end of lists of millions of items."""
    for n in [(2_000_000, 60_000, 60_000, 1), (5, 16_000_000, 3, 12_345_678)]:
        total = sum(n)
        for first in (0, total // 3, total - 5000):
            cls, item = hsp.hsp_gram_items(n, first, 5000)
            assert np.all((item >= 0) & (item < np.array(n)[cls]))
            for c in range(4):
                assert np.all(np.diff(item[cls == c]) == 1)


def test_bad_arguments():
    for n, first, count in [((-1, 0, 0, 1), 0, 1), ((1, 0, 0, 1), 0, 3), ((1 << 24, 0, 0, 1), 0, 1)]:
        with pytest.raises(hsp.HspError):
            hsp.hsp_gram_items(n, first, count)
