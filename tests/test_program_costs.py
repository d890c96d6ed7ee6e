"""The multiply-adds that the bench's rooflines are computed from (no GPU)."""
import numpy as np
import pytest

from paper_2410_03348_amd import programs as GP


def counted(symbols):
    """Tuple by tuple: every (i, j) of every stage forward; backward the tuples of the columns that reach a target, most of any target."""
    rows = [symbols[0]]
    for nb in symbols[1:]:
        rows.append(rows[-1] + nb - 1)
    n, best = len(symbols), [0] * len(symbols)
    for target in range(rows[-1]):
        seen = {target}
        for t in range(n - 1, -1, -1):
            best[t] = max(best[t], len(seen))
            if t:
                seen = {c - j for c in seen for j in range(symbols[t]) if 0 <= c - j < rows[t - 1]}
    return sum(nb * (rows[t] + best[t] + best[t + 1]) for t, nb in enumerate(symbols[1:]))


@pytest.mark.parametrize("symbols", [[10, 10], [10] * 3, [10] * 15, [3, 7, 1, 4], [40, 2, 2], [1, 1, 5], [16] * 9])
def test_multiply_adds_of_a_fold_under_a_target(symbols):
    assert GP.target_fold_macs(symbols) == counted(symbols)


def test_the_headline_fold_is_not_priced_at_the_full_reverse_sweep():
    full = 3 * sum(10 * (9 * t + 1) for t in range(1, 15))
    assert 2 * GP.target_fold_macs([10] * 15) == 39720 < 2 * full == 57540
