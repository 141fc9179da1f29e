"""The tile finish in bits (csrc/nf_kernels.hip) at the ends of its range: slacks
of the whole tile width and of 0, rows that rise everywhere and nowhere, partial
last tiles, one to a few tiles per side.  Every table must equal the oracle's."""

import numpy as np
import pytest

import oracle
from paper_1307_7820_amd import gen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nf():
    from paper_1307_7820_amd import nf as m
    m.nf_init(0)
    return m


def _patterns(n):
    h = n // 2
    return {
        "halves": "A" * h + "U" * (n - h),                       # every row rises in every column to its right
        "one letter": "G" * n,                                   # nothing ever rises
        "letters apart": "A" * (n - 1) + "U",                    # one column pairs, at the far end
        "alternating": ("AU" * n)[:n],                           # slacks of 0 and 1 only
        "quarters": ("A" * (n // 4) + "C" * (n // 4) + "G" * (n // 4) + "U" * n)[:n],
        "stretches": "".join("ACGU"[(k // 64) % 4] for k in range(n)),  # one letter per tile
        "stems": gen.stem_sequence(n, [77, n]) if n > 80 else gen.iid_sequence(n, [77, n]),
    }


@pytest.mark.parametrize("q", [1, 3, 4, 5, 8, 9])
@pytest.mark.parametrize("n", [63, 64, 126, 191, 192, 321, 449])
def test_finish_extremes(nf, n, q):
    for name, s in _patterns(n).items():
        score, T = nf.nf_fold(s, q, table=True)
        want = oracle.fold_table(s)
        assert score == int(want[0, n - 1]), (name, n, q)
        assert np.array_equal(T, want), (name, n, q)
