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


@pytest.mark.parametrize("target", ["1", "37", "4096"])
@pytest.mark.parametrize("n", [383, 1090, 1500])
def test_sparse_between(nf, monkeypatch, n, target):
    """The between-group lookups at q = 8 walk only the groups the finish marks:
    few and many marked groups in a row, chunks of one to many tiles (whole
    fours and remainders), every table against the oracle's."""
    monkeypatch.setenv("NF_BETWEEN_TARGET", target)  # part of a workspace's key
    for name, s in {
        "iid": gen.iid_sequence(n, [78, n]),
        "stems": gen.stem_sequence(n, [79, n]),
        "repeats": ("GGGAAACCCUUU" * n)[:n],          # a third of all groups
        "two letters": gen.iid_sequence(n, [80, n], (0.5, 0.0, 0.0, 0.5)),
        "halves": "C" * (n // 2) + "G" * (n - n // 2),
    }.items():
        score, T = nf.nf_fold(s, 8, table=True)
        want = oracle.fold_table(s)
        assert score == int(want[0, n - 1]), (name, n, target)
        assert np.array_equal(T, want), (name, n, target)


@pytest.mark.parametrize("n", [127, 128, 192, 449, 1090])
def test_walked_end_tiles(nf, monkeypatch, n):
    """Staged steps at q = 8 look up only the marked groups of the end tiles:
    no end tile, one and two (the first three diagonals), rows with none to all
    of their groups marked, the last row block, every table against the
    oracle's.  Several folds in one step, so that the wavefronts' roles are
    taken both ways."""
    monkeypatch.setenv("NF_MODE", "staged")  # part of a workspace's key
    seqs = list(_patterns(n).values()) + [("GGGAAACCCUUU" * n)[:n], gen.iid_sequence(n, [81, n])]
    scores, tables = nf.nf_fold_batch(seqs, q=8, tables=True)
    for k, s in enumerate(seqs):
        want = oracle.fold_table(s)
        assert scores[k] == int(want[0, n - 1]), (k, n)
        assert np.array_equal(tables[k], want), (k, n)


@pytest.mark.parametrize("n", [5567, 5568])
def test_short_and_long_single_folds(nf, n):
    """A single fold at q = 8 looks every group up below 88 tiles per side and
    only the marked ones from there on: both sides of the line."""
    s = gen.stem_sequence(n, [82, n])
    score, T = nf.nf_fold(s, 8, table=True)
    want = oracle.fold_table(s)
    assert score == int(want[0, n - 1])
    assert np.array_equal(T, want)


@pytest.mark.parametrize("target", ["1", "37", "4096"])
@pytest.mark.parametrize("n", [383, 1090])
def test_marks_in_fused_batches(nf, monkeypatch, n, target):
    """Several folds in a fused step take the marks at any length: chunks of one
    to many tiles, every table against the oracle's."""
    monkeypatch.setenv("NF_MODE", "fused")
    monkeypatch.setenv("NF_BETWEEN_TARGET", target)
    seqs = [gen.iid_sequence(n, [83, n]), gen.stem_sequence(n, [84, n]), ("GGGAAACCCUUU" * n)[:n],
            gen.iid_sequence(n, [85, n], (0.5, 0.0, 0.0, 0.5)), "C" * (n // 2) + "G" * (n - n // 2)]
    scores, tables = nf.nf_fold_batch(seqs, q=8, tables=True)
    for k, s in enumerate(seqs):
        want = oracle.fold_table(s)
        assert scores[k] == int(want[0, n - 1]), (k, n, target)
        assert np.array_equal(tables[k], want), (k, n, target)
