"""The between-group lookups over marks (q = 8) in the shapes that a short single
fold takes only when it is told to: the wide fused step (two workgroups a chunk,
four rows a wavefront, eight tiles at a time) and the staged steps (k_between,
and the walk of the end tiles in the finish).  Rows with no marked group and with
many, chunks of one to many tiles that are no multiple of what a turn takes;
every table must equal the oracle's."""

import numpy as np
import pytest

import oracle
from paper_1307_7820_amd import gen

pytestmark = pytest.mark.gpu

SHAPES = {"wide": {"NF_MODE": "fused", "NF_STAGE_WIDE": "1"}, "staged": {"NF_MODE": "staged"}}


@pytest.fixture(params=sorted(SHAPES))
def nf(request, monkeypatch):
    from paper_1307_7820_amd import nf as m
    for k, v in SHAPES[request.param].items():  # part of a workspace's key
        monkeypatch.setenv(k, v)
    m.nf_init(0)
    return m


def _inputs(n):
    return {
        "iid": gen.iid_sequence(n, [78, n]),
        "stems": gen.stem_sequence(n, [79, n]),
        "repeats": ("GGGAAACCCUUU" * n)[:n],  # a third of all groups marked
        "two letters": gen.iid_sequence(n, [80, n], (0.5, 0.0, 0.0, 0.5)),
        "halves": "C" * (n // 2) + "G" * (n - n // 2),
        "one letter": "G" * n,                # none
    }


@pytest.mark.parametrize("target", ["1", "37", "4096"])
@pytest.mark.parametrize("n", [383, 640, 1090, 1500])
def test_marked_walk(nf, monkeypatch, n, target):
    monkeypatch.setenv("NF_BETWEEN_TARGET", target)
    for name, s in _inputs(n).items():
        score, T = nf.nf_fold(s, 8, table=True)
        want = oracle.fold_table(s)
        assert score == int(want[0, n - 1]), (name, n, target)
        assert np.array_equal(T, want), (name, n, target)


@pytest.mark.parametrize("seed", [1, 2, 3])
def test_marked_walk_under_perturbed_schedules(nf, monkeypatch, seed):
    """The items of a step in other orders, the staged launches delayed."""
    monkeypatch.setenv("NF_BETWEEN_TARGET", "37")
    lib = nf.load()
    want = {name: oracle.fold_table(s) for name, s in _inputs(1090).items()}
    assert lib.nf_test_set_perturb(seed) == 0
    try:
        for name, s in _inputs(1090).items():
            assert np.array_equal(nf.nf_fold(s, 8, table=True)[1], want[name]), (name, seed)
    finally:
        lib.nf_test_set_perturb(0)


def test_one_workspace_over_many_folds(nf):
    """A workspace keeps the marks of the fold before: each fold writes all those
    that it reads."""
    n = 1283
    for k in range(2):
        for name, s in _inputs(n).items():
            assert np.array_equal(nf.nf_fold(s, 8, table=True)[1], oracle.fold_table(s)), (name, k)
