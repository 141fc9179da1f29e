"""What a fold takes on the device (host arithmetic, no GPU): the bytes a served
fold is charged, and where the marks of q = 8 lie."""

import ctypes

import pytest


@pytest.fixture(scope="module")
def nf():
    from paper_1307_7820_amd import nf as m
    m.load()
    return m


@pytest.mark.parametrize("q", range(1, 10))
@pytest.mark.parametrize("n", [0, 1, 63, 64, 500, 6000, 16000, 65534])
def test_fold_bytes_are_table_words_and_accumulators(nf, n, q):
    """Codes, the dense table, one row and one column block a tile, two
    accumulators a tile row: nothing else, so a serving budget holds the folds
    that this sum says it holds."""
    up = lambda x: (x + 255) // 256 * 256  # noqa: E731
    G = 64 // q
    T = G * q
    NT = (n + T) // T
    tiles = NT * (NT + 1) // 2
    want = up(NT * T + 64) + up((NT * T) ** 2 * 2) + 2 * up(tiles * G * 64 * 4) + 2 * NT * 64 * 64 * 4
    assert nf.nf_fold_bytes(n, q) == want


def test_marks_lie_in_the_unused_half_of_the_table(nf):
    """The schedule hook checks their place for a single fold of NT tiles a side."""
    msg = ctypes.create_string_buffer(256)
    for NT in list(range(1, 200)) + [251, 512, 1023, 1024]:
        assert nf.load().nf_test_schedule((ctypes.c_int * 1)(NT), 1, 1024, msg, 256) == 0, (NT, msg.value)
