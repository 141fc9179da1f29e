"""Streams under capture into a HIP graph: nf_fold_dev and nf_batch_run refuse
them at every length and leave the capture whole; nf_fold_dev_noalloc is
recorded, and each replay folds what the codes buffer then holds."""

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


@pytest.mark.parametrize("n", [60, 500, 2000])
def test_capture(nf, n):
    import torch
    seqs = [gen.iid_sequence(n, [93, n, k]) for k in range(4)]
    want = [oracle.fold_table(s) for s in seqs]
    codes = [torch.from_numpy(nf.encode(s).copy()).cuda() for s in seqs]
    buf = torch.zeros_like(codes[0])
    score = torch.zeros(1, dtype=torch.int32, device="cuda")
    S = torch.zeros((n, n), dtype=torch.int16, device="cuda")
    stream = torch.cuda.Stream()
    batch = nf.Batch(seqs, q=8)

    def eager(call, k):
        with torch.cuda.stream(stream):
            score.fill_(-5)
            S.fill_(-9)
            buf.copy_(codes[k])
            call(buf, n, 8, score, S, stream)
        torch.cuda.synchronize()
        assert int(score.item()) == int(want[k][0, n - 1])
        assert np.array_equal(S.cpu().numpy(), want[k])

    eager(nf.nf_fold_dev, 0)
    batch.run()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(stream):
        g.capture_begin(capture_error_mode="thread_local")
        score.fill_(-3)
        for call in (lambda: nf.nf_fold_dev(buf, n, 8, score, S, stream), lambda: batch.run(stream)):
            with pytest.raises(nf.NFError) as e:
                call()
            assert e.value.code == nf.NF_E_INVAL
        nf.nf_fold_dev_noalloc(buf, n, 8, score, S, stream)
        g.capture_end()
    torch.cuda.synchronize()
    for k in (1, 2, 3):
        score.fill_(-5)
        S.fill_(-9)
        buf.copy_(codes[k])
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert int(score.item()) == int(want[k][0, n - 1]), k
        assert np.array_equal(S.cpu().numpy(), want[k]), k
        eager(nf.nf_fold_dev, k)
        eager(nf.nf_fold_dev_noalloc, 0)
    batch.run()
    assert [int(x) for x in batch.scores()] == [int(w[0, n - 1]) for w in want]
    batch.close()
