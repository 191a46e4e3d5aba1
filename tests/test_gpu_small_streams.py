"""Access streams and folded partitions of small jobs against the oracle.

Jobs of few scatter chunks take smaller chunks (8,192 ids instead of 24,576)
and smaller sort buckets; jobs that would be left with fewer than 64
sub-chunks keep their epochs apart. The shapes sit on the edges: an id more
or less than a chunk, chunk counts on both sides of the rule (48 full chunks
over all epochs), bucket counts on both sides of theirs (512), and row
lengths that give 63, 64 and 65 sub-chunks.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2101_08734_amd import nopfs  # noqa: E402

STREAMS = [
    # F, E, N, B, drop_last, seed
    (2, 2, 1, 1, 0, 1),
    (1_023, 3, 2, 1, 0, 2), (1_025, 3, 2, 1, 0, 3),
    (8_191, 2, 3, 4, 0, 4), (8_192, 2, 3, 4, 1, 5), (8_193, 2, 3, 4, 0, 6),
    (24_575, 5, 4, 1, 0, 7), (24_577, 5, 4, 1, 1, 8),
    (9_000, 47, 2, 1, 0, 9), (9_000, 48, 2, 1, 0, 10),
    (24_576 * 47, 1, 5, 3, 0, 11), (24_576 * 47 + 1, 1, 5, 3, 0, 12),
    (120_001, 9, 7, 2, 0, 13), (600, 255, 3, 1, 0, 14),
]
FOLDS = [
    # N rows of E * L reads: 63, 64 and 65 sub-chunks; short epochs, 64 and 48
    (8_000 * 63, 2, 63, 1, 1, 1), (8_000 * 64, 2, 64, 1, 1, 2), (8_000 * 65, 2, 65, 1, 1, 3),
    (16 * 300, 200, 16, 1, 0, 4), (16 * 200, 240, 16, 1, 0, 5),
]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nopfs.lib()
    yield
    torch.cuda.empty_cache()


def _ids(shapes):
    return [f"F{s[0]}E{s[1]}N{s[2]}" for s in shapes]


@pytest.mark.parametrize("shape", STREAMS, ids=_ids(STREAMS))
def test_streams(oracle, shape):
    R = nopfs.access_streams(nopfs.Job(*shape))
    torch.cuda.synchronize()
    assert np.array_equal(R.cpu().numpy(), oracle.access_streams(oracle.make_job(*shape)))


@pytest.mark.parametrize("shape", FOLDS, ids=_ids(FOLDS))
def test_folds(oracle, shape):
    rjob, job = oracle.make_job(*shape), nopfs.Job(*shape)
    want = oracle.access_streams(rjob)
    count_o, first_o = oracle.access_stats(rjob, want)
    R = torch.from_numpy(want).cuda()
    count, first = nopfs.access_stats(job, R)
    nxt = nopfs.reuse_next(job, R)
    tier = np.random.default_rng(shape[-1]).integers(-1, 2, (shape[2], shape[0])).astype(np.int8)
    tier[count_o == 0] = -1
    order_o, qlen_o = oracle.prefetch_order(rjob, want, first_o, tier, 2)
    order, qlen = nopfs.prefetch_order(job, R, torch.from_numpy(tier).cuda(), 2)
    torch.cuda.synchronize()
    assert np.array_equal(count.cpu().numpy(), count_o)
    assert np.array_equal(first.cpu().numpy(), first_o)
    assert np.array_equal(nxt.cpu().numpy(), oracle.reuse_next(rjob, want))
    assert np.array_equal(qlen.cpu().numpy(), qlen_o)
    assert np.array_equal(order.cpu().numpy(), order_o)
