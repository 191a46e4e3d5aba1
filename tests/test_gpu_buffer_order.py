"""The buffer's replay in the order of next uses against the oracle.

Jobs with enough reuse per epoch for that path, at the sizes of its pieces: a
window of 4,096 positions and rows just below and above it, more candidates
in a window than its list of 2,048, time blocks of 64 positions and of more
(rows above 2^19 positions), capacities from one sample to everything, equal
sizes (every discard a tie in size), and sizes of which a few fill the buffer.
Flags and sums are integer decisions and must be equal.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2101_08734_amd import nopfs  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nopfs.lib()
    yield
    torch.cuda.empty_cache()


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


SHAPES = [
    # F, E, N, B, drop_last, seed
    (1_023, 4, 1, 1, 0, 1),      # 4,092 reads: less than a window
    (1_024, 4, 1, 1, 1, 2),      # exactly one window
    (4_097, 3, 1, 1, 0, 3),      # dense: every read of epochs 2 and 3 is a candidate
    (10_001, 9, 4, 3, 0, 4),     # ragged rows
    (60_000, 6, 3, 8, 1, 5),
    (200_000, 3, 1, 64, 1, 6),   # 600,000 reads: blocks of 128 positions
    (350_001, 5, 1, 1, 0, 7),    # 1.75M reads: blocks of 256
    (2_000, 200, 3, 1, 0, 8),    # many short epochs
]
SIZES = {
    "uniform": lambda rng, F: rng.integers(1_000, 2_000_000, F),
    "equal": lambda rng, F: np.full(F, 16_777_216),
    "unit": lambda rng, F: np.ones(F),
    "few_huge": lambda rng, F: np.where(rng.random(F) < 0.01, 50_000_000, rng.integers(1, 1_000, F)),
}


@pytest.mark.parametrize("shape", SHAPES, ids=[f"F{s[0]}E{s[1]}N{s[2]}" for s in SHAPES])
@pytest.mark.parametrize("kind", list(SIZES))
def test_matches_oracle(oracle, shape, kind):
    rjob, job = oracle.make_job(*shape), nopfs.Job(*shape)
    F, N = shape[0], shape[2]
    R = oracle.access_streams(rjob)
    nx = oracle.reuse_next(rjob, R)
    sizes = SIZES[kind](np.random.default_rng(shape[-1]), F).astype(np.int64)
    Rd, nd, sd = _dev(R), _dev(nx), _dev(sizes)
    epoch, largest = int(sizes.sum()) // N, int(sizes.max())
    # the last two: just below and at the largest capacity the path takes
    caps = [largest - 1, largest, 3 * largest, epoch // 50, epoch // 4, epoch - 1, 3 * epoch,
            (1 << 50) - 1, 1 << 50]
    for d0 in caps:
        hit_o, hits_o = oracle.buffer_sim(rjob, R, nx, sizes, d0)
        hit_g, hits_g = nopfs.buffer_sim(job, Rd, nd, sd, d0)
        torch.cuda.synchronize()
        bad = np.argwhere(hit_g.cpu().numpy() != hit_o)
        assert len(bad) == 0, (d0, len(bad), bad[:3].tolist())
        assert np.array_equal(hits_g.cpu().numpy(), hits_o), d0
