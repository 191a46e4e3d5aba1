"""Fetch model over rows of few and of many spans of 16,384 reads.

A span's start is chained from the spans before it, looked at 64 at a time:
rows of one, two, 64, 65 and 140 spans, spans of one read, more rows than
workgroups, rows of unequal length, and the same call twice with the same bits.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2101_08734_amd import nopfs  # noqa: E402
from paper_2101_08734_amd import workloads as wl  # noqa: E402

SHAPES = [
    # F, E, N, B, drop_last, seed
    (16_384, 1, 1, 1, 0, 1), (16_385, 1, 1, 1, 0, 2), (1, 2, 1, 1, 0, 3),
    (16_384 * 64, 1, 1, 1, 0, 4), (16_384 * 64 + 1, 1, 1, 1, 0, 5),
    (1_146_881, 2, 1, 4, 0, 6), (900_001, 3, 2, 1, 0, 7), (500_003, 4, 3, 7, 0, 8),
    (20_011, 5, 700, 1, 0, 9), (700_001, 30, 300, 1, 1, 10),
]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nopfs.lib()
    yield
    torch.cuda.empty_cache()


@pytest.mark.parametrize("shape", SHAPES, ids=[f"F{s[0]}E{s[1]}N{s[2]}" for s in SHAPES])
def test_spans(oracle, shape):
    F, E, N = shape[:3]
    rjob, job = oracle.make_job(*shape), nopfs.Job(*shape)
    R = oracle.access_streams(rjob)
    tier = np.random.default_rng(shape[-1]).integers(-1, 2, (N, F)).astype(np.int8)
    sizes = wl.random_sizes(F, shape[-1], 1, 1 << 24)
    prm = wl.LASSEN_MODEL
    src_o, t_o = oracle.fetch_model(rjob, R, tier, sizes, oracle.make_model(**prm))
    Rd, td, sd = (torch.from_numpy(a).cuda() for a in (R, tier, sizes))
    src, t = nopfs.fetch_model(job, Rd, td, sd, nopfs.make_model(**prm))
    src2, t2 = nopfs.fetch_model(job, Rd, td, sd, nopfs.make_model(**prm))
    torch.cuda.synchronize()
    assert torch.equal(src, src2) and torch.equal(t, t2)
    assert np.array_equal(src.cpu().numpy(), src_o)
    t = t.cpu().numpy()
    pad = src_o < 0
    assert (t[pad] == -1.0).all()
    # sums of n positive terms in different orders: see the bound in test_gpu_model.py
    for i in range(N):
        n = int((~pad[i]).sum())
        if n:
            tol = 8 * (n + 2) * 2.0**-53 * t_o[i, n - 1]
            assert np.abs(t[i, :n] - t_o[i, :n]).max() <= tol, i
