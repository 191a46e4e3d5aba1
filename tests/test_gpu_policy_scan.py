"""The scanned policy chains against the oracle where a scan has to stop.

The policy kernel scans each chain on the bit patterns of its values and
steps a read with ordinary operations where that does not hold: a value that
leaves its binade, an addend exactly halfway between two multiples of the
ulp, operands that are zero or not finite, a wait for a read of the same
scan. The comparison is bit for bit, as the chains' order is fixed.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2101_08734_amd import nopfs  # noqa: E402
from paper_2101_08734_amd import workloads as wl  # noqa: E402

POLICIES = (nopfs.POLICY_PERFECT, nopfs.POLICY_NAIVE, nopfs.POLICY_STAGING, nopfs.POLICY_NOPFS)
POW2 = dict(c=1.0, beta=2.0 ** 10, b_c=2.0 ** 9, pfs_t=2.0 ** 8, pfs_gamma=2, w0=2.0 ** 12, p0=2,
            r=(2.0 ** 11, 2.0 ** 7), p=(4, 2))


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nopfs.lib()
    yield
    torch.cuda.empty_cache()


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _check(oracle, shape, R, sizes, fill, prm, seed):
    rjob, job = oracle.make_job(*shape), nopfs.Job(*shape)
    rng = np.random.default_rng(seed)
    src = rng.choice(np.array([0, 128, 129, 256, 257], np.int16), size=R.shape)
    m_o, m_g = oracle.make_model(**prm), nopfs.make_model(**prm)
    Rd, sd, srcd, filld = _dev(R), _dev(sizes), _dev(src), _dev(fill)
    for pol in POLICIES:
        with np.errstate(all="ignore"):
            want = oracle.policy_sim(rjob, R, sizes, m_o, pol, src=src, fill=fill)
        got = nopfs.policy_sim(job, Rd, sd, m_g, pol, src=srcd, fill=filld)
        torch.cuda.synchronize()
        for what, g, w in zip(("t", "finish", "io"), got, want):
            g = g.cpu().numpy()
            bad = np.argwhere(~((g == w) | (np.isnan(g) & np.isnan(w))))
            assert len(bad) == 0, (pol, what, len(bad), bad[:3].tolist(),
                                   g[tuple(bad[0])], w[tuple(bad[0])])


# rows of M reads around the chunk (2,048), its halves and the LDS ring (4,096)
@pytest.mark.parametrize("M", [1, 2, 63, 64, 65, 2047, 2048, 2049, 4095, 4097, 6143, 6145, 9001])
def test_row_lengths(oracle, M):
    shape = (2 * M + 1, 1, 2, 1, 0, M)  # the second row is one read shorter
    R = oracle.access_streams(oracle.make_job(*shape))
    sizes = wl.random_sizes(shape[0], M, 1_000, 2_000_000)
    fill = np.maximum(0, np.arange(R.shape[1]) - 700)[None].repeat(2, 0).astype(np.int32)
    _check(oracle, shape, R, sizes, fill, dict(wl.LASSEN_MODEL), M)


# windows of w reads: read by read, scans of one wave, of the workgroup, and
# waits older than the LDS ring
@pytest.mark.parametrize("w", [1, 2, 7, 8, 9, 63, 64, 65, 200, 511, 513, 2047, 2049, 4096, 5000])
def test_window_lengths(oracle, w):
    shape = (40_003, 1, 2, 3, 0, w)
    R = oracle.access_streams(oracle.make_job(*shape))
    sizes = wl.random_sizes(shape[0], w, 1_000, 2_000_000)
    fill = np.maximum(0, np.arange(R.shape[1]) - w + 1)[None].repeat(2, 0).astype(np.int32)
    for kw in (dict(), dict(c=64e9), dict(c=1e9, p0=3)):  # compute-bound, I/O-bound, in between
        _check(oracle, shape, R, sizes, fill, dict(wl.LASSEN_MODEL, **kw), w)


# more workers than compute units: the kernel's smaller workgroups (chunks of 1,024)
@pytest.mark.parametrize("w", [1, 9, 65, 511, 513, 1023, 1025, 2049])
def test_more_workers_than_units(oracle, w):
    shape = (257 * 2_100 + 5, 1, 257, 1, 0, w)
    R = oracle.access_streams(oracle.make_job(*shape))
    sizes = wl.random_sizes(shape[0], w, 1_000, 2_000_000)
    fill = np.maximum(0, np.arange(R.shape[1]) - w + 1)[None].repeat(257, 0).astype(np.int32)
    _check(oracle, shape, R, sizes, fill, dict(wl.LASSEN_MODEL, c=1e9), w)


def _sizes_halfway(R, F):
    """The first reads put t at 2^56 (ulp 16), the rest add odd multiples of 8:
    every addition is halfway and takes the even neighbour."""
    s = 8 * (2 * np.arange(F, dtype=np.int64) + 1)
    s[R[:, 0]] = 1 << 56
    return s


SIZES = {
    "halfway": lambda R, F: _sizes_halfway(R, F),
    "halfway_rare": lambda R, F: np.where(np.arange(F) % 500 == 3, _sizes_halfway(R, F) | (1 << 56),
                                          16 * (np.arange(F, dtype=np.int64) + 1)),
    "zero": lambda R, F: np.zeros(F, np.int64),
    "mostly_zero": lambda R, F: np.where(np.arange(F) % 97 == 0, 12345, 0).astype(np.int64),
    "equal": lambda R, F: np.full(F, 16_777_216, np.int64),
    "doubling": lambda R, F: np.int64(1) << (np.arange(F, dtype=np.int64) % 60),
}


@pytest.mark.parametrize("name", list(SIZES))
@pytest.mark.parametrize("model", ["pow2", "lassen", "overflow", "tiny"])
def test_sizes_that_stop_scans(oracle, name, model):
    shape = (14_001, 2, 2, 1, 0, 5)
    R = oracle.access_streams(oracle.make_job(*shape))
    sizes = SIZES[name](R, shape[0])
    prm = {"pow2": POW2, "lassen": dict(wl.LASSEN_MODEL),
           # compute times of up to 2^56 / 1e-295: t overflows to infinity
           "overflow": dict(wl.LASSEN_MODEL, c=1e-295),
           # times below the smallest normal double
           "tiny": dict(c=1e300, beta=1e300, b_c=1e300, pfs_t=1e300, pfs_gamma=1, w0=1e300, p0=1,
                        r=(1e300, 1e300), p=(1, 1))}[model]
    fill = np.maximum(0, np.arange(R.shape[1]) - 900)[None].repeat(2, 0).astype(np.int32)
    _check(oracle, shape, R, sizes, fill, prm, 3)


# the stepped first reads of a row: rows that end inside, at and behind them
# (256, 512, 768 and 1,024 reads), whole and part batches of 64, and windows
# that reach into the same batch (63), the one before (64 to 127) or none of them
@pytest.mark.parametrize("N", [2, 257])
@pytest.mark.parametrize("w", [63, 64, 127, 128, 600, 5000])
def test_first_reads(oracle, N, w):
    rows = [1, 64, 65, 255, 256, 257, 511, 513, 767, 769, 1023, 1025, 1087]
    for M in rows if N == 2 else rows[2::3]:
        shape = (N * M - 1, 1, N, 1, 0, M + w)  # the last row is one read shorter
        R = oracle.access_streams(oracle.make_job(*shape))
        sizes = wl.random_sizes(shape[0], M, 1_000, 2_000_000)
        fill = np.maximum(0, np.arange(R.shape[1]) - w + 1)[None].repeat(N, 0).astype(np.int32)
        _check(oracle, shape, R, sizes, fill, dict(wl.LASSEN_MODEL, c=1e9), M)


def test_first_reads_of_all_classes(oracle):
    """32 tiers: 65 source classes, one more than a wave has lanes."""
    shape = (3_001, 1, 2, 1, 0, 7)
    rjob, job = oracle.make_job(*shape), nopfs.Job(*shape)
    R = oracle.access_streams(rjob)
    sizes = wl.random_sizes(shape[0], 8, 1_000, 2_000_000)
    prm = dict(wl.LASSEN_MODEL, r=[1e9 + 1e7 * j for j in range(32)], p=[1 + j % 3 for j in range(32)])
    codes = np.array([0] + [128 + j for j in range(32)] + [256 + j for j in range(32)] + [127, 160, 288], np.int16)
    src = np.random.default_rng(9).choice(codes, size=R.shape)
    fill = np.maximum(0, np.arange(R.shape[1]) - 300)[None].repeat(2, 0).astype(np.int32)
    want = oracle.policy_sim(rjob, R, sizes, oracle.make_model(**prm), nopfs.POLICY_NOPFS, src=src, fill=fill)
    got = nopfs.policy_sim(job, _dev(R), _dev(sizes), nopfs.make_model(**prm), nopfs.POLICY_NOPFS,
                           src=_dev(src), fill=_dev(fill))
    torch.cuda.synchronize()
    for what, g, e in zip(("t", "finish", "io"), got, want):
        assert np.array_equal(g.cpu().numpy(), e), what


@pytest.mark.parametrize("M", [383, 384, 385, 767, 769, 1025])
def test_first_reads_of_many_workers(oracle, M):
    """More than two workgroups per compute unit: Naive steps 384 reads instead of 768."""
    shape = (513 * M - 1, 1, 513, 1, 0, M)
    R = oracle.access_streams(oracle.make_job(*shape))
    sizes = wl.random_sizes(shape[0], M, 1_000, 2_000_000)
    fill = np.maximum(0, np.arange(R.shape[1]) - 700)[None].repeat(513, 0).astype(np.int32)
    _check(oracle, shape, R, sizes, fill, dict(wl.LASSEN_MODEL, c=1e9), M)
