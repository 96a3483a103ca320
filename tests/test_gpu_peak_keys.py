"""Peak keys and crossing counts are formed only for transforms that reach the tag's best power so far or the
threshold: on every shape they are those of the powers of all lags (same FP32 values, so no tolerance)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

FS = 8e6

# (tags, chips, spc, bins, segment length, block length): 2^14-point transforms with exactly half, just over and
# just under half, few and nearly all outputs valid, ragged last segments; every Stockham size
SHAPES = [
    (3, 8192, 2, 3, 1 << 15, 70001),
    (2, 8191, 2, 3, 1 << 15, 65536),
    (2, 8193, 2, 1, 1 << 15, 60000),
    (2, 16000, 2, 1, 1 << 15, 33333),
    (2, 700, 2, 3, 1 << 15, 100000),
    (2, 8192, 1, 1, 1 << 14, 24576),
    (5, 511, 2, 3, 1 << 11, 9000),
    (5, 511, 4, 1, 1 << 13, 20001),
    (3, 1023, 4, 5, 1 << 14, 30003),
    (2, 1024, 4, 1, 1 << 15, 50000),
]


def _block(seed, n, period=0):
    g = np.random.default_rng(seed)
    x = (g.standard_normal(n) + 1j * g.standard_normal(n)).astype(np.complex64)
    return np.resize(x[:period], n).astype(np.complex64) if period else x


def _check(plan, x, theta):
    import torch
    xd = torch.from_numpy(x).cuda()
    P = plan.correlate_power(xd).cpu().numpy()
    T, K, lags = P.shape
    dets = {d.tag: d for d in plan.detect(xd)}
    assert len(dets) == T
    for t in range(T):
        d = dets[t]
        pthr = np.float32(theta * float(plan.template_len) * d.block_power)
        assert d.crossings == int(np.count_nonzero(P[t] >= pthr)), t
        flat = P[t].T.reshape(-1)                       # index lag * K + bin: ties to the smaller lag, then bin
        lag, k = divmod(int(np.argmax(flat)), K)
        assert (d.bin, abs(d.lag - lag) <= 1) == (k, True), (t, d, lag, k)


@pytest.mark.parametrize("shape", SHAPES, ids=[str(s) for s in SHAPES])
def test_keys_and_counts_match_every_lag(shape):
    from paper_2005_10445_amd import Plan
    T, C, spc, K, M, N = shape
    chips = (2 * np.random.default_rng(C).integers(0, 2, (T, C)) - 1).astype(np.int8)
    theta = 3.0                                          # low: many crossings, every tag detected
    with Plan(chips, spc, FS, num_bins=K, bin_step_hz=8000.0, max_block_len=N, fft_len=M, threshold=theta) as plan:
        for seed in (1, 2):
            _check(plan, _block(seed, N), theta)


@pytest.mark.parametrize("shape", [(2, 8192, 2, 1, 1 << 15), (2, 1023, 4, 1, 1 << 14)])
def test_ties_go_to_the_smaller_lag(shape):
    """A block with the period of the segments has the same powers in every segment."""
    import torch
    from paper_2005_10445_amd import Plan
    T, C, spc, K, M = shape
    L = C * spc
    V = M - L + 1
    N = 6 * V + L - 1
    chips = (2 * np.random.default_rng(C).integers(0, 2, (T, C)) - 1).astype(np.int8)
    x = _block(5, N, period=V)
    with Plan(chips, spc, FS, num_bins=K, max_block_len=N, fft_len=M, threshold=3.0) as plan:
        xd = torch.from_numpy(x).cuda()
        P = plan.correlate_power(xd).cpu().numpy()[:, 0]
        assert np.array_equal(P[:, :V], P[:, V:2 * V])   # equal segments, equal values
        for d in plan.detect(xd):
            assert d.lag < V
