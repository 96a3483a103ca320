"""Blocks whose powers are all equal are searched as fast as noise."""
import pytest

import siggen

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

FS = 8e6


@pytest.mark.parametrize("chips,spc,fft_len", [(8192, 2, 1 << 15), (1023, 4, 0)])
def test_time_of_a_block_of_zeros(chips, spc, fft_len):
    """Every transform of a block of zeros reaches its tag's best, and of noise few do: a
    peak key for each of them costs a fiftieth of a transform (1.04 times the kernel's time),
    and 0.6 of one where the equal lanes are looked at one after the other."""
    from paper_2005_10445_amd import Plan
    codes = siggen.make_codes(9000, 64, chips)
    n = 1 << 19
    noise = torch.randn(n, dtype=torch.complex64, generator=torch.Generator().manual_seed(9001)).to("cuda:0")
    with Plan(codes, spc, FS, num_bins=5, bin_step_hz=1000.0, max_block_len=n, fft_len=fft_len) as p:
        p.set_profiling(True)
        best = []
        for x in (noise, torch.zeros_like(noise)):
            times = []
            for _ in range(12):
                assert all(d.block_power > 0.0 for d in p.detect(x))
                times.append(p.last_kernel_times()["correlate"])
            best.append(min(times))
    assert best[1] <= 1.25 * best[0], best
