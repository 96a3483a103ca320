"""Rounding of the split inverse transform of few templates: the phases' twiddles are table values."""
import pytest

import siggen

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

FS = 8e6


def test_correlation_error_of_two_to_eight_phases():
    """RMS difference from the same correlation in 64 bits, for segments of 2^15 (two phases, each of whose
    twiddles any form reads from the table) to 2^17 points (eight).  A butterfly adds a fixed share to the
    error's variance, so 17 levels for 15 make it sqrt(17 / 15) = 1.065 times as large.  The forward combination
    of eight phases multiplies its twiddles up (products of up to 6 table values, 3.5 on average over the eight
    inputs, 2^-24 / sqrt(6) each in either part): with the 4.7e-7 of the levels about another 8 %.  1.065 * 1.08
    = 1.15, and 0.04 for the chance of 800,000 values: 1.19.  A second such product in the inverse's first step
    makes it 1.26."""
    from paper_2005_10445_amd.fsk import FskPlan
    n = 200000
    bits = siggen.make_fsk_bits(9200, 4, 1500)
    bp = siggen.fsk_bandpass(101, 600e3, FS)
    g = torch.Generator().manual_seed(9201)
    iq = (700.0 * torch.randn(n, 2, generator=g)).round().to(torch.int16).to("cuda:0")
    rms = {}
    for fft_len in (1 << 15, 1 << 16, 1 << 17):
        with FskPlan(bits, FS, 1e6, 250e3, -250e3, bp, 6, n, fft_len=fft_len) as p:
            c, (d, _) = p.xcorr(iq).double(), p.demod(iq)
            tm = torch.stack([p.template(t) for t in range(4)]).double()
        F = 1 << 18
        ref = torch.fft.irfft(torch.fft.rfft(d.double(), F) * torch.fft.rfft(tm, F).conj(), F)[:, :c.shape[1]]
        rms[fft_len] = float((c - ref).square().mean().sqrt())
    print("[fsk phase error]", rms, flush=True)
    assert rms[1 << 16] <= 1.19 * rms[1 << 15], rms
    assert rms[1 << 17] <= 1.19 * rms[1 << 15], rms
