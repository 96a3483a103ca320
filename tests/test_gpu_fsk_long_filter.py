"""FSK front end with composed filters longer than a workgroup's row of samples
(256): the block's first samples lie in the second register of a thread, and
reach the first outputs."""
import numpy as np
import pytest

import oracle.fsk as ofsk
import siggen

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

FS = 8e6


@pytest.mark.parametrize("ntaps", [252, 253, 254, 255, 256, 301, 511])      # filters of 256 .. 260, 305, 515 taps
def test_first_outputs(ntaps):
    from paper_2005_10445_amd.fsk import FskPlan
    sps, f1, f0, lo, n = 5, 400e3, -300e3, 2.0e6, 9000
    bits = siggen.make_fsk_bits(8800, 2, 300)
    bp = siggen.fsk_bandpass(ntaps, 900e3, FS)
    rng = np.random.default_rng(8801 + ntaps)
    iq = rng.integers(-2000, 2000, size=(n, 2)).astype(np.int16)
    iq[:4] = 30000                            # the first samples weigh
    with FskPlan(bits, FS, lo, f1, f0, bp, sps, n) as plan:
        d, u = (v.cpu().numpy().astype(np.float64) for v in plan.demod(torch.from_numpy(iq).to("cuda:0")))
    x = ofsk.lo_mix(ofsk.iq_to_complex(iq), lo, FS)
    s = sum(np.abs(ofsk.fir(x, ofsk.compose(bp, ofsk.tone_matched_filter(f, sps, FS)))) for f in (f1, f0))
    rd, ru = ofsk.front_end(iq, FS, lo, bp, f1, f0, sps)
    # FP32 filtering: 2e-5 of the filter outputs, as for the whole front end
    assert np.max(np.abs(u - ru)) <= 2e-5 * s.max()
    assert np.max(np.abs(d - rd) * s) <= 2e-5 * s.max()
