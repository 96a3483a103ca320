"""Launches that hand their results to the last workgroup to arrive: calls of different kinds
and sizes that share a plan's or a network's arrival counts, one after the other, give the
same results every time."""
import pytest

import siggen

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

FS = 8e6


def test_searches_of_different_sizes_in_turn():
    from paper_2005_10445_amd import Plan
    codes = siggen.make_codes(9300, 9, 600)
    xs = [torch.from_numpy(siggen.make_block(9301 + i, n, codes, 2, FS, [0.0], 2, snr_db=(0.0, 3.0))[0]).to("cuda:0")
          for i, n in enumerate((30000, 4500, 1201))]
    with Plan(codes, 2, FS, max_block_len=30000, max_batch_blocks=200) as p:
        def calls():
            yield p.detect(xs[0])
            yield p.detect_batch(xs)
            yield p.detect(xs[2])
            yield p.track([(x, t) for t, x in enumerate(xs)])
            p.set_profiling(True)                     # the block power in a launch of its own
            yield p.detect(xs[1])
            p.set_profiling(False)
            yield p.detect_batch(xs[1:] * 20)
        first = list(calls())
        assert first[0] and first[1] and first[3]
        for _ in range(4):
            assert list(calls()) == first


def test_network_calls_in_turn():
    from paper_2005_10445_amd.proposals import Network, SynthTransmission, num_params
    x = [torch.randn(n, dtype=torch.complex64, generator=torch.Generator().manual_seed(9310 + n)).to("cuda:0")
         for n in (256, 70000, 9000)]
    p = (0.05 * torch.randn(num_params(256), generator=torch.Generator().manual_seed(9311))).numpy()
    txs = [[SynthTransmission(500, 0.01, 0.5, 0.25, b)] for b in range(5)]
    with Network("bf16", max_rows=4096, max_block_len=1 << 18) as net:
        def calls():
            net.set_params(p)
            for b in x:
                yield net.power_map(b)[1]
            yield net.train_synthetic(5, 0, 20000, 700, 2, txs, 2.0, 0.0)
            yield net.power_map(x[1])[1]
        first = list(calls())
        for _ in range(4):
            assert list(calls()) == first


def test_fsk_calls_in_turn():
    from paper_2005_10445_amd.fsk import FskPlan
    bits = siggen.make_fsk_bits(9320, 12, 100)
    bp = siggen.fsk_bandpass(41, 600e3, FS)
    g = torch.Generator().manual_seed(9321)
    iq = [(700.0 * torch.randn(n, 2, generator=g)).round().to(torch.int16).to("cuda:0") for n in (9000, 1000, 2500)]
    with FskPlan(bits, FS, 1e6, 250e3, -250e3, bp, 8, 12500, max_track_tasks=8) as p:
        def calls():
            yield p.detect(iq[0])
            yield p.track([(b, 3 * i) for i, b in enumerate(iq)])
            yield p.detect(iq[1])
            yield p.track([(iq[2], 7)])
        first = list(calls())
        assert all(first)
        for _ in range(4):
            assert list(calls()) == first
