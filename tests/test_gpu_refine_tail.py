"""The refinement launch: a search of at most 1024 (block, tag) items writes its
detections from that launch and a larger one through the compaction kernel,
with the same records in the same order; an item whose FP64 maximum sits next
to its FP32 or 16-bit peak is re-centred within the launch."""
import dataclasses

import pytest

import siggen

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

FS = 8e6


@pytest.mark.parametrize("tags,capacity", [(1, 1), (8, 128), (9, 114)])     # 1, 1024 and 1026 items
def test_records_with_and_without_the_compaction_kernel(tags, capacity):
    from paper_2005_10445_amd import Plan
    codes = siggen.make_codes(8300 + tags, tags, 300)
    lens = [4000, 599, 2500, 600, 3001][:capacity]            # 599: shorter than a template
    xs = [torch.from_numpy(siggen.make_block(8310 + i, n, codes, 2, FS, [0.0], min(tags, 3) if n >= 1200 else 0,
                                             snr_db=(0.0, 3.0))[0]).to("cuda:0") for i, n in enumerate(lens)]
    with Plan(codes, 2, FS, max_block_len=4000, max_batch_blocks=capacity) as p:
        each = [p.detect(x) for x in xs]
        assert each[0]
        want = [dataclasses.replace(d, block=b) for b, dets in enumerate(each) for d in dets]
        for _ in range(3):
            assert p.detect_batch(xs) == want
        p.set_profiling(True)                                 # every kernel on its own
        assert [p.detect(x) for x in xs] == each
        assert p.detect_batch(xs) == want


@pytest.mark.parametrize("precision", ["fp16", "bf16"])
def test_recentred_window(precision):
    """Transmissions half a sample late: the powers at their two lags agree to
    1e-3, so a 16-bit search takes the wrong one of them for some tags.  The
    refined records are those of the FP32 search.  They are FP64 sums of at most
    2^13 terms split at other places: 2^13 * 2^-53 < 1e-12 of the peak power."""
    from paper_2005_10445_amd import Plan
    tags, chips, n = 24, 2000, 30000
    codes = siggen.make_codes(8400, tags, chips)
    x, _ = siggen.make_block(8401, n, codes, 2, FS, [0.0], tags, snr_db=(3.0, 3.0), tags=list(range(tags)),
                             delays=[1000 * (t + 1) for t in range(tags)], fracs=[0.5] * tags)
    xd = torch.from_numpy(x).to("cuda:0")
    with Plan(codes, 2, FS, max_block_len=n) as p32, \
            Plan(codes, 2, FS, max_block_len=n, precision=precision, refine_radius=1) as p16:
        want, got = p32.detect(xd), p16.detect(xd)
    assert len(want) == tags
    assert [(d.tag, d.bin, d.lag, d.flags) for d in got] == [(d.tag, d.bin, d.lag, d.flags) for d in want]
    for g, w in zip(got, want):
        assert abs(g.peak_power - w.peak_power) <= 1e-12 * w.peak_power
        assert abs(g.energy - w.energy) <= 1e-12 * w.energy
