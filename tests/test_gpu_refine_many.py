"""The refinement launch with 1 to 16 of an item's parts in a workgroup, which the number of
items decides: the sums are added in the same order, so records do not depend on it."""
import dataclasses

import pytest

import siggen

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

FS = 8e6


@pytest.mark.parametrize("capacity", [23, 24, 47, 48, 255, 256, 1023, 1024])      # items: 4 times as many
@pytest.mark.parametrize("kw", [dict(), dict(exact_bins=True), dict(precision="bf16", refine_radius=8),
                                dict(precision="fp16", refine_radius=8, exact_bins=True)])
def test_records_do_not_depend_on_the_number_of_items(capacity, kw):
    from paper_2005_10445_amd import Plan
    codes = siggen.make_codes(8900, 4, 512)
    args = dict(num_bins=3, bin_step_hz=1500.0, max_block_len=5000, **kw)
    lens = [5000, 1023, 1024, 1031, 3333]                     # 1023: shorter than a template; 1 and 8 lags
    xs = [torch.from_numpy(siggen.make_block(8901 + i, n, codes, 2, FS, [0.0], 2 if n >= 3000 else 0,
                                             snr_db=(0.0, 3.0))[0]).to("cuda:0") for i, n in enumerate(lens)]
    with Plan(codes, 2, FS, **args) as one, \
            Plan(codes, 2, FS, max_batch_blocks=capacity, max_batch_samples=5000 * len(lens), **args) as p:
        each = [one.detect(x) for x in xs]
        assert each[0] and each[4]
        want = [dataclasses.replace(d, block=b) for b, dets in enumerate(each) for d in dets]
        for _ in range(2):
            assert p.detect_batch(xs) == want


def test_time_of_many_items():
    """4096 items, which fill the chip many times over, against 64, which fill it once (16 workgroups
    each): about 14 times the time with the parts of an item in one workgroup, 29 with one each."""
    from paper_2005_10445_amd import Plan
    codes = siggen.make_codes(8910, 256, 512)
    x = [torch.randn(1300, dtype=torch.complex64, generator=torch.Generator().manual_seed(8911 + i)).to("cuda:0")
         for i in range(16)]
    best = {}
    for tags, blocks in ((64, 1), (256, 16)):
        with Plan(codes[:tags], 2, FS, max_block_len=1300, max_batch_blocks=blocks) as p:
            p.set_profiling(True)
            times = []
            for _ in range(12):
                p.detect_batch(x[:blocks])
                times.append(p.last_kernel_times()["refine"])
            best[tags * blocks] = min(times)
    assert best[4096] <= 21.0 * best[64], best
