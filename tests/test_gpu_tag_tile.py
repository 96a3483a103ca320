"""Tags per work item chosen from the work (plans made with no tile): records
equal those of a plan whose tile is named, for each engine length's edges: one
item per unit, a last round of one item, one tag per item, and a batch."""
import pytest

import siggen

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

FS = 8e6


@pytest.mark.parametrize("tags,chips,spc,bins,n,precision", [
    (1, 300, 1, 1, 400, "fp32"),            # one item
    (7, 8192, 2, 3, 100000, "fp32"),        # 2^14 points, one tag per item
    (13, 1023, 4, 5, 100003, "fp32"),       # 2^12 points, a last tile of three tags
    (33, 1500, 1, 3, 40001, "fp32"),        # 2^13 points
    (64, 260, 2, 5, 70000, "fp32"),         # 2^11 points
    (40, 260, 1, 3, 20000, "fp32"),         # 2^10 points
    (70, 300, 8, 3, 20000, "fp32"),         # eight phases, more tags than a tile takes
    (20, 1000, 4, 3, 30000, "fp16"),        # 16-bit storage
    (20, 8192, 2, 3, 60000, "bf16"),
])
def test_chosen_tile_gives_the_named_tiles_records(tags, chips, spc, bins, n, precision):
    from paper_2005_10445_amd import Plan
    codes = siggen.make_codes(8100 + tags, tags, chips)
    freqs = [1000.0 * (k - (bins - 1) / 2) for k in range(bins)]
    x, _ = siggen.make_block(8200 + tags, n, codes, spc, FS, freqs, min(tags, 4) if n > 1000 else 1, snr_db=(-6.0, 3.0))
    xd = torch.from_numpy(x).to("cuda:0")
    kw = dict(num_bins=bins, bin_step_hz=1000.0, max_block_len=n, max_batch_blocks=3, precision=precision)
    with Plan(codes, spc, FS, **kw) as auto, Plan(codes, spc, FS, tag_tile=16, **kw) as named:
        assert auto.tuning == named.tuning and auto.tuning["tag_tile"] == min(16, tags)
        a, b = auto.detect(xd), named.detect(xd)
        assert a and a == b
        ab, bb = auto.detect_batch([xd] * 3), named.detect_batch([xd] * 3)
        assert ab == bb and len(ab) == 3 * len(a)
        auto.set_tuning(0, 16)          # from here on the named tile
        assert auto.detect(xd) == a
