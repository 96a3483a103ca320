"""Row tiles of the bf16 convolutions: a network's logits of a batch (tiles of 64
rows above 40,960) are bit for bit those of its blocks alone (tiles of 32), for
block lengths that put block edges anywhere in a tile."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("blocks,frames", [(43, 1000), (5860, 7), (40961, 1), (2, 20481), (1, 41024), (1249, 33)])
def test_logits_do_not_depend_on_the_tile(blocks, frames):
    from paper_2005_10445_amd.proposals import Network
    rows = blocks * frames
    x = torch.randn(rows, 256, generator=torch.Generator().manual_seed(8600 + frames)).to(torch.bfloat16).to("cuda:0")
    with Network("bf16", max_rows=rows, max_block_len=256) as net:
        p = 0.05 * torch.randn(net.num_params, generator=torch.Generator().manual_seed(8601))
        net.set_params(p.numpy())
        whole = net.forward(x, nblocks=blocks)
        if blocks == 1:                                   # the rows that the cut's edge does not reach
            assert torch.equal(whole[:40960 - 30], net.forward(x[:40960])[:40960 - 30])
            return
        for b in sorted({0, 1, blocks // 2, blocks - 1}):
            own = slice(b * frames, (b + 1) * frames)
            assert torch.equal(net.forward(x[own].clone()), whole[own])
