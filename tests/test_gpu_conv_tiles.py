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


@pytest.mark.parametrize("frames", [16416, 20481])            # 513 and 641 pieces of 64 rows, two blocks
def test_gradients_of_many_rows(frames):
    """Above 2048 pieces x channel groups the weight gradients are summed in twice as many chunks: two
    blocks' gradient is the mean of each one's, which fewer chunks sum.  1/rows is a power of two apart,
    so the terms are the same; a sum takes at most 64 additions of 2^-24 of a partial sum on either
    side, partial sums within 4 of the layer's largest gradient: 2 * 64 * 4 * 2^-24 = 3.1e-5."""
    from paper_2005_10445_amd.proposals import Network
    g = torch.Generator().manual_seed(8700 + frames)
    x = torch.randn(2 * frames, 256, generator=g).to(torch.bfloat16).to("cuda:0")
    lab = (torch.rand(2 * frames, generator=g) < 0.3).float().to("cuda:0")
    with Network("bf16", max_rows=2 * frames, max_block_len=256) as net:
        p = 0.05 * torch.randn(net.num_params, generator=torch.Generator().manual_seed(8701))
        net.set_params(p.numpy())
        loss, whole = net.gradients(x, lab, 2.0, nblocks=2)
        parts = [net.gradients(x[o:o + frames].clone(), lab[o:o + frames].clone(), 2.0) for o in (0, frames)]
    mean = (parts[0][1].double() + parts[1][1].double()) / 2
    assert abs(loss - (parts[0][0] + parts[1][0]) / 2) <= 1e-5 * loss
    bounds = [0]
    for cin in (256, 64, 64, 64):
        bounds += [bounds[-1] + 5 * cin * 64, bounds[-1] + 5 * cin * 64 + 64]
    bounds.append(net.num_params)
    for a, b in zip(bounds, bounds[1:]):
        assert (whole[a:b].double() - mean[a:b]).abs().max() <= 3.1e-5 * mean[a:b].abs().max(), (a, b)
