"""The power map's median: exact (a value of the map's own powers, at the lower
middle rank) at the edges of its workgroups' shares, for equal powers, and on
repeated calls of one network."""
import numpy as np
import pytest

import oracle.learned as ol

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("frames", [1, 4, 5, 32, 33, 2049])       # 4 frames a workgroup, 32 a median one
@pytest.mark.parametrize("kind", ["noise", "constant", "zero"])
def test_median_of_a_block(frames, kind):
    from paper_2005_10445_amd.proposals import Network
    n = 256 + 128 * (frames - 1)
    rng = np.random.default_rng(8500 + frames)
    x = {"noise": rng.standard_normal(n) + 1j * rng.standard_normal(n), "constant": np.full(n, 0.5 - 0.25j),
         "zero": np.zeros(n)}[kind].astype(np.complex64)
    xd = torch.from_numpy(x).to("cuda:0")
    with Network("fp32", max_rows=4096, max_block_len=n) as net:
        got = [net.power_map(xd) for _ in range(3)]
        maps = [m.float().cpu().numpy().reshape(-1).copy() for m, _ in got]
    meds = [med for _, med in got]
    assert meds[0] == meds[1] == meds[2]
    assert all((m == maps[0]).all() for m in maps)
    if kind == "zero":
        assert meds[0] == 0.0 and (maps[0] == 0.0).all()
        return
    _, want = ol.power_map(x)
    if kind == "noise":
        # FP32 transforms of 256 points: 1e-5 covers 16 roundings of 2^-24 at
        # powers no smaller than 1/16 of the mean, where the middle lies
        assert abs(meds[0] - want) <= 1e-5 * want
        # ln(P / median): the middle rank's own entry is ln 1
        assert np.sort(maps[0])[(maps[0].size - 1) // 2] == 0.0
