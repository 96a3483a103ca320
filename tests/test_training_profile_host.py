"""Summary of a training trace: every kernel whose work is known gets its rate, and a trace
whose kernels go by other names is refused."""
import csv

import pytest

from paper_2005_10445_amd import profiling

KERNELS = ("k_stft(BlockSource, long)", "k_conv_tile<true, 4>(void const*)", "k_conv_tile<false, 4>(void const*)",
           "k_conv_dw_taps<1>(int)", "k_conv_dw_taps<2>(int)", "k_conv_dw_taps<4>(int)", "k_conv_dw_taps<8>(int)",
           "k_head<true>(void const*)", "k_adam(float*)")


def _trace(path, kernels, steps):
    with open(path / "t_kernel_trace.csv", "w", newline="") as f:
        w = csv.writer(f)
        w.writerow(["Kernel_Name", "Start_Timestamp", "End_Timestamp"])
        t = 0
        for _ in range(steps):
            for k in kernels:
                w.writerow([f"void acq::learned::(anonymous namespace)::{k}", t, t + 10000])
                t += 20000


def test_every_known_kernel_has_its_rate(tmp_path):
    _trace(tmp_path, KERNELS, 4)
    lines = profiling.learned_summary(str(tmp_path), "cmd", 8, 1 << 20, 4, 1).splitlines()
    rows = {ln.split("  ")[0]: ln for ln in lines if ln.startswith("k_")}
    assert len(rows) == len(KERNELS)
    for name, ln in rows.items():
        assert ("TFLOP/s)" in ln) == (not name.startswith("k_adam")), ln
    frames = ((1 << 20) - 256) // 128 + 1
    gflop = 2.0 * 8 * frames * 64 * 5 * (256 + 3 * 64) / 1e9
    assert f"{gflop:.2f}" in rows["k_conv_tile<true, 4>"] and f"{gflop / 10e-3:.1f}" in rows["k_conv_tile<true, 4>"]


@pytest.mark.parametrize("change", [("k_conv_tile<true, 4>", "k_conv_rows<true>"), ("k_stft", "k_frames")])
def test_renamed_kernels_are_refused(tmp_path, change):
    _trace(tmp_path, [k.replace(*change) for k in KERNELS], 3)
    with pytest.raises(ValueError, match="belongs to one kernel"):
        profiling.learned_summary(str(tmp_path), "cmd", 8, 1 << 20, 3, 1)
