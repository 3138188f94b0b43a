"""bench.py's names and bounds of the step kernels, from the statistics of a call (CPU)."""
import pytest

import bench

STENCIL = {"ms_steps1": 0.86, "launches1": 14, "bytes1": 14 * 165e6, "ms_steps23": 1.18, "launches23": 28,
           "bytes23": 28 * 164e6, "dia_diagonals": 5, "dia_constant": 1, "degree": 80, "k": 20, "k_G": 20,
           "block_cols1": 20, "block_cols23": 20, "dot_mode_used": 2, "n": 1 << 20}
SMALL = {"ms_steps1": 0.055, "launches1": 1, "bytes1": 1e5, "ms_steps23": 0.075, "launches23": 1, "bytes23": 1e5,
         "dia_diagonals": 5, "dia_constant": 1, "degree": 40, "k": 10, "k_G": 10, "block_cols1": 10,
         "block_cols23": 20, "dot_mode_used": 2, "n": 1024}
LARGE = {**STENCIL, "ms_steps1": 10.9, "bytes1": 14 * 2004e6, "ms_steps23": 13.0, "launches23": 14,
         "bytes23": 14 * 3907e6, "k": 10, "k_G": 10, "block_cols1": 10, "n": 25000000}   # beyond the Infinity Cache
SINGLE = {**STENCIL, "launches1": 80, "launches23": 80, "block_cols23": 20, "dia_constant": 0}


@pytest.mark.parametrize("st,name,bound,unit", [
    (STENCIL, "fused_kernel", "valu", "TFLOP/s"),
    (LARGE, "fused_kernel", "hbm", "GB/s"),
    (SMALL, "resident_kernel", "lds_latency", "TFLOP/s"),
    ({**SMALL, "dia_diagonals": 0, "dia_constant": 0}, "resident_kernel", "lds_latency", "TFLOP/s"),
    (SINGLE, "step_kernel", "infinity_cache", "GB/s"),
])
def test_kernel_names_and_bounds(st, name, bound, unit):
    rec = bench.kernel_records(st)["quadform"]
    assert rec["kernel"] == name and bench.step_bound(rec) == bound
    r = bench.roofline("quadform", rec, st, 5 * st["n"])
    assert r["unit"] == unit and r["bound"] == bound and r["frac"] == pytest.approx(r["achieved"] / r["peak"])
    assert 0 < r["frac"] < 1
    assert (name == "fused_kernel") == ("moves once per launch" in bench.working_set(rec))


def test_useful_flops_of_a_phase():
    rec = bench.kernel_records(STENCIL)["quadform"]
    steps, cols, n = 40, 40, 1 << 20   # ceil(80 / 2) steps of k + k_G columns
    want = steps * cols * (2 * 5 * n + 4 * n) / (STENCIL["ms_steps23"] * 1e-3) / 1e12
    assert bench.step_tflops("quadform", rec, STENCIL, 5 * n) == pytest.approx(want)
