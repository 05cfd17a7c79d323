"""Slice counts between the powers of two (single add-ons that leave compute units free): edges of the rule."""
import pytest

import oracle
import sgmv_workloads as wl
from test_gpu_parity import _dev, assert_parity

pytestmark = pytest.mark.gpu


# 33 .. 48 and 49 items are padded to 40, 48 and 56; one segment or row per item; widths that leave the last slice short
# or empty of columns; the eight slices of a very wide input on more workgroups than units
@pytest.mark.parametrize("dtype,lens,h_in,h_out,r,slices", [
    ("f16", [1] * 33, 5120, 5120, 16, 5), ("bf16", [1] * 48, 5120, 5128, 32, 5), ("f16", [1] * 49, 5120, 5120, 32, 4),
    ("bf16", [1] * 40, 11000, 4104, 16, 6), ("f16", [1] * 40, 4104, 11016, 8, 6), ("f16", [1] * 48, 5120, 2056, 64, 5),
    ("bf16", [20, 1, 3, 0, 11, 10], 5120, 5120, 64, 5), ("f16", [1] * 41, 11008, 520, 32, 8)])
def test_add_on_with_odd_slice_counts(dtype, lens, h_in, h_out, r, slices):
    from paper_2310_18547_amd import binding as B
    w = wl.custom(lens, h_in, h_out, r, dtype, seed=77 + r, scale=0.5)
    d = _dev(w)
    plan = B.sgmv_plan_add_lora(d.problem, w.n_segs, 1)
    assert (plan.kernel, plan.slices) == (B.KERNEL_FUSED, slices)
    d.add_lora()
    assert_parity(d.y_bits(), oracle.run_workload(w, n_threads=8), dtype, f"{len(lens)} segments, {slices} slices")
