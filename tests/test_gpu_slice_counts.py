"""Slice counts between the powers of two (single add-ons that leave compute units free) and the sizes from which the
one-row kernels read their weights past the caches: edges of both rules."""
import numpy as np
import pytest
import torch

import oracle
import sgmv_workloads as wl
from test_gpu_parity import _dev, assert_parity

pytestmark = pytest.mark.gpu


# 33 .. 48 and 49 items are padded to 40, 48 and 56; one segment or row per item; widths that leave the last slice short
# or empty of columns; the eight slices of a very wide input on more workgroups than units
@pytest.mark.parametrize("dtype,lens,h_in,h_out,r,slices", [
    ("f16", [1] * 33, 5120, 5120, 16, 5), ("bf16", [1] * 48, 5120, 5128, 32, 5), ("f16", [1] * 49, 5120, 5120, 32, 4),
    ("bf16", [1] * 40, 11000, 4104, 16, 6), ("f16", [1] * 40, 4104, 11016, 8, 6), ("f16", [1] * 48, 5120, 2056, 64, 5),
    ("bf16", [20, 1, 3, 0, 11, 10], 5120, 5120, 64, 5), ("f16", [1] * 41, 11008, 520, 32, 8),
    ("bf16", [9, 6, 4, 4, 3, 3, 3, 3] + [1] * 10, 13824, 520, 64, 8)])
def test_add_on_with_odd_slice_counts(dtype, lens, h_in, h_out, r, slices):
    from paper_2310_18547_amd import binding as B
    w = wl.custom(lens, h_in, h_out, r, dtype, seed=77 + r, scale=0.5)
    d = _dev(w)
    plan = B.sgmv_plan_add_lora(d.problem, w.n_segs, 1)
    assert (plan.kernel, plan.slices) == (B.KERNEL_FUSED, slices)
    d.add_lora()
    assert_parity(d.y_bits(), oracle.run_workload(w, n_threads=8), dtype, f"{len(lens)} segments, {slices} slices")


# 4 Mi weights on either side, and three rows an adapter on either side of the per-row launches
@pytest.mark.parametrize("dtype,lens,h_in,r,by_rows", [
    ("f16", [2] * 24, 8192, 32, True), ("bf16", [2] * 15, 8192, 32, True), ("bf16", [4] * 16, 8192, 32, True),
    ("f16", [3] * 18, 11008, 64, True), ("bf16", [1] * 63, 4096, 16, False), ("f16", [1] * 64, 4096, 16, False)])
def test_shrink_around_the_size_that_streams(dtype, lens, h_in, r, by_rows):
    from paper_2310_18547_amd import binding as B
    w = wl.custom(lens, h_in, 64, r, dtype, seed=90 + r, num_layers=2, seg_adapter=[i % 7 for i in range(len(lens))])
    d = _dev(w)
    plan = B.sgmv_plan_shrink(d.problem, w.n_segs)
    assert plan.launches == 1 and plan.kernel == (B.KERNEL_FUSED if by_rows or dtype == "bf16" else B.KERNEL_WHOLE)
    v = torch.ones(w.n_tokens, r, dtype=torch.float32, device="cuda:0")
    d.shrink(v, 1)
    ref = oracle.run_workload(w, op="shrink", layer_idx=1, v=np.ones((w.n_tokens, r), np.float32), n_threads=8)
    assert np.all(np.abs(v.cpu().numpy() - ref) <= 2e-3 + 2e-2 * np.abs(ref))


@pytest.mark.parametrize("dtype,lens,P,r", [("f16", [3] * 20, 2, 32), ("bf16", [3] * 16, 2, 32), ("bf16", [4] * 15, 2, 32), ("f16", [2] * 9, 2, 64)])
def test_several_add_ons_around_the_size_that_streams(dtype, lens, P, r):
    from paper_2310_18547_amd import binding as B
    ws = [wl.custom(lens, 4096, 4104, r, dtype, seed=97 + k, scale=0.5, seg_adapter=[(i + k) % 5 for i in range(len(lens))]) for k in range(P)]
    ds = [_dev(w, n_proj=P) for w in ws]
    plan = B.sgmv_plan_add_lora(ds[0].problem, len(lens), P)
    assert (plan.kernel, plan.launches) == (B.KERNEL_MULTI_SIDE, 1)
    B.sgmv_add_lora_multi(ds[0].problem, [d.y[0] for d in ds], [d.x[0] for d in ds], [d.A_ptrs for d in ds], [d.B_ptrs for d in ds],
                          ds[0].seg_starts, len(lens), 0, 0.5)
    for k, (d, w) in enumerate(zip(ds, ws)):
        assert_parity(d.y_bits(), oracle.run_workload(w, n_threads=8), dtype, f"add-on {k} of {P}")
