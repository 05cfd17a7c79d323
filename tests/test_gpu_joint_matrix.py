"""Several add-ons of rank 64 on segments of a few rows: the MFMA kernels together, on both sides of the rule's edges."""
import pytest

import oracle
import sgmv_workloads as wl
from test_gpu_parity import _dev, assert_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,lens,P,matrix", [
    ("f16", [8] * 16, 3, True), ("bf16", [4] * 32, 2, True), ("f16", [3] * 60, 3, False), ("bf16", [9, 0, 1, 17, 5, 33, 2, 61], 4, True),
    ("f16", [4] * 99 + [3], 2, False), ("bf16", [4] * 100, 2, True)])
def test_several_add_ons_of_rank_64(dtype, lens, P, matrix):
    from paper_2310_18547_amd import binding as B
    ws = [wl.custom(lens, 4096, 4104, 64, dtype, seed=17 + k, scale=0.5, seg_adapter=[(i + k) % 6 - (i % 7 == 3) for i in range(len(lens))])
          for k in range(P)]
    ds = [_dev(w, n_proj=P) for w in ws]
    plan = B.sgmv_plan_add_lora(ds[0].problem, len(lens), P)
    assert (plan.kernel == B.KERNEL_MATRIX) == matrix
    B.sgmv_add_lora_multi(ds[0].problem, [d.y[0] for d in ds], [d.x[0] for d in ds], [d.A_ptrs for d in ds], [d.B_ptrs for d in ds],
                          ds[0].seg_starts, len(lens), 0, 0.5)
    for k, (d, w) in enumerate(zip(ds, ws)):
        assert_parity(d.y_bits(), oracle.run_workload(w, n_threads=8), dtype, f"add-on {k} of {P}")
