"""Several add-ons of rank 64 on segments of a few rows: the MFMA kernels together, on both sides of the rule's edges."""
import numpy as np
import pytest

import oracle
import sgmv_workloads as wl
from helpers import decode64
from test_gpu_parity import _dev, assert_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,lens,P,matrix", [
    ("f16", [8] * 16, 3, True), ("bf16", [4] * 32, 2, True), ("f16", [3] * 60, 3, False), ("bf16", [9, 0, 1, 17, 5, 33, 2, 61], 4, True),
    ("f16", [4] * 99 + [3], 2, False), ("bf16", [4] * 100, 2, False), ("f16", [8] * 16, 4, True), ("f16", [8, 4], 4, False)])
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


# Calls that keep v in fp32 add-on by add-on keep it there together.  v is about 2^-18, where binary16 has six bits left: as 16-bit
# operands it gives y a relative error of 2^-8.  Here y (y0 = 0) is rounded once: 2^-11 at most, beside 2^-20 for the fp32 sums.
@pytest.mark.parametrize("lens,h_in,h_out", [([4] * 100, 4096, 520), ([30], 4096, 1608), ([9, 0, 1, 17, 5, 33, 2, 61], 4096, 1024)])
def test_small_intermediate_results(lens, h_in, h_out):
    from paper_2310_18547_amd import binding as B
    P, scale = 3, 2.0 ** 15
    ws, ds = [], []
    for k in range(P):
        w = wl.custom(lens, h_in, h_out, 64, "f16", seed=40 + k, scale=scale, seg_adapter=[i % 6 for i in range(len(lens))])
        for bits, size in [(w.x, 2.0 ** -9)] + [(a, 2.0 ** -15) for a in w.A]:
            values = decode64(bits, "f16")
            bits[...] = wl.encode((values * size / np.std(values)).astype(np.float32), "f16")
        w.y0[...] = 0
        ws.append(w)
        ds.append(_dev(w, n_proj=P))
    B.sgmv_add_lora_multi(ds[0].problem, [d.y[0] for d in ds], [d.x[0] for d in ds], [d.A_ptrs for d in ds], [d.B_ptrs for d in ds],
                          ds[0].seg_starts, len(lens), 0, scale)
    for d, w in zip(ds, ws):
        x = decode64(w.x, "f16")
        exact = np.zeros((w.n_tokens, h_out))
        for i, a in enumerate(w.seg_adapter):
            rows = slice(w.seg_starts[i], w.seg_starts[i + 1])
            exact[rows] = scale * (x[rows] @ decode64(w.A[a][0], "f16") @ decode64(w.B[a][0], "f16"))
        error = np.linalg.norm(decode64(d.y_bits(), "f16") - exact) / np.linalg.norm(exact)
        assert 2.0 ** -4 < np.std(exact) < 2.0 ** 8 and error <= 2.0 ** -11, error
