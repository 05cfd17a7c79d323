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
    ("f16", [4] * 99 + [3], 2, False), ("bf16", [4] * 100, 2, True), ("f16", [8] * 16, 4, True), ("f16", [8, 4], 4, False)])
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


# Add-ons that keep v in fp32 one by one lose no bit of it together: y0 is the result negated and rounded, so that what is left shows errors
# far below y's rounding, and v lies about 2^-18 (binary16 has six bits of it left: two 16-bit parts gave 2^-8), 1 or 2^18.  The sums are
# taken in another order, on the matrix cores in chains of up to h_in / 32 = 128 roundings of a running sum: sqrt(128 / 3) / 2 times 2^-24 as
# a root mean square, 2^-22, for v and less for its 64 products: twice that, or a quarter more than the separate calls.
@pytest.mark.parametrize("dtype,v_size", [("f16", -18), ("f16", 0), ("f16", 18), ("bf16", -18), ("bf16", 0)])
@pytest.mark.parametrize("lens,h_in,h_out", [([4] * 100, 2048, 520), ([30], 4096, 1608), ([9, 0, 1, 17, 5, 33, 2, 61], 4096, 1024),
                                             ([1, 2] * 7 + [30, 13], 2048, 11008)])      # strips of one and two rows
def test_no_bits_of_v_are_lost(dtype, v_size, lens, h_in, h_out):
    from paper_2310_18547_amd import binding as B
    P, scale = 3, 2.0 ** -v_size
    ws, exact = [], []
    for k in range(P):
        w = wl.custom(lens, h_in, h_out, 64, dtype, seed=40 + k, scale=scale, seg_adapter=[i % 6 for i in range(len(lens))])
        for bits, size in [(w.x, 2.0 ** (v_size // 2))] + [(a, 2.0 ** (v_size // 2) * h_in ** -0.5) for a in w.A]:
            values = decode64(bits, dtype)
            bits[...] = wl.encode((values * size / np.std(values)).astype(np.float32), dtype)
        x, delta = decode64(w.x, dtype), np.zeros((w.n_tokens, h_out))
        for i, a in enumerate(w.seg_adapter):
            rows = slice(w.seg_starts[i], w.seg_starts[i + 1])
            delta[rows] = scale * (x[rows] @ decode64(w.A[a][0], dtype) @ decode64(w.B[a][0], dtype))
        w.y0[...] = wl.encode(-delta.astype(np.float32), dtype)
        ws.append(w)
        exact.append(delta + decode64(w.y0, dtype))
    ds = [_dev(w, n_proj=P) for w in ws]
    assert B.sgmv_plan_add_lora(ds[0].problem, len(lens), P).kernel == B.KERNEL_MATRIX
    assert B.sgmv_plan_add_lora(ds[0].problem, len(lens), 1).kernel != B.KERNEL_MATRIX
    error = lambda: np.array([np.linalg.norm(decode64(d.y_bits(), dtype) - e) for d, e in zip(ds, exact)])
    for d in ds:
        d.add_lora(0)
    apart = error()
    for d in ds:
        d.y[0].copy_(d.y0)
    B.sgmv_add_lora_multi(ds[0].problem, [d.y[0] for d in ds], [d.x[0] for d in ds], [d.A_ptrs for d in ds], [d.B_ptrs for d in ds],
                          ds[0].seg_starts, len(lens), 0, scale)
    assert np.all(error() <= np.maximum(1.25 * apart, [2.0 ** -21 * np.linalg.norm(e - decode64(w.y0, dtype)) for w, e in zip(ws, exact)]))
