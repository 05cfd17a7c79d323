"""Per-row launches that take two rows of a segment to an item: odd and even segment lengths, empty segments, segments
without an adapter, more segments than a wave has lanes, the slices of a width that leave the last one short."""
import numpy as np
import pytest
import torch

import oracle
import sgmv_workloads as wl
from test_gpu_parity import _dev, assert_parity

pytestmark = pytest.mark.gpu

MIXED = [7, 0, 1, 2, 0, 0, 3, 20, 1, 1, 0, 4, 0, 5, 16, 68]   # 128 rows
MANY = [2, 0, 3, 1, 0, 2, 1, 2] * 9                            # 72 segments, 99 rows


def _workload(lens, h_in, h_out, r, dtype):
    adapters = [-1 if i % 9 == 4 else i % 11 for i in range(len(lens))]
    return wl.custom(lens, h_in, h_out, r, dtype, seed=60 + r, num_layers=2, seg_adapter=adapters, scale=0.5)


def _is_paired(plan, w, slices):
    from paper_2310_18547_amd import binding as B
    places = -(-((w.n_tokens + w.n_segs) // 2) // 8) * 8
    return (plan.kernel, plan.launches, plan.slices, plan.workgroups) == (B.KERNEL_FUSED, 1, slices, slices * places)


@pytest.mark.parametrize("dtype,lens,h_in,h_out,r,slices", [
    ("f16", MIXED, 11008, 520, 8, 8), ("bf16", MIXED, 9992, 2056, 8, 8), ("f16", [2] * 64, 11008, 4104, 16, 8),
    ("bf16", [2, 2, 1, 3] * 16, 11008, 8192, 16, 8), ("f16", MANY, 11000, 264, 8, 8), ("bf16", [50, 19] + [3, 0, 2, 1] * 4 + [3], 6152, 4096, 32, 4),
    ("f16", [50, 19] + [3, 0, 2, 1] * 4 + [3], 5120, 1032, 32, 4), ("bf16", [200] + [0, 7, 1, 3, 1, 2] * 4, 8192, 1024, 8, 4),
    # rank 8 with one lane group (slices of more than 1024 columns), rank 32 with eight and with two passes over B_i
    ("f16", [200] + [0, 7, 1, 3, 1, 2] * 4, 8192, 8192, 8, 4), ("bf16", MIXED, 11008, 11000, 8, 8),
    ("bf16", [50, 19] + [3, 0, 2, 1] * 4 + [3], 5120, 1024, 32, 4), ("f16", [50, 19] + [3, 0, 2, 1] * 4 + [3], 8192, 8192, 32, 4),
    ("bf16", [50, 19] + [3, 0, 2, 1] * 4 + [3], 8192, 5000, 32, 4)])
def test_add_on(dtype, lens, h_in, h_out, r, slices):
    from paper_2310_18547_amd import binding as B
    w = _workload(lens, h_in, h_out, r, dtype)
    d = _dev(w)
    assert _is_paired(B.sgmv_plan_add_lora(d.problem, w.n_segs, 1), w, slices)
    ref = oracle.run_workload(w, layer_idx=1, n_threads=8)
    d.add_lora(1)
    assert_parity(d.y_bits(), ref, dtype, "pairs of rows")
    d.y[0].copy_(d.y0)
    d.add_lora(1)                            # the workspace's second generation
    assert_parity(d.y_bits(), ref, dtype, "pairs of rows, again")
    assert d.check() == 0


@pytest.mark.parametrize("dtype,lens,h_in,r,slices", [
    ("f16", MIXED, 11008, 8, 8), ("bf16", MANY, 9992, 16, 8), ("f16", [96, 32], 13824, 16, 8), ("bf16", [2, 2, 1, 3] * 16, 11008, 32, 8),
    ("f16", [2, 1, 2] * 20, 8200, 16, 8), ("bf16", [100, 0, 100, 55], 9000, 16, 5)])
def test_shrink(dtype, lens, h_in, r, slices):
    from paper_2310_18547_amd import binding as B
    w = _workload(lens, h_in, 64, r, dtype)
    d = _dev(w)
    assert _is_paired(B.sgmv_plan_shrink(d.problem, w.n_segs), w, slices)
    v = torch.ones(w.n_tokens, r, dtype=torch.float32, device="cuda:0")
    d.shrink(v, 1)
    ref = oracle.run_workload(w, op="shrink", layer_idx=1, v=np.ones((w.n_tokens, r), np.float32), n_threads=8)
    assert np.all(np.abs(v.cpu().numpy() - ref) <= 2e-3 + 2e-2 * np.abs(ref))
    assert d.check() == 0


# The bounded wait, forced from the host: workgroup 0 tags its partial sums with a generation that its neighbours do not expect, so the
# first pair is given up: both its rows stay as they were, all others are finished.
@pytest.mark.parametrize("op", ["add_lora", "shrink"])
def test_a_pair_that_is_given_up_stays_as_it_was(op):
    from paper_2310_18547_amd import binding as B
    lens = [3, 48] + [3, 0, 2, 1] * 7 + [3]                        # 96 rows
    w = _workload(lens, 6152, 4096, 32, "f16") if op == "add_lora" else _workload([3, 56] + lens[2:], 11008, 64, 8, "f16")
    d = _dev(w, spin_limit=5000)
    plan = (B.sgmv_plan_add_lora(d.problem, w.n_segs, 1) if op == "add_lora" else B.sgmv_plan_shrink(d.problem, w.n_segs))
    assert _is_paired(plan, w, 4 if op == "add_lora" else 8)
    v0 = np.full((w.n_tokens, w.r), 3.0, np.float32)
    ref = oracle.run_workload(w, layer_idx=1, n_threads=8) if op == "add_lora" else oracle.run_workload(w, op="shrink", layer_idx=1, v=v0.copy())
    v = torch.from_numpy(v0.copy()).to("cuda:0")
    d.workspace[0:4].view(torch.int32).fill_(77)
    torch.cuda.synchronize()
    if op == "add_lora":
        d.add_lora(1)
    else:
        d.shrink(v, 1)
    assert d.check() == 8                                          # SGMV_ERR_TIMEOUT
    if op == "add_lora":
        got = d.y_bits()
        assert np.array_equal(got[:2], w.y0[:2])
        assert_parity(got[2:], ref[2:], "f16", "the other rows")
    else:
        got = v.cpu().numpy()
        assert np.all(got[:2] == 3.0)
        assert np.all(np.abs(got[2:] - ref[2:]) <= 2e-3 + 2e-2 * np.abs(ref[2:]))
