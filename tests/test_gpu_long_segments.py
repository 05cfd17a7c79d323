"""The MFMA kernels where their lists of work have edges, and the rounding of bfloat16 stores."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import sgmv_workloads as wl
from helpers import decode64
from test_gpu_parity import _dev, assert_parity

pytestmark = pytest.mark.gpu

# both sides of: a few-row segment (4 rows), a tile (16), two and four tiles of a block, a block (64) and the rows of
# a shrink workgroup (64, 128); empty segments; more segments than a wave looks at in one round (64)
LENS = [1, 4, 5, 0, 16, 17, 2, 32, 33, 63, 64, 65, 3, 128, 129] + [1] * 48 + [70, 0, 6]


@pytest.mark.parametrize("dtype,r,P,same_x,h_in,h_out", [
    ("f16", 8, 1, True, 136, 264), ("bf16", 16, 1, True, 1032, 2056), ("f16", 64, 1, True, 264, 256),   # one add-on
    ("bf16", 8, 3, True, 520, 264), ("f16", 16, 2, True, 136, 2056), ("bf16", 32, 3, True, 1032, 264),  # one pass over x
    ("f16", 64, 3, True, 264, 520), ("bf16", 16, 3, False, 520, 776),                                   # side by side
    ("f16", 32, 4, True, 264, 264), ("bf16", 64, 5, False, 136, 264)])                                  # in groups of three
def test_every_edge_of_the_work_lists(dtype, r, P, same_x, h_in, h_out):
    from paper_2310_18547_amd import binding as B
    n = len(LENS)
    ws = [wl.custom(LENS, h_in, h_out, r, dtype, seed=900 + r + k, num_layers=2, scale=0.5,
                    seg_adapter=[-1 if k == P - 1 and i in (6, 11, n - 1) else i for i in range(n)]) for k in range(P)]
    ds = [_dev(w, path=B.PATH_MATRIX, n_proj=P) for w in ws]
    xs = [ds[0 if same_x else k].x[0] for k in range(P)]
    if P == 1:
        ds[0].add_lora(1)
    else:
        B.sgmv_add_lora_multi(ds[0].problem, [d.y[0] for d in ds], xs, [d.A_ptrs for d in ds], [d.B_ptrs for d in ds],
                              ds[0].seg_starts, n, 1, 0.5)
    got = [d.y_bits() for d in ds]
    for k, w in enumerate(ws):
        if same_x:
            w.x[...] = ws[0].x
        assert_parity(got[k], oracle.run_workload(w, layer_idx=1, n_threads=8), dtype, f"add-on {k} of {P}")


# The same where the expand adds the partial sums up itself: one slice, as many as it requests at a time (eight), one more,
# twice as many; binary16 with rows of v on both sides of the range factor.
@pytest.mark.parametrize("dtype,r,P,h_in,h_out,slices,large", [
    ("bf16", 8, 1, 136, 264, 1, False), ("f16", 16, 1, 1152, 2056, 8, True), ("bf16", 16, 3, 1152, 264, 9, False),
    ("f16", 8, 2, 2048, 520, 16, True), ("bf16", 16, 1, 2048, 256, 16, False)])
def test_expand_that_adds_the_partial_sums_up(dtype, r, P, h_in, h_out, slices, large):
    from paper_2310_18547_amd import binding as B
    n = len(LENS)
    scale = 2.0 ** -13 if large else 0.5
    ws = [wl.custom(LENS, h_in, h_out, r, dtype, seed=950 + r + k, num_layers=2, scale=scale,
                    seg_adapter=[-1 if k == P - 1 and i in (6, 11, n - 1) else i for i in range(n)]) for k in range(P)]
    if large:  # |v| about 2^13 in every other row, the largest of a row on both sides of 2^14
        x = decode64(ws[0].x, dtype) * np.where(np.arange(ws[0].n_tokens) % 2, 2.0 ** 13, 1.0)[:, None]
        ws[0].x[...] = wl.encode(x.astype(np.float32), dtype)
    for w in ws[1:]:
        w.x[...] = ws[0].x
    ds = [_dev(w, n_proj=P, ksplit=slices) for w in ws]
    plan = B.sgmv_plan_add_lora(ds[0].problem, n, P)
    assert (plan.kernel, plan.launches) == (B.KERNEL_MATRIX, 2)
    if P == 1:
        ds[0].add_lora(1)
    else:
        B.sgmv_add_lora_multi(ds[0].problem, [d.y[0] for d in ds], [ds[0].x[0]] * P, [d.A_ptrs for d in ds],
                              [d.B_ptrs for d in ds], ds[0].seg_starts, n, 1, scale)
    for k, w in enumerate(ws):
        assert_parity(ds[k].y_bits(), oracle.run_workload(w, layer_idx=1, n_threads=8), dtype, f"add-on {k} of {P}")


# The same at rank 8 where segments of up to four rows are strips, three and four as two pairs (63 segments to 8200 columns, 315 strips),
# the split-K factor the library's own.
@pytest.mark.parametrize("dtype,h_in", [("f16", 4104), ("bf16", 8192)])
def test_strips_of_three_and_four_rows_add_the_partial_sums_up(dtype, h_in):
    from paper_2310_18547_amd import binding as B
    lens = [3, 4, 1, 2, 4, 3, 0, 150] + [4, 3, 1, 2, 3] * 11
    w = wl.custom(lens, h_in, 8200, 8, dtype, seed=31, num_layers=2, scale=0.5, seg_adapter=[-1 if i == 4 else i % 9 for i in range(len(lens))])
    d = _dev(w)
    plan = B.sgmv_plan_add_lora(d.problem, len(lens), 1)
    assert len(lens) == 63 and (plan.kernel, plan.launches) == (B.KERNEL_MATRIX, 2)
    d.add_lora(1)
    assert_parity(d.y_bits(), oracle.run_workload(w, layer_idx=1, n_threads=8), dtype, "strips")


# The launches of a call are those of its plan, whichever of the add-ons read one x (900 rows of inputs of their own take fewer slices).
@pytest.mark.parametrize("r,P,one_x", [(16, 3, True), (16, 3, False), (8, 2, False), (16, 4, False), (64, 3, False)])
def test_launches_are_those_of_the_plan(r, P, one_x):
    from paper_2310_18547_amd import binding as B
    lens = [520, 180, 20, 180]
    ws = [wl.custom(lens, 4096, 4096, r, "bf16", seed=70 + k, scale=0.5) for k in range(P)]
    if one_x:
        for w in ws[1:]:
            w.x[...] = ws[0].x
    ds = [_dev(w, n_proj=P) for w in ws]
    plan = B.sgmv_plan_add_lora(ds[0].problem, len(lens), P)
    assert plan.kernel == B.KERNEL_MATRIX
    def call(stream=None):
        B.sgmv_add_lora_multi(ds[0].problem, [d.y[0] for d in ds], [(ds[0] if one_x else d).x[0] for d in ds], [d.A_ptrs for d in ds],
                              [d.B_ptrs for d in ds], ds[0].seg_starts, len(lens), 0, 0.5, stream)
    call()                                              # kernels loaded
    for k, w in enumerate(ws):
        assert_parity(ds[k].y_bits(), oracle.run_workload(w, n_threads=8), "bf16", f"add-on {k} of {P}")
    graph, nodes = ctypes.c_void_p(), ctypes.c_size_t()
    stream = torch.cuda.Stream(device="cuda:0")
    assert B.lib.hipStreamBeginCapture(ctypes.c_void_p(stream.cuda_stream), 1) == 0
    call(stream.cuda_stream)
    assert B.lib.hipStreamEndCapture(ctypes.c_void_p(stream.cuda_stream), ctypes.byref(graph)) == 0
    assert B.lib.hipGraphGetNodes(graph, None, ctypes.byref(nodes)) == 0
    assert B.lib.hipGraphDestroy(graph) == 0
    assert nodes.value == plan.launches


# Every kernel that stores y, by path and segment lengths: with one term per sum the fp32 result is exact, so that y is
# its rounding to nearest even, bit for bit (the operands lie within a factor of four: many ties).
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("path,lens", [("PATH_VECTOR", [1, 3, 2]), ("PATH_MATRIX", [1, 3, 2, 5, 40, 64]), ("PATH_FUSED", [1, 1, 1]),
                                       ("PATH_FUSED", [4, 20]), ("PATH_WHOLE", [1, 1, 1]), ("PATH_ROWS", [1, 3, 2])])
def test_y_is_rounded_to_nearest_even(path, lens, dtype):
    from paper_2310_18547_amd import binding as B
    w = wl.custom(lens, 256, 2056, 16, dtype, seed=31)
    rng = np.random.Generator(np.random.PCG64(32))

    def values(shape):
        sign = rng.choice([-1.0, 1.0], shape)
        return wl.encode((sign * rng.uniform(0.5, 2.0, shape)).astype(np.float32), dtype)

    one = wl.encode(np.ones(1, np.float32), dtype)[0]
    w.x[...] = one
    for a in w.A:
        a[...] = 0
        a[0, 5, 3] = one
    for b in w.B:
        b[...] = values(b.shape)
    w.y0[...] = values(w.y0.shape)
    d = _dev(w, path=getattr(B, path))
    d.add_lora()
    assert np.array_equal(d.y_bits(), oracle.run_workload(w))


# Adding nothing keeps every value of the type, subnormals, infinities and NaN (as a NaN) among them.
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("path,lens", [("PATH_VECTOR", [1, 7]), ("PATH_MATRIX", [2, 6]), ("PATH_FUSED", [1] * 8)])
def test_adding_nothing_keeps_every_value(path, lens, dtype):
    from paper_2310_18547_amd import binding as B
    w = wl.custom(lens, 256, 8192, 16, dtype, seed=33)
    w.y0[...] = np.arange(1 << 16, dtype=np.uint32).astype(np.uint16).reshape(8, 8192)
    for b in w.B:
        b[...] = 0
    d = _dev(w, path=getattr(B, path))
    d.add_lora()
    with np.errstate(invalid="ignore"):
        got, kept = decode64(d.y_bits(), dtype), decode64(w.y0, dtype)
    assert np.array_equal(got, kept, equal_nan=True)    # -0 + 0 is +0, which compares equal


# How a workgroup finds its segment: 64 segments in one round of a wave, 256 at four per lane, a search beyond, whose
# first guess is right for equal lengths and whose further rounds take 64 and 4096 segments at once
MANY = {
    "65": [3] * 65, "256": [1, 0, 7, 2] * 64, "257": [1, 0, 70, 2] * 64 + [5], "equal": [9] * 300, "empty": [0] * 400 + [20] + [0] * 200,
    "front": [3000] + [2] * 700, "back": [1, 0, 3] * 250 + [2500, 4], "far": [0, 1, 2] * 1500 + [4000] + [3, 80] * 100,
}


@pytest.mark.parametrize("lens,dtype,r,P,h_in,h_out", [
    ("65", "f16", 8, 3, 136, 264), ("65", "bf16", 64, 1, 264, 4104), ("256", "bf16", 16, 1, 136, 2056), ("256", "f16", 64, 2, 264, 264),
    ("257", "f16", 16, 1, 264, 4104), ("257", "bf16", 32, 3, 136, 264), ("equal", "bf16", 8, 1, 136, 520), ("empty", "f16", 32, 2, 136, 264),
    ("front", "bf16", 64, 1, 136, 264), ("front", "f16", 16, 3, 136, 2048), ("back", "f16", 64, 1, 264, 2048), ("back", "bf16", 16, 1, 136, 264),
    ("far", "bf16", 8, 1, 136, 264), ("far", "f16", 64, 2, 136, 264)])
def test_many_segments(lens, dtype, r, P, h_in, h_out):
    from paper_2310_18547_amd import binding as B
    lens = MANY[lens]
    n = len(lens)
    # five adapters, one segment in seven has none
    ws = [wl.custom(lens, h_in, h_out, r, dtype, seed=60 + r + k, scale=0.5,
                    seg_adapter=[-1 if i % 7 == 3 else (i * 3 + k) % 5 for i in range(n)]) for k in range(P)]
    ds = [_dev(w, path=B.PATH_MATRIX, n_proj=P) for w in ws]
    if P == 1:
        ds[0].add_lora()
    else:
        B.sgmv_add_lora_multi(ds[0].problem, [d.y[0] for d in ds], [d.x[0] for d in ds], [d.A_ptrs for d in ds],
                              [d.B_ptrs for d in ds], ds[0].seg_starts, n, 0, 0.5)
    for k, (d, w) in enumerate(zip(ds, ws)):
        assert_parity(d.y_bits(), oracle.run_workload(w, n_threads=8), dtype, f"add-on {k} of {P}")


def test_more_workgroups_than_one_dimension_of_a_grid_holds():
    """65535 segments x 257 strips of columns x 256 threads is more than 2^32."""
    from paper_2310_18547_amd import binding as B
    n, h_in, h_out, r = 65535, 8, 257 * 256, 8
    gen = torch.Generator("cuda:0").manual_seed(3)
    x, A, Bw = (torch.empty(s, dtype=torch.bfloat16, device="cuda:0").normal_(generator=gen) for s in ((n, h_in), (h_in, r), (r, h_out)))
    y = torch.ones(n, h_out, dtype=torch.bfloat16, device="cuda:0")
    seg_starts = torch.arange(n + 1, dtype=torch.int32, device="cuda:0")
    A_ptrs, B_ptrs = (torch.full((n,), t.data_ptr(), dtype=torch.int64, device="cuda:0") for t in (A, Bw))
    size = B.sgmv_workspace_bytes(n, r)
    workspace = torch.empty(size, dtype=torch.uint8, device="cuda:0")
    p = B.make_problem(B.BF16, h_in, h_out, r, 1, n, workspace=workspace, workspace_bytes=size, path=B.PATH_MATRIX)
    B.sgmv_add_lora(p, y, x, A_ptrs, B_ptrs, seg_starts, n, 0, 0.25)
    rows = torch.arange(0, n, 37, device="cuda:0")
    want = 1 + 0.25 * (x[rows].double() @ A.double() @ Bw.double())
    # y is rounded once to 8 bits; v keeps 16
    assert torch.all((y[rows].double() - want).abs() <= 2.0 ** -8 * want.abs() + 2.0 ** -13 * 8 * 4)
