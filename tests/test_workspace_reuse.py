"""One backward workspace for several sequence lengths: what the size function
reports for a longer sequence is enough for a shorter one, whose work is then
split only as far as its partial sums fit."""

import ctypes

import pytest
import torch

import parity as P
from paper_2507_02754_amd import binding, load_library
from paper_2507_02754_amd import (simplicial_attn_bwd, simplicial_attn_bwd_fused, simplicial_attn_bwd_fused_reduce,
                                  simplicial_attn_bwd_gqa,
                                  simplicial_attn_bwd_gqa_workspace_size, simplicial_attn_bwd_key_side,
                                  simplicial_attn_bwd_noalloc, simplicial_attn_bwd_preprocess,
                                  simplicial_attn_bwd_query_side, simplicial_attn_bwd_workspace_size,
                                  simplicial_attn_det_bwd, simplicial_attn_det_bwd_workspace_size,
                                  simplicial_attn_det_fwd, simplicial_attn_fwd, simplicial_attn_fwd_gqa)
from paper_2507_02754_amd.workloads import draw

BF16, FP32 = torch.bfloat16, torch.float32
A = ctypes.c_void_p(0x10000)  # never touched: without a GPU no kernel is launched


@pytest.mark.skipif(torch.cuda.device_count() > 0, reason="fake-pointer checks run only where no GPU is visible")
@pytest.mark.parametrize("h,d,w1,w2,dtype", [
    (8, 128, 512, 32, BF16), (8, 128, 256, 32, BF16), (1, 64, 128, 5, BF16), (2, 128, 1024, 64, BF16),
    (16, 64, 512, 24, BF16), (4, 128, 128, 128, FP32), (4, 64, 256, 16, FP32), (64, 32, 100, 32, BF16)])
def test_a_longer_sequence_covers_shorter_ones(h, d, w1, w2, dtype):
    """Sizes alone, no launch: SA_ERR_WORKSPACE (3) for none of the pairs."""
    lib = load_library()
    dt, scale = binding._DTYPES[dtype], ctypes.c_float(0.1)
    lengths = [1, 31, 33, 64, 100, 129, 200, 300, 515, 700, 1021, 1500, 2000, 3000, 4096, 6001, 8192]
    size = ctypes.c_size_t
    for hi, longer in enumerate(lengths):
        ws = simplicial_attn_bwd_workspace_size(1, longer, h, d, w1, w2, dtype)
        det = simplicial_attn_det_bwd_workspace_size(1, longer, h, d, w1, w2, dtype)
        gqa = simplicial_attn_bwd_gqa_workspace_size(1, longer, 2 * h, h, d, w1, w2, dtype)
        for n in lengths[:hi + 1]:
            args = (d, w1, w2, scale, dt, None)
            assert lib.simplicial_attn_bwd(*[A] * 14, size(ws), 1, n, h, *args) != 3, (longer, n)
            if w2 <= 32:  # (one kernel path for every length)
                assert lib.simplicial_attn_det_bwd(*[A] * 14, size(det), 1, n, h, *args) != 3, (longer, n)
            assert lib.simplicial_attn_bwd_gqa(*[A] * 14, size(gqa), 1, n, 2 * h, h, *args) != 3, (longer, n)
            assert lib.simplicial_attn_bwd_preprocess(*[A] * 3, size(ws), 1, n, h, d, w1, w2, dt, None) != 3
            assert lib.simplicial_attn_bwd_query_side(*[A] * 11, size(ws), 1, n, h, *args) != 3, (longer, n)
            assert lib.simplicial_attn_bwd_key_side(*[A] * 10, size(ws), 1, n, h, *args) != 3, (longer, n)


def _least(n, h, d, w2, dtype):
    """Delta, and for the bf16 kernels the boundary sums of chunks of 128 queries."""
    delta = (4 * n * h + 255) // 256 * 256
    if dtype == FP32 or d < 64 or w2 > 64:
        return delta
    return delta + 16 * h * -(-n // 128) * (31 if w2 <= 32 else 63) * d


def _order_bound(r, dtype):
    """The same float32 terms in another order: a few hundred roundings of 2^-24 of
    the largest sum; with bf16 results the last rounding may then fall the other
    way, one unit in the last of 8 bits (2^-7 of the element where its mantissa
    is 1). grouped-query dK', dV': of each query head, then summed."""
    return 2.0 ** -7 * r.abs() + 2.0 ** -13 * r.abs().max() if dtype == BF16 else 1e-5 * r.abs().max()


@pytest.mark.gpu
@pytest.mark.parametrize("kind,n,longer,h,d,w1,w2,dtype", [
    ("plain", 3000, 4096, 8, 128, 512, 32, BF16),   # query chunks of 32, key blocks in 4 shares: 146 MB, 16 MB given
    ("plain", 1021, 4096, 8, 128, 256, 32, BF16),
    ("plain", 700, 0, 4, 64, 300, 64, BF16),        # 0: no more than is needed without a split
    ("stages", 1021, 0, 8, 128, 256, 17, BF16),
    ("det", 1021, 0, 8, 128, 256, 32, BF16),
    ("gqa", 1100, 0, 2, 128, 200, 32, BF16),
    ("gqa", 200, 0, 2, 64, 70, 9, FP32),
    ("plain", 1500, 1536, 4, 128, 60, 128, FP32),
    ("plain", 700, 0, 2, 64, 90, 33, FP32),
    ("stages", 300, 0, 3, 32, 50, 8, FP32),
    ("plain", 300, 0, 9, 32, 50, 16, FP32),         # one chunk per head (the rows above: plain kernels)
    ("plain", 500, 0, 4, 128, 64, 96, BF16),
])
def test_results_with_a_smaller_workspace(kind, n, longer, h, d, w1, w2, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    print(f"\n[workspace] {kind} N={n} of {longer} H={h} D={d} w1={w1} w2={w2} {dtype}", flush=True)
    group = 3 if kind == "gqa" else 1
    x = [t.cuda() for t in draw((1, n, h, d), seed=n + d, dtype=dtype)]
    if group > 1:
        x[0], x[5] = (t.cuda() for t in draw((1, n, h * group, d), seed=n, dtype=dtype)[:2])
    scale = d ** -0.5
    fwd = {"det": simplicial_attn_det_fwd, "gqa": simplicial_attn_fwd_gqa}.get(kind, simplicial_attn_fwd)
    o, lse = fwd(*x[:5], w1, w2, scale)

    def size(length):
        if kind == "gqa":
            return simplicial_attn_bwd_gqa_workspace_size(1, length, h * group, h, d, w1, w2, dtype)
        if kind == "det":
            return simplicial_attn_det_bwd_workspace_size(1, length, h, d, w1, w2, dtype)
        return simplicial_attn_bwd_workspace_size(1, length, h, d, w1, w2, dtype)

    if longer:
        given = size(longer)
    elif kind == "gqa":
        per = (n * h * group * d * dtype.itemsize + 255) // 256 * 256
        given = max(_least(n, h * group, d, w2, dtype), 4 << 20 if dtype == BF16 else 0) + (2 if dtype == BF16 else 8) * per
    else:
        given = _least(n, h, d, w2, dtype)
        if kind != "stages" and given < 4 << 20 and dtype == BF16 and d >= 64 and w2 <= 64:
            given = 4 << 20
    assert given < size(n)
    # bytes past the workspace stay as they are
    buf = torch.full((given + 65536,), 0x5A, dtype=torch.uint8, device="cuda")
    ws = buf[:given]

    def run(w):
        if kind == "stages":
            w = w if w is not None else torch.empty(size(n), dtype=torch.uint8, device="cuda")
            simplicial_attn_bwd_preprocess(o, x[5], w1, w2, w)
            dq, dkp, dvp = simplicial_attn_bwd_query_side(*x, lse, w1, w2, w, scale)
            dk, dv = simplicial_attn_bwd_key_side(*x, lse, w1, w2, w, scale)
            return dq, dk, dkp, dv, dvp
        bwd = {"det": simplicial_attn_det_bwd, "gqa": simplicial_attn_bwd_gqa}.get(kind, simplicial_attn_bwd)
        return bwd(*x[:5], o, x[5], lse, w1, w2, scale, workspace=w)

    got, again, ref = run(ws), run(ws), run(None)
    torch.cuda.synchronize()
    assert bool((buf[given:] == 0x5A).all())
    for name, a, b, r in zip(P.GRAD_NAMES, got, again, ref):
        assert torch.equal(a, b), name
        a, r = a.double(), r.double()
        assert bool(((a - r).abs() <= _order_bound(r, dtype)).all()), (name, float((a - r).abs().max()))


@pytest.mark.gpu
@pytest.mark.parametrize("n,h,d,w1,w2,dtype,changed", [
    (2000, 4, 128, 60, 128, FP32, ("dkp", "dvp")),  # longer chunks
    (3000, 8, 128, 128, 32, BF16, ("dk", "dv")),    # fewer shares of a key block
])
def test_noalloc_with_a_smaller_split(n, h, d, w1, w2, dtype, changed):
    """The allocation-free entry where the reported workspace passes its array:
    within the order of float32 sums of the whole split, and bit for bit the
    workspace entry's with a workspace of the array's size."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    print(f"\n[workspace] noalloc N={n} H={h} D={d} w1={w1} w2={w2} {dtype}", flush=True)
    cap, scale = 64 << 20, d ** -0.5
    assert simplicial_attn_bwd_workspace_size(1, n, h, d, w1, w2, dtype) > cap
    x = [t.cuda() for t in draw((1, n, h, d), seed=n + w2, dtype=dtype)]
    o, lse = simplicial_attn_fwd(*x[:5], w1, w2, scale)
    ref = simplicial_attn_bwd(*x[:5], o, x[5], lse, w1, w2, scale)
    ws = torch.empty(cap, dtype=torch.uint8, device="cuda")
    same = simplicial_attn_bwd(*x[:5], o, x[5], lse, w1, w2, scale, workspace=ws)
    got = simplicial_attn_bwd_noalloc(*x[:5], o, x[5], lse, w1, w2, scale)
    torch.cuda.synchronize()
    for name, a, b, r in zip(P.GRAD_NAMES, got, same, ref):
        assert torch.equal(a, b), name
        assert torch.equal(a, r) == (name not in changed), name
        a, r = a.double(), r.double()
        assert bool(((a - r).abs() <= _order_bound(r, dtype)).all()), name


@pytest.mark.gpu
@pytest.mark.parametrize("n,h,w1,w2", [(100, 2, 7, 5), (64, 1, 16, 32), (700, 4, 100, 17)])
def test_fused_stages_with_the_fused_plans_bytes(n, h, w1, w2):
    """Delta and the fused kernel's partial sums are enough for its three calls, also
    where the two-kernel backward's whole split takes more."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    print(f"\n[workspace] fused N={n} H={h} w1={w1} w2={w2}", flush=True)
    d, scale = 128, 128 ** -0.5
    need = (4 * n * h + 255) // 256 * 256 + 4 * h * -(-n // 64) * ((63 + w1) + 2 * (94 + w1)) * d
    x = [t.cuda() for t in draw((1, n, h, d), seed=n)]
    o, lse = simplicial_attn_fwd(*x[:5], w1, w2, scale)
    buf = torch.full((need + 65536,), 0x5A, dtype=torch.uint8, device="cuda")
    ws = buf[:need]
    simplicial_attn_bwd_preprocess(o, x[5], w1, w2, ws)
    dk, dv = simplicial_attn_bwd_fused(*x, lse, w1, w2, ws, scale)
    dq, dkp, dvp = simplicial_attn_bwd_fused_reduce(x[0], w1, w2, ws, scale)
    ref = simplicial_attn_bwd(*x[:5], o, x[5], lse, w1, w2, scale)
    torch.cuda.synchronize()
    assert bool((buf[need:] == 0x5A).all())
    P.check_grads([P.to64(g) for g in (dq, dk, dkp, dv, dvp)], [P.to64(g) for g in ref], "bf16", "fused")
