"""GPU test of the bf16 backward's work splits: the same head computed alone (short
query chunks, a key block's rows shared by several workgroups) and among enough
heads that neither is split."""

import pytest
import torch

from paper_2507_02754_amd import (load_library, simplicial_attn_bwd, simplicial_attn_bwd_gqa,
                                  simplicial_attn_bwd_workspace_size, simplicial_attn_det_bwd,
                                  simplicial_attn_det_fwd, simplicial_attn_fwd, simplicial_attn_fwd_gqa)
from paper_2507_02754_amd.workloads import draw

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    load_library()


@pytest.mark.parametrize("kind,n,d,w1,w2,group", [
    ("plain", 515, 128, 300, 32, 1),   # a ragged last key block and chunk
    ("plain", 1021, 64, 1100, 17, 1),  # w1 past the sequence
    ("plain", 383, 128, 64, 64, 1),    # w2 = 64: two row blocks per query
    ("plain", 130, 64, 5, 40, 1),      # fewer row blocks than an even share needs
    ("det", 515, 128, 300, 32, 1),
    ("gqa", 515, 128, 300, 32, 3),     # splits that begin inside a head's row blocks
    ("gqa", 260, 64, 100, 48, 4),
])
def test_backward_splits_agree(kind, n, d, w1, w2, group):
    print(f"\n[splits] {kind} N={n} D={d} w1={w1} w2={w2} group={group}", flush=True)
    many = 96  # K-side heads: more than one workgroup per CU without any split
    q, k, kp, v, vp, do = draw((1, n, many, d), seed=n + d)
    if kind == "gqa":
        q, do = (torch.cat([x] * group, 3).view(1, n, many * group, d) for x in (q, do))
    fwd, bwd = {"plain": (simplicial_attn_fwd, simplicial_attn_bwd),
                "det": (simplicial_attn_det_fwd, simplicial_attn_det_bwd),
                "gqa": (simplicial_attn_fwd_gqa, simplicial_attn_bwd_gqa)}[kind]

    def grads(x):
        x = [t.contiguous().cuda() for t in x]
        o, lse = fwd(*x[:5], w1, w2, d ** -0.5)
        g = bwd(*x[:5], o, x[5], lse, w1, w2, d ** -0.5)
        again = bwd(*x[:5], o, x[5], lse, w1, w2, d ** -0.5)
        torch.cuda.synchronize()
        assert all(torch.equal(a, c) for a, c in zip(g, again))
        return g

    all_g = grads([q, k, kp, v, vp, do])
    one = grads([q[:, :, :group], *(x[:, :, :1] for x in (k, kp, v, vp)), do[:, :, :group]])
    if kind == "plain":  # the split shows in the workspace: more than one share of it per head
        alone = simplicial_attn_bwd_workspace_size(1, n, 1, d, w1, w2, torch.bfloat16)
        assert alone > simplicial_attn_bwd_workspace_size(1, n, many, d, w1, w2, torch.bfloat16) / many
    for a, c in zip(all_g, one):
        a = a[:, :, :c.shape[2]].double()
        c = c.double()
        # same products, float32 sums in another order, one bf16 rounding: 2^-8 of
        # the element, and the order's error against the tensor's largest element
        assert bool(((a - c).abs() <= 2.0 ** -8 * a.abs() + 2.0 ** -12 * a.abs().max()).all())


@pytest.mark.parametrize("d,w2", [(64, 5), (128, 5), (64, 31), (128, 31)])
def test_determinant_rows_outside_the_window_stay_out(d, w2):
    """The determinant backward's dq and dk' epilogue: a k' row that is not finite
    reaches no query past its window, bit for bit (rows of a query's 32 that are
    no pair's must not enter its sums, not even as zero times that row)."""
    print(f"\n[det rows] D={d} w2={w2}", flush=True)
    n, w1 = 150, 40
    q, k, kp, v, vp, do = (x.cuda() for x in draw((1, n, 2, d), seed=900 + d + w2))
    bad = kp.clone()
    bad[:, 0] = float("nan")
    runs = []
    for x in (kp, bad):
        o, lse = simplicial_attn_det_fwd(q, k, x, v, vp, w1, w2, d ** -0.5)
        g = simplicial_attn_det_bwd(q, k, x, v, vp, o, do, lse, w1, w2, d ** -0.5)
        torch.cuda.synchronize()
        runs.append((o, g[0], g[2]))
    for a, c in zip(*runs):
        assert torch.isfinite(a).all()
        assert torch.equal(a[:, w2:], c[:, w2:])
