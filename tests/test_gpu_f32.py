"""GPU tests of the float32 MFMA kernels (float32 data; bf16 with head_dim 16 / 32
or w2 > 64) against the oracle, at the edges of their row packing, key blocks,
query chunks and workspace splits, and with infinities and NaN in the inputs."""

import pytest
import torch

import parity as P
from paper_2507_02754_amd import (load_library, simplicial_attn_bwd, simplicial_attn_bwd_noalloc,
                                  simplicial_attn_bwd_preprocess, simplicial_attn_bwd_workspace_size,
                                  simplicial_attn_fwd, simplicial_attn_path_name)
from paper_2507_02754_amd.workloads import draw

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    load_library()


SHAPES = [
    # (B, H, N, D, w1, w2, dtype): 8, 4, 2 and 1 queries per wavefront, one to
    # four row groups, chunks longer and shorter than the k-row window
    (1, 1, 1, 16, 1, 1, "fp32"),
    (1, 2, 70, 16, 31, 8, "fp32"),
    (2, 1, 97, 32, 33, 9, "fp32"),
    (1, 1, 130, 64, 64, 16, "fp32"),
    (1, 2, 101, 128, 32, 17, "fp32"),
    (1, 1, 75, 128, 1, 32, "fp32"),      # w1 = 1: one key per query
    (1, 1, 90, 64, 500, 33, "fp32"),     # w1 past the sequence
    (1, 1, 140, 32, 50, 96, "fp32"),     # three row groups
    (1, 1, 150, 16, 40, 127, "fp32"),
    (1, 1, 160, 128, 20, 128, "fp32"),
    (1, 1, 150, 64, 24, 129, "fp32"),    # query side on the plain kernels
    (1, 1, 70, 128, 64, 65, "bf16"),
    (1, 2, 131, 32, 100, 16, "bf16"),
    (1, 1, 33, 16, 32, 32, "bf16"),
    (1, 1, 150, 64, 24, 130, "bf16"),    # query side on the plain kernels
    (1, 2, 210, 128, 40, 300, "bf16"),
    (1, 1, 300, 16, 1, 100, "fp32"),     # chunks of one query or two, 16 workgroups per key block
    (1, 1, 140, 128, 2, 128, "bf16"),
    (1, 2, 90, 64, 9, 12, "fp32"),       # chunks of one step of eight queries
]


@pytest.mark.parametrize("shape", SHAPES, ids=[str(s) for s in SHAPES])
def test_f32_kernels_against_oracle(shape):
    b, h, n, d, w1, w2, dt = shape
    dtype = torch.float32 if dt == "fp32" else torch.bfloat16
    assert simplicial_attn_path_name(0, b, n, h, d, w1, w2, dtype) == "generic"
    print(f"\n[f32] {shape}", flush=True)
    inputs = draw((b, n, h, d), seed=n + d + w2, dtype=dtype)
    scale = d ** -0.5
    o, lse = P.gpu_forward(inputs, w1, w2, scale)
    grads = P.gpu_backward(inputs, o, lse, w1, w2, scale)
    o_ref, lse_ref, g_ref = P.full_oracle(inputs, w1, w2, scale)
    P.check_forward(P.to64(o), P.to64(lse), o_ref, lse_ref, dt, str(shape))
    if w1 == 1 and min(n, w2) == 1:
        # one pair per query: dQ, dK, dK' vanish in exact arithmetic; what is left
        # is the rounding of dP - Delta (D terms each) times a unit-scale operand
        bound = 64 * 2.0 ** -24 * d ** 0.5
        assert all(float(g.abs().max()) <= bound for g in grads[:3])
        P.check_grads([P.to64(g) for g in grads[3:]], g_ref[3:], dt, str(shape))
    else:
        P.check_grads([P.to64(g) for g in grads], g_ref, dt, str(shape))


@pytest.mark.parametrize("h,n,d,w2", [(1, 300, 64, 16), (16, 640, 32, 32), (1, 257, 32, 128), (40, 520, 16, 8)])
def test_f32_splits_agree(h, n, d, w2):
    """Few and many workgroups take different chunk lengths and key-side splits;
    the allocation-free entry runs the same split, which fits its 64 MiB here.
    Run twice: bitwise the same."""
    w1 = 70
    print(f"\n[f32] splits H={h} N={n} D={d} w2={w2}", flush=True)
    x = [t.cuda() for t in draw((1, n, h, d), seed=5 + n, dtype=torch.float32)]
    o, lse = simplicial_attn_fwd(*x[:5], w1, w2)
    ref = simplicial_attn_bwd(*x[:5], o, x[5], lse, w1, w2)
    again = simplicial_attn_bwd(*x[:5], o, x[5], lse, w1, w2)
    noalloc = simplicial_attn_bwd_noalloc(*x[:5], o, x[5], lse, w1, w2)
    torch.cuda.synchronize()
    assert simplicial_attn_bwd_workspace_size(1, n, h, d, w1, w2, torch.float32) <= 64 << 20
    for a, c, e in zip(ref, again, noalloc):
        assert torch.equal(a, c)
        assert torch.equal(a, e)
    one = [t[:, :, :1].contiguous() for t in x]  # head 0 alone: fewer workgroups
    o1, lse1 = simplicial_attn_fwd(*one[:5], w1, w2)
    g1 = simplicial_attn_bwd(*one[:5], o1, one[5], lse1, w1, w2)
    torch.cuda.synchronize()
    for a, c in zip(ref, g1):
        # the same sums in another order: a few hundred float32 additions
        assert float((a[:, :, :1] - c).abs().max()) <= 1e-5 * float(c.abs().max())


@pytest.mark.parametrize("w2,d", [(5, 64), (16, 128), (16, 16), (32, 32)])
def test_f32_rows_outside_the_window_do_not_matter(w2, d):
    """Infinities and NaN in one row of K / V (or of dO, K', V', Q) reach only the
    outputs whose windows include that row: everything else is finite and agrees
    with the run on clean inputs."""
    n, w1, r = 150, 40, 77
    x = [t.cuda() for t in draw((1, n, 1, d), seed=w2 + d, dtype=torch.float32)]
    o, lse = simplicial_attn_fwd(*x[:5], w1, w2)
    g = simplicial_attn_bwd(*x[:5], o, x[5], lse, w1, w2)
    idx = torch.arange(n, device="cuda")
    for t, name in enumerate(("q", "k", "kp", "v", "vp", "do")):
        print(f"\n[f32] non-finite row in {name} w2={w2} D={d}", flush=True)
        y = [z.clone() for z in x]
        y[t][0, r, 0, :3] = torch.tensor([float("inf"), float("nan"), -float("inf")], device="cuda")
        win = {"k": w1, "v": w1, "kp": w2, "vp": w2}.get(name, 1)
        seen = (idx >= r) & (idx < r + win)  # queries that read the row
        o2, l2 = simplicial_attn_fwd(*y[:5], w1, w2)
        g2 = simplicial_attn_bwd(*y[:5], o, y[5], lse, w1, w2)  # clean O, LSE: the operands alone
        torch.cuda.synchronize()
        assert torch.allclose(o2[0, ~seen], o[0, ~seen], rtol=1e-4, atol=1e-5), name
        assert torch.allclose(l2[0, :, ~seen], lse[0, :, ~seen], rtol=1e-4, atol=1e-5), name
        qs = torch.nonzero(seen).flatten()
        lo, hi = int(qs.min()), int(qs.max())
        reach = {0: ~seen,
                 1: (idx <= lo - w1) | (idx > hi), 3: (idx <= lo - w1) | (idx > hi),
                 2: (idx <= lo - w2) | (idx > hi), 4: (idx <= lo - w2) | (idx > hi)}
        for gi, keep in reach.items():
            assert torch.allclose(g2[gi][0, keep], g[gi][0, keep], rtol=1e-4, atol=1e-5), (name, gi)


@pytest.mark.parametrize("d,w2,n", [(16, 8, 70), (32, 32, 131), (64, 65, 90), (128, 128, 160), (128, 97, 75)])
@pytest.mark.parametrize("bad", ["", "k", "v", "q", "do"])
def test_bf16_products_in_parts_equal_float32(d, w2, n, bad):
    """bf16 data multiplies float32 values as three bf16 parts: the same sums as
    with float32 products of the widened data (the float32 entry), so the LSE
    agrees to float32 rounding, outputs to one bf16 rounding (2^-8), and
    infinities give the same infinities and NaN."""
    w1, scale = 40, d ** -0.5
    print(f"\n[f32] parts D={d} w2={w2} N={n} infinity in {bad or 'nothing'}", flush=True)
    x = [t.cuda() for t in draw((1, n, 2, d), seed=n + w2, dtype=torch.bfloat16)]
    o, lse = simplicial_attn_fwd(*x[:5], w1, w2, scale)
    if bad:
        x[("q", "k", "kp", "v", "vp", "do").index(bad)][0, n // 2, 1, d // 3] = float("inf")
    wide = [t.float() for t in x]
    got = [*simplicial_attn_fwd(*x[:5], w1, w2, scale),
           *simplicial_attn_bwd(*x[:5], o, x[5], lse, w1, w2, scale)]
    ref = [*simplicial_attn_fwd(*wide[:5], w1, w2, scale),
           *simplicial_attn_bwd(*wide[:5], o.float(), wide[5], lse, w1, w2, scale)]
    torch.cuda.synchronize()
    for t, (a, r) in enumerate(zip(got, ref)):
        assert torch.equal(torch.isfinite(a), torch.isfinite(r)), t
        assert torch.equal(torch.isnan(a), torch.isnan(r)), t
        ok = torch.isfinite(r)
        big = float(r[ok].abs().max()) if bool(ok.any()) else 0.0
        err = (a.float()[ok] - r[ok]).abs()
        # LSE: a few float32 roundings of sums of up to 5120 terms; the others one
        # bf16 rounding plus float32 sums of the size of the largest
        bound = 4e-6 * max(big, 1.0) if t == 1 else 2.0 ** -8 * r[ok].abs() + 4e-6 * big
        assert bool((err <= bound).all()), (t, float(err.max()))


@pytest.mark.parametrize("h,n,w1,w2", [
    (33026, 129, 3, 128),   # 128 k-rows span more than 2^31 bytes: query side
    (105000, 41, 41, 5),    # so do 32 keys: forward and both sides
])
def test_f32_strides_past_32_bit_offsets(h, n, w1, w2):
    """Many heads: rows of one head lie so far apart that those of a block span
    more than a 32-bit offset. First, middle and last head against the oracle."""
    d, scale = 128, 128 ** -0.5
    print(f"\n[f32] strides H={h} N={n} w2={w2}", flush=True)
    assert n * h * d * 4 > 1 << 31
    g = torch.Generator(device="cuda").manual_seed(h)
    x = [torch.randn((1, n, h, d), generator=g, device="cuda") for _ in range(6)]
    o, lse = simplicial_attn_fwd(*x[:5], w1, w2, scale)
    grads = simplicial_attn_bwd(*x[:5], o, x[5], lse, w1, w2, scale)
    torch.cuda.synchronize()
    for head in (0, h // 2, h - 1):
        one = [t[:, :, head:head + 1].cpu() for t in x]
        o_ref, lse_ref, g_ref = P.full_oracle(one, w1, w2, scale)
        P.check_forward(P.to64(o[:, :, head:head + 1]), P.to64(lse[:, head:head + 1]), o_ref, lse_ref, "fp32",
                        f"head {head}")
        P.check_grads([P.to64(t[:, :, head:head + 1]) for t in grads], g_ref, "fp32", f"head {head}")


def test_f32_logits_in_two_chains():
    """The rounding of a logit's running sum is the largest error of the float32
    forward. One chain of D products of rms t carries u t D / sqrt(6) of it (u =
    2^-24), two chains of D / 2 and their sum sqrt(1/2 + 2/D) = 0.73 of that; the
    operands' rounding adds 2%. Emulated on the CPU with everything else exact,
    O at this shape is 1.9e-7 off with one chain and 1.3e-7 with two. With the
    kernel's other roundings 2.31e-7 and 1.62e-7: the bound lies between."""
    n, h, d, w1, w2 = 400, 4, 64, 256, 16
    err = ref = 0.0
    for seed in range(2):
        inputs = draw((1, n, h, d), seed=1000 + seed, dtype=torch.float32)
        o, _ = simplicial_attn_fwd(*(t.cuda() for t in inputs[:5]), w1, w2, d ** -0.5)
        o_ref = P.full_oracle(inputs, w1, w2, d ** -0.5)[0]
        o = P.to64(o)
        err += float(((o - o_ref) ** 2).sum())
        ref += float((o_ref ** 2).sum())
    rel = (err / ref) ** 0.5
    print(f"\n[f32] O against float64: {rel:.3e}", flush=True)
    assert rel <= 2.0e-7


@pytest.mark.parametrize("n,h,d,dt", [(4194304 + 77, 1, 16, "bf16"), (300001, 2, 128, "fp32"), (1, 1, 16, "fp32"),
                                      (65, 3, 64, "fp32")])
def test_f32_delta_of_many_rows(n, h, d, dt):
    """Delta where its launch has fewer workgroups than runs of rows (more than
    2^26 elements), and of few rows."""
    dtype = torch.float32 if dt == "fp32" else torch.bfloat16
    print(f"\n[f32] delta N={n} H={h} D={d} {dt}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(n)
    o, do = (torch.randn((1, n, h, d), generator=g, device="cuda").to(dtype) for _ in range(2))
    ws = torch.empty(simplicial_attn_bwd_workspace_size(1, n, h, d, 1, 1, dtype), dtype=torch.uint8, device="cuda")
    simplicial_attn_bwd_preprocess(o, do, 1, 1, ws)
    delta = ws[:4 * n * h].view(torch.float32).view(h, n)
    ref = (o.double() * do.double()).sum(-1)[0].t()
    # D products and D - 1 sums, each 2^-24 of at most the sum of magnitudes
    bound = d * 2.0 ** -24 * (o.double() * do.double()).abs().sum(-1)[0].t()
    assert bool(((delta.double() - ref).abs() <= bound).all())


def test_f32_delta_of_2_to_the_30_rows():
    """Sizes whose Delta would take 2^32 threads at four elements each."""
    n, d = (1 << 30) + 5, 16
    print(f"\n[f32] delta N={n}", flush=True)
    if torch.cuda.mem_get_info()[0] < 100 << 30:
        pytest.skip("needs 73 GB of GPU memory")
    o, do = (torch.empty((1, n, 1, d), dtype=torch.bfloat16, device="cuda").fill_(x) for x in (0.5, 0.25))
    rows = torch.tensor([0, 1, n // 2, n - 2, n - 1], device="cuda")
    o[0, rows] = torch.arange(1, 6, dtype=torch.bfloat16, device="cuda").view(5, 1, 1)
    ws = torch.empty(simplicial_attn_bwd_workspace_size(1, n, 1, d, 1, 1, o.dtype), dtype=torch.uint8, device="cuda")
    simplicial_attn_bwd_preprocess(o, do, 1, 1, ws)
    delta = ws[:4 * n].view(torch.float32)
    assert delta[rows].tolist() == [4.0 * x for x in range(1, 6)]
    delta[rows] = 2.0
    assert float(delta.min()) == 2.0 and float(delta.max()) == 2.0


@pytest.mark.parametrize("n,d,w1,w2,dt", [(150, 64, 40, 16, "fp32"), (90, 128, 30, 40, "bf16"), (100, 32, 50, 5, "bf16"),
                                          (80, 16, 20, 130, "fp32")])
def test_f32_infinite_lse_leaves_a_query_out(n, d, w1, w2, dt):
    """An LSE of +inf makes a query's probabilities 0, as a huge one does: it adds
    nothing to any gradient, and its own dq is 0."""
    dtype = torch.float32 if dt == "fp32" else torch.bfloat16
    print(f"\n[f32] infinite LSE N={n} D={d} w2={w2} {dt}", flush=True)
    x = [t.cuda() for t in draw((1, n, 2, d), seed=n + w2, dtype=dtype)]
    o, lse = simplicial_attn_fwd(*x[:5], w1, w2)
    runs = []
    for big in (1e30, float("inf")):
        l2 = lse.clone()
        l2[:, 1, ::7] = big
        runs.append(simplicial_attn_bwd(*x[:5], o, x[5], l2, w1, w2))
    torch.cuda.synchronize()
    for name, a, b in zip(P.GRAD_NAMES, *runs):
        assert torch.isfinite(a).all() and torch.equal(a, b), name
    assert bool((runs[1][0][:, ::7, 1] == 0).all())
