"""GPU test of the bf16 kernels at the start of the sequence, where a tile leaves
out the key blocks that hold no key: it still reads no key later than it would
with the whole window walked. Where the window of a tile fills its blocks (w1 a
multiple of 32 for one query position, 3 or 1 less for a tile of 4 or 2
queries) that is no key after its own queries, so that a row of K or V that is
not finite (padding, say) reaches no earlier tile, although a masked pair's
probability of 0 times such a row is NaN."""

import pytest
import torch

from paper_2507_02754_amd import (load_library, simplicial_attn_bwd, simplicial_attn_bwd_gqa,
                                  simplicial_attn_fwd, simplicial_attn_fwd_gqa)
from paper_2507_02754_amd.workloads import draw

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    load_library()


# group: query heads per K-side head (4: tiles of one position and four heads in
# the forward); tile: positions of a tile in the forward and in the query side
@pytest.mark.parametrize("group,d,w1,w2,fwd_tile,bwd_tile", [
    (4, 128, 64, 32, 1, 0), (4, 64, 96, 17, 1, 0), (8, 128, 160, 32, 1, 0),
    (1, 128, 61, 32, 4, 4), (1, 64, 125, 9, 4, 4), (1, 128, 63, 64, 2, 2), (1, 64, 95, 40, 2, 2),
])
@pytest.mark.parametrize("row", [1, 13, 44])
def test_keys_after_a_tile_do_not_matter(group, d, w1, w2, fwd_tile, bwd_tile, row):
    print(f"\n[window start] group={group} D={d} w1={w1} w2={w2} row {row}", flush=True)
    n, hkv = 170, 2
    q, _, _, _, _, do = (x.cuda() for x in draw((1, n, hkv * group, d), seed=n + d + w1))
    _, k, kp, v, vp, _ = (x.cuda() for x in draw((1, n, hkv, d), seed=n + d + w2))
    fwd, bwd = ((simplicial_attn_fwd, simplicial_attn_bwd) if group == 1
                else (simplicial_attn_fwd_gqa, simplicial_attn_bwd_gqa))
    bad = v.clone()
    bad[0, row, :, :3] = torch.tensor([float("inf"), float("nan"), -float("inf")], device="cuda")
    o, lse = fwd(q, k, kp, v, vp, w1, w2)
    ob, lb = fwd(q, k, kp, bad, vp, w1, w2)
    dq = bwd(q, k, kp, v, vp, o, do, lse, w1, w2)[0]
    dqb = bwd(q, k, kp, bad, vp, o, do, lse, w1, w2)[0]
    torch.cuda.synchronize()
    first = row // fwd_tile * fwd_tile  # first query of the first tile that sees the row
    assert torch.equal(ob[:, :first], o[:, :first])
    assert torch.equal(lb, lse)  # V enters no logit
    if bwd_tile:
        first = row // bwd_tile * bwd_tile
        assert torch.equal(dqb[:, :first], dq[:, :first])
    assert not torch.isfinite(ob[:, row]).all()  # the row does reach its own query
