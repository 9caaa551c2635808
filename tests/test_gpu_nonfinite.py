"""NaN and infinity in q, k and v where a row's keys are worked off in parts: a
part that holds one shows in the row's result, cut or not, and a key that a row
does not take part in shows in none."""
import pytest

import oracle as O

pytestmark = pytest.mark.gpu

HEADS = 7  # of 159 blocks: 1,113 rows, of which the dense call cuts the last 43 of every eighth


@pytest.fixture(scope="module")
def workload():
    import torch
    import paper_2608_02504_amd as tra
    plan = tra.Plan(tra.Config(1, HEADS, 13, 30, 52, 128))
    assert plan.n_blocks == 159
    g = torch.Generator(device="cuda").manual_seed(2)
    # small scores: every weight stays far above the smallest bf16 number
    q, k, v = (0.3 * torch.randn(1, HEADS, plan.n_tokens, 128, generator=g, device="cuda") for _ in range(3))
    pos = torch.tensor(O.tile_major_order(13, 30, 52, 8, 16), device="cuda")  # position -> token
    return plan, q.bfloat16(), k.bfloat16(), v.bfloat16(), pos


def _lists(call):
    """Rows' lists [HEADS, 159]: every block (dense), or every block in each fifth
    row (cut: 159 entries against a piece length of 48) and two blocks, one row in
    five with block 7, in the others."""
    import torch
    NB = 159
    u = torch.arange(NB, device="cuda")
    cols = u.expand(NB, NB).clone()
    cnt = torch.full((NB,), NB, device="cuda")
    if call != "dense":
        short = u % 5 != 0
        cnt[short] = 2
        cols[short, 0] = torch.where(u % 5 == 1, 7, 20)[short]
        cols[short, 1] = 21
    takes = torch.zeros(NB, NB, dtype=torch.bool, device="cuda")
    for r in range(NB):
        takes[r, cols[r, :cnt[r]]] = True
    return (cnt.int().expand(1, HEADS, NB).contiguous(), cols.int().expand(1, HEADS, NB, NB).contiguous(), takes)


@pytest.mark.parametrize("call", ["dense", "sparse", "token"])
def test_cut_rows_keep_nan_and_infinity(workload, call):
    import torch
    import paper_2608_02504_amd as tra
    plan, q, k, v, pos = workload
    S = plan.n_tokens
    cnt, cols, takes = _lists(call)
    q, k, v = q.clone(), k.clone(), v.clone()
    key = pos[7 * 128 + 40]                 # a key of block 7
    queries = pos[torch.arange(50, S, 128, device="cuda")]  # a query of every row
    k[0, 1, key] = float("nan")
    q[0, 2, queries] = float("nan")
    v[0, 3, key, 5] = float("inf")
    o, lse = torch.empty_like(q), torch.empty(1, HEADS, S, device="cuda")
    if call == "dense":
        tra.tra_dense_attention(plan, q, k, v, o, lse)
    elif call == "sparse":
        tra.tra_sparse_attention(plan, q, k, v, cnt, cols, None, o, lse)
    else:
        full = torch.full((1, HEADS, S), tra.TRA_RADIUS_FULL, dtype=torch.int32, device="cuda")
        tra.tra_token_attention(plan, q, k, v, full, cnt, cols, None, o, lse)
    block = torch.empty(S, dtype=torch.long, device="cuda")
    block[pos] = torch.arange(S, device="cuda") // 128
    touched = takes[block, 7]               # tokens whose row takes block 7
    nan = torch.zeros(HEADS, S, 128, dtype=torch.bool, device="cuda")
    nan[1, touched] = True
    nan[2, queries] = True
    assert torch.equal(o[0].isnan(), nan)
    inf = torch.zeros_like(nan)
    inf[3, touched, 5] = True
    assert torch.equal(o[0] == float("inf"), inf)
    assert (o[0] != -float("inf")).all() and lse[0, [0, 3, 4, 5, 6]].isfinite().all()


@pytest.mark.parametrize("head_dim", [64, 128])
def test_fp32_infinite_last_value(head_dim):
    """An infinite value in the last token of a partial 32-key tile (45 and 77
    tokens: 13 in the last) makes its component infinite, not NaN."""
    import torch
    import paper_2608_02504_amd as tra
    for h in (5, 7):
        plan = tra.Plan(tra.Config(1, 1, 1, h, 9 if h == 5 else 11, head_dim, block=64, tile_h=8, tile_w=8, dtype="fp32"))
        S, NB = plan.n_tokens, plan.n_blocks
        assert S % 32 == 13
        g = torch.Generator(device="cuda").manual_seed(1)
        q, k, v = (torch.randn(1, 1, S, head_dim, generator=g, device="cuda") for _ in range(3))
        last = int(O.tile_major_order(1, h, 9 if h == 5 else 11, 8, 8)[-1])
        v[0, 0, last, 3] = float("inf")
        want = torch.zeros(S, head_dim, dtype=torch.bool, device="cuda")
        want[:, 3] = True
        cnt = torch.full((1, 1, NB), NB, dtype=torch.int32, device="cuda")
        cols = torch.arange(NB, dtype=torch.int32, device="cuda").expand(1, 1, NB, NB).contiguous()
        full = torch.full((1, 1, S), tra.TRA_RADIUS_FULL, dtype=torch.int32, device="cuda")
        for call in ("dense", "entropy", "sparse", "token"):
            o = torch.empty_like(q)
            if call == "dense":
                tra.tra_dense_attention(plan, q, k, v, o)
            elif call == "entropy":
                tra.tra_entropy(plan, q, k, v, o, torch.empty(1, 1, S, device="cuda"))
            elif call == "sparse":
                tra.tra_sparse_attention(plan, q, k, v, cnt, cols, None, o)
            else:
                tra.tra_token_attention(plan, q, k, v, full, cnt, cols, None, o)
            assert not o.isnan().any(), (call, h)
            assert torch.equal(o[0, 0] == float("inf"), want), (call, h)


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("mixed", [False, True])
def test_fp32_token_value_out_of_reach(head_dim, mixed):
    """Token-level call, a column of 8 blocks of 8 x 8, every block listed: an infinite
    value in the last block reaches no query of short radius in the others, also where
    one query among its 32 has the full radius (mixed) and gets it."""
    import torch
    import paper_2608_02504_amd as tra
    plan = tra.Plan(tra.Config(1, 1, 1, 64, 8, head_dim, block=64, tile_h=8, tile_w=8, dtype="fp32"))
    S, NB = plan.n_tokens, plan.n_blocks  # (raster order is the tile-major order here)
    g = torch.Generator(device="cuda").manual_seed(1)
    q, k, v = (torch.randn(1, 1, S, head_dim, generator=g, device="cuda") for _ in range(3))
    v[0, 0, S - 5, 3] = float("inf")
    cnt = torch.full((1, 1, NB), NB, dtype=torch.int32, device="cuda")
    cols = torch.arange(NB, dtype=torch.int32, device="cuda").expand(1, 1, NB, NB).contiguous()
    rad = torch.full((1, 1, S), 2, dtype=torch.int32, device="cuda")
    if mixed:
        rad[0, 0, 5::32] = tra.TRA_RADIUS_FULL
    o = torch.empty_like(q)
    tra.tra_token_attention(plan, q, k, v, rad, cnt, cols, None, o)
    far = o[0, 0, :S - 64]
    inf = torch.zeros_like(far, dtype=torch.bool)
    if mixed:
        inf[5::32, 3] = True
    assert not far.isnan().any()
    assert torch.equal(far == float("inf"), inf)
