"""The bf16 calls' pre-pass where one workgroup rewrites several heads' keys and
values in turn and the last one has fewer: every head of a many-head plan bit
for bit equal to a one-head plan's call (one head a workgroup)."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,head_dim", [(17, 128), (33, 64)])
def test_heads_in_turn_equal_one_head(heads, head_dim):
    import torch
    import paper_2608_02504_amd as tra
    cfg = dict(frames=9, height=45, width=80, head_dim=head_dim)   # 32,400 tokens, a ragged last block
    plan, one = tra.Plan(tra.Config(1, heads, **cfg)), tra.Plan(tra.Config(1, 1, **cfg))
    S, NB = plan.n_tokens, plan.n_blocks
    # two heads a workgroup at least (256 CUs, 64 tokens of 128 components a workgroup)
    assert (NB * 2 * head_dim // 128) * heads // (16 * 256) >= 2 and heads % 2
    g = torch.Generator(device="cuda").manual_seed(3)
    q, k, v = (torch.randn(1, heads, S, head_dim, generator=g, device="cuda").bfloat16() for _ in range(3))
    u = torch.arange(NB, device="cuda")
    pair = torch.stack([u, (7 * u + 3) % NB], 1).sort(1).values
    pair = torch.where((pair[:, :1] == pair[:, 1:]) & (torch.arange(2, device="cuda") == 1), -1, pair)
    cols = torch.full((1, heads, NB, NB), -1, dtype=torch.int32, device="cuda")
    cols[..., :2] = pair.int()
    cnt = (pair >= 0).sum(1).int().expand(1, heads, NB).contiguous()
    o, o1 = torch.empty_like(q), torch.empty_like(q[:, :1])
    tra.tra_sparse_attention(plan, q, k, v, cnt, cols, None, o)
    for h in range(heads):
        tra.tra_sparse_attention(one, *(t[:, h:h + 1].contiguous() for t in (q, k, v, cnt, cols)), None, o1)
        assert torch.equal(o[:, h:h + 1], o1), h


@pytest.mark.parametrize("heads,whole", [(3, False), (8, True)])
def test_piece_length_follows_the_rows(heads, whole):
    """Rows of 61 blocks, every block kept: 183 of them are cut in two (the
    pieces cost less than the longer tail), 488 are not (cutting them all would
    cost more than it evens out) and equal the dense call bit for bit."""
    import torch
    import paper_2608_02504_amd as tra
    plan = tra.Plan(tra.Config(1, heads, 5, 30, 52, 128))
    S, NB = plan.n_tokens, plan.n_blocks
    g = torch.Generator(device="cuda").manual_seed(4)
    q, k, v = (torch.randn(1, heads, S, 128, generator=g, device="cuda").bfloat16() for _ in range(3))
    cnt = torch.full((1, heads, NB), NB, dtype=torch.int32, device="cuda")
    cols = torch.arange(NB, dtype=torch.int32, device="cuda").expand(1, heads, NB, NB).contiguous()
    o, d = torch.empty_like(q), torch.empty_like(q)
    lse, lse_d = (torch.empty(1, heads, S, device="cuda") for _ in range(2))
    tra.tra_sparse_attention(plan, q, k, v, cnt, cols, None, o, lse)
    tra.tra_dense_attention(plan, q, k, v, d, lse_d)
    assert torch.equal(o, d) == whole
    # bf16 outputs of the same sums: an ulp or two of values below 1
    assert (o.float() - d.float()).abs().max() <= 2 ** -7
    assert (lse - lse_d).abs().max() <= 1e-5 * lse_d.abs().max()


@pytest.mark.parametrize("head_dim,frames", [(128, 13), (64, 13), (128, 21)])
def test_dense_cut_rows(head_dim, frames):
    """A dense call whose last rows are cut into pieces (159 blocks x 2 heads: every
    row; 256 x 5 heads: the rows past the GPU's last full round) against the
    oracle on blocks at both ends of the queues' ranges, and against one-head
    plans, which the key-splitting kernel takes or cut elsewhere."""
    import numpy as np
    import torch
    import paper_2608_02504_amd as tra
    import synth
    from _pipeline import TOL_O_BF16, OracleTables, dense_reference, torch_inputs
    import oracle as O
    heads = 2 if frames == 13 else 5
    w = synth.Workload("dense_cut", 1, heads, head_dim, "bf16", frames, 30, 52, 128, 0.25, 4.0, 0.6, seed=41,
                       tile_h=8, tile_w=16)
    inputs = synth.generate(w)
    q, k, v = torch_inputs(w, *inputs)
    plan, one = (tra.Plan(tra.Config.from_workload(w.replace(heads=n))) for n in (heads, 1))
    o, lse = torch.empty_like(q), torch.empty(1, heads, w.n_tokens, device="cuda")
    tra.tra_dense_attention(plan, q, k, v, o, lse)
    o1, lse1 = torch.empty_like(q[:, :1]), torch.empty(1, 1, w.n_tokens, device="cuda")
    perm, NB = OracleTables(w).perm, plan.n_blocks
    for h in range(heads):
        tra.tra_dense_attention(one, *(t[:, h:h + 1].contiguous() for t in (q, k, v)), o1, lse1)
        assert (o[:, h:h + 1].float() - o1.float()).abs().max() <= TOL_O_BF16
        assert (lse[:, h:h + 1] - lse1).abs().max() <= 1e-4 + 1e-5 * lse1.abs().max()
        if h in (0, heads - 1):
            rows = np.concatenate([O.block_tokens(perm, 128, u) for u in (0, NB // 2, NB - 1)])
            _, want, want_lse = dense_reference(*(synth.to_f64(a[0, h], "bf16") for a in inputs), rows)
            assert np.abs(o[0, h].float().cpu().numpy()[rows] - want).max() <= TOL_O_BF16
            assert np.abs(lse[0, h].cpu().numpy()[rows] - want_lse).max() <= 1e-4 + 1e-5 * np.abs(want_lse).max()


@pytest.mark.parametrize("heads", [620, 700])
def test_plan_of_many_rows(heads):
    """31,000 rows, whose lengths the plan of the work units keeps in LDS (62 KB
    of them), and 35,000, which it reads from memory: short rows and, every 97th,
    one of all 50 blocks, which is cut.  First, middle and last head against a
    one-head plan."""
    import torch
    import paper_2608_02504_amd as tra
    cfg = dict(frames=5, height=32, width=40, head_dim=64)
    plan, one = tra.Plan(tra.Config(1, heads, **cfg)), tra.Plan(tra.Config(1, 1, **cfg))
    S, NB = plan.n_tokens, plan.n_blocks
    assert NB == 50 and plan.rows == 50 * heads
    g = torch.Generator(device="cuda").manual_seed(9)
    q, k, v = (torch.randn(1, heads, S, 64, generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(3))
    long = (torch.arange(heads * NB, device="cuda") % 97 == 0).view(1, heads, NB)
    cnt = torch.where(long, NB, 2).int()
    u = torch.arange(NB, device="cuda")
    cols = u.expand(1, heads, NB, NB).clone().int()
    cols[..., :2] = torch.where(long[..., None], cols[..., :2], torch.stack([u.clamp(max=NB - 2), u.clamp(max=NB - 2) + 1], 1).int())
    o, o1 = torch.empty_like(q), torch.empty_like(q[:, :1])
    tra.tra_sparse_attention(plan, q, k, v, cnt, cols, None, o)
    for h in (0, heads // 2, heads - 1):
        tra.tra_sparse_attention(one, *(t[:, h:h + 1].contiguous() for t in (q, k, v, cnt, cols)), None, o1)
        # bf16 outputs of the same sums in another order (|v| up to 5): two ulps
        assert (o[:, h:h + 1].float() - o1.float()).abs().max() <= 2 ** -4, h
        assert (o[:, h:h + 1].float() - o1.float()).norm() <= 1e-2 * o1.float().norm()
