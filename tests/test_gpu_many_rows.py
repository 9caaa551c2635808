"""The kernels of bf16 calls with many rows (attn_k64, attn_bf16, attn_fused: work
units, pieces, row queues, orders) on ragged, padded, joint and split workloads: the
same shapes at one or two heads are the key-splitting kernel's, which takes up to
three quarters of the CUs in rows."""
import numpy as np
import pytest

import oracle as O
import synth
from _pipeline import (TOL_H_ABS, TOL_H_REL, TOL_O_BF16, OracleTables, Run, check_head, check_lists, dense_reference,
                       log)

pytestmark = pytest.mark.gpu

W = {
    # 16 blocks, the last of 4 tokens
    "ragged_d128": synth.Workload("many_d128", 1, 14, 128, "bf16", 4, 13, 37, 128, 0.25, 4.0, 0.6, seed=78,
                                  tile_h=8, tile_w=16),
    "ragged_d64": synth.Workload("many_d64", 2, 14, 64, "bf16", 3, 11, 29, 128, 0.1, 8.0, 0.95, seed=79,
                                 tile_h=8, tile_w=16),
    "joint_d64": synth.Workload("many_joint", 1, 22, 64, "bf16", 3, 11, 29, 128, 0.25, 4.0, 0.6, seed=80,
                                tile_h=8, tile_w=16, text_tokens=200),
    # 61 blocks: rows of more than 48 are cut
    "split_d128": synth.Workload("many_split", 1, 4, 128, "bf16", 5, 30, 52, 128, 0.25, 4.0, 0.6, seed=88,
                                 tile_h=8, tile_w=16),
    "split_d64": synth.Workload("many_split64", 1, 4, 64, "bf16", 5, 30, 52, 128, 0.25, 4.0, 0.6, seed=89,
                                tile_h=8, tile_w=16),
}
CASES = [(n, "packed", r) for n in W for r in (None, 40)] + [("ragged_d128", "tiles", 40), ("joint_d64", "tiles", 40)]


def many(plan):
    """The plan has more rows than the key-splitting kernel takes."""
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert 4 * plan.cfg.batch * plan.cfg.heads * -(-plan.n_tokens // 128) > 3 * cus
    assert 4 * plan.rows > 3 * cus
    return plan


def _mixed(name):
    """Radii of 40; in split workloads, half of the heads' rows keep all 61 blocks
    (122 rows, of which two pieces each cost less than their longer tail)."""
    import paper_2608_02504_amd as tra
    run = Run(W[name], radius_override=40)
    if name.startswith("split"):
        run.rad[:, ::2] = tra.TRA_RADIUS_FULL
        tra.tra_build_block_mask(run.plan, run.rad, run.mask, run.cnt, run.cols, run.order)
        assert (run.cnt[:, ::2] == 61).all() and (run.cnt[:, 1::2] <= 48).all()
    many(run.plan)
    return run


@pytest.mark.parametrize("name,layout,radius", CASES, ids=str)
def test_many_rows(name, layout, radius):
    """Every call of the path: first and last head against the oracle (packed), every
    head against a one-head plan's calls; the heaviest-first order (Run's), none, and
    a random one with entries that are skipped."""
    import torch
    import paper_2608_02504_amd as tra
    w = W[name]
    run = Run(w, radius_override=radius, block_layout=layout)
    plan, S, NB, d = many(run.plan), w.n_tokens, run.plan.n_blocks, w.head_dim
    if layout == "packed":
        tabs = OracleTables(w)
        blocks = np.arange(NB) if NB <= 16 else np.array([0, 7, 30, NB - 1])
        for b, h in ((0, 0), (w.batch - 1, w.heads - 1)):
            check_head(run, tabs, b, h, blocks, TOL_O_BF16, {})
        check_lists(run)
    # the three orders: bit for bit where no row is cut
    o, lse = torch.empty_like(run.O_sp), torch.empty_like(run.lse_sp)
    tra.tra_sparse_attention(plan, run.q, run.k, run.v, run.cnt, run.cols, None, o, lse)
    rng = np.random.default_rng(3)
    shuffled = rng.permutation(plan.rows).astype(np.int32)
    shuffled[::9] = rng.choice([-1, plan.rows, 1 << 30], len(shuffled[::9]))
    o2, lse2 = torch.full_like(o, 9.0), torch.full_like(lse, 9.0)
    tra.tra_sparse_attention(plan, run.q, run.k, run.v, run.cnt, run.cols, torch.tensor(shuffled, device="cuda"), o2, lse2)
    tabs = OracleTables(w, block_layout=layout)
    taken = np.zeros((w.batch * w.heads, S), bool)
    for r in shuffled[(shuffled >= 0) & (shuffled < plan.rows)]:
        taken[r // NB, O.block_tokens(tabs.perm, 128, r % NB)] = True
    taken = torch.tensor(taken.reshape(w.batch, w.heads, S), device="cuda")
    assert (o2[~taken] == 9.0).all() and (lse2[~taken] == 9.0).all()
    if NB <= 48:
        assert torch.equal(o, run.O_sp) and torch.equal(lse, run.lse_sp)
        assert torch.equal(o2[taken], o[taken]) and torch.equal(lse2[taken], lse[taken])
    else:
        assert (o2[taken].float() - o[taken].float()).abs().max() <= TOL_O_BF16
        assert (o.float() - run.O_sp.float()).abs().max() <= TOL_O_BF16
    # one-head plans
    tok = torch.empty_like(o)
    token = w.height * w.width >= 128 or layout == "tiles"
    if token:
        tra.tra_token_attention(plan, run.q, run.k, run.v, run.rad, run.cnt, run.cols, run.order, tok)
    one = tra.Plan(tra.Config.from_workload(w.replace(batch=1, heads=1), block_layout=layout))
    o1, e1, l1 = torch.empty_like(o[:1, :1]), torch.empty(1, 1, S, device="cuda"), torch.empty(1, 1, S, device="cuda")
    for b in range(w.batch):
        for h in range(w.heads):
            cut = lambda t: t[b:b + 1, h:h + 1].contiguous()
            q, k, v, cnt, cols, rad = (cut(t) for t in (run.q, run.k, run.v, run.cnt, run.cols, run.rad))
            near = lambda got, want: (got[b, h].float() - want[0, 0].float()).abs().max() <= TOL_O_BF16
            tra.tra_sparse_attention(one, q, k, v, cnt, cols, None, o1, l1)
            assert near(o, o1) and (lse[b, h] - l1).abs().max() <= 1e-4 + 1e-5 * l1.abs().max(), (b, h)
            tra.tra_dense_attention(one, q, k, v, o1, l1)
            assert near(run.O_d, o1) and (run.lse_d[b, h] - l1).abs().max() <= 1e-4 + 1e-5 * l1.abs().max(), (b, h)
            tra.tra_entropy(one, q, k, v, o1, e1)
            assert near(run.O_ent, o1) and (run.H[b, h] - e1).abs().max() <= TOL_H_REL * e1.abs().max(), (b, h)
            assert (run.H_only[b, h] - e1).abs().max() <= TOL_H_REL * e1.abs().max(), (b, h)
            if token:
                tra.tra_token_attention(one, q, k, v, rad, cnt, cols, None, o1)
                assert near(tok, o1), (b, h)


@pytest.mark.parametrize("name", ["ragged_d128", "ragged_d64", "split_d128", "split_d64"])
@pytest.mark.parametrize("call", ["sparse", "token"])
def test_many_rows_list_entries(name, call):
    """Block ids outside [0, NB), empty lists and lengths outside [0, NB]: as the
    call with the valid entries alone, an empty row 0 with lse -inf."""
    import torch
    import paper_2608_02504_amd as tra
    w = W[name]
    run = _mixed(name)
    plan, NB, S = run.plan, run.plan.n_blocks, w.n_tokens
    rng = np.random.default_rng(7)
    cnt, cols = run.cnt.cpu().numpy(), run.cols.cpu().numpy()
    cnt2, cols2 = cnt.copy(), cols.copy()
    empty = np.zeros((w.batch, w.heads, S), bool)
    perm = OracleTables(w).perm
    for i, idx in enumerate(np.ndindex(cnt.shape)):
        ids = []
        for c in cols[idx][:cnt[idx]]:
            ids += [-1, NB, -7, 1 << 20][:rng.integers(0, 3)] + [c]
        ids = (ids + [NB, -5])[:NB]
        if i % 11 == 3:
            ids = [-1, NB][:i % 3]                  # nothing valid
        kept = [c for c in ids if 0 <= c < NB]
        cols[idx], cols2[idx] = -1, -1
        cnt[idx], cols[idx][:len(kept)] = len(kept), kept
        cnt2[idx], cols2[idx][:len(ids)] = len(ids), ids
        if not ids:
            cnt2[idx] = -3
        if not kept:
            empty[idx[0], idx[1], O.block_tokens(perm, 128, idx[2])] = True
    out = []
    for c, l in ((cnt, cols), (cnt2, cols2)):
        c, l = torch.tensor(c, device="cuda"), torch.tensor(l, device="cuda")
        o, lse = torch.full_like(run.q, 9.0), torch.full_like(run.lse_sp, 9.0)
        if call == "sparse":
            tra.tra_sparse_attention(plan, run.q, run.k, run.v, c, l, None, o, lse)
        else:
            tra.tra_token_attention(plan, run.q, run.k, run.v, run.rad, c, l, None, o, lse)
        out.append((o, lse))
    empty = torch.tensor(empty, device="cuda")
    assert empty.any() and not empty.all()
    for o, lse in out:
        assert (o[empty] == 0).all() and (lse[empty] == -float("inf")).all()
        assert o.isfinite().all()
        # (a token-level row can list no block that its queries cover)
        assert call == "token" or lse[~empty].isfinite().all()
    (o, lse), (o2, lse2) = out
    live = lse.isfinite()
    assert torch.equal(live, lse2.isfinite())
    if NB <= 48:
        assert torch.equal(o, o2) and torch.equal(lse, lse2)
    else:
        assert (o.float() - o2.float()).abs().max() <= TOL_O_BF16
        assert (lse[live] - lse2[live]).abs().max() <= 1e-4 + 1e-5 * lse[live].abs().max()


def _calls(tra, run, plan, out):
    q, k, v = run.q, run.k, run.v
    tra.tra_sparse_attention(plan, q, k, v, run.cnt, run.cols, None, out["sp"], out["lse"])
    tra.tra_sparse_attention(plan, q, k, v, run.cnt, run.cols, run.order, out["sp_order"])
    tra.tra_dense_attention(plan, q, k, v, out["d"], out["lse_d"])
    tra.tra_token_attention(plan, q, k, v, run.rad, run.cnt, run.cols, None, out["tok"])
    tra.tra_entropy(plan, q, k, v, out["ent_o"], out["H"])
    tra.tra_entropy(plan, q, k, None, None, out["H_only"])


def _outs(run):
    import torch
    return ({n: torch.empty_like(run.q) for n in ("sp", "sp_order", "d", "tok", "ent_o")} |
            {n: torch.empty_like(run.H) for n in ("lse", "lse_d", "H", "H_only")})


@pytest.mark.parametrize("name", ["split_d128", "ragged_d64"])
def test_many_rows_graph_and_streams(name):
    """Captured calls (queue counters, unit tables, pieces and their merge) replayed
    with eager work between, and two streams at once on one plan: bit for bit the
    eager calls."""
    import torch
    import paper_2608_02504_amd as tra
    run = _mixed(name)
    plan = run.plan
    out = _outs(run)
    _calls(tra, run, plan, out)
    torch.cuda.synchronize()
    eager = {n: t.clone() for n, t in out.items()}
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        _calls(tra, run, plan, out)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        _calls(tra, run, plan, out)
    for rep in range(3):
        for t in out.values():
            t.fill_(float("nan"))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for n in eager:
            assert torch.equal(out[n], eager[n]), (rep, n)
    streams, got = [torch.cuda.Stream(), torch.cuda.Stream()], [_outs(run), _outs(run)]
    for s in streams:
        s.wait_stream(torch.cuda.current_stream())
    for _ in range(3):
        for s, o in zip(streams, got):
            with torch.cuda.stream(s):
                _calls(tra, run, plan, o)
    torch.cuda.synchronize()
    for o in got:
        for n in eager:
            assert torch.equal(o[n], eager[n]), n


@pytest.mark.parametrize("head_dim", [64, 128])
def test_many_rows_scores_jumping(head_dim):
    """Scores that rise by 5, 15 and 35 nats from block to block: the entropy pass's
    tiles taken against the reference and redone from their max, the fused kernel's
    and the dense kernel's rescaling, against the oracle; 26 pairs of heads with the
    same inputs, whose rows are equal wherever they run."""
    import torch
    import paper_2608_02504_amd as tra
    heads = 52
    w = synth.Workload("jumps", 1, heads, head_dim, "bf16", 2, 12, 20, 128, 0.25, 4.0, 0.6, tile_h=8, tile_w=16)
    plan = many(tra.Plan(tra.Config.from_workload(w)))
    N, d = w.n_tokens, head_dim
    perm = O.tile_major_order(w.frames, w.height, w.width, w.tile_h, w.tile_w)
    rng = np.random.default_rng(5)
    level = np.array([0.0, 5.0, 15.0, 35.0])[np.arange(N) // 128]
    q = np.zeros((2, N, d), np.float32)
    k = rng.standard_normal((2, N, d)).astype(np.float32) * 0.5
    v = rng.standard_normal((2, N, d)).astype(np.float32)
    q[:, :, 0] = 1.0
    q[1, :, 0] = rng.uniform(0.5, 1.0, N)
    k[:, perm, 0] = (level + 0.3 * rng.uniform(0, 1, N)) * np.sqrt(d)
    bits = [synth.bf16_bits_from_f32(a) for a in (q, k, v)]
    qt, kt, vt = (torch.from_numpy(a.view(np.int16)).view(torch.bfloat16).reshape(1, 2, N, d).cuda()
                  .repeat(1, heads // 2, 1, 1) for a in bits)
    H, Hf = torch.empty(1, heads, N, device="cuda"), torch.empty(1, heads, N, device="cuda")
    Of, Od = torch.empty_like(qt), torch.empty_like(qt)
    tra.tra_entropy(plan, qt, kt, None, None, H)
    tra.tra_entropy(plan, qt, kt, vt, Of, Hf)
    tra.tra_dense_attention(plan, qt, kt, vt, Od)
    for t in (H, Hf, Of, Od):
        assert torch.equal(t[:, 2:], t[:, :2].repeat(1, heads // 2 - 1, *[1] * (t.dim() - 2)))
    for h in range(2):
        H_ref, O_ref, _ = dense_reference(*(synth.to_f64(a[h], "bf16") for a in bits), np.arange(N))
        tol = np.maximum(TOL_H_REL * np.abs(H_ref), TOL_H_ABS)
        for got in (H, Hf):
            assert (np.abs(got[0, h].double().cpu().numpy() - H_ref) <= tol).all(), h
        for got in (Of, Od):
            assert np.abs(got[0, h].double().cpu().numpy() - O_ref).max() <= TOL_O_BF16, h
    log(f"score jumps d {head_dim}: H in [{H_ref.min():.3f}, {H_ref.max():.3f}] nats")
