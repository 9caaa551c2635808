"""GPU parity of token-level TRA attention (tra_token_attention: Eq. 16 with
the token mask of Eq. 15 applied inside the retained blocks) against the
oracle's token_attention_rows, through the C ABI.  Radii and block lists come
from the GPU path (they are checked bit-exact against the oracle elsewhere);
the oracle then takes the same radii and rows.  Bars as for block-sparse
attention: 2e-2 max-abs for bf16 I/O, 1e-5 for fp32."""
import numpy as np
import pytest

import oracle as O
import synth
from _pipeline import TOL_O_BF16, TOL_O_FP32, OracleTables, Run, log, sample_blocks

pytestmark = pytest.mark.gpu


def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


W = {
    "tiny": synth.workload("tiny"),
    "ragged_fp32_d128_b128": synth.Workload("ragged_fp32_d128_b128", 1, 2, 128, "fp32", 3, 7, 19, 128,
                                            0.25, 4.0, 0.6, seed=77, tile_h=8, tile_w=16),
    "ragged_bf16_d128": synth.Workload("ragged_bf16_d128", 1, 2, 128, "bf16", 4, 13, 37, 128,
                                       0.25, 4.0, 0.6, seed=78, tile_h=8, tile_w=16),
    "ragged_bf16_d64": synth.Workload("ragged_bf16_d64", 2, 2, 64, "bf16", 3, 11, 29, 128,
                                      0.1, 8.0, 0.95, seed=79, tile_h=8, tile_w=16),
    "aligned_bf16": synth.Workload("aligned_bf16", 1, 2, 128, "bf16", 5, 16, 32, 128,
                                   0.25, 4.0, 0.6, seed=80, tile_h=8, tile_w=16),
    "fp32_b64_d128": synth.Workload("fp32_b64_d128", 1, 1, 128, "fp32", 2, 9, 11, 64,
                                    0.25, 4.0, 0.6, seed=82, tile_h=8, tile_w=8),
}
W["joint_bf16_d128"] = W["ragged_bf16_d128"].replace(name="joint_bf16_d128", text_tokens=77)
W["joint_fp32"] = W["ragged_fp32_d128_b128"].replace(name="joint_fp32", text_tokens=50)


def _token_call(run, cnt=None, cols=None, order=None):
    import torch
    import paper_2608_02504_amd as tra
    o = torch.empty_like(run.q)
    lse = torch.empty_like(run.lse_sp)
    tra.tra_token_attention(run.plan, run.q, run.k, run.v, run.rad,
                            run.cnt if cnt is None else cnt, run.cols if cols is None else cols,
                            order, o, lse)
    torch.cuda.synchronize()
    return o, lse


def _check_against_oracle(run, o, lse, tol):
    """Every query row of every (batch, head) against token_attention_rows."""
    w = run.w
    tabs = OracleTables(w)
    NB = run.plan.n_blocks
    worst = 0.0
    for b in range(w.batch):
        for h in range(w.heads):
            q, k, v = (synth.to_f64(a[b, h], w.dtype) for a in (run.q_np, run.k_np, run.v_np))
            M = run.mask[b, h].cpu().numpy().astype(bool)
            n_tok = run.rad[b, h].cpu().numpy()
            rows, o_ref, lse_ref = O.token_attention_rows(
                q, k, v, tabs.perm, w.block, list(range(NB)), M, n_tok, tabs.F, tabs.H, tabs.W,
                w.gamma, distance=run.cfg.distance, return_lse=True)
            o_gpu = o[b, h].double().cpu().numpy()[rows]
            err = np.abs(o_gpu - o_ref).max()
            assert err <= tol, f"token attention max-abs {err:.3e} (b={b}, h={h})"
            lse_gpu = lse[b, h].double().cpu().numpy()[rows]
            assert np.abs(lse_gpu - lse_ref).max() <= 1e-4 + 1e-5 * np.abs(lse_ref).max(), "token lse"
            worst = max(worst, float(err))
    return worst


@pytest.mark.parametrize("name", list(W))
@pytest.mark.parametrize("rule", ["vote", "union"])
def test_token_attention_parity(name, rule):
    _gpu()
    w = W[name]
    run = Run(w, rule=rule)
    o, lse = _token_call(run, order=run.order)
    tol = TOL_O_BF16 if w.dtype == "bf16" else TOL_O_FP32
    err = _check_against_oracle(run, o, lse, tol)
    log(f"{name} {rule}: token attention max-abs {err:.2e}")


@pytest.mark.parametrize("name", ["ragged_bf16_d128", "ragged_bf16_d64", "tiny"])
@pytest.mark.parametrize("radius", [0, 3, 40])
def test_token_attention_forced_radii_1d_and_2d(name, radius):
    """Fixed radii for every video query, both distances: masks with many
    partially covered tiles, tiles no query of a wave covers, and (radius 0)
    rows whose only key is the query itself."""
    _gpu()
    w = W[name]
    tol = TOL_O_BF16 if w.dtype == "bf16" else TOL_O_FP32
    for distance in ("2d", "1d"):
        run = Run(w, rule="union", radius_override=radius, distance=distance)
        o, lse = _token_call(run)
        _check_against_oracle(run, o, lse, tol)
        if radius == 0 and distance == "1d":
            # |i - j| <= 0 keeps only the query's own key: o_i = v_i exactly
            v = run.v[..., :w.n_video, :]
            assert np.array_equal(o[..., :w.n_video, :].float().cpu().numpy(), v.float().cpu().numpy())


@pytest.mark.parametrize("name", ["ragged_bf16_d128", "tiny", "joint_bf16_d128"])
def test_token_full_radius_matches_sparse(name):
    """Every radius FULL: every query covers every key of its retained blocks,
    so token-level attention computes the block-sparse call.  The bf16 kernels
    walk the keys in tiles of different sizes (the softmax reference moves at
    different points), so the two agree to rounding, not bit for bit; fp32
    shares one kernel and stays bitwise."""
    _gpu()
    import torch
    w = W[name]
    run = Run(w, radius_override=2 ** 31 - 1)
    o, lse = _token_call(run)
    if w.dtype == "fp32":
        assert torch.equal(o, run.O_sp) and torch.equal(lse, run.lse_sp)
        return
    err = (o.float() - run.O_sp.float()).abs().max().item()
    assert err <= TOL_O_BF16, f"token vs sparse max-abs {err:.3e}"
    lerr = (lse - run.lse_sp).abs().max().item()
    assert lerr <= 1e-4 + 1e-5 * run.lse_sp.abs().max().item(), f"token vs sparse lse {lerr:.3e}"


@pytest.mark.parametrize("head_dim,text", [(128, 0), (64, 40)])
@pytest.mark.parametrize("radius", [None, 120])
def test_token_split_rows(head_dim, text, radius):
    """Rows of more than 48 blocks (61 or 62 here, lists that keep every block)
    are cut into pieces and merged: outputs against the oracle under the
    method's own radii and under short forced ones, where a query covers no key
    of some pieces, and bitwise the same under a row order."""
    _gpu()
    import torch
    w = synth.Workload("token_split", 1, 1, head_dim, "bf16", 5, 30, 52, 128, 0.25, 4.0, 0.6, seed=88,
                       tile_h=8, tile_w=16, text_tokens=text)
    run = Run(w, rule="union", radius_override=radius)
    NB = run.plan.n_blocks
    run.mask.fill_(1)
    run.cnt.fill_(NB)
    run.cols.copy_(torch.arange(NB, dtype=torch.int32, device="cuda").expand_as(run.cols))
    assert NB > 48
    o, lse = _token_call(run)
    _check_against_oracle(run, o, lse, TOL_O_BF16)
    o2, lse2 = _token_call(run, order=torch.arange(NB - 1, -1, -1, dtype=torch.int32, device="cuda"))
    assert torch.equal(o, o2) and torch.equal(lse, lse2)


@pytest.mark.parametrize("name", ["ragged_bf16_d128", "tiny"])
def test_token_out_of_range_column_ids_are_skipped(name):
    """Lists padded with -1 / NB entries give the same output as clean lists."""
    _gpu()
    import torch
    run = Run(W[name], radius_override=40)
    NB = run.plan.n_blocks
    cnt, cols = run.cnt.cpu().numpy(), run.cols.cpu().numpy()
    cnt2, cols2 = np.zeros_like(cnt), np.full_like(cols, -1)
    for idx in np.ndindex(cnt.shape):
        valid = cols[idx][:cnt[idx]].tolist()
        out = []
        for c in valid:
            out += [-1, c]
        out = (out + [NB])[:NB]
        kept = [c for c in out if 0 <= c < NB]
        cnt2[idx], cols2[idx][:len(out)] = len(out), out
        cnt[idx], cols[idx][:len(kept)] = len(kept), kept
    dev = run.q.device
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    ref = _token_call(run, cnt=t(cnt), cols=t(cols))
    got = _token_call(run, cnt=t(cnt2), cols=t(cols2))
    assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1])


def test_token_unsupported_shapes_are_rejected():
    """bf16 token attention needs thresholds below 65536 and H*W >= block."""
    _gpu()
    import torch
    import paper_2608_02504_amd as tra
    for cfg in (tra.Config(batch=1, heads=1, frames=1, height=300, width=300, head_dim=64),
                tra.Config(batch=1, heads=1, frames=3, height=8, width=8, head_dim=64)):
        plan = tra.Plan(cfg)
        S, NB = cfg.n_tokens, plan.n_blocks
        x = torch.zeros(1, 1, S, 64, dtype=torch.bfloat16, device="cuda")
        rad = torch.zeros(1, 1, S, dtype=torch.int32, device="cuda")
        cnt = torch.zeros(1, 1, NB, dtype=torch.int32, device="cuda")
        cols = torch.zeros(1, 1, NB, NB, dtype=torch.int32, device="cuda")
        with pytest.raises(tra.TraError, match="UNSUPPORTED"):
            tra.tra_token_attention(plan, x, x, x, rad, cnt, cols, None, torch.empty_like(x))


@pytest.mark.parametrize("radius", [3000, 20000])
def test_token_attention_largest_frame(radius):
    """The largest frame bf16 token attention takes (thresholds below 65,536:
    182 x 182, n_cap = 65,522), two frames: the 2-D key test's vectors reach
    their largest coordinates and thresholds.  Forced radii leave most tiles
    partially covered; 24 sampled query blocks (the last included) against the
    oracle's token_attention_rows."""
    _gpu()
    w = synth.Workload("frame182_bf16", 1, 1, 64, "bf16", 2, 182, 182, 128, 0.25, 4.0, 0.6, seed=84,
                       tile_h=8, tile_w=16)
    run = Run(w, rule="union", radius_override=radius)
    o, lse = _token_call(run)
    tabs = OracleTables(w)
    q, k, v = (synth.to_f64(a[0, 0], w.dtype) for a in (run.q_np, run.k_np, run.v_np))
    blocks = sample_blocks(w, 24, seed=11)[(0, 0)]
    M = run.mask[0, 0].cpu().numpy().astype(bool)[blocks]
    rows, o_ref, lse_ref = O.token_attention_rows(
        q, k, v, tabs.perm, w.block, list(blocks), M, run.rad[0, 0].cpu().numpy(), tabs.F, tabs.H, tabs.W,
        w.gamma, distance="2d", return_lse=True)
    err = np.abs(o[0, 0].double().cpu().numpy()[rows] - o_ref).max()
    assert err <= TOL_O_BF16, f"token attention max-abs {err:.3e}"
    lse_gpu = lse[0, 0].double().cpu().numpy()[rows]
    assert np.abs(lse_gpu - lse_ref).max() <= 1e-4 + 1e-5 * np.abs(lse_ref).max(), "token lse"
    log(f"182 x 182 frames, radius {radius}: kept {run.cnt.float().mean().item():.1f} blocks per row, "
        f"token attention max-abs {err:.2e}")


@pytest.mark.slow
def test_token_attention_720p_sampled_at_paper_density():
    """Token-level attention at the headline shape with about 15 % of the blocks
    kept (one constant entropy ln(7997 / tau) for every token), without a row
    order as the benchmark runs it: 8 sampled query blocks in each of 4 heads
    against the oracle's token_attention_rows, outputs and lse."""
    _gpu()
    w = synth.workload("wan14b_720p")
    run = Run(w, with_order=False, entropy_override=float(np.log(7997 / w.tau)))
    o, lse = _token_call(run)
    tabs = OracleTables(w)
    worst = 0.0
    for (b, h), blocks in sample_blocks(w, 8, seed=7).items():
        if h not in (0, 13, 26, 39):
            continue
        q, k, v = (synth.to_f64(a[b, h], w.dtype) for a in (run.q_np, run.k_np, run.v_np))
        M = run.mask[b, h].cpu().numpy().astype(bool)[blocks]
        n_tok = run.rad[b, h].cpu().numpy()
        rows, o_ref, lse_ref = O.token_attention_rows(
            q, k, v, tabs.perm, w.block, list(blocks), M, n_tok, tabs.F, tabs.H, tabs.W, w.gamma,
            distance=run.cfg.distance, return_lse=True)
        err = np.abs(o[b, h].double().cpu().numpy()[rows] - o_ref).max()
        assert err <= TOL_O_BF16, f"token attention max-abs {err:.3e} (b={b}, h={h})"
        lse_gpu = lse[b, h].double().cpu().numpy()[rows]
        assert np.abs(lse_gpu - lse_ref).max() <= 1e-4 + 1e-5 * np.abs(lse_ref).max(), "token lse"
        worst = max(worst, float(err))
        log(f"wan14b_720p token-level: batch {b} head {h} checked")
    log(f"wan14b_720p token-level at the paper's density: max-abs {worst:.2e}")
