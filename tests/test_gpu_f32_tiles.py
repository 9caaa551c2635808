"""fp32 attention at the edges of its 32-token tiles: fewer tokens than one
tile, exactly one, one more, one tile per wave and a remainder, padded blocks.
Every output is held to the fp32 bar of the parity tests (1e-5 max-abs)."""
import numpy as np
import pytest

import oracle as O
import synth
from _pipeline import TOL_O_FP32, OracleTables, Run, check_head, check_lists, to_np_f64

pytestmark = pytest.mark.gpu

# frames, height, width, text tokens, head_dim, block
SHAPES = [(1, 4, 5, 0, 128, 64), (1, 4, 8, 0, 64, 64), (1, 3, 11, 0, 128, 128), (2, 9, 14, 5, 128, 64),
          (2, 9, 15, 3, 64, 128), (3, 10, 18, 40, 128, 128)]


def _workload(shape):
    f, h, w, text, d, b = shape
    return synth.Workload(f"f32_{f}x{h}x{w}+{text}_d{d}_b{b}", 1, 2, d, "fp32", f, h, w, b, 0.25, 4.0, 0.6, seed=77,
                          tile_h=8, tile_w=b // 8, text_tokens=text)


@pytest.mark.parametrize("shape", SHAPES, ids=str)
@pytest.mark.parametrize("radius", [None, 3])
def test_fp32_tile_edges(shape, radius):
    """Entropy, dense, fused and block-sparse calls (own radii, and short forced
    ones whose rows keep few blocks) against the oracle, every row."""
    w = _workload(shape)
    run = Run(w, rule="union", radius_override=radius)
    tabs = OracleTables(w)
    for h in range(w.heads):
        check_head(run, tabs, 0, h, np.arange(w.n_blocks), TOL_O_FP32, {})
    check_lists(run)


@pytest.mark.parametrize("shape", SHAPES[3:], ids=str)
def test_fp32_padded_blocks(shape):
    """Tile-aligned blocks, whose clipped tiles leave query tiles without a
    token and key tiles with few."""
    w = _workload(shape)
    run = Run(w, rule="union", radius_override=3, block_layout="tiles")
    tabs = OracleTables(w, block_layout="tiles")
    for h in range(w.heads):
        M = run.mask[0, h].cpu().numpy().astype(bool)
        q, k, v = (synth.to_f64(a[0, h], "fp32") for a in (run.q_np, run.k_np, run.v_np))
        rows, o_ref = O.masked_attention_rows(q, k, v, tabs.perm, w.block, list(range(tabs.n_blocks)), M)
        assert np.abs(to_np_f64(run.O_sp[0, h])[rows] - o_ref).max() <= TOL_O_FP32


@pytest.mark.parametrize("call", ["entropy", "sparse"])
def test_fp32_more_tiles_than_a_launch_holds(call):
    """2^21 + 2^10 one-token heads of 128-token blocks: 2^23 + 2^12 query tiles of 512
    threads, more than the 2^32 threads of one launch.  A lone key's output is its
    value and its entropy 0, whatever the score."""
    import torch
    import paper_2608_02504_amd as tra
    n = (1 << 21) + (1 << 10)
    assert n * 4 * 512 > 1 << 32
    plan = tra.Plan(tra.Config(1 << 10, n >> 10, 1, 1, 1, 64, dtype="fp32"))
    g = torch.Generator(device="cuda").manual_seed(1)
    q, v = (torch.randn(1 << 10, n >> 10, 1, 64, generator=g, device="cuda") for _ in range(2))
    o = torch.full_like(v, -1.0)
    per = torch.full((1 << 10, n >> 10, 1), -1.0, device="cuda")
    if call == "entropy":
        tra.tra_entropy(plan, q, q, v, o, per)
        assert (per == 0).all()
    else:
        cnt = torch.ones(1 << 10, n >> 10, 1, dtype=torch.int32, device="cuda")
        cols = torch.zeros(1 << 10, n >> 10, 1, 1, dtype=torch.int32, device="cuda")
        tra.tra_sparse_attention(plan, q, q, v, cnt, cols, None, o, per)
        want = (q.double() ** 2).sum(-1) / 8
        assert ((per.double() - want).abs() <= 1e-5 * want).all()
    assert torch.equal(o, v)
