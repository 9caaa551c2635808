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
