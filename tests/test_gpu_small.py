"""The key-splitting kernel of bf16 calls with few rows: fewer key tiles than
waves, sub-tiles without a token, lists whose entries leave waves without a tile,
both head sizes, against the oracle; and, on each side of the line where the
other kernels take over, a plan's heads against the same heads alone."""
import numpy as np
import pytest

import oracle as O
import synth
from _pipeline import TOL_O_BF16, OracleTables, Run, check_head, to_np_f64

pytestmark = pytest.mark.gpu

# frames, height, width, text tokens, head_dim
SHAPES = [(1, 4, 5, 0, 128), (1, 8, 16, 0, 64), (1, 8, 17, 0, 128), (2, 9, 23, 20, 64), (3, 11, 29, 0, 128),
          (9, 16, 32, 7, 64)]


@pytest.mark.parametrize("shape", SHAPES, ids=str)
@pytest.mark.parametrize("radius", [None, 2])
def test_small_calls(shape, radius):
    f, h, w, t, d = shape
    wl = synth.Workload("small", 1, 2, d, "bf16", f, h, w, 128, 0.25, 4.0, 0.6, seed=31, tile_h=8, tile_w=16,
                        text_tokens=t)
    run = Run(wl, rule="union", radius_override=radius)
    tabs = OracleTables(wl)
    for hd in range(2):
        check_head(run, tabs, 0, hd, np.arange(wl.n_blocks), TOL_O_BF16, {})


def test_small_padded_blocks():
    """Tile-aligned blocks of 32 to 128 tokens: sub-tiles and query tiles without one."""
    wl = synth.Workload("small_tiles", 1, 2, 128, "bf16", 3, 12, 24, 128, 0.25, 4.0, 0.6, seed=32, tile_h=8, tile_w=16,
                        text_tokens=40)
    run = Run(wl, rule="union", radius_override=30, block_layout="tiles")
    tabs = OracleTables(wl, block_layout="tiles")
    for h in range(2):
        q, k, v = (synth.to_f64(a[0, h], "bf16") for a in (run.q_np, run.k_np, run.v_np))
        M = run.mask[0, h].cpu().numpy().astype(bool)
        rows, o_ref = O.masked_attention_rows(q, k, v, tabs.perm, 128, list(range(tabs.n_blocks)), M)
        assert np.abs(to_np_f64(run.O_sp[0, h])[rows] - o_ref).max() <= TOL_O_BF16


@pytest.mark.parametrize("head_dim,heads", [(128, 8), (128, 9), (128, 4), (128, 5), (64, 12), (64, 13)])
def test_small_at_the_line(head_dim, heads):
    """16 blocks a head: 128 and 144 rows (the line of the dense, sparse and
    entropy calls on 256 CUs), 64 and 80 (fused), 192 and 208 (head_dim 64).
    Every head against a one-head plan's call, which the small kernel takes."""
    import torch
    import paper_2608_02504_amd as tra
    cfg = dict(frames=4, height=16, width=32, head_dim=head_dim)
    plan, one = tra.Plan(tra.Config(1, heads, **cfg)), tra.Plan(tra.Config(1, 1, **cfg))
    S, NB = plan.n_tokens, plan.n_blocks
    g = torch.Generator(device="cuda").manual_seed(6)
    q, k, v = (torch.randn(1, heads, S, head_dim, generator=g, device="cuda").bfloat16() for _ in range(3))
    cnt = torch.full((1, heads, NB), NB - 3, dtype=torch.int32, device="cuda")
    cols = torch.arange(NB, dtype=torch.int32, device="cuda").expand(1, heads, NB, NB).contiguous()

    def outputs(p, q, k, v, cnt, cols):
        n = q.shape[1]
        o = [torch.empty_like(q) for _ in range(3)]
        f = [torch.empty(1, n, S, device="cuda") for _ in range(4)]
        tra.tra_dense_attention(p, q, k, v, o[0], f[0])
        tra.tra_entropy(p, q, k, v, o[1], f[1])
        tra.tra_entropy(p, q, k, None, None, f[2])
        tra.tra_sparse_attention(p, q, k, v, cnt, cols, None, o[2], f[3])
        return o, f

    o, f = outputs(plan, q, k, v, cnt, cols)
    for h in range(heads):
        o1, f1 = outputs(one, *(t[:, h:h + 1].contiguous() for t in (q, k, v, cnt, cols)))
        for a, b in zip(o, o1):  # bf16 outputs below 1 of the same sums in another order: an ulp or two
            assert (a[:, h:h + 1].float() - b.float()).abs().max() <= 2 ** -7
        for a, b in zip(f, f1):
            assert (a[:, h:h + 1] - b).abs().max() <= 1e-5 * b.abs().max()
