"""The block mask's three filters (box against box, query against box, pair by
pair on the matrix cores) against the oracle's literal Alg. 1, bit for bit, at
the edges where one hands over to the next: mixed radii from 0 to FULL in one
block, out-of-range ones, blocks that span two frames and more, ragged last
blocks of fewer than 64 and 32 keys, clipped tiles, both block sizes."""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu

# frames, height, width, text tokens, block, block layout
GRIDS = [(3, 16, 32, 0, 128, "packed"),    # whole tiles, one frame a block
         (4, 13, 27, 0, 128, "packed"),    # blocks over two frames, last one 124 tokens
         (2, 9, 23, 0, 128, "packed"),     # last block 30 tokens
         (5, 10, 17, 30, 64, "packed"),    # block 64, text, a mixed block
         (6, 5, 9, 0, 128, "packed"),      # blocks over more than two frames
         (3, 13, 27, 40, 128, "tiles"),    # clipped tiles of 44 to 128 tokens
         (3, 30, 52, 0, 128, "packed")]    # 37 blocks: more than eight undecided per wave


@pytest.mark.parametrize("grid", GRIDS, ids=str)
@pytest.mark.parametrize("rule", ["vote", "union"])
@pytest.mark.parametrize("distance", ["2d", "1d"])
def test_mask_filters(grid, rule, distance):
    import torch
    import paper_2608_02504_amd as tra
    F, H, W, T, b, layout = grid
    gamma = 0.3
    plan = tra.Plan(tra.Config(1, 4, F, H, W, 64, block=b, tile_h=8, tile_w=b // 8, dtype="bf16" if b == 128 else "fp32",
                               rule=rule, gamma=gamma, distance=distance, text_tokens=T, block_layout=layout))
    S, NB, cap = plan.n_tokens, plan.n_blocks, plan.n_cap
    rng = np.random.default_rng(5)
    rad = np.stack([rng.integers(0, 40, S),                                       # short
                    np.floor(np.exp(rng.uniform(0, np.log(cap + 1), S))) - 1,     # 0 to the cap
                    rng.choice([-7, 0, 1, cap, cap + 1, 2 ** 31 - 1], S),         # the extremes
                    np.where(rng.random(S) < 0.34, 2 ** 31 - 1, 9)]).astype(np.int64)  # about a third FULL
    r = torch.tensor(rad[None], dtype=torch.int32, device="cuda")
    mask = torch.empty(1, 4, NB, NB, dtype=torch.uint8, device="cuda")
    cnt = torch.empty(1, 4, NB, dtype=torch.int32, device="cuda")
    cols = torch.empty(1, 4, NB, NB, dtype=torch.int32, device="cuda")
    order = torch.empty(4 * NB, dtype=torch.int32, device="cuda")
    tra.tra_build_block_mask(plan, r, mask, cnt, cols, order)
    if layout == "tiles":
        perm = O.tile_aligned_order(F, H, W, 8, b // 8, b, text_tokens=T)
    else:
        perm = O.joint_order(O.tile_major_order(F, H, W, 8, b // 8), T)
    M = mask[0].cpu().numpy().astype(bool)
    for h in range(4):
        n = np.where(rad[h] > cap, O.RADIUS_FULL, np.maximum(rad[h], 0))
        n[F * H * W:] = O.RADIUS_FULL
        want = O.block_mask_rows(n, perm, b, F, H, W, gamma, list(range(NB)), rule=rule, distance=distance)
        assert np.array_equal(M[h], want), f"head {h}: {np.argwhere(M[h] != want)[:5]}"
        for u in range(NB):
            keep = np.nonzero(want[u])[0]
            assert int(cnt[0, h, u]) == len(keep)
            assert np.array_equal(cols[0, h, u].cpu().numpy(), np.r_[keep, np.full(NB - len(keep), -1)])
    c = cnt.cpu().numpy().reshape(-1)
    assert np.array_equal(order.cpu().numpy(), np.argsort(-c, kind="stable"))
