"""The radius search through the count table's index at row lengths around its
line (32), group (512) and run (8,192) sizes, budgets from 1 past the largest count, against
the oracle's search, integer for integer."""
import math

import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu


# n_cap = (H-1)^2 + (W-1)^2: 0, 26, 32, 128, 493, 512, 545, 8,177; 8,200 (two runs of the index's first
# level), 16,385 (three), 39,602 (five)
@pytest.mark.parametrize("grid", [(3, 1, 1, 200), (5, 2, 6, 9), (4, 5, 5, 0), (3, 9, 9, 0), (2, 4, 23, 3), (3, 17, 17, 0),
                                  (2, 17, 18, 0), (3, 45, 80, 5), (2, 91, 11, 3), (2, 129, 2, 0), (1, 2, 200, 7)], ids=str)
@pytest.mark.parametrize("gamma", [0.0, 0.6])
def test_radius_index(grid, gamma):
    import torch
    import paper_2608_02504_amd as tra
    F, H, W, T = grid
    plan = tra.Plan(tra.Config(1, 3, F, H, W, 64, block=64, tile_h=8, tile_w=8, dtype="fp32", gamma=gamma, text_tokens=T))
    S, N = plan.n_tokens, F * H * W
    rng = np.random.default_rng(8)
    budgets = np.stack([rng.integers(1, S + 1, S), np.minimum(S, np.floor(np.exp(rng.uniform(0, math.log(S + 1), S)))),
                        rng.choice([1, 2, F, min(F + 1, S), max(1, N - 1), N, S], S)])
    # K = ceil(0.9 e^H): H a little below log(K / 0.9), K - 1/2 of the way up
    ent = np.log((budgets - 0.5) / 0.9).astype(np.float32)
    khat = np.clip(np.ceil(0.9 * np.exp(ent.astype(np.float64))), 1, S).astype(np.int64)
    r = torch.empty(1, 3, S, dtype=torch.int32, device="cuda")
    b = torch.empty_like(r)
    tra.tra_budget_radius(plan, torch.tensor(ent[None], device="cuda"), b, r)
    f, x, y = O.grid_coords(F, H, W)
    cap = O.n_cap(H, W)
    thr, disk = O.threshold_table(cap, F, gamma), O.disk_count_table(H, W, cap)
    for h in range(3):
        assert np.array_equal(b[0, h, :N].cpu().numpy(), khat[h, :N])
        want = O.select_radius(khat[h, :N], f, x, y, F, thr, disk)
        assert np.array_equal(r[0, h, :N].cpu().numpy(), want)
        assert (r[0, h, N:] == O.RADIUS_FULL).all() and (b[0, h, N:] == S).all()
