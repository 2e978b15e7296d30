"""2D Euler stages in FP64 by pairs of waves against one wave per run.

Grids whose runs are short take a pair of waves per run (one for each
direction's sweep); a launch shape set by hand takes one wave.  Both
evaluate the same expressions on the same values, so they agree bitwise: at the
edges of the strips, with one row and with several per run, at every boundary,
with several grids in one launch and over whole steps."""
import numpy as np
import pytest
import torch

import paper_2402_03074_amd as H

pytestmark = pytest.mark.gpu

# a strip is 62 columns; 3 rows or columns are the fewest; (400, 203) and the 24 grids
# have several rows per run, those of the 24 going on in the next grid
GRIDS = [[(3, 3)], [(62, 5)], [(63, 4)], [(125, 3)], [(131, 97)], [(400, 203)],
         [(40, 40), (63, 21), (5, 130)], [(60, 61)] * 24]
SIDES = ["periodic", ("transmissive", "reflective", "reflective", "transmissive")]


def _state(grids, seed):
    rng = np.random.default_rng(seed)
    u, m = [], []
    for nx, ny in grids:
        n = nx * ny
        rho, p = rng.uniform(0.8, 0.9, n), rng.uniform(0.7, 0.9, n)
        vx, vy = rng.uniform(-0.2, 0.2, n), rng.uniform(-0.2, 0.2, n)
        u.append(np.stack([rho, rho * vx, rho * vy, p / 0.4 + 0.5 * rho * (vx * vx + vy * vy)]))
        m.append(0.005 * rng.uniform(-1, 1, (2, 4, n)))
    return np.concatenate(u, axis=1), np.concatenate(m, axis=2)


@pytest.mark.parametrize("weights", ["scale_invariant", "zq"])
@pytest.mark.parametrize("sides", SIDES, ids=["periodic", "walls"])
@pytest.mark.parametrize("grids", GRIDS, ids=lambda g: f"{len(g)}x{g[0]}")
def test_pairs_equal_single_waves(grids, sides, weights):
    print(f"[gpu] pairs {grids} {sides} {weights}", flush=True)
    u0, m0 = _state(grids, 11)
    insts, off = [], 0
    for nx, ny in grids:
        insts.append(H.make_inst(nx, ny, (0.0, 1.0, 0.0, 1.5), sides, offset=off))
        off += nx * ny
    out = []
    for shape in (None, (4, 0)):
        S = H.Solver(2, "euler", insts, weights=weights)
        if shape:
            S.set_launch(*shape)
        u = torch.tensor(u0, device="cuda")
        m = torch.tensor(m0, device="cuda").to(S.mom_dtype)
        a = S.max_wavespeed(u)
        h = torch.tensor([[I.nx / 1.0, I.ny / 1.5] for I in insts], dtype=torch.float64,
                         device="cuda")
        dt = 0.4 / (a * h).sum(1)
        b = [(u, m)] + [S.empty_state() for _ in range(3)]
        for s in range(3):
            S.stage(s, dt, a, *b[s], *b[s + 1])
        torch.cuda.synchronize()
        out.append([x for y in b[1:] for x in y])
        out[-1] += [u, m] + [S.advance(u, m, 0.4, 1e30, 2)]
        S.close()
    (*x, rx), (*y, ry) = out
    assert all(torch.equal(a, b) for a, b in zip(x, y))
    assert rx == ry and rx[1] == [2] * len(grids)
