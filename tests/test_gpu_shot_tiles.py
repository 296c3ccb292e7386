"""Shooting decisions at the edges of the map's tiles of 32 positions (1, 31,
32, 33, 65 positions; 0, 1, 15 and 16 opponents; every sample count; robots
faster than vmax): against the oracle, and the same bytes for a window that
travels with the launch, for one of several windows and within a larger one."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1909_07717_amd.framegen import Params, random_frame
from tests.test_gpu_shot import _close

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

H = np.float32(0.1)
SIZES = [(1, 1), (31, 1), (8, 4), (11, 3), (5, 13)]


def _frame(n_opp, fast, seed):
    f = random_frame(np.random.default_rng(seed), 3, n_opp, Params())
    if fast:
        f.opp[:, 2:] *= 3.0
    return f


@pytest.mark.parametrize("K", [64, 128, 192, 256])
@pytest.mark.parametrize("n_opp,fast", [(0, False), (1, False), (8, True), (15, False),
                                        (16, True)])
def test_shot_tiles(K, n_opp, fast):
    from paper_1909_07717_amd import binding as B
    print(f"[shot tiles] K={K} n_opp={n_opp} fast={fast}", flush=True)
    p = Params(n_samples=K).as_f32()
    s = B.Searcher(p)
    f = _frame(n_opp, fast, 40 + n_opp)
    i0, j0, nx, ny = 70, 40, 13, 13
    f.windows = [(H, i0, j0, nx, ny)]
    _, mp = s.shot([f], 6.5, 0.05, 0.0)
    torch.cuda.synchronize()
    g = B.shots_host(mp)[:nx * ny].copy()
    o = O.shot_search(f, p, v_shot=6.5, min_angle=0.05, margin_s=0.0, bands=True)
    ok = o["ambig"] == 0
    assert ok.mean() > 0.9
    assert (g["shoot"][ok] == o["shoot"][ok]).all()
    assert (g["reachable"][ok] == o["reachable"][ok]).all()
    for k in ("gap", "open_angle", "aim"):
        assert _close(g[k][ok], o[k][ok], 2e-5), k
    cond = ok & (o["length_sens"] < 1e-4)
    assert _close(g["length"][cond], o["length"][cond], 2e-4)
    assert _close(g["t_goal"][cond], o["t_goal"][cond], 1e-4)
    well = ok & (o["slack_sens"] < 5e-5)
    assert _close(g["slack"][well], o["slack"][well], 1e-4)
    whole = g.reshape(ny, nx)
    if n_opp:  # the sizes as windows of their own, alone and together
        wins = [(H, i0 + 1, j0, a, b) for a, b in SIZES if a < nx and b <= ny]
        f.windows = wins
        _, mp = s.shot([f], 6.5, 0.05, 0.0)
        torch.cuda.synchronize()
        many = B.shots_host(mp)
        off = 0
        for w in wins:
            a, b = w[3], w[4]
            part = many[off:off + a * b]
            off += a * b
            assert part.tobytes() == whole[:b, 1:1 + a].tobytes()
            f.windows = [w]
            ball, mp = s.shot([f], 6.5, 0.05, 0.0)
            torch.cuda.synchronize()
            assert B.shots_host(mp)[:a * b].tobytes() == part.tobytes()
            alone, _ = s.shot([f], 6.5, 0.05, 0.0, map=False)
            assert B.shots_host(alone)[:1].tobytes() == B.shots_host(ball)[:1].tobytes()
    # a row longer than a tile
    f.windows = [(H, 50, 50, 31, 1), (H, 50, 50, 33, 1), (H, 50, 50, 65, 1)]
    _, mp = s.shot([f], 6.5, 0.05, 0.0)
    torch.cuda.synchronize()
    r = B.shots_host(mp)
    assert r[:31].tobytes() == r[31 + 33:31 + 33 + 31].tobytes() == r[31:62].tobytes()
    assert r[31:64].tobytes() == r[64:97].tobytes()
    s.close()
