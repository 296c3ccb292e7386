"""A frame's ball is decided by a wave of its own, window points by tiles: on a
lattice of 0.25 m, whose points are exact, the ball's record is byte for byte
that of the map's point it lies on, alone, in a batch and beside a map, for no
opponent to 16, robots faster than vmax, positions inside a robot, on the goal
line and past every gap, and every sample count."""
import numpy as np
import pytest

from paper_1909_07717_amd.framegen import Params, random_frame

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

H, NX, NY = 0.25, 49, 37


def _cases(n_opp, fast):
    f = random_frame(np.random.default_rng(300 + n_opp), 3, n_opp)
    if fast:
        f.opp[:, 2:] *= np.float32(3.0)
    if n_opp:
        f.opp[0, :2] = (1.0, 0.25)  # a lattice point is inside this robot
    spots = [(28, 19), (48, 18), (48, 25), (0, 0), (24, 18), (47, 16), (40, 3), (36, 30)]
    out = []
    for i, j in spots:
        g = f.copy()
        g.ball = np.float32([H * (i - (NX - 1) / 2), H * (j - (NY - 1) / 2)])
        g.windows = [(H, 0, 0, NX, NY)]
        out.append((g, j * NX + i))
    return out


@pytest.mark.parametrize("K", [64, 128, 192, 256])
@pytest.mark.parametrize("n_opp,fast", [(0, False), (1, False), (7, True), (15, False),
                                        (16, True)])
def test_ball_equals_the_map_there(K, n_opp, fast):
    from paper_1909_07717_amd import binding as B
    print(f"[shot ball] K={K} n_opp={n_opp} fast={fast}", flush=True)
    s = B.Searcher(Params(n_samples=K).as_f32())
    cases = _cases(n_opp, fast)
    frames = [f for f, _ in cases]
    balls, maps = s.shot(frames, 5.0, 0.05, 0.0)
    only, _ = s.shot(frames, 5.0, 0.05, 0.0, map=False)
    torch.cuda.synchronize()
    balls, only, maps = (B.shots_host(t) for t in (balls, only, maps))
    for q, (f, at) in enumerate(cases):
        want = maps[q * NX * NY + at].tobytes()
        one, one_map = s.shot([f], 5.0, 0.05, 0.0)
        alone, _ = s.shot([f], 5.0, 0.05, 0.0, map=False)
        torch.cuda.synchronize()
        got = [balls[q].tobytes(), only[q].tobytes()] + \
              [B.shots_host(t)[0].tobytes() for t in (one, alone)]
        assert got == [want] * 4, (q, f.ball, balls[q], maps[q * NX * NY + at])
        assert B.shots_host(one_map)[at].tobytes() == want
    s.close()
