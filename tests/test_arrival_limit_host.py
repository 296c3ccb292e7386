"""The arrival limit that lets the point search leave robots out of a quarter
of a path: 1.03 times the time, to the quarter's end, of the slowest ball
that gets to the end of the path.  A robot at or past the limit must not be
able to intercept any kick that reaches the path's end, by a clear margin in
kick speed where the ball still moves, so that which later time stands in
for it decides nothing."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1909_07717_amd.framegen import CHIP, FLAT, Params


def _range(p, typ):
    """Stopping distance of a 1 m/s kick."""
    if typ == CHIP:
        vh = np.cos(p.chip_angle)
        return np.sin(2 * p.chip_angle) / p.gravity + vh * vh / (2 * p.roll_decel)
    return ((1 - p.slide_ratio ** 2) / (2 * p.slide_decel)
            + p.slide_ratio ** 2 / (2 * p.roll_decel))


@pytest.mark.parametrize("typ", [FLAT, CHIP])
@pytest.mark.parametrize("p", [Params(), Params(slide_decel=3.0, roll_decel=1.5, slide_ratio=0.4),
                               Params(roll_decel=0.1, chip_angle=1.2)])
@pytest.mark.parametrize("d", [0.3, 2.0, 9.0])
def test_no_reaching_kick_is_met_past_the_limit(typ, p, d):
    v = np.sqrt(d / _range(p, typ)) * (1 + 1e-12)  # stops at the path's end
    for q in range(1, 5):
        end = d * q / 4
        limit = 1.03 * O.ball_time(p, typ, v, min(end, d))
        assert np.isfinite(limit)
        for s in np.linspace(0.02, 1.0, 12) * end:
            for f in (1.0, 1.3, 3.0):
                assert O.ball_time(p, typ, f * v, s) < limit
            if q < 4:  # even a slightly slower kick has passed (or stopped short)
                t = O.ball_time(p, typ, v * (1 - 2e-3), s)
                assert t < limit
        if q == 4:     # past the stop of every kick that stops on the path
            for s in np.linspace(0.05, 1.0, 12) * d:
                u = np.sqrt(s / _range(p, typ))
                assert O.ball_time(p, typ, u * (1 + 1e-9), s) < limit
