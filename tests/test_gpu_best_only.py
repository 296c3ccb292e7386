"""The surrogate search leaves out points whose score bound is below the best
found: the records are those, byte for byte, of the search that evaluates every
point, for every sample count, speeds in and out of reach, weights of both
signs (a negative weight of the angle or the margin has no such bound) and
frames without a pass."""
import dataclasses

import numpy as np
import pytest

from paper_1909_07717_amd.framegen import (Params, full_window, random_frame, speeds_linear,
                                           variants_for)
from tests.test_gpu_mlp import _windows_of_cells

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

WEIGHTS = [(0.5, 0.3, 0.2), (0.0, 0.0, 0.2), (0.7, -0.3, 0.0), (-0.2, 0.3, 0.2), (0.5, 0.3, -0.1)]


def _frames(n, seed):
    out = []
    for i in range(n):
        rng = np.random.default_rng(seed + i)
        f = random_frame(rng, int(rng.integers(2, 9)), int(rng.integers(0, 9)))
        f.windows = [full_window(0.2)]
        flat, chip = [(1, 0), (8, 0), (0, 3), (32, 32)][i % 4]
        lo = 0.2 if i % 3 == 0 else 1.5  # some frames reach a few metres only
        hi = 1.2 if i % 3 == 0 else 6.5
        f.variants = (variants_for(speeds_linear(flat, lo, hi), True, False) if flat else []) + \
                     (variants_for(speeds_linear(chip, lo, hi), False, True) if chip else [])
        out.append(f)
    return out


@pytest.mark.parametrize("K,weights", [(64, w) for w in WEIGHTS] +
                         [(k, WEIGHTS[0]) for k in (128, 192, 256)])
def test_best_only_equals_the_whole_search(K, weights):
    from paper_1909_07717_amd import binding as B
    print(f"[best only] K={K} weights={weights}", flush=True)
    p = dataclasses.replace(Params(n_samples=K), w_angle=weights[0], w_dist=weights[1],
                            w_margin=weights[2]).as_f32()
    s = B.Searcher(p)
    net = B.Mlp(s, 16, seed=7)
    frames = _frames(12, 4000)
    bt = s.batch(frames)
    raw = B.best_records(net.search(bt, k=64, fallback=False)[0]).copy()
    all_t, nfb = net.search(bt, k=64, fallback=True)
    full = B.best_records(all_t).copy()
    net.forward(bt)
    cells = net.topk(len(frames), 64).cpu().numpy()
    redo = 0
    for i, f in enumerate(frames):
        g = f.copy()
        g.windows = _windows_of_cells(cells[i])
        _, ref = s.search(g)
        assert raw[i].tobytes() == ref.tobytes(), i
        if not ref["found"]:
            redo += 1
            g.windows = [full_window(0.05)]
            _, ref = s.search(g)
        assert full[i].tobytes() == ref.tobytes(), i
        one, _ = net.search_frames([f], k=64, fallback=True)
        torch.cuda.synchronize()
        assert B.best_records(one).tobytes() == ref.tobytes(), i
    assert nfb == redo > 0
    bt.close(); net.close(); s.close()
