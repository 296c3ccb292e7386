"""The best-only searches split their tiles by how many there are per workgroup
(all its own, a quarter and then groups from the counter): the records of a
batch are, byte for byte, those of the same frames in batches of 8, from less
than one tile a workgroup to many, for the re-scored windows and for the exact
fallback of few and of many frames."""
import numpy as np
import pytest

from paper_1909_07717_amd.framegen import (Params, full_window, random_frame, speeds_linear,
                                           variants_for)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _frames(n):
    out = []
    for i in range(n):
        rng = np.random.default_rng(7000 + i)
        f = random_frame(rng, int(rng.integers(3, 9)), int(rng.integers(2, 9)))
        f.windows = [full_window(0.2)]
        f.variants = variants_for(speeds_linear(1 + i % 2, lo=3.0), True, False)
        out.append(f)
    return out


@pytest.mark.parametrize("n,k,below", [(17, 64, None), (24, 100, None), (40, 128, 0.30),
                                       (104, 64, 0.25), (200, 64, None), (600, 32, 0.15)])
def test_records_do_not_depend_on_the_batch(n, k, below):
    from paper_1909_07717_amd import binding as B
    print(f"[claims] n={n} k={k} below={below}", flush=True)
    p = Params(n_samples=64).as_f32()
    s = B.Searcher(p)
    net = B.Mlp(s, n, max_k=k, seed=3)
    frames = _frames(n)
    kw = dict(k=k, fallback_below=float("-inf") if below is None else below)
    got, n_fb = net.search(s.batch(frames), **kw)
    got = B.best_records(got).copy()
    parts, want_fb = [], 0
    for i in range(0, n, 8):
        r, c = net.search(s.batch(frames[i:i + 8]), **kw)
        parts.append(B.best_records(r).copy())
        want_fb += c
    want = np.concatenate(parts)
    assert got.tobytes() == want.tobytes()
    assert n_fb == want_fb
    print(f"[claims] fallbacks {n_fb} of {n}, found {int((got['found'] != 0).sum())}", flush=True)
    s.close()
