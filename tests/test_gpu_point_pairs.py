"""The point search evaluates two neighbouring points per wave, 32 lanes each:
parity with the oracle at the edges of that split (odd point counts, one
point, one variant, 32 / 33 / 64 variants, 16 / 17 / 31 interceptors, every
sample count), and the reduced output against the full maps."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1909_07717_amd.framegen import (Params, full_window, random_frame, speeds_linear,
                                           variants_for)
from tests.parity import BandPool, compare_maps

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CASES = [
    # n_team, n_opp, K, flat speeds, chip speeds, window
    (8, 8, 256, 16, 16, (0.05, 100, 60, 7, 3)),   # 32 variants, 21 points
    (8, 8, 256, 17, 16, (0.05, 3, 5, 5, 5)),      # 33 variants
    (9, 8, 192, 32, 32, (0.1, 40, 20, 9, 7)),     # 64 variants, 16 interceptors
    (10, 8, 128, 8, 0, (0.1, 10, 70, 11, 3)),     # 17 interceptors
    (16, 16, 64, 5, 4, (0.2, 0, 0, 13, 5)),       # 31 interceptors
    (2, 1, 64, 1, 0, (0.2, 30, 22, 1, 1)),        # one point
    (1, 3, 128, 4, 2, (0.2, 20, 10, 3, 3)),       # no receiver
    (4, 0, 256, 0, 3, (0.2, 50, 40, 5, 2)),       # chips only, no opponent
]


def _frame(n_team, n_opp, flat, chip, win, seed):
    f = random_frame(np.random.default_rng(seed), n_team, n_opp)
    f.windows = [(float(np.float32(win[0])),) + win[1:]]
    f.variants = (variants_for(speeds_linear(flat, lo=1.5), True, False) if flat else []) + \
                 (variants_for(speeds_linear(chip, lo=1.5), False, True) if chip else [])
    return f


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c[:5])))
def test_pairs_match_oracle(case):
    from paper_1909_07717_amd import binding as B
    n_team, n_opp, K, flat, chip, win = case
    p = Params(n_samples=K).as_f32()
    s = B.Searcher(p)
    r = B.Searcher(p, out_flags=B.DPPS_OUT_REDUCED)
    for seed in range(4):
        print(f"[pairs] {case} seed={seed}", flush=True)
        f = _frame(n_team, n_opp, flat, chip, win, 900 + seed)
        out, best = s.search(f, times=True)
        red, rbest = r.search(f)
        torch.cuda.synchronize()
        g = {k: getattr(out, k).cpu().numpy() for k in ("mask", "score", "t_team", "t_opp")}
        compare_maps(g, O.search_frame(f, p, bands=True), f"{case} {seed}",
                     pool=BandPool("pairs"))
        sc = g["score"].reshape(len(f.variants), -1)
        assert np.array_equal(red.score.cpu().numpy(), sc.max(0))
        top = np.where(np.isneginf(sc.max(0)), 255, sc.argmax(0))
        assert np.array_equal(red.mask.cpu().numpy(), top)
        assert bool(best["found"]) == bool(np.isfinite(sc).any()) == bool(rbest["found"])
        if best["found"]:
            assert best["score"] == sc.max() == rbest["score"]
    s.close()
    r.close()


def test_window_inside_a_batch():
    """Frames of different sizes in one launch equal each frame alone (the
    staged maps' rows are sized by the frame with the most variants)."""
    from paper_1909_07717_amd import binding as B
    p = Params(n_samples=128).as_f32()
    s = B.Searcher(p)
    frames = []
    for i, (v, h) in enumerate(((1, 0.2), (33, 0.5), (4, 0.1), (16, 0.2))):
        f = random_frame(np.random.default_rng(40 + i), 6 + i % 3, 5 + i)
        f.windows = [full_window(h)]
        f.variants = variants_for(speeds_linear(v, lo=2.0))
        frames.append(f)
    pk, out = s.search_batch(frames, times=True)
    torch.cuda.synchronize()
    for i, f in enumerate(frames):
        one, _ = s.search(f, times=True)
        a, n = int(pk.frames["out_off"][i]), int(pk.frame_elems[i])
        for k in ("mask", "score", "t_team", "t_opp"):
            assert torch.equal(getattr(one, k), getattr(out, k)[a:a + n]), (i, k)
    s.close()
