"""A request of one frame travels with the launch (one window) or through the
staged tables (several windows): both give, bit for bit, what a batch of the
same frame gives, at the smallest and largest counts and when requests of
different sizes follow each other."""
import numpy as np
import pytest

from paper_1909_07717_amd.framegen import Params, random_frame, speeds_linear, variants_for

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

H = float(np.float32(0.1))
CASES = [
    # n_team, n_opp, flat speeds, chip speeds, windows
    (1, 0, 1, 0, [(H, 0, 0, 1, 1)]),
    (16, 16, 32, 32, [(H, 3, 2, 31, 17)]),
    (11, 11, 3, 2, [(H, 0, 0, 40, 30), (H, 60, 40, 1, 5)]),
    (2, 5, 0, 4, [(H, 70, 50, 9, 1)]),
]


@pytest.mark.parametrize("K", [64, 256])
def test_one_frame_equals_its_batch(K):
    from paper_1909_07717_amd import binding as B
    p = Params(n_samples=K).as_f32()
    s = B.Searcher(p)
    for seed, (nt, no, flat, chip, wins) in enumerate(CASES + CASES[::-1]):
        print(f"[one frame] K={K} {nt}-{no}-{flat}-{chip} {wins}", flush=True)
        f = random_frame(np.random.default_rng(70 + seed), nt, no)
        f.windows = wins
        f.variants = (variants_for(speeds_linear(flat, lo=1.5), True, False) if flat else []) + \
                     (variants_for(speeds_linear(chip, lo=1.5), False, True) if chip else [])
        one, best = s.search(f, times=True)
        pk = B.pack([f], p)
        out = s.outputs_for(pk, times=True)
        bt = B.Batch(s, pk)
        bt.run(out)
        torch.cuda.synchronize()
        for k in ("mask", "score", "t_team", "t_opp"):
            assert torch.equal(getattr(one, k).view(torch.uint8), getattr(out, k).view(torch.uint8)), k
        ref = out.best_host()[0]
        assert np.array(best).tobytes() == ref.tobytes()
        bt.close()
    s.close()
