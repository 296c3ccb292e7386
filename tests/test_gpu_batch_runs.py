"""Tiles of several frames are split over the workgroups by their number (all a
workgroup's own, one and the rest from the counter, a halved grid, three
quarters and groups): the outputs are, byte for byte, those of each frame alone,
for host requests and resident batches, at the default launch, with a fixed
number of workgroups per CU and with one workgroup per tile."""
import numpy as np
import pytest

from paper_1909_07717_amd.framegen import (Params, full_window, random_frame, speeds_linear,
                                           variants_for)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _frames(n):
    out = []
    for i in range(n):
        f = random_frame(np.random.default_rng(8100 + i), 4 + i % 5, 3 + i % 6)
        f.windows = [full_window(0.2 if i % 4 else 0.5)]
        f.variants = variants_for(speeds_linear(2 + i % 3, lo=2.0), True, False)
        out.append(f)
    return out


@pytest.mark.parametrize("K", [64, 128, 256])
@pytest.mark.parametrize("n", [2, 4, 7, 11, 15, 40])
def test_outputs_do_not_depend_on_the_split(K, n):
    from paper_1909_07717_amd import binding as B
    print(f"[runs] K={K} n={n}", flush=True)
    s = B.Searcher(Params(n_samples=K).as_f32())
    frames = _frames(n)
    alone = [s.search(f, times=True)[0] for f in frames]
    for shape in ((0, 0, 0), (8, 4, 2), (16, 4, -2), (8, 2, -1)):
        s.set_launch(*shape)
        pk, out = s.search_batch(frames, times=True)
        bt = s.batch(frames)
        res = s.outputs_for(bt.pk, True, True, True)
        bt.run(res)
        torch.cuda.synchronize()
        for i in range(n):
            a, m = int(pk.frame_elems[:i].sum()), int(pk.frame_elems[i])
            for k in ("mask", "score", "t_team", "t_opp"):
                want = getattr(alone[i], k)
                assert torch.equal(want, getattr(out, k)[a:a + m]), (shape, i, k)
                assert torch.equal(want, getattr(res, k)[a:a + m]), (shape, i, k)
    s.close()
