"""Running points take more threads per zone the fewer zones there are: scores
and records are, byte for byte, those of the same frame in batches of one zone
per CU and less, of two, and of many, for zones of one point, of less points than
threads and of many, and for a zone without a usable point."""
import numpy as np
import pytest

from paper_1909_07717_amd.framegen import Params, random_frame

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

H = float(np.float32(0.1))
ZONES = [(H, 60, 0, 61, 45), (H, 0, 0, 1, 1), (H, 100, 30, 17, 31), (H, 111, 35, 8, 20)]


@pytest.mark.parametrize("n_opp", [0, 2, 9])
def test_records_do_not_depend_on_the_batch(n_opp):
    from paper_1909_07717_amd import binding as B
    s = B.Searcher(Params(n_samples=64).as_f32())
    f = random_frame(np.random.default_rng(50 + n_opp), 5, n_opp)
    f.windows = list(ZONES)
    want = None
    for n in (1, 50, 64, 65, 110, 128, 129, 300):
        print(f"[run blocks] n_opp={n_opp} n={n}", flush=True)
        best, sc = s.running_points([f] * n)
        torch.cuda.synchronize()
        rec = B.run_best_host(best)[:4 * n].tobytes()
        one, pts = len(rec) // n, sc.numel() // n
        got = (rec[:one], sc[:pts].cpu().numpy().tobytes())
        want = want or got
        assert got == want
        assert rec == want[0] * n and sc.cpu().numpy().tobytes() == want[1] * n
    assert B.run_best_host(best)[3]["found"] == 0
    s.close()
