"""GPU parity at the sizes where a kernel's split of the work changes: edges
of tiles, blocks and parts, remainders, the smallest and largest of a range.
Every case is compared with the CPU oracle, bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from test_gpu_parity import SOLVERS, both  # noqa: E402

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


@pytest.mark.parametrize("solver", sorted(SOLVERS))
@pytest.mark.parametrize("R,G,E,N,counts", [
    (8, 4, 256, 3, (0, 1, 15, 16, 17, 63, 64, 65, 127, 128)),   # half the waves per domain
    (32, 1, 64, 5, (1, 16, 17, 62)),                              # more domains than waves
    (6, 2, 192, 70, (33, 128)),                                   # more slots than candidates
])
def test_stage1_candidate_counts(R, G, E, N, counts, solver):
    """Exactly c stage-1 candidates in domain 0 (W = 0: an expert is one when
    the domain has any load on it), with loads that tie in pairs: the ranks
    are counted for 64 candidates against 16 at a time."""
    P = E // R
    for c in counts:
        rng = np.random.default_rng(c)
        omega = rng.integers(0, 3, size=(R, E)).astype(np.int32)
        omega[:G] = 0
        outside = np.arange(G * P, E)
        hot = rng.choice(outside, size=c, replace=False)
        omega[rng.integers(0, G), hot] = 1 + (np.arange(c) // 2).astype(np.int32)
        s = R - 1
        tk = np.repeat(np.arange(E, dtype=np.int32), omega[s]).reshape(-1, 1)
        both(R, G, E, s, 1, 8, 64, 0, N, omega, np.ascontiguousarray(tk), launch=SOLVERS[solver],
             what="stage 1, %d candidates R=%d G=%d E=%d N=%d %s" % (c, R, G, E, N, solver))
