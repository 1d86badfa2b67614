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


def _zipf_case(R, G, E, N, n, k, seed, S=4096, W=9 << 20):
    """One plan of n = T k local ids (Zipf over E) and rows of Omega drawn
    around their counts, so that replicated experts split their shares."""
    rng = np.random.default_rng(seed)
    p = np.arange(1, E + 1, dtype=np.float64) ** -1.1
    p = p[rng.permutation(E)] / p.sum()
    tk = rng.choice(E, size=(n // k, k), p=p).astype(np.int32)
    omega = rng.poisson(np.maximum(n * p, 0.01), size=(R, E)).astype(np.int32)
    s = int(rng.integers(R))
    omega[s] = np.bincount(tk.ravel(), minlength=E)
    return R, G, E, s, 1, 8, S, W, N, omega, tk


@pytest.mark.parametrize("n", [(1 << 20) + 1, (1 << 20) + 8192, 3 * 8192 * 512 - 64, 512 * 8192 + 1, 5 * (1 << 20) + 7])
@pytest.mark.parametrize("R,G,E,N", [(32, 8, 128, 2), (64, 1, 64, 1), (6, 2, 30, 3)])
def test_large_batches(R, G, E, N, n):
    """Blocks of 1024 threads above 2^20 ids: one tile, the last block of one
    id, and chunks of several tiles; experts whose share ends inside a chunk
    (their ids are ranked) beside those that one destination serves."""
    both(*_zipf_case(R, G, E, N, n, 1, n % 97 + R), what="large batch R=%d E=%d n=%d" % (R, E, n))


@pytest.mark.parametrize("offset", [0, 1, 3])
def test_large_batch_unaligned(offset):
    """ids and destinations that do not start on a 16-byte boundary."""
    from test_gpu_parity import DEV, assert_same, ref_plan, topoep
    R, G, E, s, cI, cX, S, W, N, omega, tk = args = _zipf_case(32, 8, 128, 2, (1 << 20) + 77, 1, 5)
    topo = topoep.topology(R, G, E, s, cI, cX, S, W)
    p = topoep.Planner(topo, tk.shape[0], 1, N, device=DEV)
    ids = torch.zeros(tk.size + 4, dtype=torch.int32, device=DEV)
    ids[offset:offset + tk.size] = torch.from_numpy(tk.ravel()).to(DEV)
    dest = torch.full((tk.size + 4,), -9, dtype=torch.int32, device=DEV)
    p.token_dest = dest[offset:offset + tk.size].view(tk.shape)
    p.plan(torch.from_numpy(omega).to(DEV), ids[offset:offset + tk.size].view(tk.shape))
    torch.cuda.synchronize()
    got = dict(replica_slots=p.replica_slots.cpu().numpy(), token_dest=p.token_dest.cpu().numpy(),
               send_counts=p.send_counts.cpu().numpy(), status=int(p.status[0]), move_count=int(p.status[1]))
    assert_same(got, ref_plan(*args), "unaligned by %d" % offset)
    rest = torch.cat([dest[:offset], dest[offset + tk.size:]])
    assert bool((rest == -9).all())
