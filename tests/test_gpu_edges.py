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
    (8, 4, 640, 3, (129, 192, 193, 256, 319, 320)),               # three to five times 64 candidates
    (24, 1, 192, 2, (65, 129, 184)),                              # those, and more domains than waves
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


@pytest.mark.parametrize("c", [1, 63, 64, 65, 127, 129, 300, 512, 577])
def test_stage1_candidate_counts_general(c):
    """The same under a general cost model, where the candidates are ranked by
    benefits that tie in pairs and follow the experts' sizes."""
    from test_gpu_costs import both as both_costs
    R, G, E, N, S = 8, 4, 1280, 3, 64
    rng = np.random.default_rng(c)
    omega = rng.integers(0, 3, size=(R, E)).astype(np.int32)
    omega[:G] = 0
    hot = rng.choice(np.arange(E // 2, E), size=c, replace=False)
    omega[rng.integers(0, G), hot] = 1 + (np.arange(c) // 2).astype(np.int32)
    near = rng.integers(1, 4, size=(R, R))
    cost = np.triu(near, 1) + np.triu(near, 1).T
    sizes = 2 * S * rng.integers(0, 2, size=E)
    sizes[hot[omega[:G, hot].sum(0) < 2]] = 0   # every hot expert's benefit is positive
    s = R - 1
    tk = np.repeat(np.arange(E, dtype=np.int32), omega[s]).reshape(-1, 1)
    both_costs(R, G, E, s, 1, 8, S, 0, N, omega, np.ascontiguousarray(tk), C=cost.astype(np.int32),
               We=sizes.astype(np.int64), what="general stage 1, %d candidates" % c)


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


@pytest.mark.parametrize("n", [(1 << 20) + 1, (1 << 20) + 8192, 3 * 8192 * 512 - 64, 512 * 8192 + 1, 5 * (1 << 20) + 7,
                               (1 << 24) + 9])
@pytest.mark.parametrize("R,G,E,N", [(32, 8, 128, 2), (64, 1, 64, 1), (6, 2, 30, 3)])
def test_large_batches(R, G, E, N, n):
    """Blocks of 1024 threads above 2^20 ids: one tile, the last block of one
    id, and chunks of several tiles; experts whose share ends inside a chunk
    (their ids are ranked) beside those that one destination serves."""
    both(*_zipf_case(R, G, E, N, n, 1, n % 97 + R), what="large batch R=%d E=%d n=%d" % (R, E, n))


def _check_at_offset(args, offset, launch, what):
    """A plan whose ids and destinations start `offset` words past a 16-byte
    boundary, against the oracle; the words around the destinations stay."""
    from test_gpu_parity import DEV, assert_same, ref_plan, topoep
    R, G, E, s, cI, cX, S, W, N, omega, tk = args
    topo = topoep.topology(R, G, E, s, cI, cX, S, W)
    p = topoep.Planner(topo, tk.shape[0], 1, N, device=DEV, launch=launch)
    ids = torch.zeros(tk.size + 4, dtype=torch.int32, device=DEV)
    ids[offset:offset + tk.size] = torch.from_numpy(tk.ravel()).to(DEV)
    dest = torch.full((tk.size + 4,), -9, dtype=torch.int32, device=DEV)
    p.token_dest = dest[offset:offset + tk.size].view(tk.shape)
    p.plan(torch.from_numpy(omega).to(DEV), ids[offset:offset + tk.size].view(tk.shape))
    torch.cuda.synchronize()
    got = dict(replica_slots=p.replica_slots.cpu().numpy(), token_dest=p.token_dest.cpu().numpy(),
               send_counts=p.send_counts.cpu().numpy(), status=int(p.status[0]), move_count=int(p.status[1]))
    assert_same(got, ref_plan(*args), what)
    rest = torch.cat([dest[:offset], dest[offset + tk.size:]])
    assert bool((rest == -9).all()), what


@pytest.mark.parametrize("offset", [0, 1, 3])
def test_large_batch_unaligned(offset):
    """ids and destinations that do not start on a 16-byte boundary."""
    _check_at_offset(_zipf_case(32, 8, 128, 2, (1 << 20) + 77, 1, 5), offset, None, "unaligned by %d" % offset)


@pytest.mark.parametrize("ipt", [1, 2, 4, 8])
@pytest.mark.parametrize("threads,tiles", [(64, 1), (64, 3), (256, 1), (1024, 2)])
def test_ids_per_thread(ipt, threads, tiles):
    """One, two and four ids a load: edges of the wave's piece and of the
    block's chunk, aligned and not; experts whose share ends in a chunk."""
    chunk = ipt * threads * tiles
    for n in (1, 64 * ipt - 1, 64 * ipt + 1, chunk - 1, chunk, 3 * chunk + 5):
        for offset in (0, 2):
            _check_at_offset(_zipf_case(32, 8, 128, 2, n, 1, n % 97 + ipt), offset, (ipt, threads, tiles, 0, 1),
                             "%d ids per thread, %d x %d, n=%d offset %d" % (ipt, threads, tiles, n, offset))


def _domain_case(name, seed=3):
    """Plans that run the per-domain solver and the chunks as one launch by
    default: a large group (Stress-like) and many experts over a few nodes."""
    if name == "stress":
        return _zipf_case(256, 8, 512, 4, 131072, 8, seed)
    if name == "experts":
        return _zipf_case(32, 8, 1024, 2, 20000, 4, seed)
    if name == "refine":
        return _zipf_case(64, 8, 512, 4, 3001, 1, seed, W=1 << 20)
    if name == "empty":
        R, G, E, s, cI, cX, S, W, N, omega, _ = _zipf_case(256, 8, 512, 4, 64, 8, seed)
        omega[s] = 0
        return R, G, E, s, cI, cX, S, W, N, omega, np.zeros((0, 8), np.int32)
    return _zipf_case(256, 8, 512, 4, int(name), 1, seed)


DOMAIN_CASES = ["stress", "experts", "refine", "empty", "1", "1023", "1024", "1025", "32768", "32769", "131073"]


@pytest.mark.parametrize("name", DOMAIN_CASES)
def test_per_domain_one_launch(name):
    """The default launch against the oracle and against the three kernels of
    solver 2, at the edges of the chunks (2 and 8 ids per thread) and just
    beyond the most ids that one launch takes; then with a row self that is
    not the histogram (stage 1 again), a bad id and a refused Omega."""
    args = _domain_case(name)
    got, _ = both(*args, what="per-domain one launch %s" % name)
    three, _ = both(*args, launch=SOLVERS["perdomain"], what="three kernels %s" % name)
    for k in got:
        assert np.array_equal(got[k], three[k]), k
    R, G, E, s, cI, cX, S, W, N, omega, tk = args
    other = omega.copy()
    other[s] = np.roll(omega[s], 7) * 2 + 1
    both(R, G, E, s, cI, cX, S, W, N, other, tk, what="row self differs %s" % name)
    other = omega.copy()
    other[s, 1] = -3
    both(R, G, E, s, cI, cX, S, W, N, other, tk, what="negative in row self %s" % name)
    other = omega.copy()
    other[(s + 1) % R, 1] = -3
    both(R, G, E, s, cI, cX, S, W, N, other, tk, what="negative elsewhere %s" % name)
    if tk.size:
        bad = tk.copy()
        bad[-1, -1] = E
        both(R, G, E, s, cI, cX, S, W, N, omega, bad, what="bad id %s" % name)


@pytest.mark.parametrize("name", ["stress", "refine"])
def test_per_domain_one_launch_reuse(name):
    """One workspace, plan after plan: other inputs, a plan whose every wait
    gives up (SYNC), the stages run alone in between, HIP graph replays."""
    from test_gpu_parity import DEV, assert_same, ref_plan, topoep
    a, b = _domain_case(name, 3), _domain_case(name, 4)
    R, G, E, s, cI, cX, S, W, N, _, tk = a
    b = (R, G, E, s) + b[4:9] + (b[9].copy(), b[10])
    b[9][s] = np.bincount(b[10].ravel(), minlength=E)
    other = b[9].copy()
    other[s] = np.roll(other[s], 5)
    c = b[:9] + (other, b[10])
    p = topoep.Planner(topoep.topology(R, G, E, s, cI, cX, S, W), tk.shape[0], tk.shape[1], N, device=DEV)
    dev = [(torch.from_numpy(x[9]).to(DEV), torch.from_numpy(x[10]).to(DEV)) for x in (a, b, c)]
    refs = [ref_plan(*x) for x in (a, b, c)]

    def check(i, what):
        torch.cuda.synchronize()
        assert_same(dict(replica_slots=p.replica_slots.cpu().numpy(), token_dest=p.token_dest.cpu().numpy(),
                         send_counts=p.send_counts.cpu().numpy(), status=int(p.status[0]),
                         move_count=int(p.status[1])), refs[i], what)

    for rnd in range(3):
        for i in (0, 1, 2, 1):
            p.token_dest.fill_(-9)
            p.plan(*dev[i])
            check(i, "%s round %d input %d" % (name, rnd, i))
        p.plan(*dev[2], launch=(0, 0, 0, 0, 0, -1, 0))
        torch.cuda.synchronize()
        assert int(p.status[0]) & topoep.ST_SYNC and bool((p.token_dest == -1).all())
        p.plan(*dev[0])
        check(0, "%s after SYNC, round %d" % (name, rnd))
        for stage in range(3):
            p.stage(stage, *dev[1])
        check(1, "%s stages, round %d" % (name, rnd))
        p.plan(*dev[2])
        check(2, "%s after stages, round %d" % (name, rnd))
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(stream):
        with torch.cuda.graph(graph, stream=stream):
            p.plan(*dev[0])
    torch.cuda.current_stream().wait_stream(stream)
    for i in range(4):
        p.token_dest.fill_(-9)
        graph.replay()
        check(0, "%s replay %d" % (name, i))
        p.plan(*dev[1 + i % 2])
        check(1 + i % 2, "%s eager after replay %d" % (name, i))


def test_per_domain_three_kernel_workspace():
    """A workspace of the three-kernel plan's size: the same plan, as three
    kernels."""
    from test_gpu_parity import DEV, assert_same, ref_plan, topoep
    args = _domain_case("refine")
    R, G, E, s, cI, cX, S, W, N, omega, tk = args
    topo = topoep.topology(R, G, E, s, cI, cX, S, W)
    p = topoep.Planner(topo, tk.shape[0], tk.shape[1], N, device=DEV)
    three = topoep.workspace_bytes(topo, tk.shape[0], tk.shape[1], N, launch=SOLVERS["perdomain"])
    assert three < p.ws_bytes
    p.ws_bytes = three
    p.workspace_view().zero_()
    p.plan(torch.from_numpy(omega).to(DEV), torch.from_numpy(tk).to(DEV))
    torch.cuda.synchronize()
    assert_same(dict(replica_slots=p.replica_slots.cpu().numpy(), token_dest=p.token_dest.cpu().numpy(),
                     send_counts=p.send_counts.cpu().numpy(), status=int(p.status[0]), move_count=int(p.status[1])),
                ref_plan(*args), "three-kernel workspace")
    p.ws_bytes = three - 256
    with pytest.raises(topoep.TopoepError):
        p.plan(torch.from_numpy(omega).to(DEV), torch.from_numpy(tk).to(DEV))


@pytest.mark.parametrize("name", ["stress", "refine"])
def test_per_domain_mixed_launches(name):
    """One workspace, launches of one shape in every order: the default (one
    kernel), the per-domain solver named (three kernels), the default's
    blocks and solver threads named, and a workspace_bytes without room for
    the one kernel's buffers.  A three-kernel plan leaves that kernel's words
    as they were."""
    from test_gpu_parity import DEV, assert_same, ref_plan, topoep
    a, b = _domain_case(name, 3), _domain_case(name, 4)
    R, G, E, s, cI, cX, S, W, N, _, tk = a
    b = (R, G, E, s) + b[4:9] + (b[9].copy(), b[10])
    b[9][s] = np.bincount(b[10].ravel(), minlength=E)
    topo = topoep.topology(R, G, E, s, cI, cX, S, W)
    T, k = tk.shape
    p = topoep.Planner(topo, T, k, N, device=DEV)
    full, three = p.ws_bytes, topoep.workspace_bytes(topo, T, k, N, launch=SOLVERS["perdomain"])
    dev = [(torch.from_numpy(x[9]).to(DEV), torch.from_numpy(x[10]).to(DEV)) for x in (a, b)]
    refs = [ref_plan(*x) for x in (a, b)]
    ways = [("default", None, full), ("solver 2", SOLVERS["perdomain"], full), ("4 x 256", (4, 256), full),
            ("512 solver threads", (0, 0, 0, 512), full), ("fewer bytes", None, three)]
    assert all(topoep.plan_shape(topo, T, k, N, launch).as_dict() == p.shape.as_dict() for _, launch, _ in ways)
    view = p.workspace_view()
    order = [i for x in range(len(ways)) for y in range(len(ways)) for i in (x, y)]
    for step, i in enumerate(order):
        what, launch, p.ws_bytes = ways[i]
        own = view[three:full].clone()
        p.token_dest.fill_(-9)
        p.plan(*dev[step % 2], launch=launch)
        torch.cuda.synchronize()
        assert_same(dict(replica_slots=p.replica_slots.cpu().numpy(), token_dest=p.token_dest.cpu().numpy(),
                         send_counts=p.send_counts.cpu().numpy(), status=int(p.status[0]),
                         move_count=int(p.status[1])), refs[step % 2], "%s step %d: %s" % (name, step, what))
        assert i == 0 or torch.equal(own, view[three:full]), (step, what)


@pytest.mark.parametrize("name", ["stress", "refine"])
def test_per_domain_one_launch_single_stages(name):
    """After one plan that ran as one launch, each stage alone reproduces the
    outputs, on the same inputs and after a plan of others."""
    from test_gpu_parity import DEV, assert_same, ref_plan, topoep
    a = _domain_case(name, 3)
    R, G, E, s, cI, cX, S, W, N, omega, tk = a
    other = omega.copy()
    other[(s + 1) % R] += 100
    dev = [(torch.from_numpy(x).to(DEV), torch.from_numpy(tk).to(DEV)) for x in (omega, other)]
    refs = [ref_plan(*a), ref_plan(*(a[:9] + (other, tk)))]
    p = topoep.Planner(topoep.topology(R, G, E, s, cI, cX, S, W), tk.shape[0], tk.shape[1], N, device=DEV)
    assert p.shape.kernels == 3
    for step, stage in enumerate((2, 1, 2, 0, 1, 2)):
        i = step % 2
        p.plan(*dev[i])
        for out in (p.token_dest, p.replica_slots, p.send_counts, p.status):
            if stage == 2 or (stage == 1 and out is not p.token_dest):
                out.fill_(-9)
        p.stage(stage, *dev[i])
        torch.cuda.synchronize()
        assert_same(dict(replica_slots=p.replica_slots.cpu().numpy(), token_dest=p.token_dest.cpu().numpy(),
                         send_counts=p.send_counts.cpu().numpy(), status=int(p.status[0]),
                         move_count=int(p.status[1])), refs[i], "%s stage %d alone, step %d" % (name, stage, step))


def test_per_domain_launch_count():
    """The floor of a plan is one empty kernel where the plan is one launch:
    its graph takes the time of one, not of three, and plan_launches says so."""
    from test_gpu_parity import DEV, topoep
    R, G, E, s, cI, cX, S, W, N, omega, tk = _domain_case("stress")
    topo = topoep.topology(R, G, E, s, cI, cX, S, W)
    dev = torch.from_numpy(omega).to(DEV), torch.from_numpy(tk).to(DEV)
    count = {}
    for launch in (None, SOLVERS["perdomain"]):
        p = topoep.Planner(topo, tk.shape[0], tk.shape[1], N, device=DEV, launch=launch)
        assert p.shape.kernels == 3
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=stream):
                for _ in range(200):
                    p.stage(topoep.STAGE_FLOOR, *dev)
            for _ in range(3):
                graph.replay()
            a.record()
            graph.replay()
            b.record()
        torch.cuda.synchronize()
        count[launch] = topoep.plan_launches(topo, tk.shape[0], tk.shape[1], N, launch), a.elapsed_time(b)
    (one, t1), (three, t3) = count[None], count[SOLVERS["perdomain"]]
    assert one == 1 and three == 3
    assert t1 < 0.6 * t3   # (a third, were the launches alike)


def test_noalloc_per_domain_one_launch():
    """The library's array, dirty from a plan of another shape, before each
    per-domain plan in one launch."""
    from test_gpu_parity import DEV, assert_same, ref_plan, topoep
    for name in ("refine", "large", "stress", "1025", "large", "refine"):
        args = _zipf_case(32, 8, 128, 2, 200000, 4, 9) if name == "large" else _domain_case(name)
        R, G, E, s, cI, cX, S, W, N, omega, tk = args
        out = [torch.full(sh, -9, dtype=torch.int32, device=DEV) for sh in ((R, N), tk.shape, (R,), (2,))]
        topoep.plan_noalloc(topoep.topology(R, G, E, s, cI, cX, S, W), torch.from_numpy(omega).to(DEV),
                            torch.from_numpy(tk).to(DEV), N, *out)
        torch.cuda.synchronize()
        slots, dest, send, status = [x.cpu().numpy() for x in out]
        assert_same(dict(replica_slots=slots, token_dest=dest, send_counts=send, status=int(status[0]),
                         move_count=int(status[1])), ref_plan(*args), "no-alloc %s" % name)


@pytest.mark.parametrize("name", ["stress", "experts", "refine", "empty", "1025"])
def test_per_domain_one_launch_dispatch(name):
    """Receive counts, send offsets and slots of the one-launch plan."""
    from test_gpu_dispatch import check
    check(_domain_case(name), "per-domain one launch %s" % name)


@pytest.mark.parametrize("solver", sorted(SOLVERS))
@pytest.mark.parametrize("R,G,P,N,cI", [
    (8, 8, 7, 1, 1), (8, 8, 8, 1, 1),       # 8 and 9 instances per rank: one and two pairs a lane
    (16, 8, 13, 3, 1), (16, 8, 13, 4, 1),   # 16 and 17: pairs, one lane per instance
    (4, 2, 62, 2, 1), (4, 4, 63, 2, 0),     # 64 and 65: one and two rounds of instances
    (10, 5, 3, 3, 2), (72, 8, 2, 3, 1),     # ranks that fill no group of lanes; more than 64 sources
    (24, 12, 10, 4, 1), (24, 12, 10, 5, 1),  # 14 and 15 instances on more than 8 ranks: lanes, LDS form
    (24, 12, 2, 2, 1), (32, 16, 3, 2, 1),   # 4 and 5: one and two pairs a lane
    (18, 9, 5, 3, 0), (80, 16, 6, 3, 2),    # 8 and 9: pairs, one lane per instance
])
def test_refinement_forms(R, G, P, N, cI, solver):
    """Moves at the edges of the refinement's forms, with hot experts on one
    rank of each node, equal loads in half of the cases."""
    from test_gpu_parity import topoep
    E = R * P
    for seed in range(4):
        rng = np.random.default_rng(1000 * R + 10 * P + seed)
        omega = rng.integers(0, 30, size=(R, E)).astype(np.int32)
        hot = rng.integers(0, R // G, size=3) * G * P + rng.integers(0, P, size=3)
        omega[:, hot] += rng.integers(100, 900, size=(R, 3)).astype(np.int32)
        if seed % 2:
            omega = omega // 16 * 16
        s = int(rng.integers(R))
        tk = np.repeat(np.arange(E, dtype=np.int32), omega[s]).reshape(-1, 1)
        W = int(omega.sum()) * 2   # few stage-1 replicas: slots stay free
        try:
            got, _ = both(R, G, E, s, cI, 8, 64, W, N, omega, np.ascontiguousarray(tk), launch=SOLVERS[solver],
                          what="forms R=%d G=%d P=%d N=%d seed %d %s" % (R, G, P, N, seed, solver))
        except topoep.TopoepError as ex:
            if ex.rc != topoep.ELIMIT:
                raise
            pytest.skip("the %s solver's state does not fit one workgroup's LDS here" % solver)
        assert got["move_count"] > 0


LAYOUT_SIZES = [1, 1024, 1025, 15 * 1024, 15 * 1024 + 1, 16 * 1024, 16 * 1024 + 1, 32 * 1024, 65536, 65537, 262144,
                262145, 1 << 20, (1 << 20) + 1, 1 << 21, (1 << 21) + 1, 3 << 20, 4 << 20, (4 << 20) + 3]


def _layout(planner, R, n, seed, skew):
    import oracle
    from test_gpu_dispatch import layout_case
    dest, send = layout_case(R, n, np.random.default_rng(seed), skew=skew)
    d, s = torch.from_numpy(dest).cuda(), torch.from_numpy(send).cuda()
    offs, slot = planner.layout(d, s)
    torch.cuda.synchronize()
    ref_offs, ref_slot = oracle.layout_ref(R, dest, send)
    assert int(planner.status[0]) == 0
    assert np.array_equal(offs.cpu().numpy(), ref_offs) and np.array_equal(slot.cpu().numpy(), ref_slot), (R, n)
    return dest.shape


@pytest.mark.parametrize("R", [1, 3, 64, 128, 160, 1024])
def test_layout_edges(R):
    """One, two, four and eight ids per thread, groups of 16 workgroups, one
    less and one more, 256 and 512 workgroups; twice on each workspace, which
    is zero again after every call."""
    from test_gpu_parity import DEV, topoep
    for n in LAYOUT_SIZES:
        p = None
        for seed, skew in ((n, 0.0), (n + 1, 1.5)):
            from test_gpu_dispatch import layout_case
            T, k = layout_case(R, n, np.random.default_rng(seed), skew=skew)[0].shape
            if p is None:
                p = topoep.LayoutPlanner(topoep.topology(R, 1, R, 0, 1, 1, 1, 0), T, k, device=DEV)
            _layout(p, R, n, seed, skew)
        assert not bool(p._ws.any()), (R, n)


def test_layout_one_workspace_many_sizes():
    """A workspace of the largest size serves every smaller one in turn, and
    one of a grid of four ids per thread is still enough for that grid."""
    from test_gpu_parity import DEV, topoep
    R = 48
    topo = topoep.topology(R, 1, R, 0, 1, 1, 1, 0)
    from test_gpu_dispatch import layout_case
    shape = lambda n: layout_case(R, n, np.random.default_rng(1), skew=0.0)[0].shape  # noqa: E731
    big = topoep.LayoutPlanner(topo, *shape(4 * (1 << 20) + 3), device=DEV)
    for i, n in enumerate(LAYOUT_SIZES + LAYOUT_SIZES[::-1]):
        p = topoep.LayoutPlanner(topo, *shape(n), device=DEV)
        assert p.ws_bytes <= big.ws_bytes
        p.ws_ptr, p.ws_bytes = big.ws_ptr, big.ws_bytes
        _layout(p, R, n, i, 1.0)
    n = 65536
    p = topoep.LayoutPlanner(topo, *shape(n), device=DEV)
    p.ws_bytes = 256 + 256 + 2 * (n // 4096 * R * 4)
    _layout(p, R, n, 5, 1.0)
