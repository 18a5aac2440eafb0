"""The step loops that keep a class's gains in registers against the loops that keep them in memory (RCD_RESIDENT = 0).  The
oracle referees both in test_gpu_incremental.py and test_gpu_graph_cut.py.  Here: same assignment, order and objectives to the bit, at the edges of every
variant's sample and block range, with zero quotas and samples left over, with groups of identical samples (exact
ties), with the state stored and loaded again in mid-run, and for classes of unequal size in one launch."""
import ctypes

import numpy as np
import pytest

import synth_inputs as si

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def rcd():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU: there is no CPU path")
    import paper_2211_00839_amd as m

    m.load_library()
    return m


def both(monkeypatch, call):
    got = []
    for on in ("1", "0"):
        monkeypatch.setenv("RCD_RESIDENT", on)
        assign, order, obj = call()
        got.append((assign.cpu().numpy(), order.cpu().numpy(), obj))
    for x, y in zip(*got):
        assert np.array_equal(x, y)
    return got[0]


def quotas(rng, n, K, full):
    w = rng.integers(0, 5, K) + (np.arange(K) == rng.integers(0, K))
    cap = (n * w // w.sum()).astype(np.int64)
    if full:
        cap[int(np.argmax(cap))] += n - int(cap.sum())
    return cap


# (n, K): both sides of every variant's last sample, and its most blocks
EDGES = [(1, 1), (2, 3), (255, 2), (256, 16), (257, 5), (512, 16), (513, 3), (1024, 16), (1025, 8), (2048, 16), (2049, 4),
         (3072, 8), (3072, 16), (3073, 12), (4096, 9), (4096, 12), (4097, 4), (5120, 8), (5121, 8), (6144, 5), (6144, 8),
         (6145, 3), (8192, 4), (8193, 2), (16383, 2)]


@pytest.mark.parametrize("n,K", EDGES)
def test_graph_cut_class(rcd, monkeypatch, n, K):
    print(f"resident graph cut n={n} K={K}", flush=True)
    rng = np.random.default_rng(n + K)
    X = torch.from_numpy(si.make_class(seed=n, n=n, d=64)).cuda()
    if n % 2 == 0:
        X[n // 2:] = X[: n - n // 2]                     # every sample twice: exact ties
    S = rcd.similarity(X, 64.0)
    cap = quotas(rng, n, K, full=K % 2 == 0)
    # a few steps per launch as well: the state goes through memory in between
    for steps in ("", "7") if n < 1000 else ("", "1000"):
        monkeypatch.setenv("RCD_GC_STEPS", steps)
        assign, order, _ = both(monkeypatch, lambda: rcd.partition_class_graph_cut(S, cap))
        assert np.bincount(assign[assign >= 0], minlength=K).tolist() == cap.tolist()
        assert sorted(order[order >= 0].tolist()) == list(range(int(cap.sum())))


# ((3072, 16), (5121, 8) and (6144, 5) lie just outside the variants: there both runs take the loop in memory)
INC_EDGES = [(1, 1), (2, 3), (255, 2), (256, 16), (257, 5), (512, 16), (513, 3), (1024, 16), (1025, 8), (2048, 16), (2049, 4),
             (3072, 8), (3072, 16), (3073, 3), (5120, 4), (5120, 8), (5121, 8), (6144, 5), (6145, 3), (8192, 4)]


@pytest.mark.parametrize("n,K", INC_EDGES)
def test_incremental_class(rcd, monkeypatch, n, K):
    print(f"resident incremental n={n} K={K}", flush=True)
    rng = np.random.default_rng(n + K)
    X = torch.from_numpy(si.make_class(seed=n, n=n, d=64)).cuda()
    if n % 2 == 0:
        X[n // 2:] = X[: n - n // 2]                     # every sample twice: exact ties
    S = rcd.similarity(X, 64.0)
    cap = quotas(rng, n, K, full=K % 2 == 0)
    # as it is; every list of more than four rows handed out, to one helper; the state through memory in mid-run
    for env in ({}, {"RCD_INC_SMALL_KB": "1", "RCD_HELPERS": "1"}, {"RCD_INC_STEPS": "7" if n < 1000 else "1000"}):
        with monkeypatch.context() as m:
            for k, v in env.items():
                m.setenv(k, v)
            assign, order, _ = both(m, lambda: rcd.partition_class(S=S, cap=cap, mode=rcd.MODE_INCREMENTAL))
        assert np.bincount(assign[assign >= 0], minlength=K).tolist() == cap.tolist()
        assert sorted(order[order >= 0].tolist()) == list(range(int(cap.sum())))


# (the later ones: classes far smaller than the variant that the largest one takes, so that whole pieces of a wave lie
# outside their rows)
@pytest.mark.parametrize("sizes,K", [((1, 700, 256, 90), 4), ((2500, 300, 40), 8), ((4000, 5000), 3), ((300,) * 40, 16),
                                     ((5000, 40), 4), ((5000, 40), 1), ((8000, 60, 500), 3), ((12000, 50, 1), 2)])
def test_data_set_of_unequal_classes(rcd, monkeypatch, sizes, K):
    print(f"resident classes {sizes[:4]} K={K}", flush=True)
    rng = np.random.default_rng(K)
    X = np.concatenate([si.make_class(seed=i, n=n, d=32) for i, n in enumerate(sizes)])
    labels = np.concatenate([np.full(n, i, np.int32) for i, n in enumerate(sizes)])
    at = rng.permutation(len(X))
    Xd, yd = torch.from_numpy(X[at]).cuda(), torch.from_numpy(labels[at]).cuda()
    r = rng.integers(1, 5, K).astype(np.int32)
    _, full = rcd.dataset_workspace_bytes(len(X), len(sizes), max(sizes), K, rcd.MODE_STORED)
    ws = torch.empty(full, dtype=torch.uint8, device="cuda")
    both(monkeypatch, lambda: rcd.partition_dataset(Xd, yd, len(sizes), r, 32.0, workspace=ws, graph_cut=True))
    both(monkeypatch, lambda: rcd.partition_dataset(Xd, yd, len(sizes), r, 32.0, rcd.MODE_INCREMENTAL, ws))


@pytest.mark.parametrize("sizes,K", [((2000,) + (90,) * 60, 4), ((30,) * 50 + (1500, 1500, 1400), 2), ((300,) * 60, 3)])
def test_helpers_dealt_by_size(rcd, monkeypatch, sizes, K):
    # many small classes beside a few large ones: the helpers go to the large ones, the rest get one or none; lists of more
    # than four rows are handed out
    print(f"helpers dealt to {len(sizes)} classes", flush=True)
    rng = np.random.default_rng(len(sizes))
    X = torch.from_numpy(np.concatenate([si.make_class(seed=i, n=n, d=16) for i, n in enumerate(sizes)])).cuda()
    y = np.repeat(np.arange(len(sizes)), sizes).astype(np.int32)
    at = rng.permutation(len(y))
    X, y = X[torch.from_numpy(at).cuda()].contiguous(), torch.from_numpy(y[at]).cuda()
    r = rng.integers(1, 5, K).astype(np.int32)
    _, full = rcd.dataset_workspace_bytes(len(at), len(sizes), max(sizes), K, rcd.MODE_STORED)
    ws = torch.empty(full, dtype=torch.uint8, device="cuda")
    for kb in ("", "1"):
        monkeypatch.setenv("RCD_INC_SMALL_KB", kb)
        both(monkeypatch, lambda: rcd.partition_dataset(X, y, len(sizes), r, 16.0, rcd.MODE_INCREMENTAL, ws))


# more classes than half the compute units: with helpers because several workgroups fit one, with a few or without any
# because the classes are small, in two lanes with the gains in memory; and more classes than compute units
@pytest.mark.parametrize("L,n,K", [(130, 450, 16), (140, 40, 4), (200, 200, 16), (256, 30, 2), (150, 700, 16), (280, 40, 4)])
def test_many_classes(rcd, monkeypatch, L, n, K):
    print(f"resident, {L} classes of {n} K={K}", flush=True)
    rng = np.random.default_rng(L)
    X = torch.from_numpy(rng.standard_normal((n * L, 16)).astype(np.float32)).cuda()
    y = torch.from_numpy(rng.permutation(np.repeat(np.arange(L), n)).astype(np.int32)).cuda()
    _, full = rcd.dataset_workspace_bytes(n * L, L, n, K, rcd.MODE_STORED)
    ws = torch.empty(full, dtype=torch.uint8, device="cuda")
    r = rng.integers(1, 4, K).astype(np.int32)
    both(monkeypatch, lambda: rcd.partition_dataset(X, y, L, r, 16.0, rcd.MODE_INCREMENTAL, ws))


@pytest.mark.parametrize("route", ["incremental", "graph cut"])
@pytest.mark.parametrize("n,bad", [(300, float("nan")), (3000, 1.5)])
def test_no_step_is_taken_on_a_refused_matrix(rcd, route, n, bad):
    print(f"refused matrix n={n} {route}", flush=True)
    S = rcd.similarity(torch.from_numpy(si.make_class(seed=n, n=n, d=32)).cuda(), 32.0)
    S[n - 1, n // 2] = bad
    lib, K = rcd.load_library(), 3
    cap, obj = rcd.quota(n, [1, 2, 1]), np.zeros(K)
    assign = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    order = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    size = rcd.class_workspace_bytes(n, K, rcd.MODE_INCREMENTAL)
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    capp, objp = cap.ctypes.data_as(ctypes.c_void_p), obj.ctypes.data_as(ctypes.c_void_p)
    if route == "incremental":
        status = lib.rcd_partition_class_mode(S.data_ptr(), n, None, 0, 0, 0, 1.0, n, K, capp, rcd.MODE_INCREMENTAL,
                                              assign.data_ptr(), order.data_ptr(), objp, ws.data_ptr(), size, None)
    else:
        status = lib.rcd_partition_class_graph_cut(S.data_ptr(), n, n, K, capp, assign.data_ptr(), order.data_ptr(), objp,
                                                   ws.data_ptr(), size, None)
    assert status == 7
    assert bool((assign < 0).all()) and bool((order < 0).all())


def test_launches_are_counted_as_made(rcd, monkeypatch):
    # three launches to start with, a batch of step launches that the host waits for and one queued behind it, the
    # objective; the loop in memory has an update launch beside every step launch
    S = rcd.similarity(torch.from_numpy(si.make_class(seed=5, n=200, d=32)).cuda(), 32.0)
    monkeypatch.setenv("RCD_ROUNDS_PER_BATCH", "5")
    for on, per_round in (("1", 1), ("0", 2)):
        monkeypatch.setenv("RCD_RESIDENT", on)
        rcd.partition_class(S=S, cap=rcd.quota(200, [1, 1]), mode=rcd.MODE_INCREMENTAL)
        launches = rcd.last_stats()["launches"] - 4
        assert launches % (5 * per_round) == 0 and launches >= 10 * per_round
        if on == "1":
            assert launches == 10


def test_a_wait_for_a_helper_that_runs_out_is_reported(rcd, monkeypatch):
    # the bound set to zero from the host: helpers leave at once, and the first wave of the class that finds another one's
    # part of a list unfinished raises the flag; every kernel exits, and the next call with the default bound works
    S = rcd.similarity(torch.from_numpy(si.make_class(seed=6, n=2000, d=32)).cuda(), 32.0)
    cap = rcd.quota(2000, [1, 1])
    with monkeypatch.context() as m:
        m.setenv("RCD_MW_SPIN_MS", "0")
        with pytest.raises(rcd.RcdError) as e:
            rcd.partition_class(S=S, cap=cap, mode=rcd.MODE_INCREMENTAL)
        assert e.value.status == 6 and "helper" in str(e.value)
    torch.cuda.synchronize()
    both(monkeypatch, lambda: rcd.partition_class(S=S, cap=cap, mode=rcd.MODE_INCREMENTAL))


@pytest.mark.parametrize("route", ["incremental", "graph cut"])
def test_the_timing_knows_the_first_step_launch(rcd, route):
    # one launch makes every step: its time has to be in the sum (step_ticks: 10 ns units inside the one class's loop)
    S = rcd.similarity(torch.from_numpy(si.make_class(seed=7, n=2000, d=32)).cuda(), 32.0)
    cap = rcd.quota(2000, [1, 2])
    rcd.profile(True)
    if route == "incremental":
        rcd.partition_class(S=S, cap=cap, mode=rcd.MODE_INCREMENTAL)
    else:
        rcd.partition_class_graph_cut(S, cap)
    ms, ticks = rcd.profile_read()["steps_ms"], rcd.last_stats()["step_ticks"]
    rcd.profile(False)
    assert ms >= 0.9e-5 * ticks > 0
