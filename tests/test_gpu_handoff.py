"""GPU parity of the hand-off to Algorithm 2: rcd_worker_shards against the oracle bit for bit (ragged
sizes around the 1024-sample chunks, leftovers, empty workers, full-size assignment of a real run),
rcd_batch_sizes against the oracle (host only, checked here too so that both sit together)."""
import ctypes

import numpy as np
import pytest

import oracle
import synth_inputs as si

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def rcd():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU: there is no CPU path")
    import paper_2211_00839_amd as m

    m.load_library()
    return m


def dev(a):
    if a.dtype == np.uint16:
        return torch.from_numpy(a.view(np.int16)).cuda().view(torch.bfloat16)
    return torch.from_numpy(a).cuda()


@pytest.mark.gpu
@pytest.mark.parametrize("N,K", [(1, 1), (63, 2), (1023, 3), (1024, 4), (1025, 5), (5000, 16), (70001, 8)])
def test_worker_shards_bit_exact(rcd, N, K):
    print(f"worker shards N={N} K={K}", flush=True)
    rng = np.random.default_rng(N + K)
    for low in (0, -1):                      # everyone assigned / some left over
        a = rng.integers(low, K, size=N).astype(np.int32)
        if K > 2:
            a[a == 1] = 0                    # a worker with an empty list
        index, offset = rcd.worker_shards(torch.from_numpy(a).cuda(), K)
        ref_index, ref_offset = oracle.worker_shards(a, K)
        assert offset.tolist() == ref_offset.tolist()
        assert np.array_equal(index.cpu().numpy()[: offset[K]], ref_index)


@pytest.mark.gpu
def test_worker_shards_of_a_real_partition_and_errors(rcd):
    ds = si.make_dataset(si.WORKLOADS["hetero8"], L=4, n_c=600, d=64)
    N = ds.X.shape[0]
    K = len(ds.r)
    _, full = rcd.dataset_workspace_bytes(N, ds.L, 600, K, rcd.MODE_STORED)
    ws = torch.empty(full, dtype=torch.uint8, device="cuda")
    assign, _, _ = rcd.partition_dataset(dev(ds.X), dev(ds.labels), ds.L, ds.r, ds.sigma2, rcd.MODE_STORED, ws)
    index, offset = rcd.worker_shards(assign, K)
    a = assign.cpu().numpy()
    ref_index, ref_offset = oracle.worker_shards(a, K)
    assert offset.tolist() == ref_offset.tolist() and np.array_equal(index.cpu().numpy(), ref_index)
    # every worker's shard holds its quota of every class (the point of the class-wise partition)
    idx = index.cpu().numpy()
    for k in range(K):
        shard = idx[offset[k]:offset[k + 1]]
        per_class = np.bincount(ds.labels[shard], minlength=ds.L)
        assert per_class.tolist() == [int(oracle.quota(600, ds.r)[k])] * ds.L
    lib = rcd.load_library()
    bad = assign.clone()
    bad[17] = K
    off = np.zeros(K + 1, dtype=np.int64)
    out = torch.empty(N, dtype=torch.int32, device="cuda")
    wsz = lib.rcd_worker_shards_workspace_bytes(N, K)
    w2 = torch.empty(wsz, dtype=torch.uint8, device="cuda")
    offp = off.ctypes.data_as(ctypes.c_void_p)
    assert lib.rcd_worker_shards(bad.data_ptr(), N, K, out.data_ptr(), offp, w2.data_ptr(), wsz, None) == 2
    bad[17] = -2
    assert lib.rcd_worker_shards(bad.data_ptr(), N, K, out.data_ptr(), offp, w2.data_ptr(), wsz, None) == 2
    assert lib.rcd_worker_shards(assign.data_ptr(), N, K, out.data_ptr(), offp, w2.data_ptr(), wsz - 256, None) == 5
    assert lib.rcd_worker_shards(None, N, K, out.data_ptr(), offp, w2.data_ptr(), wsz, None) == 1
    assert lib.rcd_worker_shards(assign.data_ptr(), N, 17, out.data_ptr(), offp, w2.data_ptr(), wsz, None) == 4
    assert lib.rcd_worker_shards(None, 0, K, None, offp, None, 0, None) == 0 and off.tolist() == [0] * (K + 1)


@pytest.mark.gpu
@pytest.mark.parametrize("N,at,value", [(1, 0, 3), (5000, 4999, 3), (5000, 0, -2), (300000, 1025, 77)])
def test_a_refused_assignment_leaves_the_lists_alone(rcd, N, at, value):
    print(f"shards, refused N={N}", flush=True)
    K = 3
    a = np.random.default_rng(N).integers(-1, K, size=N).astype(np.int32)
    a[at] = value
    a = torch.from_numpy(a).cuda()
    lib = rcd.load_library()
    index = torch.full((N,), -7, dtype=torch.int32, device="cuda")
    offset = np.full(K + 1, -7, dtype=np.int64)
    size = lib.rcd_worker_shards_workspace_bytes(N, K)
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    offp = offset.ctypes.data_as(ctypes.c_void_p)
    assert lib.rcd_worker_shards(a.data_ptr(), N, K, index.data_ptr(), offp, ws.data_ptr(), size, None) == 2
    assert bool((index == -7).all()) and offset.tolist() == [0] * (K + 1)


def test_batch_sizes_match_the_oracle():
    import paper_2211_00839_amd as m

    rng = np.random.default_rng(2)
    assert m.batch_sizes(64, [1, 1, 2, 4]).tolist() == [64, 64, 128, 256]
    assert m.batch_sizes(3, [2, 1]).tolist() == [3, 2]
    for _ in range(300):
        K = int(rng.integers(1, 17))
        r = rng.integers(1, 9, size=K)
        B = int(rng.integers(1, 100000))
        assert m.batch_sizes(B, r).tolist() == oracle.batch_sizes(B, r).tolist()
    with pytest.raises(m.RcdError):
        m.batch_sizes(0, [1, 2])
    with pytest.raises(m.RcdError):
        m.batch_sizes(8, [1, 0])


@pytest.mark.gpu
@pytest.mark.parametrize("K", [1, 2, 3, 7, 16])
@pytest.mark.parametrize("N", [1, 64, 1023, 1024, 1025, 65536, 262144, 262145, 600001])
def test_shards_at_the_edges_of_chunks_and_scan_runs(rcd, N, K):
    # chunks of 1024 samples, one thread of the scan per run of ceil(chunks / 256) of them
    print(f"shards edges N={N} K={K}", flush=True)
    assign = np.random.default_rng(N + K).integers(-1, K, N).astype(np.int32)
    index, offset = rcd.worker_shards(torch.from_numpy(assign).cuda(), K)
    order = np.argsort(assign, kind="stable")
    left = int(np.sum(assign < 0))
    assert offset.tolist() == [int(np.sum((assign >= 0) & (assign < k))) for k in range(K + 1)]
    assert np.array_equal(index.cpu().numpy()[: N - left], order[left:])


@pytest.mark.gpu
@pytest.mark.parametrize("L", [1, 2, 63, 64, 65, 129, 1000])
def test_class_split_of_many_classes(rcd, L):
    # every class is its own run of steps: the order inside a class counts 0, 1, ... and the quotas are the class's own
    print(f"class split L={L}", flush=True)
    rng = np.random.default_rng(L)
    N = 3 * L + 1500
    labels = rng.integers(0, L, N).astype(np.int32)
    X = torch.from_numpy(rng.standard_normal((N, 8)).astype(np.float32)).cuda()
    r = np.array([1, 2, 2], np.int32)
    most = int(np.bincount(labels).max())
    _, full = rcd.dataset_workspace_bytes(N, L, most, 3, rcd.MODE_STORED)
    ws = torch.empty(full, dtype=torch.uint8, device="cuda")
    assign, order, _ = rcd.partition_dataset(X, torch.from_numpy(labels).cuda(), L, r, 8.0, workspace=ws, graph_cut=True)
    assign, order = assign.cpu().numpy(), order.cpu().numpy()
    for c in range(L):
        at = np.flatnonzero(labels == c)
        assert sorted(order[at].tolist()) == list(range(len(at)))
        assert np.array_equal(np.bincount(assign[at], minlength=3), rcd.quota(len(at), r))


@pytest.mark.gpu
@pytest.mark.parametrize("where", [0, 1023, 1024, 4999])
@pytest.mark.parametrize("K", [1, 4, 16])
def test_a_bad_worker_anywhere_is_told_and_writes_nothing(rcd, K, where):
    # the split carries a bad label in the sign of a chunk's first count (zero there or not), -1 stays nobody's
    print(f"bad worker K={K} at {where}", flush=True)
    assign = np.random.default_rng(where + K).integers(-1, K, 5000).astype(np.int32)
    assign[1024:2048] = -1                       # a chunk without a single count
    for bad in (K, -2):
        assign[where] = bad
        with pytest.raises(rcd.RcdError) as e:
            rcd.worker_shards(torch.from_numpy(assign).cuda(), K)
        assert e.value.status == 2
    assign[where] = -1
    _, offset = rcd.worker_shards(torch.from_numpy(assign).cuda(), K)
    assert offset.tolist() == [int(np.sum((assign >= 0) & (assign < k))) for k in range(K + 1)]


@pytest.mark.gpu
@pytest.mark.parametrize("where", [0, 1024, 4999])
@pytest.mark.parametrize("L", [16, 17, 100])
def test_a_bad_label_on_either_side_of_the_counting_by_ballots(rcd, L, where):
    print(f"bad label L={L} at {where}", flush=True)
    N = 5000
    labels = np.random.default_rng(L).integers(0, L, N).astype(np.int32)
    X = torch.zeros((N, 8), dtype=torch.float32, device="cuda")
    ws = torch.empty(rcd.dataset_workspace_bytes(N, L, N, 2, rcd.MODE_STORED)[0], dtype=torch.uint8, device="cuda")
    for bad in (L, -1):
        labels[where] = bad
        with pytest.raises(rcd.RcdError) as e:
            rcd.partition_dataset(X, torch.from_numpy(labels).cuda(), L, np.array([1, 1], np.int32), 8.0, workspace=ws)
        assert e.value.status == 2
