"""The two tilings of the update launches (64 and 256 samples to a wave, RCD_INC_NARROW) give the same bits: lists about as long as
the chunk of a list that is held in LDS and as the longest that the narrow tiles take, in one segment and in many, and classes of
unequal size in one launch.  A class's first lists are as long as the class."""
import numpy as np
import pytest

import oracle
import synth_inputs as si

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def rcd():
    import paper_2211_00839_amd as m

    m.load_library()
    return m


def use(monkeypatch, loop, narrow):
    monkeypatch.setenv("RCD_INC_NARROW", str(narrow))
    monkeypatch.setenv("RCD_INC_FUSE_MIN_N", "0")
    monkeypatch.setenv("RCD_INC_SMALL_KB", "1")          # every list goes to the update launch
    monkeypatch.setenv("RCD_MW_SLICE", "256")
    monkeypatch.setenv("RCD_MW_MIN_N", "0" if loop == "one workgroup" else "1")
    monkeypatch.setenv("RCD_RESIDENT", "1" if loop == "sliced" else "0")


@pytest.mark.parametrize("loop", ["one workgroup", "shared", "sliced"])
@pytest.mark.parametrize("n", [63, 1023, 1024, 1025, 2049, 8191, 8192, 8193])
def test_narrow_and_wide_tiles_give_the_same_bits(rcd, monkeypatch, loop, n):
    print(f"update tiles n={n} loop={loop}", flush=True)
    X = torch.from_numpy(si.make_class(seed=n, n=n, d=16, G=5)).cuda()
    S = rcd.similarity(X, 16.0)
    cap = np.array([20, 13, 9] if n > 63 else [20, 13], dtype=np.int64)
    results = []
    for narrow in (1, 0):
        use(monkeypatch, loop, narrow)
        a, o, f = rcd.partition_class(S=S, cap=cap, mode=rcd.MODE_INCREMENTAL)
        results.append((a.cpu().numpy(), o.cpu().numpy(), f, rcd.last_stats()["entries_streamed"]))
    for x, y in zip(*results):
        assert np.array_equal(x, y)
    assert results[0][3] >= n * n                       # the first list, at least, was the whole class


@pytest.mark.parametrize("loop", ["one workgroup", "shared", "sliced"])
def test_classes_of_unequal_size_in_one_launch(rcd, monkeypatch, loop):
    print(f"update tiles, unequal classes, loop={loop}", flush=True)
    sizes, d, r = [1100, 40, 2305, 257, 1], 16, [1, 2, 1, 3, 1]
    X = torch.from_numpy(si.make_class(seed=9, n=sum(sizes), d=d, G=5)).cuda()
    labels = torch.from_numpy(np.repeat(np.arange(len(sizes)), sizes).astype(np.int32)).cuda()
    size = rcd.dataset_workspace_bytes(sum(sizes), len(sizes), max(sizes), len(r), rcd.MODE_STORED)[1]
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    results = []
    for narrow in (1, 0):
        use(monkeypatch, loop, narrow)
        a, o, f = rcd.partition_dataset(X, labels, len(sizes), r, float(d), rcd.MODE_INCREMENTAL, ws)
        results.append((a.cpu().numpy(), o.cpu().numpy(), f))
    for x, y in zip(*results):
        assert np.array_equal(x, y)
    at = 0
    for n in sizes[:2]:
        idx = np.arange(at, at + n)
        S = rcd.similarity(X, float(d), row_index=torch.from_numpy(idx.astype(np.int32)).cuda()).cpu().numpy()
        res = oracle.lockstep(S, oracle.quota(n, r), results[0][1][idx], results[0][0][idx], rel_tol=1e-5, objective="fl")
        assert res["rc"] == 0 and res["checked"] == n, res
        at += n
