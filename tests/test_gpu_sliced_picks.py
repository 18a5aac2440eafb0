"""The sliced step loop with up to eight picks to a trip: the picks of a trip are made on the gains at its start, and those for a
block that has one already are guesses.  Same bits as the one-workgroup loop with its gains in memory (itself refereed by the
oracle, tests/test_gpu_incremental.py), where guesses fail often, where candidates tie, where posts and trips overflow, and with
the most workgroups a class can have."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rcd():
    import paper_2211_00839_amd as m

    m.load_library()
    return m


def features(kind, n, seed, d=32):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    if kind == "mixture":
        c = torch.randn(4, d, generator=g, device="cuda")
        return c[torch.randint(0, 4, (n,), generator=g, device="cuda")] + 0.5 * torch.randn(n, d, generator=g, device="cuda")
    base = torch.randn(max(1, n // 3 if kind == "triples" else 40), d, generator=g, device="cuda")
    X = base[torch.randint(0, base.shape[0], (n,), generator=g, device="cuda")]
    # triples: a pick lowers its neighbours' gains, which are the next best; repeated: whole groups tie exactly
    return X + 0.02 * torch.randn(n, d, generator=g, device="cuda") if kind == "triples" else X


def compare(rcd, monkeypatch, S, cap, slice_, small_kb=None):
    results = []
    for shared in (True, False):
        monkeypatch.setenv("RCD_MW_MIN_N", "1" if shared else "0")
        monkeypatch.setenv("RCD_RESIDENT", "1" if shared else "0")
        monkeypatch.setenv("RCD_MW_SLICE", str(slice_))
        if small_kb and shared:
            monkeypatch.setenv("RCD_INC_SMALL_KB", str(small_kb))
        else:
            monkeypatch.delenv("RCD_INC_SMALL_KB", raising=False)
        a, o, f = rcd.partition_class(S=S, cap=np.asarray(cap, dtype=np.int64), mode=rcd.MODE_INCREMENTAL)
        results.append((a.cpu().numpy(), o.cpu().numpy(), f))
    for x, y in zip(*results):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("K", [1, 2, 3, 5, 8, 9, 16])
@pytest.mark.parametrize("kind", ["triples", "repeated"])
def test_guesses_that_fail_and_candidates_that_tie(rcd, monkeypatch, kind, K):
    n = 1500
    print(f"sliced picks {kind} K={K}", flush=True)
    S = rcd.similarity(features(kind, n, 11 + K), 32.0)
    cap = oracle.quota(n, [1 + (5 * k) % 4 for k in range(K)])
    compare(rcd, monkeypatch, S, cap, 256)


@pytest.mark.parametrize("small_kb", [1, 16, 4096])
@pytest.mark.parametrize("n,slice_,K", [(1300, 256, 1), (3000, 1024, 4), (3000, 1536, 8), (2900, 2048, 16)])
def test_lists_that_do_not_fit_a_post_or_a_trip(rcd, monkeypatch, n, slice_, K, small_kb):
    # from lists of four rows on to the update launch, to lists of 512 rows applied in the loop, 1024 entries to a trip at most
    print(f"sliced lists n={n} slice={slice_} K={K} small={small_kb}", flush=True)
    S = rcd.similarity(features("mixture", n, n), 32.0)
    compare(rcd, monkeypatch, S, oracle.quota(n, [1 + k % 3 for k in range(K)]), slice_, small_kb)


def test_quotas_of_zero_and_leftovers(rcd, monkeypatch):
    S = rcd.similarity(features("mixture", 1100, 5), 32.0)
    for cap in ([0, 40, 0, 300, 7], [1, 0, 0, 0, 0, 0, 0, 0, 0], [1100], [0, 0, 0]):
        compare(rcd, monkeypatch, S, cap, 256)


@pytest.mark.parametrize("n,K", [(16384, 5), (16000, 16)])
def test_the_most_workgroups(rcd, monkeypatch, n, K):
    # 64 and 63 slices of 256 samples
    S = rcd.similarity(features("mixture", n, n), 32.0)
    compare(rcd, monkeypatch, S, oracle.quota(n, [1 + k % 3 for k in range(K)]), 256)


@pytest.mark.parametrize("K,slice_", [(1, 1024), (5, 1024), (12, 1024), (7, 2048), (12, 2048)])
def test_a_wait_that_runs_out_in_the_middle_of_a_run(rcd, monkeypatch, K, slice_):
    # the bound set to a millisecond of a launch's ten or more from the host: some wait between the workgroups runs out, whichever
    # it is, every kernel ends and the call is run again by the loops that wait for nobody
    n = 6000
    print(f"a wait runs out, K={K} slice={slice_}", flush=True)
    S = rcd.similarity(features("mixture", n, 3), 32.0)
    cap = np.asarray(oracle.quota(n, [1 + k % 3 for k in range(K)]), dtype=np.int64)
    monkeypatch.setenv("RCD_MW_SLICE", str(slice_))
    results = []
    for ms in ("1", "2000"):
        monkeypatch.setenv("RCD_MW_SPIN_MS", ms)
        a, o, f = rcd.partition_class(S=S, cap=cap, mode=rcd.MODE_INCREMENTAL)
        results.append((a.cpu().numpy(), o.cpu().numpy(), f))
    for x, y in zip(*results):
        assert np.array_equal(x, y)
