"""The dispatch of several classes to slices on the GPU: whether a data set's call runs on another loop than with slices switched off,
seen by its number of launches, and the same bits from both, also where the slices' waits run out."""
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


# (sizes, blocks, cut into slices): from 3073 samples on with more than four blocks, 2561 with more than eight, a quarter of the work
@pytest.mark.parametrize("sizes,K,sliced", [([3073] * 3, 5, True), ([3072] * 3, 5, False), ([3073] * 3, 4, False),
                                            ([2561] * 2, 9, True), ([2560] * 2, 9, False), ([3400] + [700] * 20, 5, True),
                                            ([3400] + [2000] * 12, 5, False)])
def test_several_classes_are_cut_by_the_rule_and_give_the_same_bits(rcd, monkeypatch, sizes, K, sliced):
    print(f"dispatch of {len(sizes)} classes, the largest {sizes[0]}, K={K}", flush=True)
    d, r = 32, [1 + k % 3 for k in range(K)]
    X = torch.from_numpy(si.make_class(seed=sum(sizes), n=sum(sizes), d=d, G=5)).cuda()
    labels = torch.from_numpy(np.repeat(np.arange(len(sizes)), sizes).astype(np.int32)).cuda()
    size = rcd.dataset_workspace_bytes(sum(sizes), len(sizes), max(sizes), K, rcd.MODE_STORED)[1]
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")

    def call():
        a, o, f = rcd.partition_dataset(X, labels, len(sizes), r, float(d), rcd.MODE_INCREMENTAL, ws)
        return (a.cpu().numpy(), o.cpu().numpy(), f), rcd.last_stats()["launches"]

    default, launches = call()
    monkeypatch.setenv("RCD_MW_MIN_N", "0")
    whole, few = call()
    monkeypatch.delenv("RCD_MW_MIN_N")
    assert (launches != few) == sliced, (launches, few)
    results = [whole]
    if sliced:
        # as where others hold the device: a wait between slices runs out (its bound, a millisecond from a launch's start, in a launch
        # that lasts longer), and the answer is the other loop's
        monkeypatch.setenv("RCD_MW_SPIN_MS", "1")
        monkeypatch.setenv("RCD_INC_STEPS", "4096")
        results.append(call()[0])
    for other in results:
        for x, y in zip(default, other):
            assert np.array_equal(x, y)
