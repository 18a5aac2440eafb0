"""The similarity kernel for few tiles (32 x 32 per wave, operands straight from memory) against the 256 x 256 and 256 x 128
ones that the oracle's tests cover: the same bits over every form a call can have, alone and in a data set's batch."""
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


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n,d,pad,shift,picked", [(1, 1, 0, 0, False), (31, 7, 1, 0, False), (32, 8, 0, 0, True), (33, 63, 0, 1, False),
                                                  (64, 64, 0, 0, False), (65, 65, 3, 0, True), (255, 128, 0, 0, False),
                                                  (257, 300, 4, 0, True), (300, 511, 0, 0, False), (601, 512, 0, 4, False),
                                                  (601, 777, 0, 0, True), (130, 2048, 8, 0, False), (97, 1032, 0, 0, False)])
def test_same_bits_as_the_large_tiles(rcd, monkeypatch, dtype, n, d, pad, shift, picked):
    print(f"similarity few tiles n={n} d={d} pad={pad} shift={shift} {dtype}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(n * 1000 + d)
    rows = 2 * n if picked else n
    flat = torch.randn(rows * (d + pad) + shift, generator=g, device="cuda").to(torch.float32 if dtype == "f32" else torch.bfloat16)
    X = flat[shift:].view(rows, d + pad)[:, :d]
    index = torch.randperm(rows, generator=g, device="cuda")[:n].to(torch.int32) if picked else None
    got = []
    for mode in ("2", "0"):
        monkeypatch.setenv("RCD_SIM_FEW", mode)
        out = torch.full((n, n + 5), -1.0, device="cuda")
        rcd.similarity(X, float(d), row_index=index, out=out[:, :n])
        assert bool((out[:, n:] == -1.0).all())
        got.append(out[:, :n].clone())
    assert torch.equal(got[0].view(torch.int32), got[1].view(torch.int32))
    assert torch.equal(got[0], got[0].T) and bool((got[0].diagonal() == 1.0).all())


@pytest.mark.parametrize("dtype,d", [("f32", 64), ("f32", 50), ("bf16", 128), ("bf16", 33)])
def test_batch_of_classes(rcd, monkeypatch, dtype, d):
    print(f"similarity few tiles, classes d={d} {dtype}", flush=True)
    rng = np.random.default_rng(d)
    sizes = [1, 3, 64, 65, 300, 17, 256, 700] * 9            # more than one launch's 64 classes
    X = torch.from_numpy(np.concatenate([si.make_class(seed=i, n=n, d=d) for i, n in enumerate(sizes)])).cuda()
    X = X.to(torch.float32 if dtype == "f32" else torch.bfloat16)
    y = np.repeat(np.arange(len(sizes)), sizes).astype(np.int32)
    at = rng.permutation(len(y))
    X, y = X[torch.from_numpy(at).cuda()].contiguous(), torch.from_numpy(y[at]).cuda()
    _, full = rcd.dataset_workspace_bytes(len(at), len(sizes), 700, 3, rcd.MODE_STORED)
    ws = torch.empty(full, dtype=torch.uint8, device="cuda")
    got = []
    for mode in ("2", "0"):
        monkeypatch.setenv("RCD_SIM_FEW", mode)
        a, o, f = rcd.partition_dataset(X, y, len(sizes), [1, 2, 1], float(d), workspace=ws, graph_cut=True)
        got.append((a.cpu().numpy(), o.cpu().numpy(), f))
    for p, q in zip(*got):
        assert np.array_equal(p, q)
