"""The batched BMU of the smallest calls (direct distances of every unit) and of
large ones (products on the fp16 matrix instructions, every
operand in two halves) against the oracle at the edges of its tiles, and
against the fp32 products (som_bmu2_noalloc) for rows that cannot be split."""
import numpy as np
import pytest

import oracle
import paper_1905_09598_amd as som
import workloads
from gpu_util import dev, rel_gap, say, torch_cuda

pytestmark = pytest.mark.gpu

GAP = 1e-4


def _case(rows, cols, d, n, seed):
    X = workloads.gaussian_mixture(n, d, 8, 0.2, seed)
    W = workloads.random_weights(rows * cols, d, seed + 1, -1.0, 1.0)
    k = rows * cols // 2
    W[:k] = 0.6 * X[:k] + 0.4 * W[:k]
    return X, W


# sample tiles of 256, unit tiles of 128, slabs of 32 columns; the larger
# shapes take several unit groups, the longer rows split columns (all in one chunk
# of samples: test_chunks_of_samples has several)
@pytest.mark.parametrize("rows,cols,d,n,offset", [
    (32, 40, 700, 12032, 0),      # whole tiles
    (31, 41, 701, 12033, 0),      # remainders everywhere, rows not whole float4s
    (32, 40, 703, 12031, 1),      # misaligned samples
    (50, 50, 96, 33000, 0),
    (1, 1281, 640, 9000, 3),
    (70, 72, 1025, 4200, 0),
    (25, 41, 4000, 2600, 0),
])
def test_large_calls_match_oracle(rows, cols, d, n, offset):
    say("half products", rows, cols, d, n, offset)
    torch = torch_cuda()
    X, W = _case(rows, cols, d, n, d)
    m = som.Map(rows, cols, d, seed=0)
    m.weights = dev(W)
    flat = dev(np.concatenate([np.zeros(offset, np.float32), X.reshape(-1)]))
    Xd = flat[offset:].view(n, d)
    idx, idx2, d1 = m.bmu(Xd, second=True)
    again, qe, te = m.evaluate(Xd)
    assert torch.equal(idx, again)
    o = oracle.evaluate(W, rows, cols, X)
    gap = rel_gap(o["d1"], o["d2"])
    clear = gap > GAP
    assert clear.mean() > 0.9
    idx = idx.cpu().numpy()
    assert np.array_equal(idx[clear], o["c1"][clear])
    # the distances are direct fp32 sums
    same = idx == o["c1"]
    got = d1.cpu().numpy()
    assert np.abs(got[same] - o["d1"][same]).max() <= 1e-5 * o["d1"].max()
    assert abs(qe - o["qe"]) <= 1e-5 * o["qe"]
    m.close()


@pytest.mark.parametrize("where", ["samples", "prototypes", "both"])
def test_rows_that_cannot_be_split_match_the_fp32_products(where):
    rows, cols, d, n = 32, 40, 700, 12000
    X, W = _case(rows, cols, d, n, 11)
    special = [np.inf, -np.inf, np.nan, 3e38, -1e30, 1e-30, 1e-42, 2.0 ** 41, 2.0 ** -45]
    if where in ("samples", "both"):
        for k, v in enumerate(special):
            X[100 * k + 7, 3 * k] = v
            X[100 * k + 8] = 0.0
            X[100 * k + 8, 5 * k + 1] = v        # the row's only entry
            X[100 * k + 9] *= np.float32(v if np.isfinite(v) and abs(v) < 1e20 else 1e-20)
    if where in ("prototypes", "both"):
        few = special if where == "both" else special[5:7] + special[8:]
        for k, v in enumerate(few):
            W[50 * k + 3] *= np.float32(1e-20)
            W[50 * k + 4, 2 * k] = v
            W[50 * k + 5] = 0.0
    m = som.Map(rows, cols, d, seed=0)
    m.weights = dev(W)
    Xd = dev(X)
    a = [t.cpu().numpy() for t in m.bmu(Xd, second=True)]
    torch = torch_cuda()
    b = [torch.empty(n, dtype=t, device="cuda") for t in (torch.int32, torch.int32, torch.float32)]
    som.som_bmu2_noalloc(m.handle, Xd, n, *b)
    m.synchronize()
    b = [t.cpu().numpy() for t in b]
    differ = np.nonzero(a[0] != b[0])[0]
    say("unsplittable", where, "differing BMUs", differ.size, "of", n)
    # equal units, or distances equal within fp32 rounding of a direct sum
    for i in differ:
        assert np.isfinite(a[2][i]) and abs(a[2][i] - b[2][i]) <= 1e-5 * abs(b[2][i]), i
    both = np.isfinite(a[2]) & np.isfinite(b[2])
    assert np.array_equal(np.isfinite(a[2]), np.isfinite(b[2]))
    assert np.allclose(a[2][both], b[2][both], rtol=1e-5)
    m.close()


# Fewer samples than one tile on a large map, still in halves.
@pytest.mark.parametrize("n", [106, 200, 255])
def test_fewer_samples_than_a_tile(n, monkeypatch):
    rows, cols, d = 100, 100, 1000
    X = workloads.gaussian_mixture(n, d, 8, 0.2, 5)
    W = workloads.random_weights(rows * cols, d, 6, -1.0, 1.0)
    W[::50] = X[np.arange(200) % n] + 0.3 * W[::50]
    monkeypatch.setenv("SOM_BMU_ROUTE", "2")
    m = som.Map(rows, cols, d, seed=0)
    m.weights = dev(W)
    assert m.bmu_route(n) == "halves"
    idx, idx2, d1 = [t.cpu().numpy() for t in m.bmu(dev(X), second=True)]
    m.close()
    o = oracle.evaluate(W, rows, cols, X)
    clear = rel_gap(o["d1"], o["d2"]) > GAP
    assert np.array_equal(idx[clear], o["c1"][clear])
    same = idx == o["c1"]
    assert np.abs(d1[same] - o["d1"][same]).max() <= 1e-5 * o["d1"].max()


# Several chunks of samples, the last one short, with rows without halves in the
# first and in a later one: by a memory cap that holds 512 rows (unit groups), and
# by the chunk size itself (split columns: two chunks of 3,072 rows).
@pytest.mark.parametrize("rows,cols,d,n,rows_in_cap", [(32, 40, 96, 3001, 512),
                                                       (31, 41, 203, 1543, 300),
                                                       (5, 25, 12000, 6000, 0)])
@pytest.mark.parametrize("special", [False, True])
def test_chunks_of_samples(rows, cols, d, n, rows_in_cap, special, monkeypatch):
    torch = torch_cuda()
    N = rows * cols
    g = torch.Generator(device="cuda").manual_seed(d)
    X = torch.randn(n, d, generator=g, device="cuda")
    W = torch.randn(N, d, generator=g, device="cuda")
    if special:
        X[5, 3] = float("nan")
        X[n - 2, 1] = 2.0 ** 45
        X[n - 700] = 0.0
    m = som.Map(rows, cols, d, seed=0)
    m.weights = W
    monkeypatch.setenv("SOM_BMU_ROUTE", "1")
    a = [t.cpu().numpy() for t in m.bmu(X, second=True)]
    monkeypatch.setenv("SOM_BMU_ROUTE", "2")
    if rows_in_cap:
        row, tiles = -(-d // 32) * 128, -(-N // 128)
        cap = tiles * 128 * row + 4 * N + 2048 + rows_in_cap * (row + 4 + 32 * tiles)
        monkeypatch.setenv("SOM_MAX_BYTES", str(cap))
    assert m.bmu_route(n) == "halves"
    b = [t.cpu().numpy() for t in m.bmu(X, second=True)]
    monkeypatch.delenv("SOM_MAX_BYTES", raising=False)
    say("chunks", rows, cols, d, n, "differing", int((a[0] != b[0]).sum()))
    # the same units, or distances equal within fp32 rounding of a direct sum
    for p, q in ((a[0], b[0]), (a[1], b[1])):
        assert (p != q).mean() <= 1e-3
    assert np.array_equal(np.isfinite(a[2]), np.isfinite(b[2]))
    f = np.isfinite(a[2])
    assert np.allclose(a[2][f], b[2][f], rtol=1e-5)
    m.close()


# Rows of fewer than 32 floats keep to the fp32 products, whose few roundings
# come to less than what halves leave out.
@pytest.mark.parametrize("d", [2, 3, 8, 31, 32])
def test_short_rows_keep_the_fp32_products(d):
    torch = torch_cuda()
    rows, cols, n = 32, 32, 40000
    X, W = _case(rows, cols, d, n, d)
    m = som.Map(rows, cols, d, seed=0)
    m.weights = dev(W)
    assert m.bmu_route(n) == ("fp32" if d < 32 else "halves")
    Xd = dev(X)
    a = m.bmu(Xd, second=True)
    b = [torch.empty(n, dtype=t, device="cuda") for t in (torch.int32, torch.int32, torch.float32)]
    som.som_bmu2_noalloc(m.handle, Xd, n, *b)
    m.synchronize()
    if d < 32:
        assert all(torch.equal(p, q) for p, q in zip(a, b))
    assert (a[0] == b[0]).float().mean() > 0.999
    m.close()


# Rows without halves send their tiles to the fp32 products, not every sample to a
# scan of all prototypes: the search takes no longer than a small multiple of the
# search that forms every product in fp32 (it was 10 times that and more).
@pytest.mark.parametrize("where", ["prototype", "sample", "samples"])
def test_rows_that_cannot_be_split_keep_to_tiles(where):
    torch = torch_cuda()
    rows, cols, d, n = 70, 72, 512, 60000
    g = torch.Generator(device="cuda").manual_seed(4)
    X = torch.randn(n, d, generator=g, device="cuda")
    W = torch.randn(rows * cols, d, generator=g, device="cuda")
    if where == "prototype":
        W[77, 5] = float("nan")
    elif where == "sample":
        X[4000, 3] = float("nan")
    else:
        X[:, 7] *= 1e13
        W[:, 7] *= 1e13
    m = som.Map(rows, cols, d, seed=0)
    m.weights = W
    out = [[torch.empty(n, dtype=t, device="cuda")
            for t in (torch.int32, torch.int32, torch.float32)] for _ in range(2)]
    calls = (lambda: som.som_bmu2(m.handle, X, n, *out[0]),
             lambda: som.som_bmu2_noalloc(m.handle, X, n, *out[1]))
    ms = [[], []]
    for _ in range(4):
        for k, call in enumerate(calls):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            call()
            b.record()
            b.synchronize()
            ms[k].append(a.elapsed_time(b))
    t, fp32 = min(ms[0]), min(ms[1])
    say("unsplittable", where, "ms", t, "fp32 throughout", fp32)
    assert t <= 3 * fp32
    same = out[0][0] == out[1][0]
    assert same.float().mean() > 0.999
    bad = torch.isnan(X).any(1)
    assert bool((out[0][0][bad] == -1).all())
    m.close()


@pytest.mark.parametrize("rows,cols", [(1, 1), (1, 2), (5, 1), (9, 7), (33, 31), (70, 70)])
@pytest.mark.parametrize("d,offset", [(1, 0), (3, 1), (4, 0), (255, 0), (256, 0), (1030, 3)])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 8, 9])
def test_few_samples_match_oracle(rows, cols, d, offset, n):
    rng = np.random.default_rng(rows + d + n)
    X = rng.standard_normal((n, d)).astype(np.float32)
    W = rng.standard_normal((rows * cols, d)).astype(np.float32)
    if rows * cols > 4:
        W[4] = W[2]                    # an exact tie goes to the lower unit
        X[0] = W[2]
    m = som.Map(rows, cols, d, seed=0)
    m.weights = dev(W)
    flat = dev(np.concatenate([np.zeros(offset, np.float32), X.reshape(-1)]))
    idx, idx2, d1 = [t.cpu().numpy() for t in m.bmu(flat[offset:].view(n, d), second=True)]
    m.close()
    o = oracle.evaluate(W, rows, cols, X)
    clear = rel_gap(o["d1"], o["d2"]) > GAP
    assert np.array_equal(idx[clear], o["c1"][clear])
    # a direct fp32 sum of d terms in 64 lanes and a tree
    assert np.abs(d1 - o["d1"]).max() <= 1e-5 * max(o["d1"].max(), 1e-30)
    if rows * cols == 1:
        assert (idx2 == -1).all()
    if rows * cols > 4:
        assert (idx[0], idx2[0]) == (2, 4) and d1[0] == 0.0
