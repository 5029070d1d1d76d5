"""Panel training (asked for, and where the default takes it) against the fp64 oracle at
the edges of its shapes: units per lane and per workgroup, steps per 16 and per
panel, columns per tile and per gather, one and several control workgroups;
and its error paths."""
import numpy as np
import pytest

import oracle
import paper_1905_09598_amd as som
import workloads
from gpu_util import dev, rel_gap, say

pytestmark = pytest.mark.gpu

GAP = 1e-4
ENV = ("SOM_TRAIN_VARIANT", "SOM_TRAIN_GRID", "SOM_TRAIN_BLOCK_M", "SOM_TRAIN_LDS_ROWS",
       "SOM_TRAIN_SWEEPERS")


@pytest.fixture(autouse=True)
def _panels(monkeypatch):
    for k in ENV:
        monkeypatch.delenv(k, raising=False)
    monkeypatch.setenv("SOM_TRAIN_VARIANT", "6")


def _train(rows, cols, d, n, topology=som.RECT, sched=(0.4, 0.02, None, 0.5), offset=0, seed=5,
           step0=0, total=0):
    X = workloads.gaussian_mixture(n, d, 3, 0.2, seed=seed + d)
    W0 = workloads.random_weights(rows * cols, d, seed + 1, -1.0, 1.0)
    order = workloads.epoch_orders(n, 1, seed)
    lr0, lr1, s0, s1 = sched
    s0 = max(rows, cols) / 2.0 if s0 is None else s0
    m = som.Map(rows, cols, d, seed=0, topology=topology)
    m.weights = dev(W0)
    flat = dev(np.concatenate([np.zeros(offset, np.float32), X.reshape(-1)]))
    Xd = flat[offset:].view(n, d)
    trace = dev(np.full(n, -1, np.int32))
    m.train(Xd, 1, lr0, lr1, s0, s1, order=dev(order), bmu_trace=trace, step0=step0,
            total_steps=total)
    W = m.weights.cpu().numpy().astype(np.float64)
    got = trace.cpu().numpy()
    m.close()
    s = oracle.schedule(lr0, lr1, s0, s1)
    Wo, tr = oracle.train(W0, rows, cols, X, order, s, topology=topology, trace=True, step0=step0,
                          total_steps=total or step0 + n)
    if np.array_equal(got, tr):
        # 1e-7 relative rounding per panel of values up to a few units
        assert np.abs(W - Wo).max() <= 2e-5
        return
    k = int(np.argmax(got != tr))
    Wk, _ = oracle.train(W0, rows, cols, X, order[:k], s, topology=topology, step0=step0,
                         total_steps=total or step0 + n)
    Ds = np.sort(oracle.distances(Wk, X[order[k]]))
    say(f"  identical BMUs for {k}/{n} steps")
    # (thousands of units on rows of one float lie so close together that
    # their distances, differences of fp32 sums at the scale S of squared
    # sample-to-sample distances within about 8 roundings of 2^-24 S, are not told
    # apart below 1e-6 S; neither are they by the pipelined kernels' sums)
    S = np.square(X.astype(np.float64) - X[order[0]]).sum(1).max()
    assert len(Ds) > 1 and (Ds[1] - Ds[0] <= GAP * Ds[0] or
                            (d == 1 and Ds[1] - Ds[0] <= 1e-6 * S)), "divergence without a near tie"


@pytest.mark.parametrize("rows,cols", [(1, 1), (1, 15), (4, 4), (1, 17), (8, 8), (5, 13),
                                       (15, 17), (16, 16), (1, 257), (16, 32), (27, 19),
                                       (32, 32), (5, 205), (41, 43), (50, 50), (128, 128)])
@pytest.mark.parametrize("topology", [som.RECT, som.HEX])
def test_unit_counts_follow_the_oracle(rows, cols, topology):
    say("panel units", rows, cols, topology)
    _train(rows, cols, 40, 175, topology)


@pytest.mark.parametrize("rows,cols", [(9, 11), (20, 21), (31, 30), (60, 50)])
@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 31, 47, 48, 49, 63, 64, 65, 79, 80, 81, 97, 160,
                               161, 241])
def test_step_counts_follow_the_oracle(rows, cols, n):
    say("panel steps", rows, cols, n)
    _train(rows, cols, 24, n, seed=n)


@pytest.mark.parametrize("rows,cols", [(9, 11), (60, 50)])
@pytest.mark.parametrize("d,offset", [(1, 0), (3, 0), (4, 0), (5, 1), (16, 0), (31, 0), (32, 3),
                                      (63, 0), (64, 0), (65, 0), (129, 0), (1023, 0), (1024, 1),
                                      (1025, 0), (2049, 0), (4545, 0)])
def test_row_lengths_and_alignments_follow_the_oracle(rows, cols, d, offset):
    say("panel columns", rows, cols, d, offset)
    _train(rows, cols, d, 90 if d < 2000 else 50, offset=offset)


# Both sides of the lines between panels and the persistent kernel: units of one
# workgroup, rows per workgroup at two row lengths, the longest row, and steps.
@pytest.mark.parametrize("rows,cols,d,n", [
    (20, 35, 60, 100), (1, 701, 60, 100), (80, 128, 8, 100), (19, 539, 8, 100),
    (67, 107, 516, 100), (1, 7169, 513, 100), (27, 26, 3072, 100), (27, 26, 3073, 100),
    (127, 129, 8, 95), (127, 129, 8, 96), (5, 6, 2049, 39), (5, 6, 2049, 40), (5, 6, 1025, 3),
    (5, 6, 1025, 4), (5, 6, 1024, 1)])
def test_default_path_at_its_lines(rows, cols, d, n, monkeypatch):
    monkeypatch.delenv("SOM_TRAIN_VARIANT")
    _train(rows, cols, d, n)


def _replayed_gaps(W0, rows, cols, X, order, trace, sched):
    """The training of `trace`'s BMUs in 64 bits: per step, how far the BMU's squared
    distance lies above the smallest one, relative to that; and the final map."""
    W, T = W0.astype(np.float64), len(order)
    gaps = np.empty(T)
    for k, (i, c) in enumerate(zip(order, trace)):
        D = oracle.distances(W, X[i])
        gaps[k] = (D[c] - D.min()) / max(D.min(), 1e-300)
        h = oracle.neighbourhood(rows, cols, som.RECT, int(c), *oracle.schedule_at(k, T, sched))
        W += h[:, None] * (X[i].astype(np.float64) - W)
    return gaps, W


# Maps whose persistent kernel takes its distances from direct differences stay on
# it: many units on short rows need all of their digits.
@pytest.mark.parametrize("rows,cols,d,n", [(128, 150, 2, 1500), (128, 150, 3, 1500),
                                           (181, 181, 8, 800), (51, 51, 3100, 120)])
def test_direct_differences_are_kept(rows, cols, d, n, monkeypatch):
    rng = np.random.default_rng(d)
    X = rng.random((n, d), dtype=np.float32)
    W0 = rng.random((rows * cols, d), dtype=np.float32)
    order = np.arange(n, dtype=np.int32)
    out = []
    for variant in ("", "5"):
        monkeypatch.setenv("SOM_TRAIN_VARIANT", variant)
        m = som.Map(rows, cols, d, seed=0)
        m.weights = dev(W0)
        trace = dev(np.full(n, -1, np.int32))
        m.train(dev(X), 1, 0.2, 0.05, 1.5, 0.5, order=dev(order), bmu_trace=trace)
        out.append((trace.cpu().numpy(), m.weights.cpu().numpy()))
        m.close()
    gaps, _ = _replayed_gaps(W0, rows, cols, X, order, out[0][0],
                             oracle.schedule(0.2, 0.05, 1.5, 0.5))
    say("direct differences", rows, cols, d, "steps beyond the gap", int((gaps > GAP).sum()),
        "of", n, "largest", gaps.max())
    assert gaps.max() <= GAP
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])


# One sample thousands of times as long as the others, at the first step of an
# inner panel of any of the shapes, and one within a panel: every later step finds
# its BMU by its own distances.
@pytest.mark.parametrize("rows,cols,M", [(9, 11, 80), (20, 20, 64), (24, 25, 48), (60, 50, 80)])
@pytest.mark.parametrize("factor", [1e3, 1e4])
def test_outliers_do_not_cost_the_other_steps_their_bmus(rows, cols, M, factor):
    d, n = 64, 4 * M + 30
    rng = np.random.default_rng(M)
    X = rng.standard_normal((n, d)).astype(np.float32)
    for at in (2 * M, 3 * M, M + 7):
        X[at] *= np.float32(factor)
    W0 = rng.standard_normal((rows * cols, d)).astype(np.float32)
    order = np.arange(n, dtype=np.int32)
    m = som.Map(rows, cols, d, seed=0)
    m.weights = dev(W0)
    trace = dev(np.full(n, -1, np.int32))
    m.train(dev(X), 1, 0.3, 0.1, 2.0, 1.0, order=dev(order), bmu_trace=trace)
    W = m.weights.cpu().numpy()
    m.close()
    gaps, Wk = _replayed_gaps(W0, rows, cols, X, order, trace.cpu().numpy(),
                              oracle.schedule(0.3, 0.1, 2.0, 1.0))
    say("outliers", rows, cols, factor, "steps beyond the gap", int((gaps > GAP).sum()), "of", n,
        "largest", gaps.max())
    assert gaps.max() <= GAP
    # rounding of 1e-7 per panel of the largest values a prototype passes through
    assert np.abs(W - Wk).max() <= 1e-6 * np.abs(X).max()


# Tight clusters far apart, where many units are nearly as near as the BMU: the
# rounding of a distance stays within 6 roundings 2^-24 of the largest
# sample-to-sample distance S (the pipelined kernel: 2 to 6; one chain of fp32 sums
# over a wave's columns: 12).
@pytest.mark.parametrize("rows,cols,d", [(100, 100, 2048), (30, 30, 5000)])
def test_rounding_of_distances_on_tight_clusters(rows, cols, d):
    import torch
    n, N = 300, rows * cols
    g = torch.Generator(device="cuda").manual_seed(d)
    C = torch.randn(8, d, generator=g, device="cuda")
    pick = lambda k: C[torch.randint(0, 8, (k,), generator=g, device="cuda")]
    X = pick(n) + 0.02 * torch.randn(n, d, generator=g, device="cuda")
    W0 = pick(N) + 0.005 * torch.randn(N, d, generator=g, device="cuda")
    order = torch.arange(n, device="cuda", dtype=torch.int32)
    trace = torch.full((n,), -1, device="cuda", dtype=torch.int32)
    m = som.Map(rows, cols, d, seed=0)
    m.weights = W0
    m.train(X, 1, 0.1, 0.02, 3.0, 1.0, order=order, bmu_trace=trace)
    m.synchronize()
    m.close()
    S = float(torch.cdist(X.double(), X.double()).max()) ** 2
    W, sched = W0.double(), oracle.schedule(0.1, 0.02, 3.0, 1.0)
    worst = 0.0
    for k, c in enumerate(trace.tolist()):
        diff = X[k].double() - W
        D = diff.square().sum(1)
        worst = max(worst, float(D[c] - D.min()))
        h = oracle.neighbourhood(rows, cols, som.RECT, c, *oracle.schedule_at(k, n, sched))
        W += torch.from_numpy(h).cuda()[:, None] * diff
    say("tight clusters", rows, cols, d, "largest excess", worst / S * 2 ** 24, "x 2^-24 S")
    assert worst <= 6 * 2.0 ** -24 * S


@pytest.mark.parametrize("rows,cols", [(9, 11), (60, 50)])
def test_resumed_steps_follow_the_oracle(rows, cols):
    _train(rows, cols, 32, 100, step0=37, total=500)


@pytest.mark.parametrize("rows,cols", [(7, 9), (25, 30), (60, 50)])
def test_exact_copies_and_untouched_units(rows, cols):
    # lr = 1 and sigma = 0: the BMU becomes the sample and nothing else moves
    n, d = 170, 20
    X = workloads.gaussian_mixture(n, d, 4, 0.3, seed=8)
    W0 = workloads.random_weights(rows * cols, d, 9, -1.0, 1.0)
    order = np.arange(n, dtype=np.int32)
    m = som.Map(rows, cols, d, seed=0)
    m.weights = dev(W0)
    trace = dev(np.full(n, -1, np.int32))
    m.train(dev(X), 1, 1.0, 1.0, 0.0, 0.0, order=dev(order), bmu_trace=trace)
    got, W = trace.cpu().numpy(), m.weights.cpu().numpy()
    m.close()
    want = W0.copy()
    for k, c in enumerate(got):
        want[c] = X[k]
    assert np.array_equal(W, want)


@pytest.mark.parametrize("rows,cols", [(1, 300), (33, 32), (60, 50)])
def test_equal_units_take_the_lowest_index(rows, cols):
    # every prototype equal: each step's BMU is unit 0 while sigma is infinite
    X = workloads.gaussian_mixture(40, 12, 2, 0.3, seed=3)
    m = som.Map(rows, cols, 12, seed=0)
    m.weights = dev(np.zeros((rows * cols, 12), np.float32))
    trace = dev(np.full(40, -1, np.int32))
    m.train(dev(X), 1, 0.3, 0.3, np.inf, np.inf, order=dev(np.arange(40, dtype=np.int32)),
            bmu_trace=trace)
    assert np.array_equal(trace.cpu().numpy(), np.zeros(40, np.int32))
    m.close()


# The nearest prototypes are copies in the last units, in a row of 16 lanes of a
# wave that has fewer than four such rows with units.
@pytest.mark.parametrize("rows,cols,copies", [(3, 6, 2), (5, 5, 4), (16, 17, 16), (20, 20, 3),
                                              (21, 32, 8)])
def test_equal_units_of_a_partly_filled_wave(rows, cols, copies):
    N, d, n = rows * cols, 24, 70
    W0 = workloads.random_weights(N, d, 3, 4.0, 5.0)
    W0[-copies:] = W0[-1] - 4.0
    m = som.Map(rows, cols, d, seed=0)
    m.weights = dev(W0)
    trace = dev(np.full(n, -1, np.int32))
    X = workloads.random_weights(n, d, 4, 0.0, 1.0)
    inf = float("inf")  # every unit moves alike, so the copies stay equal
    m.train(dev(X), 1, 0.01, 0.01, inf, inf, order=dev(np.arange(n, dtype=np.int32)),
            bmu_trace=trace)
    assert np.array_equal(trace.cpu().numpy(), np.full(n, N - copies, np.int32))
    m.close()


@pytest.mark.parametrize("rows,cols", [(1, 1), (4, 4), (8, 8), (10, 10), (16, 17), (23, 23)])
def test_long_runs_with_waves_without_units(rows, cols):
    # sigma = inf: each prototype is the moving average of the samples, whatever
    # the BMUs.  2e-5: rounding of 1e-7 per panel at values of a few units,
    # shrunk by (1 - lr) a step.
    d, n, epochs, lr = 128, 640, 10, 0.05
    X = workloads.gaussian_mixture(n, d, 3, 0.2, seed=9)
    W0 = workloads.random_weights(rows * cols, d, 2, -1.0, 1.0)
    order = np.concatenate([np.arange(n, dtype=np.int32)] * epochs)
    m = som.Map(rows, cols, d, seed=0)
    m.weights = dev(W0)
    inf = float("inf")
    m.train(dev(X), epochs, lr, lr, inf, inf, order=dev(order))
    W = m.weights.cpu().numpy().astype(np.float64)
    m.close()
    want = W0.astype(np.float64)
    for k in order:
        want += lr * (X[k].astype(np.float64) - want)
    assert np.abs(W - want).max() <= 2e-5


@pytest.mark.parametrize("rows,cols", [(9, 11), (25, 30), (60, 50)])
def test_unusable_input_leaves_the_prototypes(rows, cols):
    n, d = 200, 37
    X = workloads.gaussian_mixture(n, d, 3, 0.2, seed=d)
    W = workloads.random_weights(rows * cols, d, 4)
    bad = X.copy()
    bad[150, 36] = np.inf
    wrong = np.arange(n, dtype=np.int32)
    wrong[120] = n
    for data, order, name in ((bad, np.arange(n, dtype=np.int32), "SOM_E_NONFINITE"),
                              (X, wrong, "SOM_E_BAD_ORDER")):
        m = som.Map(rows, cols, d, seed=0)
        m.weights = dev(W)
        m.train(dev(data), 1, 0.5, 0.05, 3.0, 0.5, order=dev(order))
        with pytest.raises(som.SomError) as e:
            m.synchronize()
        assert e.value.name == name
        assert np.array_equal(m.weights.cpu().numpy(), W)
        m.close()


def test_exchange_timeout_ends_the_grid_and_is_reported(monkeypatch):
    rows, cols, d, n = 60, 50, 64, 200
    X = workloads.gaussian_mixture(n, d, 3, 0.2, seed=7)
    W = workloads.random_weights(rows * cols, d, 8)
    order = dev(workloads.epoch_orders(n, 1, 9))
    m = som.Map(rows, cols, d, seed=0)
    m.weights = dev(W)
    monkeypatch.setenv("SOM_DEBUG_EXCHANGE_TIMEOUT_US", "5000")
    monkeypatch.setenv("SOM_DEBUG_ABSENT_WORKGROUP", "1")
    m.train(dev(X), 1, 0.5, 0.05, 3.0, 0.5, order=order)
    with pytest.raises(som.SomError) as e:
        m.synchronize()
    assert e.value.name == "SOM_E_TIMEOUT"
    m.synchronize()
    monkeypatch.delenv("SOM_DEBUG_ABSENT_WORKGROUP")
    monkeypatch.delenv("SOM_DEBUG_EXCHANGE_TIMEOUT_US")
    out = []
    for _ in range(2):
        m.weights = dev(W)
        m.train(dev(X), 1, 0.5, 0.05, 3.0, 0.5, order=order)
        m.synchronize()
        out.append(m.weights.cpu().numpy())
    assert np.array_equal(out[0], out[1])
    m.close()


# On one workgroup a wave waits for the others through LDS: those waits end too,
# and the panels behind the one that was given up leave at once.
@pytest.mark.parametrize("rows,cols", [(9, 11), (16, 17), (30, 31)])
def test_wave_timeout_ends_the_call_and_is_reported(rows, cols, monkeypatch):
    d, n = 64, 1000
    X = dev(workloads.gaussian_mixture(n, d, 3, 0.2, seed=7))
    W = workloads.random_weights(rows * cols, d, 8)
    order = dev(workloads.epoch_orders(n, 1, 9))
    m = som.Map(rows, cols, d, seed=0)
    m.weights = dev(W)
    monkeypatch.setenv("SOM_DEBUG_EXCHANGE_TIMEOUT_US", "5000")
    monkeypatch.setenv("SOM_DEBUG_ABSENT_WORKGROUP", "1")
    m.train(X, 1, 0.5, 0.05, 3.0, 0.5, order=order)
    with pytest.raises(som.SomError) as e:
        m.synchronize()
    assert e.value.name == "SOM_E_TIMEOUT"
    m.synchronize()
    monkeypatch.delenv("SOM_DEBUG_ABSENT_WORKGROUP")
    monkeypatch.delenv("SOM_DEBUG_EXCHANGE_TIMEOUT_US")
    out = []
    for _ in range(2):
        m.weights = dev(W)
        m.train(X, 1, 0.5, 0.05, 3.0, 0.5, order=order)
        m.synchronize()
        out.append(m.weights.cpu().numpy())
    assert np.array_equal(out[0], out[1]) and np.isfinite(out[0]).all()
    m.close()


@pytest.mark.parametrize("rows,cols,d,n", [(10, 10, 500, 400), (30, 30, 300, 300),
                                           (60, 50, 300, 300)])
def test_memory_cap_takes_the_grid_kernels(rows, cols, d, n, monkeypatch):
    # below the panels' buffers the call still trains, on the kernels that
    # need none
    X = workloads.gaussian_mixture(n, d, 3, 0.2, seed=2)
    W = workloads.random_weights(rows * cols, d, 3)
    order = dev(workloads.epoch_orders(n, 1, 1))
    traces = []
    for cap in (None, "100000"):
        m = som.Map(rows, cols, d, seed=0)
        m.weights = dev(W)
        if cap:
            monkeypatch.setenv("SOM_MAX_BYTES", cap)
        t = dev(np.full(n, -1, np.int32))
        m.train(dev(X), 1, 0.4, 0.05, 4.0, 0.7, order=order, bmu_trace=t)
        traces.append(t.cpu().numpy())
        monkeypatch.delenv("SOM_MAX_BYTES", raising=False)
        m.close()
    o = oracle.train(W, rows, cols, X, workloads.epoch_orders(n, 1, 1),
                     oracle.schedule(0.4, 0.05, 4.0, 0.7), trace=True)[1]
    k = min(int(np.argmax(t != o)) if np.any(t != o) else n for t in traces)
    if k < n:
        Wk, _ = oracle.train(W, rows, cols, X, workloads.epoch_orders(n, 1, 1)[:k],
                             oracle.schedule(0.4, 0.05, 4.0, 0.7), total_steps=n)
        D = np.sort(oracle.distances(Wk, X[workloads.epoch_orders(n, 1, 1)[k]]))
        assert rel_gap(D[:1], D[1:2])[0] <= GAP
