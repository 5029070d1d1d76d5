"""GPU parity of the principal components, the size heuristic and the linear
initialisation (Sec. 6D, Fig. 2) against the fp64 oracle."""
import numpy as np
import pytest

import oracle
import paper_1905_09598_amd as som
import workloads
from gpu_util import config, dev, say

pytestmark = pytest.mark.gpu


def _gpu_pca(X):
    l1, l2, mean, v1, v2 = som.pca2(dev(X))
    return (np.array([l1, l2]), mean.cpu().numpy().astype(np.float64),
            np.stack([v1.cpu().numpy(), v2.cpu().numpy()], axis=1).astype(np.float64))


def _spectrum(X):
    X64 = X.astype(np.float64)
    Xc = X64 - X64.mean(0)
    return np.linalg.eigvalsh(Xc.T @ Xc / X.shape[0])[::-1]


def test_planar_data_axes_on_gpu():
    i = np.arange(64)
    s = np.where((i & 1) == 0, 1.0, -1.0)
    t = np.where((i & 2) == 0, 1.0, -1.0)
    mu = np.array([1.0, 2.0, -3.0, 4.0, 0.5, 6.0])
    X = (mu + 3.0 * np.outer(s, np.eye(6)[1]) + np.outer(t, np.eye(6)[4])).astype(np.float32)
    lam, mean, V = _gpu_pca(X)
    assert np.allclose(lam, [9.0, 1.0], rtol=1e-5, atol=0)
    assert np.allclose(mean, mu, atol=1e-6)
    assert np.allclose(V[:, 0], np.eye(6)[1], atol=1e-5)
    assert np.allclose(V[:, 1], np.eye(6)[4], atol=1e-5)


@pytest.mark.parametrize("n,d", [(500, 37), (200, 3000), (2000, 64)])
def test_components_match_oracle(n, d):
    rng = np.random.default_rng(d)
    k = min(d, 12)
    A = rng.standard_normal((k, d)) * (0.6 ** np.arange(k))[:, None]
    X = (rng.standard_normal((n, k)) @ A + rng.standard_normal(d) * 0.1).astype(np.float32)
    lam_o, V_o, mu_o = oracle.pca_top2(X)
    lam, mean, V = _gpu_pca(X)
    say(f"pca n={n} d={d}: gpu {lam} oracle {lam_o}")
    assert np.allclose(lam, lam_o, rtol=1e-4)
    assert np.allclose(mean, mu_o, atol=1e-5)
    assert np.abs(V - V_o).max() <= 1e-3


@pytest.mark.parametrize("ci", [0, 1])
def test_workload_components_and_sizes(ci):
    cfg = config(ci)
    X = workloads.make_data(cfg)
    lam_o, V_o, mu_o = oracle.pca_top2(X)
    lam, mean, V = _gpu_pca(X)
    ev = _spectrum(X)
    say(f"{cfg.name}: gpu {lam} oracle {lam_o} third {ev[2]:.6g}")
    assert np.allclose(lam, lam_o, rtol=1e-4)
    size_o = oracle.suggest_size(cfg.n, *lam_o)
    size_g = som.som_suggest_size(cfg.n, *lam)
    say(f"  sizes gpu {size_g} oracle {size_o}")
    assert size_g == size_o
    # eigenvectors are only determined as well as the gap to the next value
    for a in range(2):
        gap = (ev[a] - ev[a + 1]) / ev[0]
        if gap > 0.02:
            assert np.abs(V[:, a] - V_o[:, a]).max() <= 2e-5 / gap + 1e-5


@pytest.mark.parametrize("n,d", [(40, 1), (40, 7), (33, 8), (64, 9), (31, 65), (97, 1023),
                                 (129, 1025), (300, 2049)])
def test_components_at_tile_edges(n, d):
    # edges of the covariance tiles, of the rows per workgroup and of the
    # staged columns; the data has rank min(3, d), so most of the iterated
    # directions vanish
    rng = np.random.default_rng(n + d)
    k = min(3, d)
    A = rng.standard_normal((k, d)) * np.array([4.0, 2.0, 1.0])[:k, None]
    X = (rng.standard_normal((n, k)) @ A + 1.0).astype(np.float32)
    lam_o, V_o, mu_o = oracle.pca_top2(X) if d > 1 else (np.array([X.var(), 0.0]), None, X.mean(0))
    lam, mean, V = _gpu_pca(X)
    say(f"pca edge n={n} d={d}: gpu {lam} oracle {lam_o}")
    # fp32 covariance sums and a residual of 2e-5 of the largest eigenvalue
    assert np.allclose(lam, lam_o, rtol=1e-4, atol=2e-5 * lam_o[0])
    assert np.allclose(mean, mu_o, atol=1e-5)
    if d > 1:
        # angle error <= residual / gap to the next value
        ev = _spectrum(X)
        for a in range(2):
            gap = min(abs(ev[a] - ev[b]) for b in range(min(3, d)) if b != a) / ev[0]
            if gap > 0.02:
                assert np.abs(V[:, a] - V_o[:, a]).max() <= 2e-5 / gap + 1e-5


@pytest.mark.parametrize("n,d", [(50, 2), (50, 7), (64, 40), (300, 2049)])
@pytest.mark.parametrize("rank", [0, 1])
def test_vectors_are_unit_where_the_data_have_no_second_direction(n, d, rank):
    rng = np.random.default_rng(n + d)
    X = np.ones((n, d), np.float32)
    axis = rng.standard_normal(d)
    if rank:
        X = (X + np.outer(rng.standard_normal(n), axis)).astype(np.float32)
    lam, mean, V = _gpu_pca(X)
    say(f"rank {rank} n={n} d={d}: {lam}", V.T @ V)
    # unit and at a right angle within fp32 rounding of d components
    assert np.abs(V.T @ V - np.eye(2)).max() <= 1e-5
    assert lam[1] <= 2e-5 * max(lam[0], 1e-30)
    if rank:
        # the sums' rounding turns the axis by less than 2e-5 of the eigenvalue
        assert abs(V[:, 0] @ axis) / np.linalg.norm(axis) >= 1 - 1e-4


def test_linear_init_matches_oracle_grid():
    rng = np.random.default_rng(9)
    d = 40
    A = rng.standard_normal((6, d)) * np.array([3.0, 1.5, 0.5, 0.3, 0.2, 0.1])[:, None]
    X = (rng.standard_normal((800, 6)) @ A + 2.0).astype(np.float32)
    lam_o, V_o, mu_o = oracle.pca_top2(X)
    for rows, cols in ((7, 9), (1, 5), (4, 1)):
        m = som.Map(rows, cols, d, seed=1)
        m.init_linear(dev(X))
        W = m.weights.cpu().numpy().astype(np.float64)
        Wo = oracle.linear_init(mu_o, lam_o, V_o, rows, cols)
        err = np.abs(W - Wo).max()
        say(f"linear init {rows}x{cols}: max|dW| = {err:.2e}")
        assert err <= 1e-3 * np.sqrt(lam_o[0])
        m.close()


def test_single_sample_initialises_every_unit_at_it():
    X = np.linspace(-1.0, 2.0, 24, dtype=np.float32).reshape(1, 24)
    lam, mean, V = _gpu_pca(X)
    assert lam[0] == 0.0 and lam[1] == 0.0
    m = som.Map(3, 4, 24, seed=2)
    m.init_linear(dev(X))
    W = m.weights.cpu().numpy()
    assert np.allclose(W, np.repeat(X, 12, axis=0), atol=1e-6)
    m.close()
