"""Label recovery by spectral embedding and K-means (Appendix D) against the fp64 oracle.

The oracle runs on the GPU's own factor (downloaded after the iterations) with
the same seed rows, so the comparison isolates the label step: the labels and
the number of Lloyd passes must be identical.
"""
import numpy as np
import pytest

from gpu_util import host, log, make_ctx
from oracle import kmeans
from oracle import labels as olab
from oracle import nlr as onlr
from synth import gaussian_mixture, make_workload, standard_normal_factor

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_36074_amd import nlr
    nlr.load_library()


def _check(ctx, K, seeds, truth=None, max_iter=100):
    lab_gpu, passes = ctx.labels_spectral(K, seeds, max_iter)
    lab_gpu = lab_gpu.cpu().numpy()
    lab_ref, passes_ref = olab.spectral_labels(host(ctx.U), K, seeds, max_iter)
    mism = int((lab_gpu != lab_ref).sum())
    log(f"  passes gpu {passes} oracle {passes_ref}; mismatches {mism}")
    assert passes == passes_ref
    assert mism == 0
    if truth is not None:
        ari = kmeans.adjusted_rand_index(lab_gpu, truth)
        log(f"  ARI vs truth {ari:.6f}")
        return ari
    return None


def test_labels_spectral_tiny_converged():
    X, Z, truth, wl = make_workload("tiny")
    ctx = make_ctx(X, Z.astype(np.float64), wl.K, onlr.default_step_size(wl.K), T_min=wl.T)
    ctx.run(wl.T)
    seeds = [int(np.flatnonzero(truth == k)[0]) for k in range(wl.K)]
    _check(ctx, wl.K, seeds, truth)


def test_labels_spectral_exact_recovery_factor():
    """U = H, the normalised membership matrix of the true partition (exact recovery, Appendix D):
    the labels are that partition."""
    X, Z, truth, wl = make_workload("tiny")
    H = kmeans.membership(truth.astype(np.int64), wl.K)  # in Omega: H >= 0, ||H||_F^2 = K
    ctx = make_ctx(X, H, wl.K, onlr.default_step_size(wl.K), flags=1)  # NLR_INIT_U_IN_OMEGA
    seeds = [int(np.flatnonzero(truth == k)[0]) for k in range(wl.K)]
    lab, passes = ctx.labels_spectral(wl.K, seeds)
    assert kmeans.same_partition(lab.cpu().numpy(), truth)


def test_labels_spectral_random_seeds_and_r_above_K():
    """r = 8 > K = 4 (the paper's r > K setting) and seed rows drawn at random."""
    X, truth, _ = gaussian_mixture(3000, 16, 4, 25.0, seed=9)
    Z = standard_normal_factor(3000, 8, seed=10).astype(np.float64)
    ctx = make_ctx(X, Z, 4, onlr.default_step_size(4), T_min=150)
    ctx.run(150)
    rng = np.random.default_rng(11)
    seeds = rng.choice(3000, size=4, replace=False).tolist()
    _check(ctx, 4, seeds)


def test_labels_spectral_gmm1m():
    X, Z, truth, wl = make_workload("gmm1m")
    ctx = make_ctx(X, Z.astype(np.float64), wl.K, onlr.default_step_size(wl.K), T_min=30)
    ctx.run(30)
    rng = np.random.default_rng(12)
    seeds = rng.choice(wl.n, size=wl.K, replace=False).tolist()
    _check(ctx, wl.K, seeds)


def test_labels_spectral_max_iter_and_split_path():
    X, Z, truth, wl = make_workload("tiny")
    ctx = make_ctx(X, Z.astype(np.float64), wl.K, onlr.default_step_size(wl.K), T_min=20, flags=8)
    ctx.run(20)
    seeds = [0, 1, 2, 3]
    _check(ctx, wl.K, seeds, max_iter=2)
    _check(ctx, wl.K, seeds, max_iter=100)


def test_labels_spectral_degenerate_and_errors():
    from paper_2609_36074_amd import nlr
    X, _, _ = gaussian_mixture(500, 8, 4, 16.0, seed=13)
    Z = standard_normal_factor(500, 4, seed=14).astype(np.float64)
    Z[:, 3] = -np.abs(Z[:, 3])  # projected start has a zero column: U^T U is singular
    ctx = make_ctx(X, Z, 4, 0.01)
    with pytest.raises(nlr.NlrError) as e:
        ctx.labels_spectral(4, [0, 1, 2, 3])
    assert e.value.status == nlr.NLR_EDEGENERATE
    with pytest.raises(nlr.NlrError) as e:
        ctx.labels_spectral(3, [0, 1, 500])  # seed row out of range
    assert e.value.status == nlr.NLR_EINVAL
    lab, passes = ctx.labels_spectral(3, [0, 1, 2])  # rank 3 is enough for K = 3
    assert passes >= 1


def _pattern_factor(n, K, r, seed):
    """A factor near a solution: the rows of a cluster share a non-negative pattern over the
    cluster's own columns, plus non-negative noise everywhere."""
    rng = np.random.default_rng(seed)
    own = np.arange(r) % K
    pattern = np.zeros((K, r))
    pattern[own, np.arange(r)] = 0.5 + rng.random(r)
    pattern /= np.linalg.norm(pattern, axis=1, keepdims=True)
    lab = rng.integers(0, K, n)
    lab[:K] = np.arange(K)
    return (pattern[lab] + 0.05 * np.abs(rng.standard_normal((n, r)))).astype(np.float32), lab


@pytest.mark.parametrize("n,r,K", [
    (1, 1, 1), (17, 2, 2), (300, 5, 3), (1000, 13, 4), (1029, 16, 16), (1111, 30, 17), (1500, 33, 15),
    (2000, 64, 33), (2049, 65, 48), (1800, 66, 64), (2500, 128, 100), (3001, 129, 65), (2600, 200, 100),
    (3100, 257, 113), (3333, 448, 128)])
def test_labels_spectral_shapes(n, r, K):
    """Edges of the 64-column Jacobi blocks, of the 16-row and 16-cluster tiles, 16-byte rows or
    not, ranks from 1 to 448: labels and pass counts identical to the oracle's."""
    U, lab = _pattern_factor(n, K, r, seed=100 + r)
    X, _, _ = gaussian_mixture(n, 4, 1, 1.0, seed=3) if n > 1 else (np.ones((1, 4), np.float32), None, None)
    ctx = make_ctx(X, U, K, 0.01, flags=4)  # NLR_INIT_X_NORMALISED: only the factor matters here
    rng = np.random.default_rng(7)
    seeds = rng.choice(n, size=K, replace=False).tolist()
    _check(ctx, K, seeds, max_iter=12)


def test_labels_spectral_long_chunks():
    """Row chunks of the cluster sums longer than the 2048 rows sorted at a time (128 chunks of
    2055 rows at r = 193): labels and pass counts identical to the oracle's."""
    n, r, K = 263_000, 193, 5
    U, _ = _pattern_factor(n, K, r, seed=11)
    X, _, _ = gaussian_mixture(n, 4, 1, 1.0, seed=3)
    ctx = make_ctx(X, U, K, 0.01, flags=4)  # NLR_INIT_X_NORMALISED: only the factor matters here
    seeds = np.random.default_rng(7).choice(n, size=K, replace=False).tolist()
    _check(ctx, K, seeds, max_iter=4)


def test_labels_spectral_equal_rows():
    """Every row of a cluster equal and two seeds in one cluster: two equal centroids, the lower
    index takes all of that cluster's rows and the other keeps its place without any."""
    n, K, r = 1200, 6, 9
    U, lab = _pattern_factor(n, K, r, seed=5)
    U = U[:K][lab]  # rows of a cluster bitwise equal
    X, _, _ = gaussian_mixture(n, 4, 1, 1.0, seed=3)
    ctx = make_ctx(X, U, K, 0.01, flags=4)
    seeds = [int(np.flatnonzero(lab == k)[0]) for k in range(K)]
    seeds[4] = int(np.flatnonzero(lab == 1)[1])  # cluster 4 has no seed, cluster 1 has two
    got, passes = ctx.labels_spectral(K, seeds)
    got = got.cpu().numpy()
    for k in (0, 1, 2, 3, 5):
        assert (got[lab == k] == k).all()
    assert len(set(got[lab == 4])) == 1 and not (got == 4).any()
    assert passes == 2


@pytest.mark.parametrize("n,r,K", [(900, 4, 4), (1200, 9, 6), (5003, 16, 16), (7000, 33, 20), (20011, 20, 20),
                                   (4000, 70, 40), (6000, 128, 100), (60000, 5, 3)])
def test_labels_spectral_two_seeds_in_one_cluster(n, r, K):
    """As above at more sizes: the mean of equal rows embeds exactly as the row itself does, so the
    two centroids stay equal and the second pass changes nothing, whatever the rounding."""
    rng = np.random.default_rng(n)
    own = np.arange(r) % K
    pattern = np.zeros((K, r))
    pattern[own, np.arange(r)] = 0.5 + rng.random(r)
    lab = rng.integers(0, K, n)
    lab[rng.random(n) < 0.3] = 0  # the rows without a seed of their own are nearest to the largest cluster
    U = pattern[lab].astype(np.float32)
    X, _, _ = gaussian_mixture(n, 4, 1, 1.0, seed=3)
    ctx = make_ctx(X, U, K, 0.01, flags=4)
    seeds = [int(np.flatnonzero(lab == k)[0]) for k in range(K)]
    seeds[K - 1] = int(np.flatnonzero(lab == 1)[1])
    got, passes = ctx.labels_spectral(K, seeds)
    got = got.cpu().numpy()
    log(f"  passes {passes}")
    assert np.array_equal(got, np.where(lab == K - 1, 0, lab))
    assert passes == 2


@pytest.mark.parametrize("m,r", [(2, 4), (2, 20), (6, 40), (2, 70), (6, 128)])
def test_labels_spectral_score_gaps(m, r):
    """Rows equally far from m of the K = r seeds but for a helper column of size eps that favours
    one of them, eps in decades from 1 to 1e-11: the differences of the scores run through the
    bounds at which the fp16 products, then the FP64 scores, decide.  The data is the same
    under every permutation of the m seeds (each row comes with its permuted ones), so the
    sign of eps alone decides in exact arithmetic; the FP64 route resolves 1e-15 of a
    score of order 1, and eps 1e-11 shifts them by some 1e-12."""
    import torch
    rows, want = [], []

    def add(row, lab, times=1):
        for _ in range(times):
            rows.append(row)
            want.append(lab)

    e = np.eye(r)
    helper = lambda k: e[m + k]
    for k in range(m):
        add(e[k] + 0.5 * helper(k), k, 4)
    for k in range(m):
        add(5.0 * helper(k), m + k, 2)
    for k in range(2 * m, r):
        add(5.0 * e[k], k, 2)
    for k in range(m):  # (correlates the helpers with the seeds; not compared)
        add(0.6 * e[k] - 0.7 * helper(k), r, 3)
    for dec in range(12):
        for f in (1.0, 2.7, 7.3):
            for sign in (1.0, -1.0):
                if f * 10.0 ** -dec > 1.0:
                    continue
                for j in range(m):
                    add(e[:m].sum(axis=0) / m + sign * f * 10.0 ** -dec * helper(j), j if sign > 0 else -1 - j)
    U, want = np.array(rows, dtype=np.float32), np.array(want)
    n = U.shape[0]
    seeds = [4 * k for k in range(m)] + [4 * m + 2 * k for k in range(r - m)]
    X, _, _ = gaussian_mixture(n, 4, 1, 1.0, seed=3)
    ctx = make_ctx(X, np.abs(U), r, 0.01, flags=4)
    ctx.U.copy_(torch.from_numpy(U))  # (with its negative entries)
    got = ctx.labels_spectral(r, seeds, max_iter=1)[0].cpu().numpy()
    for j in range(m):  # a negative helper: any of the others, which are equally near
        neg = want == -1 - j
        assert ((got[neg] != j) & (got[neg] < m)).all()
        if m == 2:
            assert (got[neg] == 1 - j).all()
    known = (want >= 0) & (want < r)
    assert np.array_equal(got[known], want[known])
