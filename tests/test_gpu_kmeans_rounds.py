"""Balanced k-means where its kernels change path: more rows than a price
workgroup gathers at once, one cluster holding more rows than fit its LDS
list, cluster counts that do not divide over the bid wavefronts or fill a
distance tile, the largest number of tiles, and the shortest-path finish with
its edge costs in LDS and in memory; features that are not finite and rows of
unequal norm.  Checked by the duality certificate (test_gpu_kmeans.py), exact
balance and Pi."""
import numpy as np
import pytest

import paper_2605_28283_amd as pp
from paper_2605_28283_amd.workloads import bf16_bits, bf16_to_f32, make_clustered_features
from test_gpu_kmeans import check_certificate, check_perm, run, step_parity

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    pp.load()
    torch.cuda.init()


# (130, 13): less than one bid workgroup's rows twice over, k = 13;
# (17408, 17): a second batch of rows in the price kernel; (1250, 250): two
# batches of clusters per bid wavefront, 16 distance tiles
@pytest.mark.parametrize("n,D,k", [(130, 64, 13), (17408, 64, 17), (1250, 128, 250)])
def test_kmeans_round_edges(n, D, k):
    F, _, init_rows = make_clustered_features(n, D, k, 31 + k)
    X = bf16_to_f32(F).astype(np.float64)
    r = run(F, k, X[init_rows], 1)
    check_perm(r, k)
    check_certificate(X, X[init_rows], r["assign"], r["prices"])


def test_kmeans_list_longer_than_lds():
    """20480 rows, of which all but a few first choose cluster 0 (the other
    centroids lie outside the cloud): its list is read from memory."""
    n, D, k = 20480, 64, 4
    F, _, init_rows = make_clustered_features(n, D, k, 41)
    X = bf16_to_f32(F).astype(np.float64)
    init = np.tile(X.mean(0), (k, 1)).astype(np.float32)
    init[1:] += 0.1 * np.eye(k - 1, D, dtype=np.float32)
    s = (init.astype(np.float64) ** 2).sum(1) - 2.0 * X @ init.T.astype(np.float64)
    assert (s.argmin(1) == 0).sum() > 8192
    r = run(F, k, init, 1)
    check_perm(r, k)
    check_certificate(X, init, r["assign"], r["prices"])


@pytest.mark.parametrize("what,iters,ok", [
    ("rows", 1, True), ("rows", 2, False), ("many rows", 1, False), ("row inf", 1, True),
    ("centroid", 1, False), ("centroid overflow", 1, False)])
def test_kmeans_values_that_are_not_finite(what, iters, ok):
    """Three rows of NaNs, or one of infinities (times the zero low parts of a
    bf16 centroid: NaNs again), still go somewhere; more of them than a cluster
    takes, a NaN centroid (the three rows' own one in the second iteration) or
    one whose norm overflows fp32 leave nothing to balance by: the call says so,
    with every row in some cluster, and the next call gives what it gave
    before."""
    import torch
    n, D, k = 256, 64, 8
    F, _, init_rows = make_clustered_features(n, D, k, 51)
    init = bf16_to_f32(F)[init_rows].copy()
    good = run(F, k, init, 1)
    bad = F.copy()
    free = np.setdiff1d(np.arange(n), init_rows)
    if what.endswith("rows"):
        bad[free[:40 if what == "many rows" else 3]] = 0x7FC0
    elif what == "row inf":
        bad[free[0], :2] = (0x7F80, 0xFF80)
    else:
        init[3] = float("nan") if what == "centroid" else 1e25
    if ok:
        check_perm(run(bad, k, init, iters), k)
    else:
        Fd = torch.from_numpy(bad.view(np.int16)).cuda()
        mu = torch.from_numpy(np.ascontiguousarray(init, np.float32)).cuda()
        ws = torch.empty(pp.prunepath_kmeans_workspace(n, D, k), dtype=torch.uint8, device="cuda")
        assign = torch.full((n,), -7, dtype=torch.int32, device="cuda")
        perm = torch.full((n,), -7, dtype=torch.int32, device="cuda")
        print("kmeans not finite: %s, iters=%d" % (what, iters), flush=True)
        with pytest.raises(pp.PrunePathError) as err:
            pp.prunepath_balanced_kmeans(Fd, n, D, k, mu, iters, assign, perm, torch.empty_like(mu),
                                         ws)
        assert err.value.status == pp.PP_ENOTCONVERGED
        torch.cuda.synchronize()
        a = assign.cpu().numpy()
        assert a.min() >= 0 and a.max() < k
    again = run(F, k, bf16_to_f32(F)[init_rows], 1)
    for key in ("assign", "perm", "centroids", "prices"):
        np.testing.assert_array_equal(good[key], again[key])


@pytest.mark.parametrize("n,D,k,centre_std,sigma", [
    (8192, 256, 64, 0.02, 0.2), (8192, 256, 64, 0.0, 0.2), (4096, 256, 32, 0.02, 0.3)])
def test_kmeans_rows_of_unequal_norm(n, D, k, centre_std, sigma):
    """Rows scaled by LogNormal(0, sigma), planted groups or none: the price
    rounds alone bring the excess down to a few rows (at most 8 in a simulation
    in fp64), as the shortest-path finish moves one row at a time.  Steps a
    sixth as large leave it 107 rows or more."""
    F, _, init_rows = make_clustered_features(n, D, k, 61, centre_std=centre_std)
    scale = np.random.default_rng(62).lognormal(0.0, sigma, (n, 1)).astype(np.float32)
    F = bf16_bits(bf16_to_f32(F) * scale)
    X = bf16_to_f32(F).astype(np.float64)
    r = run(F, k, X[init_rows], 1)
    assert r["rounds"][0] <= 128 + 32
    check_perm(r, k)
    check_certificate(X, X[init_rows], r["assign"], r["prices"])


# edge costs in LDS up to 126 clusters, in memory from 127 on; 160, 250, 256:
# the second half of an edge row's minima
@pytest.mark.parametrize("n,D,k", [(1008, 64, 126), (1016, 64, 127), (960, 64, 160),
                                   (1250, 128, 250), (768, 64, 256)])
def test_kmeans_finish_with_many_clusters(n, D, k):
    """Well-separated groups of which some hold several initial rows: the price
    rounds leave 17 rows or more (simulated in fp64) to the shortest-path
    finish, whose result is the exact optimum."""
    from oracle import kmeans
    F, group, init_rows = make_clustered_features(n, D, k, 12, centre_std=0.05, noise_std=0.005)
    X = bf16_to_f32(F).astype(np.float64)
    init = X[init_rows]
    r = run(F, k, init, 1)
    assert r["rounds"][0] > 128
    check_perm(r, k)
    step_parity(kmeans, X, init, r, k)
    check_certificate(X, init, r["assign"], r["prices"])
