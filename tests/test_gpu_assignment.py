"""The assignment solver behind both searches at the sizes where its launch changes: one, two, four, eight and
sixteen columns per lane, matrix in LDS or not, one and several row groups per column in the parallel start, and
columns that take one or many rows.  The searches' own parity checks are the oracle comparison."""
import numpy as np
import pytest

import hinm_synth as synth
from oracle import gyro_oracle as gyro
from oracle import hinm_oracle as orc
from tests.test_gpu_icp import _check_iteration, _gpu_search
from tests.test_gpu_ocp import _gpu_cluster

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P", [2, 64, 66, 128, 130, 136, 138, 256, 258, 512, 514, 770])
@pytest.mark.parametrize("tied", [False, True])
def test_square_problems(P, tied):
    c = synth.small_case(6, 4 * P + 8, 3, 4 * P, 1, "bf16", 300 + P)
    Wb = c.weights()
    rng = np.random.default_rng(P)
    rho = rng.integers(0, 4, size=(c.M, c.K)) if tied else rng.standard_normal((c.M, c.K)) ** 2
    rho = rho.astype(np.float32)
    vec = orc.vector_index(Wb, c.dtype, c.V, c.Kv, rho)
    samples = rng.integers(0, 4, size=(1, c.T, P))
    after, obj = _gpu_search(c, Wb, rho, vec, samples)
    _check_iteration(c, Wb, rho, vec, after, samples[0], obj[0], range(c.T))


@pytest.mark.parametrize("T,n", [(1, 5), (2, 3), (5, 130), (4, 256), (48, 8), (64, 8), (65, 15), (130, 7), (300, 3), (512, 2)])
def test_columns_that_take_several_rows(T, n):
    c = synth.small_case(T * n, 40, n, 16, 1, "f16", 400 + T)
    Wb = c.weights()
    rng = np.random.default_rng(T)
    rho = (rng.standard_normal((c.M, c.K)) ** 2).astype(np.float32)
    sampled = np.stack([rng.permutation(n) for _ in range(T)]).astype(np.int32)
    order = np.arange(c.M, dtype=np.int32)
    clusters, _, obj = _gpu_cluster(c, Wb, rho, order, sampled, 1)
    assert sorted(clusters.reshape(-1).tolist()) == list(range(T * n))
    F = gyro.sampled_features(gyro.saliency_matrix(Wb, c.dtype, rho), order.reshape(T, n), sampled)
    d = gyro.kmeans_distances(F, gyro.kmeans_initial_centroids(F, n))
    label = np.empty(T * n, dtype=np.int64)
    for k in range(T):
        label[clusters[k]] = k
    assert obj[0] == gyro.kmeans_objective(d, label)
    # both totals are sums of T n binary64 terms from potentials rounded at 2^-53: 1e-9 is far above that
    assert obj[0] <= gyro.kmeans_objective(d, gyro.kmeans_balanced_assignment(d, n)) * (1 + 1e-9)


def _moves(c, before, after, sampled, P):
    """assign[i] = whose sample sits in partition i's slot now (one tile)."""
    where = {int(before[0][4 * j + sampled[j]]): j for j in range(P)}
    return np.array([where[int(after[0][4 * i + sampled[i]])] for i in range(P)])


@pytest.mark.parametrize("P", [16, 258])                    # matrix in LDS and not
@pytest.mark.parametrize("huge", ["one", "some", "all"])
def test_costs_beyond_single_precision(P, huge):
    """Scores near the largest float (columns marked never to be pruned): the costs of their partitions, sums over the
    tile's rows, are beyond it.  The other partitions are assigned as well as if those were not there."""
    V, K = 4, 4 * P
    c = synth.small_case(V, K, V, K, 1, "f16", 500)
    Wb = c.weights()
    rng = np.random.default_rng(P)
    rho = rng.random((V, K)).astype(np.float32)
    samples = rng.integers(0, 4, size=(1, 1, P))
    vec = np.arange(K, dtype=np.int32).reshape(1, K)
    if huge == "all":
        rho *= np.float32(3e38)
    else:
        for i in (3,) if huge == "one" else range(0, P, 3):
            samples[0, 0, i] = 1
            rho[:, [4 * i, 4 * i + 2, 4 * i + 3]] = 3e38
    after, obj = _gpu_search(c, Wb, rho, vec, samples)
    _check_iteration(c, Wb, rho, vec, after, samples[0], obj[0], [0])
    cost = gyro.icp_cost_fast(gyro.kept_saliency(Wb, c.dtype, rho, V, vec[0], 0), samples[0, 0])
    assert cost.max() > 1e39
    left = cost - cost.min(axis=1, keepdims=True)           # exact where it matters: huge rows are constant or all are
    got = gyro.assignment_cost(left, _moves(c, vec, after, samples[0, 0], P))
    assert got <= gyro.assignment_cost(left, gyro.icp_assign(left)) * (1 + 1e-9)


@pytest.mark.parametrize("P", [16, 258])
@pytest.mark.parametrize("feasible", [True, False])
def test_infinite_scores_are_pairs_that_cannot_be_taken(P, feasible):
    V, K = 4, 4 * P
    c = synth.small_case(V, K, V, K, 1, "f16", 501)
    Wb = c.weights()
    rng = np.random.default_rng(P)
    rho = rng.random((V, K)).astype(np.float32)
    samples = rng.integers(0, 4, size=(1, 1, P))
    vec = np.arange(K, dtype=np.int32).reshape(1, K)
    samples[0, 0, :8] = 1
    for i in range(4):                                      # two of the three that stay, in row 0: only a finite sample fits
        rho[0, [4 * i, 4 * i + 2]] = np.inf
    for j in range(4 if feasible else 0, P if not feasible else 8):
        rho[0, 4 * j + samples[0, 0, j]] = np.inf           # samples 4..7, or all of them
    after, obj = _gpu_search(c, Wb, rho, vec, samples)
    if feasible:
        assert np.isfinite(obj[0, 0])
        _check_iteration(c, Wb, rho, vec, after, samples[0], obj[0], [0])
    else:
        assert np.isinf(obj[0, 0]) and np.array_equal(after, vec)


@pytest.mark.parametrize("T,n", [(48, 8), (130, 7)])        # matrix in LDS and not
@pytest.mark.parametrize("scale", [1e-25, 1e25])
def test_distances_beyond_single_precision(T, n, scale):
    c = synth.small_case(T * n, 40, n, 16, 1, "f16", 502)
    Wb = c.weights()
    rng = np.random.default_rng(T)
    rho = (rng.standard_normal((c.M, c.K)) ** 2 * scale).astype(np.float32)
    sampled = np.stack([rng.permutation(n) for _ in range(T)]).astype(np.int32)
    order = np.arange(c.M, dtype=np.int32)
    clusters, _, obj = _gpu_cluster(c, Wb, rho, order, sampled, 1)
    F = gyro.sampled_features(gyro.saliency_matrix(Wb, c.dtype, rho), order.reshape(T, n), sampled)
    d = gyro.kmeans_distances(F, gyro.kmeans_initial_centroids(F, n))
    label = np.empty(T * n, dtype=np.int64)
    label[clusters.reshape(-1)] = np.repeat(np.arange(T), n)
    assert obj[0] == gyro.kmeans_objective(d, label)
    assert obj[0] <= gyro.kmeans_objective(d, gyro.kmeans_balanced_assignment(d, n)) * (1 + 1e-9)


@pytest.mark.parametrize("T,n", [(2, 12), (7, 12), (8, 16), (11, 13), (32, 12), (48, 2), (49, 2), (49, 5), (64, 2), (64, 6), (64, 7), (95, 4),
                                 (96, 4), (97, 3)])
def test_edges_of_the_matrix_in_registers(T, n):
    """128 rows at a time and 6 or 12 columns a lane, up to 384 rows, 96 columns and 12 rows a column; one beyond each."""
    test_columns_that_take_several_rows(T, n)


@pytest.mark.parametrize("P", [4, 48, 50, 62, 94, 96, 98, 126])
def test_edges_of_the_square_matrix_in_registers(P):
    test_square_problems(P, False)


@pytest.mark.parametrize("T,n", [(48, 8), (96, 4)])
def test_points_that_share_their_distances(T, n):
    """Every point twice: ties in every row and column, and columns asked for by twice the rows they take."""
    c = synth.small_case(T * n, 24, n, 16, 1, "f16", 503)
    Wb = c.weights()
    rng = np.random.default_rng(T)
    rho = np.repeat(rng.integers(0, 3, size=(c.M // 2, c.K)), 2, axis=0).astype(np.float32)
    sampled = np.tile(np.arange(n, dtype=np.int32), (T, 1))
    order = np.arange(c.M, dtype=np.int32)
    clusters, _, obj = _gpu_cluster(c, Wb, rho, order, sampled, 1)
    assert sorted(clusters.reshape(-1).tolist()) == list(range(T * n))
    F = gyro.sampled_features(gyro.saliency_matrix(Wb, c.dtype, rho), order.reshape(T, n), sampled)
    d = gyro.kmeans_distances(F, gyro.kmeans_initial_centroids(F, n))
    # distances of whole numbers: every total is exact
    assert obj[0] == gyro.kmeans_objective(d, gyro.kmeans_balanced_assignment(d, n))


def test_sixteen_columns_a_lane_with_costs_of_all_kinds():
    """The path loop of its own that problems of more than 512 columns have, at its largest and next to its smallest size."""
    test_square_problems(1024, False)
    test_costs_beyond_single_precision(514, "some")
    test_infinite_scores_are_pairs_that_cannot_be_taken(514, True)
    test_infinite_scores_are_pairs_that_cannot_be_taken(514, False)
