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
