"""The SparseGPT factor's diagonal blocks and the sweep's row blocks at their edges, against
the oracle (bounds as in test_gpu_obs)."""
import numpy as np
import pytest
import torch

import oracle
from test_gpu_obs import S, U32, gpu_factor, hessian, kappa_exact, rel, run_prune, separated_weights, tol_u  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [1, 63, 65, 96, 127, 128, 129, 192, 256])
def test_factor_block_edges(S, K):  # noqa: F811
    """One block of up to 64, a pair of 65 to 128, the first recursion over pairs."""
    print(f"[obs block] K={K}", flush=True)
    H, _ = hessian(K + 7, K)
    U, _ = gpu_factor(S, H)
    ref, _ = oracle.obs_factor(H)
    U = U.cpu().numpy()
    assert np.array_equal(np.tril(U, -1), np.zeros((K, K), np.float32))
    assert rel(U, ref) <= tol_u(kappa_exact(H), K)


@pytest.mark.parametrize("K", [64, 128])
def test_bad_pivot_is_reported(S, K):  # noqa: F811
    """An indefinite matrix is refused from either half of a pair."""
    for j in (3, K - 2):
        H = np.eye(K, dtype=np.float32)
        H[j, j] = -5.0
        with pytest.raises(Exception):
            S.obs_factor(torch.from_numpy(H).cuda())


@pytest.mark.parametrize("N,K,db", [(1, 68, 64), (63, 64, 64), (64, 100, 96), (65, 132, 60), (129, 72, 68)])
def test_sweep_block_edges(S, N, K, db):  # noqa: F811
    """Row blocks of 64 and their remainders, partial column blocks, a 2:4 part that ends in one."""
    print(f"[obs sweep] N={N} K={K} db={db}", flush=True)
    H, _ = hessian(N * K, K)
    W = separated_weights(N + K, N, K, H)
    Wg, keep = run_prune(S, W, H, db)
    ref = oracle.obs_prune_24(W, H, db)
    assert np.array_equal(keep, ref["keep"])
    assert rel(Wg, ref["W"]) <= 2 * tol_u(kappa_exact(H), K) + 4 * K * U32
