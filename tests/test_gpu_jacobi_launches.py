"""Rank-deficient heads, which the Jacobi launches solve: with as many sweep logs as their rows leave room for
(two, three and four, where a launch's last replay is left to the next, five, and more than there are sweeps),
and more blocks than the device holds at once."""
import numpy as np
import pytest

from oracle import loki_oracle as O
from tests.test_gpu_calibrate import calibration_keys, fit, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hkv,N", [(2, 100), (2, 1025), (2, 2049), (2, 3073), (2, 9000), (1, 33000), (70, 200), (300, 60)])
def test_rank_deficient_heads(Hkv, N):
    say(f"case Hkv {Hkv} N {N}")
    keys = calibration_keys(300 + N, Hkv, N, "bf16")
    keys[:, :, 96:] = keys[:, :, :32]
    if Hkv > 1:
        keys[Hkv // 2, :, 20:] = 0.0
    P, lam, _ = fit(keys, "bf16")
    for h in sorted({0, Hkv // 2, Hkv - 1}):
        lam_o, _ = O.pca_basis(keys[h])
        cov = np.cov(keys[h].astype(np.float64), rowvar=False)
        # fp32 output of an orthonormal basis: 128 products of entries rounded to 2^-25 each; the Gram matrix is
        # accumulated in fp32 over at most a few thousand rows
        assert np.max(np.abs(P[h].T @ P[h] - np.eye(128))) < 1e-6
        assert np.all(np.diff(lam[h]) <= 0) and np.max(np.abs(lam[h] - lam_o)) < 5e-6 * lam_o[0]
        assert np.linalg.norm(P[h] @ np.diag(lam[h]) @ P[h].T - cov) < 2e-5 * np.linalg.norm(cov)
