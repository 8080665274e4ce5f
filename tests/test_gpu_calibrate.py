"""GPU parity of the calibration and diagnostic entry points (Section 3.1: PCA of calibration
keys, Rank@v of Eq. 2; Section 6.3: agreement of two selections) against the CPU oracle.

An eigendecomposition is unique only up to the sign of each vector (fixed here by convention)
and, numerically, up to rotations inside nearly degenerate eigenspaces, so the comparison is on
what is unique: the eigenvalues, orthonormality, the reconstruction P diag(lambda) P^T of the
oracle's covariance, and the leading subspace where the spectrum has a gap."""
import numpy as np
import pytest
import torch

from oracle import loki_oracle as O
from paper_2406_02542_amd import api, synth
from tests.parity import TORCH_DT, to_dev

pytestmark = pytest.mark.gpu


def say(msg):
    print(msg, flush=True)


def calibration_keys(seed, Hkv, N, dtype, tau=20.0, mean_scale=0.3):
    """Keys with the planted spectrum of the synthetic workloads in a per-head basis, plus a
    non-zero mean (the covariance must remove it), storage-rounded."""
    rng = np.random.default_rng(seed)
    scale = np.sqrt(synth.spectrum(128, tau) ** 2 + 0.01)
    keys = np.empty((Hkv, N, 128), np.float32)
    for h in range(Hkv):
        basis = synth.orthogonal_basis(seed, h, 128)
        c = rng.standard_normal((N, 128)) * scale[None, :]
        keys[h] = (c @ basis.T + mean_scale * rng.standard_normal(128)[None, :]).astype(np.float32)
    return synth.round_storage(keys, dtype)


def fit(keys, dtype):
    Hkv, N, _ = keys.shape
    lay = api.make_layout(1, Hkv, Hkv, 128, 32, 16, TORCH_DT[dtype])
    ws = torch.empty(api.loki_pca_workspace_bytes(lay, N), dtype=torch.uint8, device="cuda")
    P = torch.full((Hkv, 128, 128), float("nan"), device="cuda")
    lam = torch.full((Hkv, 128), float("nan"), device="cuda")
    api.loki_pca_fit(lay, to_dev(keys, dtype), N, P, lam, ws)
    torch.cuda.synchronize()
    return P.cpu().numpy().astype(np.float64), lam.cpu().numpy().astype(np.float64), (P, lam)


@pytest.mark.parametrize("dtype,Hkv,N", [("bf16", 2, 50001), ("f32", 1, 4096 + 17), ("bf16", 8, 300000)])
def test_pca_fit_matches_oracle(dtype, Hkv, N):
    keys = calibration_keys(11 + Hkv, Hkv, N, dtype)
    say(f"case dtype {dtype} Hkv {Hkv} N {N}")
    P, lam, _ = fit(keys, dtype)
    for h in range(Hkv):
        lam_o, vec_o = O.pca_basis(keys[h])
        cov_o = np.cov(keys[h].astype(np.float64), rowvar=False)
        # fp32 accumulation of the Gram matrix over runs of >= 1024 rows (fp32 keys: two bf16
        # terms, remainder x remainder dropped), fp64 from there on, fp32 output
        assert np.all(np.diff(lam[h]) <= 0)
        err = np.max(np.abs(lam[h] - lam_o)) / lam_o[0]
        orth = np.max(np.abs(P[h].T @ P[h] - np.eye(128)))
        rec = np.linalg.norm(P[h] @ np.diag(lam[h]) @ P[h].T - cov_o) / np.linalg.norm(cov_o)
        d = 16  # lambda_16 / lambda_17 = e^0.2 in the planted spectrum: a clear gap
        overlap = np.linalg.norm(vec_o[:, :d].T @ P[h][:, :d]) ** 2 / d
        say(f"   head {h}: eigenvalue err {err:.2e} (rel. to the largest), orthonormality {orth:.2e}, "
            f"reconstruction {rec:.2e}, leading-16 subspace overlap {overlap:.8f}")
        assert err < 5e-6
        assert orth < 1e-6
        assert rec < 2e-5
        assert overlap > 0.999999
        # sign convention: the largest-magnitude entry of every component is positive
        big = P[h][np.argmax(np.abs(P[h]), axis=0), np.arange(128)]
        assert np.all(big > 0)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("Hkv,N", [(1, 31), (1, 129), (3, 1153), (40, 1089), (257, 161)])
def test_covariance_at_the_edges_of_a_step(dtype, Hkv, N):
    """Rows that do not fill a 32-row step, a chunk or a round of blocks; more heads than CUs.  P diag(lambda) P^T
    against the float64 covariance: the bounds of test_pca_fit_matches_oracle (fp32 sums of at most a few
    thousand terms, remainder x remainder of fp32 keys dropped: at most 2^-18 of a term)."""
    keys = calibration_keys(5 + N, Hkv, N, dtype)
    P, lam, _ = fit(keys, dtype)
    for h in (0, Hkv // 2, Hkv - 1):
        cov = np.cov(keys[h].astype(np.float64), rowvar=False)
        rec = np.linalg.norm(P[h] @ np.diag(lam[h]) @ P[h].T - cov) / np.linalg.norm(cov)
        say(f"case {dtype} Hkv {Hkv} N {N} head {h}: reconstruction {rec:.2e}")
        assert rec < 2e-5
        assert np.max(np.abs(P[h].T @ P[h] - np.eye(128))) < 1e-6


def test_column_sums_of_fp32_keys_keep_all_their_bits():
    """One column alternates between 1 and -1, the other 127 hold x = 1 + 2^-9 - 2^-19 in each of 32 rows, so that their
    covariance is 0.  x needs 19 bits; its two bf16 terms are 1 and 2^-9, so the products the Gram pass keeps, 1 + 2^-8,
    are x^2 to 2^-27, and the sum 32 x is exact in fp32: an entry of the covariance is off by 2^-27 32 / 31 and a
    rounding, an eigenvalue by 127 times that, below 2e-6.  Sums of the two terms are 32 2^-19 too large: -5e-4."""
    keys = np.full((1, 32, 128), 1 + 2.0 ** -9 - 2.0 ** -19, np.float32)
    keys[0, :, 5] = 1 - 2.0 * (np.arange(32) % 2)
    _, lam, _ = fit(keys, "f32")
    say(f"eigenvalues {lam[0, 0]} .. {lam[0, -1]}")
    assert abs(lam[0, 0] - 32 / 31) < 2e-6
    assert np.all(np.abs(lam[0, 1:]) < 2e-6)


def test_pca_fit_then_rotate_then_decode_is_exact_attention():
    """Lemma 4.1 with the GPU's own basis: keys rotated by the fitted P, full rank and every
    row kept, give dense attention on the unrotated keys."""
    w = synth.Workload("fitchain", 1, 2, 2, 128, 900, "bf16", 128, 900, seed=12000)
    keys = calibration_keys(77, 2, 900, "bf16")
    _, _, (Pd, _) = fit(keys, "bf16")
    x = {"q": synth.make_q(w), "v": synth.make_v(w)}
    lay = api.make_layout(1, 2, 2, 128, 128, 900, torch.bfloat16)
    klo, _, v = api.alloc_cache(lay)
    v.copy_(to_dev(x["v"], "bf16"))
    K = keys[None]  # [1, Hkv, S, D]
    api.loki_rotate_keys(lay, to_dev(K, "bf16"), Pd, klo, None, 0, 900)
    ws = api.alloc_workspace(lay, 900, 128, 900, 0)
    out = torch.empty((1, 2, 128), dtype=torch.bfloat16, device="cuda")
    api.loki_decode_attn(lay, to_dev(x["q"], "bf16"), Pd, klo, None, v, 900, 128, 900, 0, ws, out)
    torch.cuda.synchronize()
    ref = O.dense_decode_batch(x["q"], K, x["v"])
    assert np.max(np.abs(out.float().cpu().numpy() - ref)) < 3e-2


def test_pca_fit_degenerate_inputs():
    """Two rows; identical rows (zero covariance): finite, orthonormal output."""
    for keys in (calibration_keys(5, 1, 2, "bf16"), np.ones((1, 100, 128), np.float32)):
        P, lam, _ = fit(keys, "bf16")
        assert np.all(np.isfinite(P)) and np.all(np.isfinite(lam))
        assert np.max(np.abs(P[0].T @ P[0] - np.eye(128))) < 1e-5
        lam_o, _ = O.pca_basis(keys[0])
        assert np.max(np.abs(lam[0] - lam_o)) <= 1e-4 * max(lam_o[0], 1e-30) + 1e-12


def test_rank_at_matches_oracle():
    rng = np.random.default_rng(3)
    spectra = np.stack([np.sort(rng.random(128))[::-1] * np.exp(-np.arange(128) / t) for t in (5.0, 20.0, 60.0, 1e6)])
    lam = torch.from_numpy(spectra.astype(np.float32)).cuda()
    for v in (50.0, 90.0, 99.0, 100.0):
        ranks = torch.zeros(4, dtype=torch.int32, device="cuda")
        api.loki_rank_at(lam, v, ranks)
        torch.cuda.synchronize()
        want = [O.rank_at(lam[i].cpu().numpy().astype(np.float64), v) for i in range(4)]
        got = ranks.cpu().tolist()
        # v = 100 sits on a rounding edge of the running sum: allow the last index either way
        for g, wv in zip(got, want):
            assert g == wv or (v == 100.0 and abs(g - wv) <= 1), (v, got, want)


def test_layer_width_matches_oracle():
    """Rank_l@v and the width policy of Appendix B.2 on spectra of 3 to 300 heads."""
    rng = np.random.default_rng(8)
    for n_heads, taus in ((3, (4.0, 30.0, 90.0)), (32, None), (300, None)):
        if taus is None:
            taus = rng.uniform(3.0, 120.0, n_heads)
        spectra = np.stack([np.sort(rng.random(128))[::-1] * np.exp(-np.arange(128) / t) for t in taus])
        lam = torch.from_numpy(spectra.astype(np.float32)).cuda()
        lam64 = lam.cpu().numpy().astype(np.float64)
        for v in (50.0, 65.0, 80.0, 90.0):
            for multiple in (1, 4, 8):
                mean = torch.full((1,), -1.0, device="cuda")
                d = torch.full((1,), -1, dtype=torch.int32, device="cuda")
                api.loki_layer_width(lam, v, multiple, mean, d)
                torch.cuda.synchronize()
                assert abs(mean.item() - O.layer_rank_at(lam64, v)) <= 1e-4
                assert d.item() == O.layer_width(lam64, v, multiple), (n_heads, v, multiple)
    d = torch.zeros(1, dtype=torch.int32, device="cuda")
    api.loki_layer_width(lam, 80.0, 8, None, d)     # the mean is optional
    torch.cuda.synchronize()
    assert d.item() == O.layer_width(lam64, 80.0, 8)
    with pytest.raises(RuntimeError):
        api.loki_layer_width(lam, 80.0, 5, None, d)  # 128 is not a multiple of 5
    with pytest.raises(RuntimeError):
        api.loki_layer_width(lam, 0.0, 8, None, d)


def test_index_jaccard_matches_oracle():
    rng = np.random.default_rng(4)
    n, k, S = 37, 500, 4000
    a = np.stack([np.sort(rng.choice(S, k, replace=False)) for _ in range(n)]).astype(np.int32)
    b = np.stack([np.sort(rng.choice(S, k, replace=False)) for _ in range(n)]).astype(np.int32)
    b[0] = a[0]                      # identical
    b[1] = np.sort((a[1] + S) % (2 * S))  # disjoint
    a[2, 400:] = -1                  # padded lists
    b[3, 123:] = -1
    out = torch.zeros(n, device="cuda")
    api.loki_index_jaccard(torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda(), out)
    torch.cuda.synchronize()
    want = np.array([O.jaccard(a[i], b[i]) for i in range(n)])
    np.testing.assert_allclose(out.cpu().numpy(), want, rtol=1e-6)
    assert out[0].item() == 1.0 and out[1].item() == 0.0


def test_loki_selection_agrees_with_exact_topk_more_as_d_grows():
    """The diagnostic of Section 6.3 on synthetic keys: Jaccard between Loki's selection at
    rank d and exact top-k (d = D) rises with d and is 1 at d = D."""
    base = synth.Workload("jac", 2, 4, 4, 128, 2048, "bf16", 128, 256, seed=13000)
    x = synth.make_inputs(base)
    q, P = to_dev(x["q"], "bf16"), torch.from_numpy(x["P"]).cuda()
    kh, vv = to_dev(x["khat"], "bf16"), to_dev(x["v"], "bf16")
    lists = {}
    for d in (16, 64, 128):
        lay = api.make_layout(2, 4, 4, 128, d, 2048, torch.bfloat16)
        ws = api.alloc_workspace(lay, 2048, d, 256, 0)
        out = torch.empty((2, 4, 128), dtype=torch.bfloat16, device="cuda")
        idx = torch.empty((2, 4, 256), dtype=torch.int32, device="cuda")
        khi = kh[..., d:].contiguous() if d < 128 else None
        api.loki_decode_attn(lay, q, P, kh[..., :d].contiguous(), khi, vv, 2048, d, 256, 0, ws, out, idx)
        lists[d] = idx
    j = {}
    for d in (16, 64, 128):
        o = torch.zeros(8, device="cuda")
        api.loki_index_jaccard(lists[d], lists[128], o)
        torch.cuda.synchronize()
        j[d] = o.mean().item()
        for i in range(8):
            assert abs(o[i].item() - O.jaccard(lists[d].view(8, 256)[i].cpu().numpy(),
                                               lists[128].view(8, 256)[i].cpu().numpy())) < 1e-6
    say(f"mean Jaccard vs exact top-k: {j}")
    assert j[16] < j[64] < j[128] == 1.0


@pytest.mark.parametrize("dtype,N", [("bf16", 3), ("f32", 127), ("bf16", 1025), ("f32", 9000)])
def test_pca_fit_mixes_regular_and_degenerate_heads(dtype, N):
    """Heads solved by the tridiagonal route next to heads whose equal eigenvalues send them to
    the Jacobi iteration: dead columns, every column twice, a steep spectrum without noise, one
    direction only; few rows (all heads rank-deficient) and many."""
    keys = calibration_keys(900 + N, 5, N, dtype)
    keys[1, :, 100:] = 0.0
    keys[2, :, 64:] = keys[2, :, :64]
    rng = np.random.default_rng(N)
    keys[3] = synth.round_storage((rng.standard_normal((N, 128)) * np.exp(-np.arange(128) / 3.0)[None, :]).astype(np.float32), dtype)
    keys[4] = synth.round_storage((rng.standard_normal((N, 1)) * np.ones((1, 128))).astype(np.float32), dtype)
    say(f"case dtype {dtype} N {N}")
    P, lam, _ = fit(keys, dtype)
    for h in range(5):
        lam_o, _ = O.pca_basis(keys[h])
        cov_o = np.cov(keys[h].astype(np.float64), rowvar=False)
        err = np.max(np.abs(lam[h] - lam_o)) / lam_o[0]
        orth = np.max(np.abs(P[h].T @ P[h] - np.eye(128)))
        rec = np.linalg.norm(P[h] @ np.diag(lam[h]) @ P[h].T - cov_o) / np.linalg.norm(cov_o)
        say(f"   head {h}: eigenvalue err {err:.2e}, orthonormality {orth:.2e}, reconstruction {rec:.2e}")
        # fp32 output of an orthonormal basis: 128 products of entries rounded to 2^-25 each
        assert orth < 1e-6
        # the bounds of test_pca_fit_matches_oracle (the Gram matrix is accumulated in fp32)
        assert np.all(np.diff(lam[h]) <= 0) and err < 5e-6 and rec < 2e-5
        # the largest entry is positive; entries of opposite sign that fp32 rounds to the same size tie
        assert np.all(P[h].max(axis=0) >= np.abs(P[h]).max(axis=0))
