"""Principal components and training targets at the edges of their kernels'
tiles: Gram tiles of 32 and 64 snapshots in 16 x 16 blocks, stages of 32
elements, the Lanczos iteration on the host and, from 128 snapshots on, on the
device, combinations in blocks of 32 rows and 128 elements, fields four at a
time; targets' rows reaching over several steps."""
import numpy as np
import pytest

import workloads as W
from oracle import cnn as ocnn
from oracle import pca

pytestmark = pytest.mark.gpu


def _snapshots(seed, D, M, r):
    """Rank r with singular values 10 to 1 and a tail of 1e-3."""
    rng = np.random.default_rng(seed)
    U, _ = np.linalg.qr(W.random_complex(rng, (D, r)))
    V, _ = np.linalg.qr(W.random_complex(rng, (M, r)))
    S = U @ np.diag(np.geomspace(10.0, 1.0, r)) @ V.conj().T
    return (S + 1e-3 / np.sqrt(D) * W.random_complex(rng, (D, M))).astype(np.complex64)


@pytest.mark.parametrize("D,M,k", [
    (33, 1, 1), (700, 31, 4), (1025, 32, 5), (999, 33, 8), (640, 48, 9), (641, 49, 16),
    (2048, 64, 17), (3000, 65, 20), (1500, 127, 24), (1501, 128, 25), (4100, 129, 3),
    (2500, 300, 30)])
def test_pca_at_tile_edges(D, M, k):
    """Singular values: FP64 sums of exact products, so an error of about
    D 2^-53 of the largest squared, (10 / 1)^2 of the smallest's.  The basis is
    stored in complex64: each vector is off by 2^-24 of its size, twice."""
    import torch
    from paper_1902_00090_amd import pca_build
    S = _snapshots(D * 1000 + M, D, M, min(k, M))
    U, sg = pca_build(torch.tensor(S.T.copy(), device="cuda"), k)
    Uo, so = pca.pca_basis(S.astype(np.complex128), k)
    np.testing.assert_allclose(sg, so, rtol=max(1e-11, 100 * D * 2.0 ** -53))
    U = U.cpu().numpy().T.astype(np.complex128)
    assert np.abs(U.conj().T @ U - np.eye(k)).max() <= 8 * 2.0 ** -24
    # the span, where the spectrum has a gap (factor 1000 after value k)
    assert np.linalg.norm(U - Uo @ (Uo.conj().T @ U), axis=0).max() <= 1e-6 + 4 * 2.0 ** -24


def test_pca_many_snapshots_of_low_rank():
    """Fewer directions than vectors asked for: an error (rounding decides which of
    the two checks sees it), as with few snapshots;
    not finite: another."""
    import torch
    from paper_1902_00090_amd import DDError, pca_build
    S = np.zeros((200, 500), np.complex64)
    S[:, 0] = 1.0
    with pytest.raises(DDError, match="rank < k|not positive definite"):
        pca_build(torch.tensor(S, device="cuda"), 4)
    S[150, 3] = np.nan
    with pytest.raises(DDError, match="non-finite"):
        pca_build(torch.tensor(S, device="cuda"), 1)


@pytest.mark.parametrize("S,D,window,k", [(1, 40, 3, 1), (2, 300, 0, 1), (5, 257, 1, 3),
                                          (9, 1000, 4, 5), (12, 511, 20, 9), (17, 300, 8, 13),
                                          (32, 513, 8, 12)])
def test_targets_at_tile_edges(S, D, window, k):
    """Targets are phase-free; their coefficients are FP64 and the result is
    rounded to complex64.  Fields with singular values within a factor of 30, so
    that a window's problem is off by less than 1e-10."""
    import torch
    from paper_1902_00090_amd import local_pca_targets
    rng = np.random.default_rng(S * 100 + D)
    Q, _ = np.linalg.qr(W.random_complex(rng, (D, S)))
    F = (Q * np.geomspace(1.0, 0.1, S)) @ W.random_complex(rng, (S, S))
    F = (F / np.linalg.norm(F, axis=0)).T.astype(np.complex64)
    T = local_pca_targets(torch.tensor(F.copy(), device="cuda"), window, k).cpu().numpy()
    F = F.astype(np.complex128)
    want = ocnn.local_pca_targets(F / np.linalg.norm(F, axis=1, keepdims=True), window, k)
    scale = np.abs(want).max()
    assert np.abs(T - want).max() <= (2.0 ** -24 + 1e-7) * scale


@pytest.mark.parametrize("S,window,k", [(2, 1, 2), (3, 1, 4), (31, 15, 5), (32, 31, 32), (32, 40, 20),
                                        (33, 15, 31), (33, 16, 12), (40, 12, 25)])
def test_targets_of_windows_up_to_32_fields(S, window, k):
    """Windows of 1 to 32 fields, odd and even, are solved on the device; of 33,
    on the host.  Singular values of a window within a factor of 30 or so: the
    bound of the test above."""
    import torch
    from paper_1902_00090_amd import local_pca_targets
    rng = np.random.default_rng(S * 100 + window)
    D = 400
    Q, _ = np.linalg.qr(W.random_complex(rng, (D, S)))
    R, _ = np.linalg.qr(W.random_complex(rng, (S, S)))
    F = (Q * np.geomspace(1.0, 0.1, S)) @ R
    F = (F * rng.uniform(0.1, 10.0, S)).T.astype(np.complex64)
    T = local_pca_targets(torch.tensor(F.copy(), device="cuda"), window, k).cpu().numpy()
    F = F.astype(np.complex128)
    want = ocnn.local_pca_targets(F / np.linalg.norm(F, axis=1, keepdims=True), window, k)
    assert np.abs(T - want).max() <= (2.0 ** -24 + 1e-7) * np.abs(want).max()


def test_targets_of_degenerate_and_broken_windows():
    """Equal fields (a window of rank one: its one target is the field, the others
    vanish), zero fields (all targets vanish), and a field that is not finite (no
    target is finite where it is not)."""
    import torch
    from paper_1902_00090_amd import local_pca_targets
    rng = np.random.default_rng(5)
    f = W.random_complex(rng, 300).astype(np.complex64)
    F = np.tile(f, (7, 1))
    T = local_pca_targets(torch.tensor(F, device="cuda"), 2, 4).cpu().numpy()
    unit = f.astype(np.complex128) / np.linalg.norm(f)
    assert np.abs(T[:, 0] - unit).max() <= 1e-6 and np.abs(T[:, 1:]).max() <= 1e-6
    assert not local_pca_targets(torch.zeros((5, 64), dtype=torch.complex64, device="cuda"), 1,
                                 2).cpu().numpy().any()
    F[3, 17] = np.inf
    T = local_pca_targets(torch.tensor(F, device="cuda"), 2, 4).cpu().numpy()
    assert not np.isfinite(T[:, :, 17]).any()


@pytest.mark.parametrize("M", [90, 200])
def test_basis_signs_do_not_depend_on_rounding(M):
    """The phase of a basis vector is fixed by the iteration's start, so that
    permuted elements (another order of every sum) give the permuted basis."""
    import torch
    from paper_1902_00090_amd import pca_build
    S = _snapshots(77 + M, 3000, M, 12).T.copy()
    perm = np.random.default_rng(3).permutation(3000)
    U, _ = pca_build(torch.tensor(S, device="cuda"), 12)
    P, _ = pca_build(torch.tensor(S[:, perm].copy(), device="cuda"), 12)
    assert np.abs(U.cpu().numpy()[:, perm] - P.cpu().numpy()).max() <= 1e-5


@pytest.mark.parametrize("M", [1, 5, 127, 128])
@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_snapshots_that_are_not_finite(M, bad):
    """Found in the Gram matrix, on the host below 128 snapshots and by the device's
    flag from there on; a finite call afterwards sees nothing of it."""
    import torch
    from paper_1902_00090_amd import DDError, pca_build
    rng = np.random.default_rng(M)
    S = W.random_complex(rng, (M, 70)).astype(np.complex64)
    S[M // 2, 69] = bad
    with pytest.raises(DDError, match="non-finite"):
        pca_build(torch.tensor(S, device="cuda"), 1)
    S[M // 2, 69] = 0.0
    U, sg = pca_build(torch.tensor(S, device="cuda"), 1)
    want = np.linalg.norm(S.astype(np.complex128), 2)
    np.testing.assert_allclose(sg, [want], rtol=1e-10)
