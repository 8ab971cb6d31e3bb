"""GPU Nystrom approximation (Sec. 5, Alg. 2) against the FP64 oracle
(oracle.nystrom), with the paper's pseudo-inverse tolerance 1e-12 (Sec. 6.2) on
both sides.  B = A Omega and C = Omega^T B come from the product kernels (FP32);
the core pseudo-inverse (block Jacobi, FP64) and the reconstruction (FP64) are
library kernels too.

Bounds:
* core pseudo-inverse on a known spectrum (C = U diag(lambda) U^T, FP64 input):
  ||Cp - U diag(mu) U^T||_F <= 64 Rp u kappa ||U diag(mu) U^T||_F, u = 2^-53,
  kappa = max|lambda| / (smallest kept |lambda|) (first-order perturbation of
  the inverse; the oracle meets the same bound in the CPU suite);
* end to end, the FP32 gap: with eps the larger relative Frobenius error of the
  device B and C against the oracle's FP64 B and C, and kappa = cond(C), the
  first-order change of B C^+ B^T is at most sqrt(r) eps (2 sqrt(kappa) + kappa)
  ||A||_2 <= sqrt(r) eps (2 sqrt(kappa) + kappa) ||A||_F (writing B = A^(1/2) G,
  C = G^T G: ||B C^-1|| <= ||A^(1/2)|| / sigma_min(G)); the device's relative
  error and its reconstructed rows stay within that distance of the oracle's;
* rank-deficient core (linear kernel of rank-40 data, r = 64): cond(C) is
  unbounded and the bound above is void; the FP32 floor is stated instead:
  relative error <= r sqrt(n) 2^-24 (FP32 rounding of A, B and C amplified by
  at most the sketch width and the row length), against the oracle's <= 1e-5.
"""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2603_20966_amd as sk
import paper_2603_20966_amd.nystrom as ny
from oracle.nystrom import core_pinv as oracle_core_pinv
from oracle.nystrom import nystrom as oracle_nystrom
from sketch_inputs import kernel_matrix

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
U64 = 2.0 ** -53
TOL = 1e-12


def known_spectrum(r, seed, lam):
    rng = np.random.default_rng(seed)
    U, _ = np.linalg.qr(rng.standard_normal((r, r)))
    C = (U * lam) @ U.T
    C = 0.5 * (C + C.T)
    cut = TOL * np.abs(lam).max()
    mu = np.where(np.abs(lam) > cut, 1.0 / np.where(lam == 0, 1.0, lam), 0.0)
    return C, (U * mu) @ U.T


@pytest.mark.parametrize("r", [1, 2, 5, 16, 31, 32, 33, 64, 100, 256])
def test_core_pinv_known_spectrum(r):
    lam = np.logspace(0, -6, r) * (1.0 + 0.1 * np.arange(r) / max(r, 1))
    if r >= 5:
        lam[1] = -0.3                       # indefinite input: kept with its sign
        lam[-1] = 0.0                       # exact null direction
        lam[-2] = 0.5 * TOL * np.abs(lam).max()    # below the cut: dropped
    C, want = known_spectrum(r, 100 + r, lam)
    Cp, info, eig = sk.sketch_core_pinv(torch.from_numpy(C).to(DEV), TOL, max_sweeps=30,
                                        eigvals=True)
    sweeps, conv = info.cpu().tolist()
    assert conv == 1 and 1 <= sweeps <= 16, (sweeps, conv)
    got = Cp.cpu().numpy()
    Rp = (r + 31) // 32 * 32
    kept = np.abs(lam) > TOL * np.abs(lam).max()
    kappa = np.abs(lam).max() / np.abs(lam[kept]).min()
    bound = 64 * Rp * U64 * kappa * np.linalg.norm(want)
    assert np.linalg.norm(got - want) <= bound, (np.linalg.norm(got - want), bound)
    assert np.array_equal(got, got.T)                       # exactly symmetric
    ref = oracle_core_pinv(C, TOL)
    assert np.linalg.norm(got - ref) <= 2 * bound
    e = np.sort(eig.cpu().numpy())
    assert np.abs(e - np.sort(lam)).max() <= 8 * Rp * U64 * np.linalg.norm(C) * 4


def test_core_pinv_fp32_input_large_r():
    """FP32 core (as sketch_gen_tmatmul returns it) at r = 1024, the widest sketch: the
    device inverts the symmetric part of the FP32 values, compared with the oracle on
    the same values."""
    r = 1024
    lam = np.logspace(0, -4, r)
    C, _ = known_spectrum(r, 7, lam)
    C32 = C.astype(np.float32)
    Cp, info = sk.sketch_core_pinv(torch.from_numpy(C32).to(DEV), TOL, max_sweeps=30)
    sweeps, conv = info.cpu().tolist()
    assert conv == 1, sweeps
    ref = oracle_core_pinv(C32.astype(np.float64), TOL)
    kappa = 1e4 * 1.05          # cond of the FP32 matrix: lambda perturbed by ~r u32
    assert np.linalg.norm(Cp.cpu().numpy() - ref) <= 64 * r * U64 * kappa * np.linalg.norm(ref)


def test_core_pinv_exact_cases():
    """A diagonal core needs no rotation: Cp = diag(1 / lambda) bitwise (IEEE division),
    with eigenvalues at or below the cut set to zero; the zero core gives zero."""
    r = 40
    lam = np.linspace(3.0, 0.1, r)
    lam[7] = 0.0
    lam[9] = 1e-13
    lam[11] = -2.5
    C = np.diag(lam)
    Cp, info = sk.sketch_core_pinv(torch.from_numpy(C).to(DEV), TOL)
    assert info.cpu().tolist() == [1, 1]
    want = np.diag(np.where(np.abs(lam) > TOL * 3.0, 1.0 / np.where(lam == 0, 1, lam), 0.0))
    assert np.array_equal(Cp.cpu().numpy(), want)
    Z = torch.zeros((33, 33), dtype=torch.float32, device=DEV)
    Cp0, info0 = sk.sketch_core_pinv(Z, TOL)
    assert info0.cpu().tolist()[1] == 1 and not Cp0.cpu().numpy().any()
    # a non-symmetric input: only its symmetric part is inverted
    rng = np.random.default_rng(3)
    M = np.diag(lam) + np.triu(rng.standard_normal((r, r)), 1) * 1e-3
    Cs, _ = sk.sketch_core_pinv(torch.from_numpy(M).to(DEV), TOL)
    Ct, _ = sk.sketch_core_pinv(torch.from_numpy(M.T.copy()).to(DEV), TOL)
    assert torch.equal(Cs, Ct)


def _device_factors(A, r, seed):
    Ad = torch.from_numpy(A).to(DEV)
    B, C, Cp = ny.nystrom(Ad, r, seed)          # paper's tolerance, 1e-12
    return Ad, B, C, Cp


@pytest.mark.parametrize("r", [16, 64])
def test_rbf_kernel_within_fp32_gap_of_oracle(r):
    A = kernel_matrix("rbf", 2000, seed=2, latent=8, dim=64)
    Ad, B, C, Cp = _device_factors(A, r, 9)
    Bo, Co, At_ref, err_ref = oracle_nystrom(A, r, 9, tol=TOL)
    eps = max(oracle.rel_fro(B.double().cpu().numpy(), Bo),
              oracle.rel_fro(C.double().cpu().numpy(), Co))
    lam = np.linalg.eigvalsh(0.5 * (Co + Co.T))
    kappa = lam.max() / lam.min()
    assert lam.min() > 0 and kappa < 1e6
    gap = math.sqrt(r) * eps * (2 * math.sqrt(kappa) + kappa)
    err = ny.relative_error(Ad, B, Cp)
    assert abs(err - err_ref) <= gap, (err, err_ref, gap)
    rows = ny.reconstruct_rows(B, Cp, slice(0, 64)).cpu().numpy()
    assert np.linalg.norm(rows - At_ref[:64]) <= gap * np.linalg.norm(A.astype(np.float64))
    # the Nystrom approximation never exceeds A: A - A~ is PSD (up to rounding)
    Atd = ny.reconstruct_rows(B, Cp, slice(0, 2000)).cpu().numpy()
    lam_min = np.linalg.eigvalsh(A.astype(np.float64) - 0.5 * (Atd + Atd.T)).min()
    assert lam_min >= -1e-4 * np.abs(A).max()


def test_low_rank_linear_kernel_fp32_floor():
    n, r = 2000, 64
    A = kernel_matrix("linear", n, seed=1, latent=40)
    Ad, B, C, Cp = _device_factors(A, r, 5)
    _, _, _, err_ref = oracle_nystrom(A, r, 5, tol=TOL)
    assert err_ref <= 1e-5
    err = ny.relative_error(Ad, B, Cp)
    assert err <= r * math.sqrt(n) * 2.0 ** -24, err


def test_reconstruction_kernels_match_fp64_formula():
    """sketch_nystrom_error and sketch_nystrom_rows against the FP64 formula evaluated on
    the host from the same device factors (B, Cp): only the summation order differs."""
    n, r = 1500, 40
    A = kernel_matrix("rbf", n, seed=4, latent=6, dim=32)
    Ad, B, C, Cp = _device_factors(A, r, 21)
    Bh = B.double().cpu().numpy()
    Cph = Cp.cpu().numpy()
    At = Bh @ Cph @ Bh.T
    A64 = A.astype(np.float64)
    sums = sk.sketch_nystrom_error(Ad, B, Cp).cpu().numpy()
    se, sa = ((A64 - At) ** 2).sum(), (A64 ** 2).sum()
    assert abs(sums[1] - sa) <= 1e-12 * sa
    assert abs(sums[0] - se) <= 1e-6 * se
    assert abs(sums[2] - math.sqrt(se / sa)) <= 1e-6 * math.sqrt(se / sa)
    for row0, mr in ((0, 1), (37, 100), (n - 70, 70)):
        rows = sk.sketch_nystrom_rows(B, Cp, row0, mr).cpu().numpy()
        assert np.abs(rows - At[row0:row0 + mr]).max() <= 1e-12 * np.abs(At).max()


@pytest.mark.parametrize("n,r", [(1, 1), (63, 5), (127, 16), (128, 17), (129, 33), (300, 100)])
@pytest.mark.parametrize("symmetric", [True, False])
def test_reconstruction_tiles_at_their_edges(n, r, symmetric):
    """Tiles of 128 x 128 with 16 contraction values at a time, and their mirror images for a
    symmetric C^+ (a C^+ that is not takes every tile), at remainders of each.  Only the
    summation order differs from the host's FP64 formula: r-term sums of products and n^2-term
    sums of squares, within 8 (r + 64) and 8 n units of FP64 rounding of their terms' size."""
    rng = np.random.default_rng(n + r)
    A = rng.standard_normal((n, n)).astype(np.float32)       # no symmetry in A itself
    B = rng.standard_normal((n, r)).astype(np.float32)
    Cp = rng.standard_normal((r, r))
    if symmetric:
        Cp = Cp + Cp.T
    Ad, Bd, Cd = (torch.from_numpy(x).to(DEV) for x in (A, B, Cp))
    B64 = B.astype(np.float64)
    At = B64 @ Cp.T @ B64.T
    size = np.abs(B64) @ np.abs(Cp.T) @ np.abs(B64.T)
    rows = sk.sketch_nystrom_rows(Bd, Cd, n // 3, n - n // 3).cpu().numpy()
    assert (np.abs(rows - At[n // 3:]) <= 8 * (r + 64) * U64 * size[n // 3:]).all()
    D = A.astype(np.float64) - At
    se, sa = (D ** 2).sum(), (A.astype(np.float64) ** 2).sum()
    got = sk.sketch_nystrom_error(Ad, Bd, Cd).cpu().numpy()
    slack = 8 * n * U64 * se + 16 * (r + 64) * U64 * (np.abs(D) * size).sum()
    assert abs(got[0] - se) <= slack and abs(got[1] - sa) <= 8 * n * U64 * sa
    assert abs(got[2] - math.sqrt(se / sa)) <= (slack / se + 16 * n * U64) * math.sqrt(se / sa)


@pytest.mark.parametrize("r", [1, 5, 31, 32, 33, 64, 65, 100, 256, 500])
@pytest.mark.parametrize("kind", ["positive", "indefinite", "singular", "below_cut"])
def test_core_pinv_inverse_or_sweeps(r, kind):
    """Without the eigenvalues asked for, a core none of whose eigenvalues is cut is inverted
    directly (0 sweeps); any other takes the Jacobi sweeps.  Both within the bound of the
    known-spectrum test, exactly symmetric, and the first equal to the spectral formula that a
    call with eigenvalues uses to within twice that bound."""
    lam = np.logspace(0, -4, r) * (1.0 + 0.1 * np.arange(r) / r)
    if kind == "indefinite":
        lam[::3] *= -1.0
    if kind == "singular":
        lam[-1] = 0.0
    if kind == "below_cut":
        lam[-1] = 0.4 * TOL * np.abs(lam).max() if r > 1 else lam[-1]
    C, want = known_spectrum(r, 300 + r, lam)
    Cd = torch.from_numpy(C).to(DEV)
    out = torch.full((r, r + 3), 7.0, dtype=torch.float64, device=DEV)
    Cp, info = sk.sketch_core_pinv(Cd, TOL, max_sweeps=30, Cp=out[:, :r])
    sweeps, conv = info.cpu().tolist()
    assert conv == 1
    if kind == "positive":
        assert sweeps == 0
    if kind in ("singular", "below_cut") and r > 1:
        assert sweeps >= 1
    got = Cp.cpu().numpy()
    assert (out[:, r:] == 7.0).all()
    Rp = (r + 31) // 32 * 32
    kept = np.abs(lam) > TOL * np.abs(lam).max()
    kappa = np.abs(lam).max() / np.abs(lam[kept]).min() if kept.any() else 1.0
    bound = 64 * Rp * U64 * kappa * np.linalg.norm(want)
    assert np.linalg.norm(got - want) <= bound
    assert np.array_equal(got, got.T)
    Ce, _, _ = sk.sketch_core_pinv(Cd, TOL, max_sweeps=30, eigvals=True)
    assert np.linalg.norm(got - Ce.cpu().numpy()) <= 2 * bound


def test_core_pinv_inverse_special_cores():
    """A diagonal core inverts to diag(1 / lambda) bitwise; tol = 1 cuts every eigenvalue but
    none is kept by the inverse path; a core with a zero pivot and a NaN take the sweeps."""
    lam = np.linspace(3.0, -2.9, 40)
    Cp, info = sk.sketch_core_pinv(torch.from_numpy(np.diag(lam)).to(DEV), TOL)
    assert info.cpu().tolist() == [0, 1]
    assert np.array_equal(Cp.cpu().numpy(), np.diag(1.0 / lam))
    C1, _ = sk.sketch_core_pinv(torch.from_numpy(np.diag(lam)).to(DEV), 1.0)
    assert not C1.cpu().numpy().any()
    P = np.array([[0.0, 1.0], [1.0, 0.0]])
    Cp, info = sk.sketch_core_pinv(torch.from_numpy(P).to(DEV), TOL)
    assert info.cpu().tolist()[0] >= 1
    assert np.abs(Cp.cpu().numpy() - P).max() <= 64 * 32 * U64


@pytest.mark.parametrize("n,r", [(3001, 64), (2900, 100)])
def test_mirrored_error_tiles(n, r):
    """Sizes whose symmetric tiles save a round of tiles (two to a compute unit): the sums of a
    bitwise symmetric C^+ against the FP64 formula, and against those of a C^+ that is not (one
    entry off by one unit), within the rounding of FP64 sums."""
    g = torch.Generator(device=DEV).manual_seed(n)
    A = torch.randn((n, (n + 3) // 4 * 4), generator=g, device=DEV)[:, :n]
    B = torch.randn((n, (r + 3) // 4 * 4), generator=g, device=DEV)[:, :r]
    Cp = torch.randn((r, r), generator=g, device=DEV, dtype=torch.float64)
    Cp = Cp + Cp.t()
    got = sk.sketch_nystrom_error(A, B, Cp).cpu().numpy()
    W = B.double() @ Cp
    D = A.double() - W @ B.double().t().contiguous()
    want = np.array([float((D * D).sum()), float((A.double() ** 2).sum())])
    assert np.abs(got[:2] / want - 1).max() <= 1e-11
    Cu = Cp.clone()
    Cu[0, 1] = torch.nextafter(Cu[0, 1], Cu[0, 1] + 1)
    other = sk.sketch_nystrom_error(A, B, Cu).cpu().numpy()
    assert np.abs(got / other - 1).max() <= 1e-11


@pytest.mark.parametrize("tol", [1e-12, 1e-6, 1e-3, 0.05])
@pytest.mark.parametrize("side", [1 - 1e-3, 1 + 1e-3])
def test_core_pinv_around_the_cut(tol, side):
    """The smallest eigenvalue just below or above tol times the largest: cut or kept, whichever
    way C^+ is formed."""
    r = 40
    lam = np.geomspace(1.0, max(10 * tol, 0.1), r)
    lam[-1] = side * tol
    Q, _ = np.linalg.qr(np.random.default_rng(7).standard_normal((r, r)))
    C = (Q * lam) @ Q.T
    Cp, info = sk.sketch_core_pinv(torch.from_numpy(0.5 * (C + C.T)).to(DEV), tol, max_sweeps=30)
    assert info.cpu().tolist()[1] == 1
    mu = np.where(lam > tol, 1.0 / lam, 0.0)
    want = (Q * mu) @ Q.T
    kappa = 1.0 / lam[lam > tol].min()
    assert np.linalg.norm(Cp.cpu().numpy() - want) <= 64 * 64 * U64 * kappa * np.linalg.norm(want)


def test_core_pinv_certificate_counts_its_rounding():
    """With a condition number whose rounding alone could hide a singular core the sweeps run,
    also at tol = 0 (a diagonal core's computed residual is exactly zero)."""
    lam = np.array([1.0, 2.0 ** -60])
    Cp, info = sk.sketch_core_pinv(torch.from_numpy(np.diag(lam)).to(DEV), 0.0)
    assert info.cpu().tolist()[0] >= 1
    assert np.array_equal(Cp.cpu().numpy(), np.diag(1.0 / lam))


def test_sweeps_beside_other_work():
    """The one-launch sweeps hand tiles from workgroup to workgroup: the same bits alone and with
    products running on a second stream, and on two streams at once."""
    cores = []
    for r in (40, 100, 256):
        F = torch.from_numpy(np.random.default_rng(r).standard_normal((r, r // 2))).to(DEV)
        cores.append(F @ F.t().contiguous())                # half the eigenvalues are cut
    A = torch.randn((8192, 8192), device=DEV)
    ws = [[torch.empty(int(sk.lib().sketch_core_pinv_workspace(C.shape[0])), dtype=torch.uint8, device=DEV)
           for C in cores] for _ in range(2)]
    alone = [sk.sketch_core_pinv(C, max_sweeps=30) for C in cores]
    torch.cuda.synchronize()
    assert all(int(info[0]) >= 1 and int(info[1]) == 1 for _, info in alone)
    s1, s2, s3 = (torch.cuda.Stream() for _ in range(3))
    outs = []
    Y = torch.empty((8192, 64), device=DEV)
    wp = torch.empty(int(sk.sketch_workspace_size(0, 0, 8192, 8192, 64, 1)), dtype=torch.uint8, device=DEV)
    torch.cuda.synchronize()
    for i in range(3):
        with torch.cuda.stream(s3):
            for _ in range(20):
                sk.sketch_gen_matmul(A, 3, 64, Y=Y, workspace=wp)
        for s, w in ((s1, ws[0]), (s2, ws[1])):
            with torch.cuda.stream(s):
                outs.append([sk.sketch_core_pinv(C, max_sweeps=30, workspace=x) for C, x in zip(cores, w)])
    torch.cuda.synchronize()
    for got in outs:
        for (Cp, info), (C0, i0) in zip(got, alone):
            assert torch.equal(Cp, C0) and torch.equal(info, i0)
