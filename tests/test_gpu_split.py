"""GPU tests of the wide FP32 sketches (k > 16) where both operands are multiplied as sums of FP16
terms with a power-of-two scale per row of A (and per column of a stored Omega).

Bars (u = 2^-24).  A term pair holds an entry of A within 2^-23 |a|, or within 2^-35 of its
row's largest entry, whichever is larger; Omega's three terms are exact; the dropped
product of the two low terms is at most 2^-22 |a omega|; the sums are bounded as a chain of
2048 FP32 additions:
    |Y - Y_ref| <= 2052 u sum_j |A_ij Omega_jc| + 2^-35 max_j |A_ij| sum_j |Omega_jc| + u |Y_ref|.
Non-finite entries give what IEEE sums of FP32 products give: infinities with their sign, NaN
where both signs or a NaN meet.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2603_20966_amd as sk
from paper_2603_20966_amd import serve as sv
from sketch_inputs import normal_matrix

pytestmark = pytest.mark.gpu

U = 2.0 ** -24
DEV = "cuda:0"


def to_dev(x):
    ld = max(4, (x.shape[1] + 3) // 4 * 4)
    buf = torch.zeros((x.shape[0], ld), dtype=torch.float32, device=DEV)
    buf[:, :x.shape[1]] = torch.from_numpy(np.ascontiguousarray(x)).to(DEV)
    return buf[:, :x.shape[1]]


def cm_dev(A):
    """Column-major device copy, the leading dimension a multiple of 4."""
    return to_dev(np.ascontiguousarray(A.T)).t()


def served(Ad, seed, k):
    Y = torch.empty((Ad.shape[0], k), device=DEV)
    torch.cuda.synchronize()
    with sk.SketchServer(1 << 28, max_slots=2, max_batch=2) as srv:
        t = srv.submit(sv.make_request(A=Ad, k=k, seed=seed, Y=Y), Ad, Y)
        assert srv.wait(t, 60.0)["state"] == sv.SK_REQ_DONE
    return Y


def uneven_rows(m, n, seed):
    """N(0,1) rows under every course a row's scale can take."""
    A = normal_matrix(m, n, seed=seed).astype(np.float64)
    A[1, 700:] *= 2.0 ** 30                  # grows inside a strip
    A[2, :300] = 0.0                         # zeros first
    A[3] *= 1e-37                            # near the smallest normal numbers
    A[4] *= 1e-42                            # subnormal
    A[5] *= 1e34
    A[6] = 0.0
    A[7, 0] = 1e6                            # one large entry first, or last
    A[8, -1] = 1e6
    A[9] *= 2.0 ** (np.arange(n) // 100)     # keeps growing
    A[10] *= 2.0 ** (-(np.arange(n) // 100))
    A[11, 1:] = 0.0
    return A.astype(np.float32)


@pytest.mark.parametrize("m,n,k", [(70, 4500, 9), (70, 2049, 24), (70, 4096, 64), (530, 2100, 130), (67, 2031, 40)])
def test_uneven_rows_on_every_route(m, n, k):
    A = uneven_rows(m, n, seed=k)
    Ad = to_dev(A)
    Y = sk.sketch_gen_matmul(Ad, 3, k)
    Yh = Y.double().cpu().numpy()
    Om = np.abs(oracle.omega_block(3, 0, n, 0, k)).astype(np.float64)
    ref = oracle.gen_matmul(A, 3, 0, 0, k)
    absA = np.abs(A).astype(np.float64)
    bound = (2052 * U * (absA @ Om) + 2.0 ** -35 * absA.max(1)[:, None] * Om.sum(0)[None, :]
             + U * np.abs(ref) + 2.0 ** -149)
    assert (np.abs(Yh - ref) <= bound).all()
    assert (Yh[6] == 0).all()
    # the scale is the row's own: row blocks, the server, column-major A and its few-row kernel
    assert torch.equal(Y[2:40], sk.sketch_gen_matmul(Ad[2:40], 3, k))
    assert torch.equal(Y, served(Ad, 3, k))
    if k > 16:
        Acm = cm_dev(A)
        assert torch.equal(Y, sk.sketch_gen_matmul_cm(Acm, 3, k))
        assert torch.equal(Y[4:40], sk.sketch_gen_matmul_cm(Acm[4:40], 3, k))


@pytest.mark.parametrize("m,n", [(5, 31), (5, 32), (6, 33), (7, 63), (515, 2047), (258, 2051),
                                 (1030, 4127)])
def test_ragged_ends(m, n):
    """Columns and rows past the last whole chunk / group of four, on the row-major and the
    column-major kernels (both loading every lane unconditionally from one whole chunk on)."""
    for k in (17, 64, 129):
        A = normal_matrix(m, n, seed=m + n)
        Y = sk.sketch_gen_matmul(to_dev(A), 6, k, omega_row0=3)
        ref = oracle.gen_matmul(A, 6, 3, 0, k)
        mag = np.abs(A).astype(np.float64) @ np.abs(oracle.omega_block(6, 3, n, 0, k))
        assert (np.abs(Y.double().cpu().numpy() - ref) <= 2052 * U * mag + U * np.abs(ref)).all()
        assert torch.equal(Y, sk.sketch_gen_matmul_cm(cm_dev(A), 6, k, omega_row0=3))


@pytest.mark.parametrize("k", [40, 130])
def test_error_is_below_the_fp32_chain(k):
    """Relative error of N(0,1), positive and scaled data below that of 512 FP32 additions of
    4-term sums (measured with the FP32 matrix instruction: 7.5e-7 to 8.4e-7)."""
    n = 8192
    for A in (normal_matrix(64, n, seed=1), np.abs(normal_matrix(64, n, seed=2)),
              normal_matrix(64, n, seed=3) * np.float32(1e20)):
        for dist in ("normal", "uniform"):
            Y = sk.sketch_gen_matmul(to_dev(A), 5, k, dist=dist, y_dtype=torch.float64)
            ref = oracle.gen_matmul(A, 5, 0, 0, k, dist)
            assert oracle.rel_fro(Y.cpu().numpy(), ref) <= 7.5e-7


@pytest.mark.parametrize("k", [9, 40, 130])
def test_non_finite_rows(k):
    n = 4100
    A = normal_matrix(80, n, seed=k)
    bad = {3: [(5, np.inf)], 17: [(4099, -np.inf)], 20: [(1, np.inf), (2, np.inf)],
           33: [(7, np.nan)], 34: [(2050, np.inf), (9, np.nan)], 79: [(0, -np.inf), (2500, np.inf)]}
    clean = to_dev(A)
    B = A.copy()
    for r, es in bad.items():
        for j, v in es:
            B[r, j] = v
    with np.errstate(invalid="ignore"):
        ref = oracle.omega_block(7, 0, n, 0, k).astype(np.float64)
        want = {r: sum((np.float64(v) * ref[j] for j, v in es), np.zeros(k)) for r, es in bad.items()}
    Yc = sk.sketch_gen_matmul(clean, 7, k)
    outs = [sk.sketch_gen_matmul(to_dev(B), 7, k), served(to_dev(B), 7, k)]
    if k > 16:
        outs += [sk.sketch_gen_matmul_cm(cm_dev(B), 7, k)]
        few = sk.sketch_gen_matmul_cm(cm_dev(B)[:40], 7, k)
        assert torch.equal(torch.nan_to_num(few, 1.0, 2.0, 3.0),
                           torch.nan_to_num(outs[0][:40], 1.0, 2.0, 3.0))
    fine = [r for r in range(80) if r not in bad]
    for Y in outs:
        assert torch.equal(Y[fine], Yc[fine])
        for r in bad:
            assert np.array_equal(Y[r].double().cpu().numpy(), want[r], equal_nan=True), r


@pytest.mark.parametrize("k", [16, 40])
def test_stored_columns_of_any_size(k):
    m, n = 65, 4200
    A = normal_matrix(m, n, seed=9)
    Om = oracle.omega_block(2, 0, n, 0, k).astype(np.float64)
    Om[:, 1] *= 1e20
    Om[:, 2] *= 1e-20
    Om[:, 3] = 0.0
    Om[:, 4] *= 1e-36
    Om[2100:, 5] *= 2.0 ** 40
    Om = Om.astype(np.float32)
    Y = sk.sketch_matmul_omega(to_dev(A), torch.from_numpy(Om).to(DEV)).double().cpu().numpy()
    ref = A.astype(np.float64) @ Om.astype(np.float64)
    absA, absO = np.abs(A).astype(np.float64), np.abs(Om).astype(np.float64)
    bound = 2052 * U * (absA @ absO) + 2.0 ** -35 * absA.max(1)[:, None] * absO.sum(0) + U * np.abs(ref)
    assert (np.abs(Y - ref) <= bound).all()
    # a non-finite entry of Omega reaches its own column only
    Om2 = Om.copy()
    Om2[10, 6], Om2[4000, 7], Om2[3, 8] = np.inf, -np.inf, np.nan
    Y2 = sk.sketch_matmul_omega(to_dev(A), torch.from_numpy(Om2).to(DEV)).double().cpu().numpy()
    keep = [c for c in range(k) if c not in (6, 7, 8)]
    assert np.array_equal(Y2[:, keep], Y[:, keep])
    assert np.array_equal(Y2[:, 6], np.copysign(np.inf, A[:, 10]))
    assert np.array_equal(Y2[:, 7], -np.copysign(np.inf, A[:, 4000]))
    assert np.isnan(Y2[:, 8]).all()


@pytest.mark.parametrize("y_dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("n,k", [(300, 24), (2048, 40), (2047, 130)])
def test_non_finite_entries_add_to_y_once(n, k, y_dtype):
    """One strip and beta = 1: the old Y plus the IEEE product, on every route."""
    m = 80
    A = normal_matrix(m, n, seed=n)
    bad = {0: [(5, np.inf)], 17: [(n - 1, -np.inf)], 33: [(7, np.nan)], 40: [(2, np.inf), (9, -np.inf)]}
    B = A.copy()
    for r, es in bad.items():
        for j, v in es:
            B[r, j] = v
    Om = oracle.omega_block(7, 0, n, 0, k)
    Y0 = torch.from_numpy(normal_matrix(m, k, seed=11)).to(DEV, y_dtype)
    with np.errstate(invalid="ignore"):
        want = {r: sum((np.float64(v) * Om[j].astype(np.float64) for j, v in es), np.zeros(k))
                for r, es in bad.items()}
    fine = [r for r in range(m) if r not in bad]

    def run(f, rows=m):
        Y = Y0[:rows].clone()
        f(Y)
        return Y

    def serve(Y):
        torch.cuda.synchronize()
        Bd = to_dev(B)
        with sk.SketchServer(1 << 28, max_slots=2, max_batch=2) as srv:
            t = srv.submit(sv.make_request(A=Bd, k=k, seed=7, Y=Y, beta=1), Bd, Y)
            assert srv.wait(t, 60.0)["state"] == sv.SK_REQ_DONE

    clean = run(lambda Y: sk.sketch_gen_matmul(to_dev(A), 7, k, Y=Y, beta=1))
    Omd = torch.from_numpy(Om).to(DEV)
    outs = [run(lambda Y: sk.sketch_gen_matmul(to_dev(B), 7, k, Y=Y, beta=1)), run(serve),
            run(lambda Y: sk.sketch_gen_matmul_cm(cm_dev(B), 7, k, Y=Y, beta=1)),
            run(lambda Y: sk.sketch_gen_matmul_cm(cm_dev(B)[:44], 7, k, Y=Y, beta=1), 44),
            run(lambda Y: sk.sketch_matmul_omega(to_dev(B), Omd, Y=Y, beta=1))]
    for Y in outs:
        rows = [r for r in fine if r < Y.shape[0]]
        assert torch.equal(Y[rows], clean[rows])
        for r in bad:
            assert np.array_equal(Y[r].double().cpu().numpy(), want[r], equal_nan=True), r
    # non-finite columns of a stored Omega, met by finite and by infinite rows
    Om2 = Om.copy()
    Om2[10, 6], Om2[n - 1, 7], Om2[3, 8] = np.inf, -np.inf, np.nan
    Y = run(lambda Y: sk.sketch_matmul_omega(to_dev(B), torch.from_numpy(Om2).to(DEV), Y=Y, beta=1))
    keep = [c for c in range(k) if c not in (6, 7, 8)]
    assert torch.equal(Y[fine][:, keep], clean[fine][:, keep])
    Yh = Y.double().cpu().numpy()
    with np.errstate(invalid="ignore"):
        ref = B.astype(np.float64) @ Om2.astype(np.float64)
    for r in range(m):
        assert np.array_equal(Yh[r, 6:9], np.where(np.isnan(ref[r, 6:9]), np.nan, np.sign(ref[r, 6:9]) * np.inf),
                              equal_nan=True), r
        if r in bad:
            assert np.array_equal(Yh[r, keep], want[r][keep], equal_nan=True), r


def test_cost_of_infinite_rows():
    """A matrix with an infinity in every row is multiplied by the FP32 instruction: at 1/16 of
    the rate for two of the FP16 instruction's four products, eight times the matrix-core time
    in addition to the first pass; 16 leaves room for generation in every wave (the server)."""
    m, n, k = 4096, 8192, 64
    A = to_dev(normal_matrix(m, n, seed=1))
    B = A.clone()
    B[:, 77] = float("inf")
    Acm, Bcm = cm_dev(A.cpu().numpy()), cm_dev(B.cpu().numpy())

    def ms(f):
        times = []
        for _ in range(4):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            f()
            e1.record()
            torch.cuda.synchronize()
            times.append(e0.elapsed_time(e1))
        return min(times[1:])

    for f, x, y in [(sk.sketch_gen_matmul, A, B), (sk.sketch_gen_matmul_cm, Acm, Bcm)]:
        for kk in (24, k):
            clean, inf = ms(lambda: f(x, 3, kk)), ms(lambda: f(y, 3, kk))
            assert inf <= 16 * clean, (f.__name__, kk, clean, inf)


def selecting_omega(n, k, seed):
    """Columns that pick out few entries of a row, or span a wide range."""
    rng = np.random.default_rng(seed)
    Om = np.zeros((n, k))
    for c in range(k):
        kind = c % 6
        if kind == 0:                                    # one entry
            Om[rng.integers(0, n), c] = 1.0
        elif kind == 1:                                  # sparse signs
            Om[:, c] = rng.choice([-1.0, 0.0, 1.0], n, p=[.05, .9, .05])
        elif kind == 2:                                  # wide range
            Om[:, c] = rng.standard_normal(n) * np.exp2(-rng.integers(0, 60, n).astype(float))
        elif kind == 3:                                  # one outlier
            Om[:, c] = rng.standard_normal(n)
            Om[0, c] = 1e20
        elif kind == 4:                                  # small everywhere, or large
            Om[:, c] = rng.standard_normal(n) * (1e-12 if c % 4 else 1e5)
        else:
            Om[:, c] = rng.standard_normal(n)
    return Om.astype(np.float32)


@pytest.mark.parametrize("m,n,k", [(70, 4500, 24), (70, 2048, 64), (530, 2100, 130), (65, 40, 40)])
def test_stored_omega_that_selects_entries(m, n, k):
    """FP32 products for columns of a stored Omega that bring out single entries of rows of a
    wide range: the bound of a chain of FP32 additions, with nothing for the terms."""
    rng = np.random.default_rng(n)
    A = normal_matrix(m, n, seed=k).astype(np.float64)
    A[:m // 2] *= np.exp2(-rng.integers(0, 90, (m // 2, n)).astype(float))
    A[0, :3], A[0, 3:] = (1e12, 1.0009765, np.pi), 0.0
    A[:, 0] = np.where(np.arange(m) % 2, 0.0, A[:, 0])
    A[1, :] = np.abs(A[1, :]) * 1e-3
    A[1, n - 1] = 1e9
    A = A.astype(np.float32)
    Om = selecting_omega(n, k, seed=m)
    Om[:, 6], Om[1, 6] = 0.0, 1.0
    Om[:, 12], Om[2, 12] = 0.0, 1.0
    Y = sk.sketch_matmul_omega(to_dev(A), torch.from_numpy(Om).to(DEV), y_dtype=torch.float64).cpu().numpy()
    ref = A.astype(np.float64) @ Om.astype(np.float64)
    mag = np.abs(A).astype(np.float64) @ np.abs(Om).astype(np.float64)
    sel = [c for c in range(k) if c % 6 != 5]            # the others are like generated ones
    assert (np.abs(Y - ref) <= 2052 * U * mag + U * np.abs(ref) + 2.0 ** -140)[:, sel].all()
    assert Y[0, 6] == A[0, 1] and Y[0, 12] == A[0, 2]
    bound = 2052 * U * mag + 2.0 ** -35 * np.abs(A).max(1)[:, None] * np.abs(Om).astype(np.float64).sum(0)
    bound += 2.0 ** -49 * np.abs(A).astype(np.float64).sum(1)[:, None]
    assert (np.abs(Y - ref) <= bound + U * np.abs(ref)).all()


@pytest.mark.parametrize("n", [1, 5, 31, 2048 + 3])
@pytest.mark.parametrize("k", [17, 40, 130])
def test_narrow_strips_are_fp32_sums(n, k):
    """Strips narrower than a chunk: at most 32 FP32 roundings of the products' sum (the first
    2048 columns of the last n are zero), the same bits on every route."""
    m, w = 80, n % 2048
    A = normal_matrix(m, n, seed=n)
    A[:, :n - w] = 0.0
    Ad = to_dev(A)
    Y = sk.sketch_gen_matmul(Ad, 3, k, y_dtype=torch.float64)
    Om = oracle.omega_block(3, 0, n, 0, k)
    ref = A.astype(np.float64) @ Om.astype(np.float64)
    mag = np.abs(A).astype(np.float64) @ np.abs(Om).astype(np.float64)
    assert (np.abs(Y.cpu().numpy() - ref) <= (w + 1) * U * mag).all()
    Y = Y.float()
    assert torch.equal(Y, served(Ad, 3, k))
    assert torch.equal(Y, sk.sketch_gen_matmul_cm(cm_dev(A), 3, k))
    assert torch.equal(Y[:40], sk.sketch_gen_matmul_cm(cm_dev(A)[:40], 3, k))
    assert torch.equal(Y[:3], sk.sketch_gen_matmul_cm(cm_dev(A)[:3], 3, k))
    assert torch.equal(Y, sk.sketch_matmul_omega(Ad, torch.from_numpy(Om).to(DEV)))


@pytest.mark.parametrize("dist", ["normal", "uniform", "rademacher"])
@pytest.mark.parametrize("n,k", [(32, 24), (33, 64), (4101, 130)])
def test_stored_copy_has_the_generated_bits(n, k, dist):
    A = to_dev(normal_matrix(70, n, seed=4))
    Om = sk.sketch_gen_omega(9, 0, n, 0, k, dist=dist)
    assert torch.equal(sk.sketch_matmul_omega(A, Om), sk.sketch_gen_matmul(A, 9, k, dist=dist))
