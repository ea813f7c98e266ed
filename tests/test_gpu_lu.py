"""GPU parity of the LU function block (fb_lu_factor) against the oracle's
Gaussian elimination with partial pivoting: the same pivots, factors within
rounding, the residual P A - L U at the level of binary64 rounding, singular
matrices reported by info; sizes with ragged panels and tiles up to the
paper's 2048 x 2048."""
import numpy as np
import pytest

import oracle
from paper_2004_09883_amd import fb

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def gpu_lu(a, lda=None):
    n = a.shape[0]
    lda = lda or n
    buf = torch.zeros((n, lda), dtype=torch.float64, device="cuda")
    buf[:, :n] = torch.from_numpy(a)
    view = buf[:, :n]
    ipiv = torch.full((n,), -1, dtype=torch.int32, device="cuda")
    info = torch.full((1,), -7, dtype=torch.int32, device="cuda")
    fb.fb_lu_factor(view, ipiv, info)
    torch.cuda.synchronize()
    return view.cpu().numpy(), ipiv.cpu().numpy(), int(info.cpu()[0]), buf.cpu().numpy()


def residual(a, lu, ipiv):
    n = a.shape[0]
    L = np.tril(lu, -1) + np.eye(n)
    U = np.triu(lu)
    perm = np.arange(n)
    for j, p in enumerate(ipiv):
        perm[[j, p]] = perm[[p, j]]
    return np.linalg.norm(a[perm] - L @ U) / np.linalg.norm(a)


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 33, 100, 257, 1000, 2048])
def test_lu_matches_oracle(n):
    print(f"lu n={n}", flush=True)
    a = np.random.default_rng(n).uniform(-1, 1, (n, n))
    lu, ipiv, info, _ = gpu_lu(a)
    lu_ref, ipiv_ref, info_ref = oracle.lu(a)
    assert info == info_ref == 0
    assert np.array_equal(ipiv, ipiv_ref)
    assert np.max(np.abs(lu - lu_ref)) <= 1e-11 * np.max(np.abs(lu_ref))
    assert residual(a, lu, ipiv) < 1e-15 * n + 1e-16
    assert np.max(np.abs(np.tril(lu, -1))) <= 1.0


def test_lu_with_row_stride_keeps_padding():
    n, lda = 300, 333
    a = np.random.default_rng(5).standard_normal((n, n))
    lu, ipiv, info, buf = gpu_lu(a, lda)
    lu_ref, ipiv_ref, _ = oracle.lu(a)
    assert np.array_equal(ipiv, ipiv_ref)
    assert np.max(np.abs(lu - lu_ref)) <= 1e-11 * np.max(np.abs(lu_ref))
    assert np.all(buf[:, n:] == 0.0)   # the padding columns are not touched


@pytest.mark.parametrize("n,lda", [(1537, 1601), (2047, 2051)])
def test_lu_large_with_row_stride(n, lda):
    """Odd row strides at sizes where the rows need 3 and 4 register slots,
    the trailing strips are ragged and the last panel is short: the rows
    past the end and the padding columns are read but never written."""
    print(f"lu n={n} lda={lda}", flush=True)
    a = np.random.default_rng(n + lda).uniform(-1, 1, (n, n))
    lu, ipiv, info, buf = gpu_lu(a, lda)
    lu_ref, ipiv_ref, info_ref = oracle.lu(a)
    assert info == info_ref == 0
    assert np.array_equal(ipiv, ipiv_ref)
    assert np.max(np.abs(lu - lu_ref)) <= 1e-11 * np.max(np.abs(lu_ref))
    assert np.all(buf[:, n:] == 0.0)


def test_lu_singular_and_special_matrices():
    a = np.arange(64.0 * 64).reshape(64, 64) % 7 - 3.0
    a[:, 20] = 0.0
    lu, ipiv, info, _ = gpu_lu(a)
    _, ipiv_ref, info_ref = oracle.lu(a)
    assert info == info_ref and info > 0
    eye = np.eye(50)
    lu, ipiv, info, _ = gpu_lu(eye)
    assert np.array_equal(lu, eye) and list(ipiv) == list(range(50)) and info == 0
    perm = np.eye(40)[np.random.default_rng(1).permutation(40)]
    lu, ipiv, info, _ = gpu_lu(perm)
    assert np.array_equal(lu, np.eye(40)) and info == 0


def test_lu_rejects_bad_arguments():
    ipiv = torch.zeros(8, dtype=torch.int32, device="cuda")
    info = torch.zeros(1, dtype=torch.int32, device="cuda")
    big = torch.zeros((4096, 4096), dtype=torch.float64, device="cuda")
    with pytest.raises(fb.FbError) as e:
        fb.fb_lu_factor(big, torch.zeros(4096, dtype=torch.int32, device="cuda"), info)
    assert e.value.code == fb.FB_ERR_UNSUPPORTED_SIZE
    with pytest.raises(fb.FbError):
        fb.fb_lu_factor(torch.zeros((8, 8), dtype=torch.float64, device="cuda"), ipiv[:4], info)


def tie_matrix(n, kind, seed):
    """Blocks of 4 (kind "equal": 4 x 4 matrices of +-1, exact in every
    elimination order) or of 2 ("low": pivots that differ in the last bits of
    the mantissa only, or not at all) on the diagonal, the rows shuffled."""
    rng = np.random.default_rng(seed)
    a = np.eye(n)
    if kind == "equal":
        h = np.array([[1, 1, 1, 1], [1, -1, 1, -1], [1, 1, -1, -1], [1, -1, -1, 1]], dtype=np.float64)
        for k in range(0, n - 3, 4):
            a[k:k + 4, k:k + 4] = h * rng.choice([-1.0, 1.0], 4)[:, None]
    else:
        for k in range(0, n - 1, 2):
            s = (1.0 + rng.integers(0, 3, 2) * 2.0**-52) * rng.choice([-1.0, 1.0], 2)
            a[k:k + 2, k:k + 2] = [[s[0], 1.0], [s[1], -s[0] * s[1] / abs(s[0] * s[1])]]
    return a[rng.permutation(n)]


@pytest.mark.parametrize("kind", ["equal", "low"])
@pytest.mark.parametrize("n", [4, 63, 66, 512, 530, 1040, 2048])
def test_lu_pivot_ties_take_the_first_row(n, kind):
    """Candidates of equal magnitude, or equal in the high word, in different
    lanes, waves and register slots: the oracle's pivots exactly."""
    print(f"lu ties n={n} {kind}", flush=True)
    a = tie_matrix(n, kind, n)
    lu, ipiv, info, _ = gpu_lu(a)
    lu_ref, ipiv_ref, info_ref = oracle.lu(a)
    assert info == info_ref == 0
    assert np.array_equal(ipiv, ipiv_ref)
    assert np.max(np.abs(lu - lu_ref)) <= 1e-11 * np.max(np.abs(lu_ref))


@pytest.mark.parametrize("e", [-900, -401, -399, 399, 401, 900])
def test_lu_column_scales(e):
    """Columns scaled by powers of two on both sides of the exponent range
    in which quotients come from the pivot's reciprocal: the same pivots and
    L, U scaled."""
    n = 150
    a = np.random.default_rng(9).uniform(-1, 1, (n, n))
    d = np.where(np.arange(n) % 3 == 1, 2.0**e, 1.0)
    lu, ipiv, info, _ = gpu_lu(a * d)
    lu_ref, ipiv_ref, _ = oracle.lu(a)
    assert info == 0 and np.array_equal(ipiv, ipiv_ref)
    lu = np.tril(lu, -1) + np.triu(lu) / d
    assert np.max(np.abs(lu - lu_ref)) <= 1e-11 * np.max(np.abs(lu_ref))


def test_lu_nan_and_inf_end_with_rows_of_the_matrix_as_pivots():
    for bad in (np.nan, np.inf):
        a = np.random.default_rng(2).uniform(-1, 1, (70, 70))
        a[40, 3] = bad
        _, ipiv, info, _ = gpu_lu(a)
        assert info == 0 and np.all(ipiv >= np.arange(70)) and np.all(ipiv < 70)


@pytest.mark.parametrize("n", [64, 600, 2048])
def test_lu_quotients_are_divisions(n):
    """Pivot rows with nothing right of the pivot, so that L is the quotients
    of the entries below by the pivots and nothing else: what a division
    gives, bit for bit, for quotients from ordinary ones down to subnormal
    ones and pivots of any exponent, the rows in any order."""
    rng = np.random.default_rng(n)
    h, m = n // 2, n - n // 2
    sign = lambda shape: rng.choice([-1.0, 1.0], shape)
    pivots = {"order 1": rng.uniform(1, 2, h) * sign(h), "all ones": (2 - 2.0**-52) * 2.0 ** rng.integers(-390, 390, h),
              "edges": rng.uniform(1, 2, h) * sign(h) * 2.0 ** rng.integers(-405, 405, h)}
    below = {"ordinary": rng.uniform(-1, 1, (m, h)), "2^-990": rng.uniform(1, 2, (m, h)) * 2.0**-990,
             "2^-1021": rng.uniform(1, 2, (m, h)) * 2.0**-1021 * sign((m, h)),
             "subnormal": rng.integers(1, 1 << 40, (m, h)) * 2.0**-1074 * sign((m, h)),
             "any": rng.uniform(1, 2, (m, h)) * 2.0 ** rng.integers(-1074, -1, (m, h)).astype(float)}
    for pname, piv in pivots.items():
        for bname, u in below.items():
            print(f"lu quotients n={n} pivots {pname} below {bname}", flush=True)
            v = u * np.abs(piv)
            a = np.zeros((n, n))
            a[:h, :h], a[h:, :h], a[h:, h:] = np.diag(piv), v, np.eye(m)
            order = rng.permutation(n)
            lu, ipiv, info, _ = gpu_lu(a[order])
            for j, p in enumerate(ipiv):
                order[[j, p]] = order[[p, j]]
            assert info == 0 and np.array_equal(order[:h], np.arange(h))
            want = v[order[h:] - h] / piv
            got = lu[h:, :h]
            where = want != 0   # (the sign of a zero also depends on the updates before)
            assert np.array_equal(got[where].view(np.int64), want[where].view(np.int64)), (pname, bname)


@pytest.mark.parametrize("col", [0, 20])
@pytest.mark.parametrize("n", [64, 600, 2048])
def test_lu_quotients_of_zeros_keep_their_sign(n, col):
    """Zeros of both signs below pivots of both signs, in the first panel and
    in one that a strip update hands over."""
    rng = np.random.default_rng(n + col)
    for piv in (1.5, -1.5, -2 + 2.0**-52):
        a = np.eye(n)
        v = rng.choice([0.0, -0.0, 0.5, -0.25, 2.0**-1070], n - col - 1)
        a[col, col], a[col + 1:, col] = piv, v
        lu, _, info, _ = gpu_lu(a)
        assert info == 0
        assert np.array_equal(lu[col + 1:, col].copy().view(np.int64), (v / piv).view(np.int64)), piv
