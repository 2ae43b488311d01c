"""The tridiagonal EVD and the split FP32 product at the edges of their tiles."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -24
FAILED = 16 | 32  # non-finite, not converged


@pytest.fixture(scope="module")
def api():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2609_32505_amd import api as _api
    return _api


def _spectrum(kind, n, rng):
    if kind == "spread":
        return rng.uniform(-1.0, 2.0, n)
    if kind == "cluster":  # half the spectrum on one value, the rest graded
        return np.where(np.arange(n) % 2 == 0, 1.0, 10.0 ** (-3.0 * np.arange(n) / n))
    return np.concatenate([[3.0, 2.0, 1.0][:n], np.zeros(max(n - 3, 0))])  # rank 3


# Edges: 32/64/128 columns per wave of the register tail, the 256 columns of the
# tail, the 512- and 1024-column forms of the blocked head, the last size of the
# tridiagonal route and the first of the sweeps.
@pytest.mark.parametrize("n", [1, 2, 3, 31, 33, 63, 64, 65, 127, 129, 255, 256, 257, 259, 383,
                               512, 513, 1023, 1024])
@pytest.mark.parametrize("kind", ["spread", "cluster", "rank3"])
def test_eigh_edges(api, n, kind):
    import torch
    print(f"eigh {kind} n={n}", flush=True)
    rng = np.random.default_rng(1000 + n)
    Q, _ = np.linalg.qr(rng.standard_normal((n, n)))
    H = ((Q * _spectrum(kind, n, rng)) @ Q.T).astype(np.float32)
    H = 0.5 * (H + H.T)
    zero = np.zeros_like(H)
    lam, V, info = api.eigh(torch.from_numpy(np.stack([H, zero, np.eye(n, dtype=np.float32)])).cuda())
    assert (api.info_to_numpy(info)["flags"] & FAILED == 0).all()
    lam, V = lam.cpu().double().numpy(), V.cpu().double().numpy()
    # n rank-one updates of a matrix of norm one, each exact to a few EPS
    tol = 8 * EPS * np.sqrt(n) + 16 * EPS
    for i, M in enumerate([H.astype(np.float64), zero.astype(np.float64), np.eye(n)]):
        scale = max(np.linalg.norm(M, 2), 1e-30)
        ref = np.linalg.eigvalsh(M)[::-1]
        assert np.abs(lam[i] - ref).max() <= tol * scale
        assert np.linalg.norm(V[i].T @ V[i] - np.eye(n), 2) <= tol
        assert np.linalg.norm((V[i] * lam[i]) @ V[i].T - M, 2) <= tol * scale


# Spectra that are narrow beside their distance from zero: the Gram matrix of a
# matrix that is orthonormal to FP32 rounding, and I + noise of FP32 rounding size,
# both signs.  Eigenvectors resolved against the offset are orthonormal to 1e-4 only.
@pytest.mark.parametrize("b,n", [(64, 128), (48, 300), (24, 512), (4, 1024)])
@pytest.mark.parametrize("kind", ["gram", "noise", "negative"])
def test_eigh_narrow_spectrum(api, b, n, kind):
    import torch
    print(f"narrow spectrum {kind} {b} x {n}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(7 * n + len(kind))
    N = torch.randn(b, n, n, generator=g, device="cuda", dtype=torch.float64)
    eye = torch.eye(n, dtype=torch.float64, device="cuda")
    if kind == "gram":
        Q = torch.linalg.qr(N)[0].float().double()
        H = Q.transpose(1, 2).contiguous() @ Q
    else:
        H = eye + 1e-7 / np.sqrt(n) * (N + N.transpose(1, 2))
    if kind == "negative":
        H = -H
    H = H.float()
    lam, V, info = api.eigh(H)
    assert (api.info_to_numpy(info)["flags"] & FAILED == 0).all()
    V, lam, H = V.double(), lam.double(), H.double()
    tol = 8 * EPS * np.sqrt(n) + 16 * EPS
    # per entry: the 2-norm bound holds for each
    assert float((V.transpose(1, 2).contiguous() @ V - eye).abs().max()) <= tol
    assert float(((V * lam[:, None, :]) @ V.transpose(1, 2).contiguous() - H).abs().max()) <= tol


def _ties(n, offset, count=None):
    """diag(1, d_i + offset) with d_i + the route's perturbation of entry i equal for
    the first count of them: eigenvalues that FP64 does not tell apart, whose vectors
    come out the same.  The others are spread over (0.2, 0.9)."""
    i = np.arange(n, dtype=np.uint64)
    h = ((i * 40503) & 0xffff) / 65536.0 - 0.5
    d = (offset - h) * 2.0 ** -25
    d[0] = 1.0
    if count is not None:
        d[count:] = np.linspace(0.2, 0.9, n - count)
    return np.diag(d).astype(np.float32)


@pytest.mark.parametrize("n", [3, 65, 130, 300])
def test_eigh_coinciding_eigenvalues(api, n):
    import torch
    print(f"ties n={n}", flush=True)
    H = _ties(n, 0.0)
    lam, V, info = api.eigh(torch.from_numpy(np.stack([H, np.eye(n, dtype=np.float32)])).cuda())
    assert (api.info_to_numpy(info)["flags"] & FAILED == 0).all()
    lam, v = lam[0].cpu().double().numpy(), V[0].cpu().double().numpy()
    tol = 8 * EPS * np.sqrt(n) + 16 * EPS
    assert np.linalg.norm(v.T @ v - np.eye(n), 2) <= tol
    assert np.linalg.norm((v * lam) @ v.T - H, 2) <= tol


# above 1024, where nothing but these vectors' own orthogonalisation solves a batch:
# ties, a few of them, half the values 1 and half 1/2, and rank 3 (W of the null
# space is arbitrary)
@pytest.mark.parametrize("n,kind", [(1100, "ties"), (2000, "halves"), (1100, "rank3"), (2300, "some")])
def test_polar_close_eigenvalues_large(api, n, kind):
    import torch
    print(f"polar close eigenvalues {kind} n={n}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(n)
    if kind in ("ties", "some"):
        A = torch.from_numpy(_ties(n, 1.0, None if kind == "ties" else 150)).cuda().expand(2, n, n).contiguous()
    else:
        Q = [torch.linalg.qr(torch.randn(n, n, generator=g, device="cuda", dtype=torch.float64))[0] for _ in range(4)]
        s = torch.ones(n, device="cuda", dtype=torch.float64)
        s[n // 2 if kind == "halves" else 3:] = 0.5 if kind == "halves" else 0.0
        A = torch.stack([(Q[2 * i] * s) @ Q[2 * i + 1] for i in range(2)]).float()
    W, H, S, V, info = api.polar_fwd(A, cache=True)
    assert (api.info_to_numpy(info)["flags"] & FAILED == 0).all()
    tol = 8 * EPS * np.sqrt(n) + 16 * EPS
    eye = torch.eye(n, dtype=torch.float64, device="cuda")
    for i in range(2):
        v, lam = V[i].double(), S[i].double()
        # Frobenius against sqrt(n) times the 2-norm bound
        assert float(torch.linalg.norm(v.T @ v - eye)) <= tol * np.sqrt(n)
        assert float(torch.linalg.norm((v * lam) @ v.T - H[i].double())) <= tol * np.sqrt(n)
    if kind != "halves":
        return
    # the gradient does not depend on the basis within an eigenspace: polar_bwd's own
    # eigendecomposition against the given one
    dH = torch.randn(2, n, n, generator=g, device="cuda")
    dA = api.polar_bwd(A, H, dH=dH)
    ref = api.polar_bwd(A, H, S=S, V=V, dH=dH)
    assert float((dA - ref).abs().max()) <= 16 * tol * float(ref.abs().max())


def test_too_many_coinciding_eigenvalues_are_flagged(api):
    import torch
    n = 2300
    ok = torch.diag(torch.linspace(0.5, 1.0, n))
    A = torch.stack([torch.from_numpy(_ties(n, 1.0)), ok]).cuda()
    W, H, S, V, info = api.polar_fwd(A, cache=True)
    assert list(api.info_to_numpy(info)["flags"] & FAILED) == [32, 0]


# Small matrices to an EPS or two: a Rayleigh quotient over v^T v has the error of the
# vector squared, which leaves the rounding of H v and of the result; a Newton-Schulz
# step leaves V orthonormal to its own rounding (2 EPS a column's norm, EPS sqrt(2) an
# angle, and the rounding of the step's sums again).
@pytest.mark.parametrize("b,n", [(256, 5), (256, 16), (128, 33), (64, 64), (64, 65), (32, 100), (32, 128)])
def test_eigh_small_accuracy(api, b, n):
    import torch
    print(f"small accuracy {b} x {n}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(n)
    Q = torch.linalg.qr(torch.randn(b, n, n, generator=g, device="cuda", dtype=torch.float64))[0]
    lo = torch.arange(n, 0, -1, device="cuda", dtype=torch.float64) / n
    H = ((Q * lo) @ Q.transpose(1, 2).contiguous()).float()
    lam, V, info = api.eigh(H)
    assert (api.info_to_numpy(info)["flags"] & FAILED == 0).all()
    ref = torch.linalg.eigvalsh(H.double().cpu()).flip(-1).cuda()
    V = V.double()
    assert float(torch.linalg.norm(lam.double() - ref) / torch.linalg.norm(ref)) <= 2 * EPS
    G = V.transpose(1, 2).contiguous() @ V - torch.eye(n, dtype=torch.float64, device="cuda")
    assert float(torch.linalg.norm(G) / np.sqrt(b * n)) <= 4 * EPS


def test_eigh_nan_is_flagged_alone(api):
    import torch
    H = torch.randn(3, 70, 70, generator=torch.Generator().manual_seed(5))
    H = 0.5 * (H + H.transpose(1, 2))
    ref, _, _ = api.eigh(H.cuda())
    bad = H.clone()
    bad[1, 4, 9] = float("nan")
    lam, _, info = api.eigh(bad.cuda())
    flags = api.info_to_numpy(info)["flags"]
    assert list(flags & FAILED != 0) == [False, True, False]
    assert torch.equal(lam[0], ref[0]) and torch.equal(lam[2], ref[2])


# dH = V diag(dlam) V^T is one product of the split kernel for any V: 64- and
# 128-wide tiles (the latter from 384 of them), remainders of tile, of the
# 32-index slice and of a 16-byte load.  Error of a K-term sum in FP32, as a
# random walk, against sum |a||b|.
@pytest.mark.parametrize("b,n", [(1, 1), (2, 5), (3, 31), (2, 64), (2, 65), (1, 130), (96, 257),
                                 (48, 384), (1, 1025)])
def test_split_product_edges(api, b, n):
    import torch
    print(f"product b={b} n={n}", flush=True)
    g = torch.Generator().manual_seed(n)
    V = torch.randn(b, n, n, generator=g)
    d = torch.randn(b, n, generator=g)
    lam = torch.arange(n, 0, -1).float().expand(b, n).contiguous()
    dH = api.eigh_bwd(lam.cuda(), V.cuda(), dlam=d.cuda())
    V, d = V.double(), d.double()
    ref = (V * d[:, None]) @ V.transpose(1, 2)
    mag = (V * d[:, None]).abs() @ V.abs().transpose(1, 2)
    assert ((dH.cpu().double() - ref).abs() <= (np.sqrt(n) + 8) * EPS * mag).all()


# the low terms of small operands underflow in 16 bits; FP32 holds them to 2^-126
@pytest.mark.parametrize("e", [-100, -107, -109, -114, -118])
@pytest.mark.parametrize("b,n", [(2, 5), (2, 64), (1, 130), (48, 384)])
def test_split_product_small_operands(api, b, n, e):
    import torch
    print(f"small operands b={b} n={n} 2^{e}", flush=True)
    g = torch.Generator().manual_seed(n)
    V = torch.randn(b, n, n, generator=g)
    d = torch.randn(b, n, generator=g) * 2.0 ** e
    lam = torch.arange(n, 0, -1).float().expand(b, n).contiguous()
    dH = api.eigh_bwd(lam.cuda(), V.cuda(), dlam=d.cuda())
    V, d = V.double(), d.double()
    ref = (V * d[:, None]) @ V.transpose(1, 2)
    mag = (V * d[:, None]).abs() @ V.abs().transpose(1, 2)
    assert bool(((dH.cpu().double() - ref).abs() <= (np.sqrt(n) + 8) * EPS * mag + n * 2.0 ** -148).all())


# the same for H = sym(W^T A) of small inputs
@pytest.mark.parametrize("e", [-100, -109, -114, -118])
@pytest.mark.parametrize("b,m,n", [(2, 9, 5), (4, 74, 64), (2, 210, 200), (16, 400, 390)])
def test_polar_h_of_small_inputs(api, b, m, n, e):
    import torch
    print(f"small inputs {b} x {m} x {n} 2^{e}", flush=True)
    g = torch.Generator().manual_seed(n)
    A = torch.randn(b, m, n, generator=g) * 2.0 ** e
    W, H, *_, info = api.polar_fwd(A.cuda(), cache=False)
    assert (api.info_to_numpy(info)["flags"] & FAILED == 0).all()
    W, H, A = W.cpu().double(), H.cpu().double(), A.double()
    ref, mag = W.transpose(1, 2) @ A, W.abs().transpose(1, 2) @ A.abs()
    ref, mag = 0.5 * (ref + ref.transpose(1, 2)), 0.5 * (mag + mag.transpose(1, 2))
    assert bool(((H - ref).abs() <= (np.sqrt(m) + 8) * EPS * mag + m * 2.0 ** -148).all())


def test_split_product_keeps_infinities(api):
    import torch
    n = 40
    g = torch.Generator().manual_seed(7)
    V = torch.randn(2, n, n, generator=g)
    d = torch.randn(2, n, generator=g)
    d[0, 3] = float("inf")
    lam = torch.arange(n, 0, -1).float().expand(2, n).contiguous()
    dH = api.eigh_bwd(lam.cuda(), V.cuda(), dlam=d.cuda())
    ref = (V * d[:, None]).double() @ V.transpose(1, 2).double()
    assert torch.equal(dH[0].cpu().double(), ref[0])
    assert torch.isfinite(dH[1]).all()


# the head of the reduction by launches per column (up to 40 matrices, all of a
# matrix on one XCD from 8) and by one workgroup per matrix (above), with
# matrices of different scales and one that splits
@pytest.mark.parametrize("b,n", [(7, 261), (9, 300), (41, 261), (9, 520), (41, 516)])
def test_eigh_reductions(api, b, n):
    import torch
    print(f"reduction b={b} n={n}", flush=True)
    g = torch.Generator().manual_seed(b * n)
    H = torch.randn(b, n, n, generator=g, dtype=torch.float64)
    H = (H + H.transpose(1, 2)) / np.sqrt(8.0 * n)
    H[1] *= 1e6
    H[2, :n // 2, n // 2:] = 0
    H[2, n // 2:, :n // 2] = 0
    H = H.float()
    lam, V, info = api.eigh(H.cuda())
    assert (api.info_to_numpy(info)["flags"] & FAILED == 0).all()
    lam, V, H = lam.cpu().double(), V.cpu().double(), H.double()
    ref = torch.linalg.eigvalsh(H).flip(-1)
    scale = ref.abs().amax(1)
    tol = 8 * EPS * np.sqrt(n) + 16 * EPS
    assert ((lam - ref).abs().amax(1) <= tol * scale).all()
    eye = torch.eye(n, dtype=torch.float64)
    assert (torch.linalg.matrix_norm(V.transpose(1, 2) @ V - eye, 2) <= tol).all()
    assert (torch.linalg.matrix_norm((V * lam[:, None, :]) @ V.transpose(1, 2) - H, 2) <= tol * scale).all()


# above 1024 in the polar factors' cached eigenpairs: the back-transformation by
# products of 128 reflectors (a last group of 1, 30 and 127 of them), two sizes of
# the column kernel, the first and last size of each padding
@pytest.mark.parametrize("b,n", [(2, 1025), (1, 1310), (1, 1536), (1, 2048), (1, 2049)])
@pytest.mark.parametrize("kind", ["flat", "cluster"])
def test_polar_eigenpairs_large(api, b, n, kind):
    import torch
    print(f"polar eigenpairs {kind} {b} x {n}", flush=True)
    rng = np.random.default_rng(n)
    Q, _ = np.linalg.qr(rng.standard_normal((n, n)))
    s = rng.uniform(0.5, 1.0, n) if kind == "flat" else np.where(np.arange(n) % 2 == 0, 1.0, 0.5)
    A = torch.from_numpy(((Q * s) @ Q.T[rng.permutation(n)]).astype(np.float32)).cuda()
    W, H, S, V, info = api.polar_fwd(torch.stack([A] * b), cache=True)
    assert (api.info_to_numpy(info)["flags"] & FAILED == 0).all()
    tol = 8 * EPS * np.sqrt(n) + 16 * EPS
    eye = torch.eye(n, dtype=torch.float64, device="cuda")
    ref = torch.linalg.svdvals(A.double().cpu())
    for i in range(b):
        L, v, h = S[i].double(), V[i].double(), H[i].double()
        # H is W^T A to a few EPS of its terms
        assert (L.cpu() - ref).abs().max() <= 2 * tol
        # Frobenius against sqrt(n) times the 2-norm bound
        assert torch.linalg.norm(v.T @ v - eye) <= tol * np.sqrt(n)
        assert torch.linalg.norm((v * L) @ v.T - h) <= tol * np.sqrt(n)


# tall matrices through the blocked QR: last blocks of 1, 4, 37, 63 and 64
# columns; the second matrix has two dependent columns in one block
@pytest.mark.parametrize("m,n", [(130, 65), (140, 68), (210, 101), (260, 127), (256, 128)])
def test_tall_qr_blocks(api, m, n):
    import torch
    print(f"tall {m} x {n}", flush=True)
    g = torch.Generator().manual_seed(m + n)
    A = torch.randn(2, m, n, generator=g)
    A[1, :, n - 1] = A[1, :, 0]
    A[1, :, n // 2] = 0.0
    U, S, V, info = api.svd_fwd(A.cuda())
    assert (api.info_to_numpy(info)["flags"] & FAILED == 0).all()
    U, S, V, A = U.cpu().double(), S.cpu().double(), V.cpu().double(), A.double()
    ref = torch.linalg.svdvals(A)
    # a few EPS per step of the polar iteration, as a random walk over n terms
    tol = 32 * EPS * np.sqrt(n)
    eye = torch.eye(n, dtype=torch.float64)
    for i in range(2):
        assert (S[i] - ref[i]).abs().max() <= tol * ref[i, 0]
        assert torch.linalg.norm(U[i].T @ U[i] - eye, 2) <= tol
        assert torch.linalg.norm(V[i].T @ V[i] - eye, 2) <= tol
        assert torch.linalg.norm((U[i] * S[i]) @ V[i].T - A[i], 2) <= tol * ref[i, 0]


# above 1024 columns the n x n core takes 64-wide tiles where the tall matrix
# takes 128-wide ones: twice the stop test's slots (4 x 3072 x 1536, 1 x 4096 x 2048)
@pytest.mark.parametrize("b,m,n", [(1, 4096, 2048), (4, 3072, 1536), (5, 2580, 1290)])
def test_tall_core_slots(api, b, m, n):
    import torch
    print(f"tall core {b} x {m} x {n}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(m)

    def orth(r, c):
        return torch.linalg.qr(torch.randn(r, c, generator=g, device="cuda", dtype=torch.float64))[0]

    s = torch.linspace(1.0, 0.1, n, device="cuda", dtype=torch.float64)
    A = torch.stack([(orth(m, n) * s) @ orth(n, n).T for _ in range(b)]).float()
    U, S, V, info = api.svd_fwd(A)
    assert (api.info_to_numpy(info)["flags"] & (FAILED | 1) == 0).all()
    tol = 32 * EPS * np.sqrt(n)
    eye = torch.eye(n, dtype=torch.float64, device="cuda")
    for i in range(b):
        u, v = U[i].double(), V[i].double()
        assert (S[i].double() - s).abs().max() <= tol
        # Frobenius against sqrt(n) times the 2-norm bound
        assert torch.linalg.norm(u.T @ u - eye) <= tol * np.sqrt(n)
        assert torch.linalg.norm(v.T @ v - eye) <= tol * np.sqrt(n)
        assert torch.linalg.norm((u * S[i].double()) @ v.T - A[i].double()) <= tol * np.sqrt(n)


# the blocked QR scales its columns in place, also where a row holds an infinity
# and the product takes its plain sums
def test_tall_infinity_is_flagged_alone(api):
    import torch
    g = torch.Generator().manual_seed(11)
    A = torch.randn(2, 300, 70, generator=g)
    ref = api.svd_fwd(A.cuda())[1]
    A[1, 5, 3] = float("inf")
    out = [api.svd_fwd(A.cuda()) for _ in range(3)]
    for U, S, V, info in out:
        flags = api.info_to_numpy(info)["flags"]
        assert list(flags & 16 != 0) == [False, True]
        assert torch.equal(S[0], ref[0])
        for x, y in zip((U, S, V), out[0]):
            assert torch.equal(x.isnan(), y.isnan()) and torch.equal(x.nan_to_num(), y.nan_to_num())


# Eigenvalues of the divide and conquer are sums over n indices of one sign; the
# running sum's rounding grows with its length.  A few EPS of the largest: the rounding
# of the result, of the shift and of eight partial sums.
@pytest.mark.parametrize("n", [1000, 2048, 4096])
def test_dc_eigenvalues(api, n):
    import torch
    print(f"dc eigenvalues {n}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(n)
    Q = torch.linalg.qr(torch.randn(n, n, generator=g, device="cuda", dtype=torch.float64))[0]
    lam = torch.linspace(1.0, 0.01, n, device="cuda", dtype=torch.float64)
    H = ((Q * lam) @ Q.T).float()
    out, V, info = api.eigh_dc(H[None])
    assert (api.info_to_numpy(info)["flags"] & FAILED == 0).all()
    assert float((out[0].double() - lam).abs().max()) <= 5 * EPS
