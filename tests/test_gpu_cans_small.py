"""CANS of small matrices in one launch: edges of its tiles and of its range."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -24
FAILED = 1 | 2 | 16  # not converged, rerun, non-finite


@pytest.fixture(scope="module")
def api():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2609_32505_amd import api as _api
    return _api


def _inputs(b, m, n, seed):
    rng = np.random.default_rng(seed)
    U, _ = np.linalg.qr(rng.standard_normal((b, m, n)))
    V, _ = np.linalg.qr(rng.standard_normal((b, n, n)))
    s = rng.uniform(0.5, 1.5, (b, 1, n))
    s[..., 0] = 1.5
    return ((U * s) @ V.transpose(0, 2, 1)).astype(np.float32)


def _check(W, H, A):
    # 15 steps, each a few EPS in every entry, at a condition of 3
    U, s, Vt = np.linalg.svd(A.astype(np.float64), full_matrices=False)
    n = A.shape[2]
    tol = 256 * EPS * np.sqrt(n)
    assert np.linalg.norm(W - U @ Vt, axis=(1, 2)).max() <= tol
    Href = (Vt.transpose(0, 2, 1) * s[:, None, :]) @ Vt
    assert np.linalg.norm(H - Href, axis=(1, 2)).max() <= 1.5 * tol


# 16 columns a tile, the 16/32/64/96/128-column forms, 16 rows a strip and 16
# strips a round, and the last and first m on either side of the LDS limit
# (1040 + 32, 528 + 64, 304 + 96, 176 + 128 rows fit).
@pytest.mark.parametrize("b,m,n", [(1, 1, 1), (3, 2, 1), (2, 15, 15), (2, 16, 16), (2, 17, 17), (2, 24, 24), (2, 25, 25), (2, 600, 24), (2, 800, 24), (3, 33, 31),
                                   (2, 33, 33), (2, 64, 64), (1, 65, 64), (2, 65, 65), (2, 97, 96), (1, 97, 97),
                                   (300, 128, 128), (1, 129, 129), (1, 257, 20), (2, 1040, 30), (1, 1300, 30),
                                   (2, 528, 61), (1, 620, 61), (2, 304, 90), (1, 330, 90), (2, 176, 127),
                                   (1, 200, 127)])
def test_polar_edges(api, b, m, n):
    import torch
    print(f"polar {b} x {m} x {n}", flush=True)
    A = _inputs(b, m, n, m * n)
    W, H, *_, info = api.polar_fwd(torch.from_numpy(A).cuda(), cache=False)
    assert (api.info_to_numpy(info)["flags"] & FAILED == 0).all()
    _check(W.cpu().double().numpy(), H.cpu().double().numpy(), A)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("b,m,n", [(1, 16, 16), (5, 40, 33), (3, 128, 128)])
def test_polar_user_bounds(api, b, m, n, precision):
    # the bounded schedule (in BF16 too) before the refinement
    import torch
    print(f"bounded polar {b} x {m} x {n} precision {precision}", flush=True)
    A = _inputs(b, m, n, m + n)
    ub = torch.tensor([[0.4, 1.6]] * b, device="cuda")
    W, H, *_, info = api.polar_fwd(torch.from_numpy(A).cuda(), cache=False, bound=2, user_bounds=ub,
                                   precision=precision)
    assert (api.info_to_numpy(info)["flags"] & FAILED == 0).all()
    Wd = W.cpu().double().numpy()
    if precision == 0:
        _check(Wd, H.cpu().double().numpy(), A)
    else:  # BF16 steps turn the factor; the refinement makes it orthonormal
        assert np.abs(Wd.transpose(0, 2, 1) @ Wd - np.eye(n)).max() <= 256 * EPS


def test_polar_nonfinite_and_zero(api):
    import torch
    A = torch.from_numpy(_inputs(4, 50, 40, 3)).cuda()
    ref = api.polar_fwd(A, cache=False)[0]
    bad = A.clone()
    bad[1, 7, 3] = float("nan")
    bad[2] = 0.0
    W, _, *_, info = api.polar_fwd(bad, cache=False)
    flags = api.info_to_numpy(info)["flags"]
    assert flags[1] & 16 and not (flags[[0, 2, 3]] & 16).any()
    assert torch.equal(W[0], ref[0]) and torch.equal(W[3], ref[3])
    assert not W[2].any()


# the stop test in the next product (up to 512 slots a matrix: 22^2 sub-tiles
# at 704) and as a launch of its own: matrices that end at different steps, one
# that holds a NaN, and a budget that ends before any converges
@pytest.mark.parametrize("n", [130, 704, 736])
@pytest.mark.parametrize("poly", [0, 2])
def test_polar_stop_test(api, n, poly):
    import torch
    print(f"stop test n={n} poly={poly}", flush=True)
    A = _inputs(4, n, n, n)
    A[1] = np.linalg.qr(A[1])[0]
    A[2] *= 1e3
    A[3, 5, 6] = np.nan
    d = torch.from_numpy(A).cuda()
    W, H, *_, info = api.polar_fwd(d, cache=False, poly=poly)
    info = api.info_to_numpy(info)
    assert list(info["flags"] & FAILED) == [0, 0, 0, 16]
    assert info["iters"][3] == 1 and 1 < info["iters"][:3].min() <= info["iters"][:3].max() < 50
    W = W.cpu().double().numpy()
    tol = 256 * EPS * np.sqrt(n)
    for i in range(3):
        U, _, Vt = np.linalg.svd(A[i].astype(np.float64))
        assert np.linalg.norm(W[i] - U @ Vt) <= tol
    alone = api.info_to_numpy(api.polar_fwd(d[2:3], cache=False, poly=poly)[-1])
    assert alone["iters"][0] == info["iters"][2]
    short = api.info_to_numpy(api.polar_fwd(d[:1], cache=False, poly=poly, max_iters=3, pre_iters=2)[-1])
    assert short["iters"][0] == 3 and short["flags"][0] & 1


# One workgroup's LDS limit is a property of the kernel: threads that launch it with
# different sizes at the same time, each on its own stream and handle
def test_small_sizes_from_two_threads():
    import threading
    import torch
    from paper_2609_32505_amd import api
    g = torch.Generator(device="cuda").manual_seed(3)
    A = [torch.randn(2, m, n, generator=g, device="cuda") for m, n in ((176, 128), (100, 100))]
    ref = [api.svd_fwd(a)[1] for a in A]
    torch.cuda.synchronize()
    bad = []

    def work(i):
        h, st = api.Handle(), torch.cuda.Stream()
        with torch.cuda.stream(st):
            for _ in range(20):
                S = api.svd_fwd(A[i], handle=h)[1]
                st.synchronize()
                if not torch.equal(S, ref[i]):
                    bad.append(i)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad
