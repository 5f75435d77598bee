"""The power iteration of one workgroup (L <= 4) product by product against the
matrix-free product on the CPU: both layouts of L = 4 (odd and even numbers of
products), both eigenvectors, both sectors; and one over several launches.

Error of a product: N <= 16 steps of 2^-53 relative each, twice, and sums of
2^16 terms; 1e-12 relative holds with a margin of 100."""
import numpy as np
import pytest

from oracle import transfer as otm
from paper_2310_07486_amd import tfim

pytestmark = pytest.mark.gpu


def _couplings(L, seed):
    rng = np.random.default_rng(seed)
    return [rng.choice([-1, 1], L * L).astype(np.int8) for _ in range(2)]


def _start(n, sign, second):
    s = np.arange(n, dtype=np.uint64)
    if second:
        h = (s * 0x9E3779B1) & 0xFFFFFFFF
        h ^= h >> np.uint64(15)
        h = (h * 0x85EBCA77) & 0xFFFFFFFF
        h ^= h >> np.uint64(13)
        v = (h & 0xFFFF).astype(np.float64) / 32768.0 - 1.0
    else:
        v = np.where((sign > 0) | (s < n // 2), 1.0, -1.0)
    return 0.5 * (v + sign * v[::-1])


@pytest.mark.parametrize("L", [2, 3, 4])
@pytest.mark.parametrize("sector", [0, 1])
@pytest.mark.parametrize("iters", [1, 2, 5])
def test_power_iteration_steps(L, sector, iters):
    Jx, Jy = _couplings(L, 10 * L + sector)
    k, sign = 0.23, 1.0 - 2.0 * sector
    print(f"power iteration L={L} sector={sector} products={iters}", flush=True)
    lam, its, vec = tfim.tm_top(L, k, Jx, Jy, sector, n_eig=2, tol=1e-300, max_iter=iters, return_vectors=True)
    assert list(its) == [iters, iters]
    z = None
    for q in range(2):
        v = _start(2 ** (L * L), sign, q == 1)
        v -= (z @ v) * z if q else 0.0
        v /= np.linalg.norm(v)
        for _ in range(iters):
            w = otm.apply(L, k, Jx, Jy, v)
            want = v @ w
            w -= (z @ w) * z if q else 0.0
            v = w / np.linalg.norm(w)
        got = np.asarray(vec[q])
        assert abs(lam[q] - want) <= 1e-12 * want
        assert np.abs(got - v).max() <= 1e-12
        assert np.array_equal(got, sign * got[::-1])
        z = v


def test_power_iteration_over_launches():
    """More products than one launch does."""
    L, k = 4, 0.01
    Jx, Jy = _couplings(L, 3)
    print("power iteration over launches", flush=True)
    lam, its, vec = tfim.tm_top(L, k, Jx, Jy, 1, n_eig=1, tol=1e-300, max_iter=4500, return_vectors=True)
    v = np.asarray(vec[0])
    assert 2048 < its[0] <= 4500
    assert abs(v @ v - 1.0) <= 1e-12
    assert abs(v @ otm.apply(L, k, Jx, Jy, v) - lam[0]) <= 1e-12 * lam[0]


def test_product_of_offset_vectors():
    """L = 5 reads and writes pairs; vectors need only the alignment of a double."""
    import torch
    L, n = 5, 2 ** 25
    Jx, Jy = _couplings(L, 8)
    print("L = 5 product of vectors at odd places", flush=True)
    g = torch.Generator(device="cuda").manual_seed(2)
    a, b = (torch.empty(n + 1, dtype=torch.float64, device="cuda") for _ in range(2))
    v = torch.randn(n, dtype=torch.float64, device="cuda", generator=g)
    w = torch.empty_like(v)
    tfim.tm_apply(L, 0.3, Jx, Jy, v, w)
    a[1:].copy_(v)
    tfim.tm_apply(L, 0.3, Jx, Jy, a[1:], b[1:])
    torch.cuda.synchronize()
    assert torch.equal(w, b[1:])
