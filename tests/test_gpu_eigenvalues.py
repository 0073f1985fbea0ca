"""Rounding of the director kernel's eigenvalues, against 80-bit arithmetic.

The largest eigenvalue is 2 p c, p = sqrt(tr(Q^2) / 6), c the largest root of
4 c^3 - 3 c = r.  At r near 1, the ordinary state, the rounding of r hardly
moves the root (by a ninth of it), and p, c and the product rounded once each leave a mean
relative error of some 7e-17 (a quarter of a spacing of 1.1e-16 to 2.2e-16
each); the bound is 0.75 times 2^-53.
"""
import numpy as np
import pytest

from paper_1911_07045_amd import lqfire

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def largest_root(q):
    """Largest eigenvalue of the tensors q [5][N] in long double."""
    a, b, c, d, e = q.astype(np.longdouble)
    f = -a - d
    p = np.sqrt((a * a + d * d + f * f + 2 * (b * b + c * c + e * e)) / 6)
    det = a * (d * f - e * e) - b * (b * f - e * c) + c * (b * e - d * c)
    r = np.clip(det / (2 * p ** 3), -1, 1)
    x = np.cos(np.arccos(r) / 3)
    for _ in range(3):
        x = x - (4 * x ** 3 - 3 * x - r) / (12 * x * x - 3)
    return 2 * p * x


@pytest.mark.parametrize("kind", ["uniaxial", "nearly uniaxial"])
def test_eigenvalues_are_rounded_once(kind):
    print(f"[eigenvalues] {kind}", flush=True)
    n = 48
    N = n ** 3
    rng = np.random.default_rng(5)
    mid = {"uniaxial": np.full(N, -0.5), "nearly uniaxial": -0.5 + 0.01 * rng.normal(size=N)}[kind]
    lam = np.stack([np.ones(N), mid, -1.0 - mid], 1)
    R = np.linalg.qr(rng.normal(size=(N, 3, 3)))[0]
    Q = np.einsum("nij,nj,nkj->nik", R, lam, R)
    q = np.stack([Q[:, 0, 0], Q[:, 0, 1], Q[:, 0, 2], Q[:, 1, 1], Q[:, 1, 2]])
    exact = largest_root(q)
    lat = lqfire.Lattice((n, n, n), prec="f64")
    _, got, _, _ = lat.director_field(torch.from_numpy(q.reshape(5, n, n, n)).cuda(), 0.1)
    err = np.abs((got.cpu().numpy().reshape(-1) - exact) / exact).astype(float)
    assert err.mean() <= 0.75 * 2.0 ** -53 and err.max() <= 6 * 2.0 ** -53
    lat.close()
