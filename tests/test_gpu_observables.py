"""Energy and director kernels where their work split or their arithmetic
changes: boxes around whole and partial blocks of 256 columns, one to many
planes a block, open axes; eigenvalues over the whole range of the cubic's
parameter and over scales.

Tolerances: energy terms to 1e-12 relative (FP64 sums, rounding order);
eigenvalues to 1e-12 relative where the largest root is simple (its condition
number, below 1e2 for r >= -0.9, times a few FP64 roundings).
"""
import numpy as np
import pytest

from paper_1911_07045_amd import lqfire, synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


@pytest.mark.parametrize("elastic", [{}, dict(L2=1.16, L3=0.7), dict(L2=0.9, L3=1.16, L4=-0.6)],
                         ids=["one", "l23", "chiral"])
@pytest.mark.parametrize("shape,periodic", [((16, 16, 5), (True, True, True)), ((257, 3, 4), (True, True, False)),
                                            ((15, 17, 1), (True, False, False)), ((300, 5, 7), (False, True, True)),
                                            ((64, 64, 300), (True, True, True)), ((3, 3, 3), (True, True, True))])
def test_energy_blocks(ora, shape, periodic, elastic):
    print(f"[energy] {shape} {periodic} {elastic}", flush=True)
    objs = []
    if min(shape) >= 5:
        objs = [dict(kind="sphere", center=tuple(0.45 * n for n in shape), radius=min(shape) / 4.0 + 0.3, law="rp", W=3.0,
                     dir="normal")]
    p = ora.Problem(shape, periodic, L1=2.32, objects=objs, **elastic)
    lat = lqfire.Lattice(shape, periodic, "f64", L1=2.32, **elastic)
    if objs:
        lat.set_boundaries(objs)
    lat.set_field([((0.2, 0.5, 0.1), 0.8)])
    pf = ora.Problem(shape, periodic, L1=2.32, objects=objs, fields=[((0.2, 0.5, 0.1), 0.8)], **elastic)
    q = synth.random_field(7, p.N).reshape(p.field_shape)
    E, terms = pf.energy(q, terms=True)
    e = lat.energy(torch.from_numpy(q).cuda())
    for k, key in enumerate(("bulk", "elastic", "anchoring", "external")):
        assert abs(e[key] - terms[k]) <= 1e-12 * max(1.0, abs(terms[k]))
    assert e["n_sim"] == pf.n_sim


@pytest.mark.parametrize("scale", [1e-120, 1e-9, 1.0, 1e90])
def test_directors_over_the_cubic(scale):
    """Eigenvalues 2p cos((phi + 2 pi m)/3) with r = cos(phi) from 1 to -1, in random frames."""
    print(f"[directors] scale {scale}", flush=True)
    n = 16
    N = n ** 3
    phi = np.concatenate([np.linspace(0.0, np.arccos(-0.9), N - 6), np.arccos([-0.95, -0.979, -0.981, -0.99, -0.999]), [np.pi]])
    rng = np.random.default_rng(4)
    R = np.linalg.qr(rng.normal(size=(N, 3, 3)))[0]
    lam = 2.0 * np.cos((phi[:, None] + 2.0 * np.pi * np.arange(3)) / 3.0)
    Q = np.einsum("nij,nj,nkj->nik", R, lam, R)
    q = scale * np.stack([Q[:, 0, 0], Q[:, 0, 1], Q[:, 0, 2], Q[:, 1, 1], Q[:, 1, 2]]).reshape(5, n, n, n)
    lat = lqfire.Lattice((n, n, n), prec="f64")
    dirs, got, defect, count = lat.director_field(torch.from_numpy(q).cuda(), 1.5 * scale)
    got = got.cpu().numpy().reshape(-1) / scale
    # the double root at r = -1 takes the square root of the rounding of r
    tol = np.where(np.cos(phi) >= -0.9, 1e-12, 3e-7)
    assert (np.abs(got - lam[:, 0]) <= tol * lam[:, 0]).all()
    d = dirs.cpu().numpy().reshape(3, -1).T
    simple = np.cos(phi) >= -0.9
    assert (np.abs(np.abs(np.einsum("ni,ni->n", d, R[:, :, 0])) - 1.0)[simple] <= 1e-12).all()
    clear = np.abs(lam[:, 0] - 1.5) > 1e-9
    assert (defect.cpu().numpy().reshape(-1)[clear] == (lam[:, 0] < 1.5)[clear]).all()
    assert count == int(defect.sum())
