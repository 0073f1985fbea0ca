"""The size of the FIRE workspace, and what lq_minimize_noalloc accepts: the
boxes whose lq_workspace_bytes fit its fixed array, whichever kernels step them.
"""
import ctypes as C

import pytest

from paper_1911_07045_amd import lqfire

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


# around 32 MiB: cubes, boxes whose bricks hang over the edge, L2/L3 (smaller
# bricks) and one-constant, in bricks and marching
BOXES = [("f64", (64, 64, 64)), ("f64", (65, 65, 66)), ("f64", (65, 66, 65)), ("f64", (65, 65, 65)), ("f64", (66, 65, 65)),
         ("f64", (17, 129, 127)), ("f64", (33, 105, 80)), ("f64", (66, 66, 66)), ("f32", (80, 80, 80)),
         ("f32", (82, 82, 83)), ("f32", (97, 77, 74)), ("f32", (83, 83, 83))]


@pytest.mark.parametrize("elastic", [{}, dict(L2=1.16, L3=0.7), dict(L2=0.9, L3=1.16, L4=-0.6)], ids=["one", "l23", "chiral"])
@pytest.mark.parametrize("prec,shape", BOXES)
def test_noalloc_accepts_what_fits(prec, shape, elastic):
    lat = lqfire.Lattice(shape, prec=prec, L1=2.32, **elastic)
    size = lat.workspace_bytes()
    print(f"[workspace] {prec} {shape} {elastic} {size}", flush=True)
    # three fields, partial sums (two slots of 32 bytes per 256 sites, up to 2048), the controller
    sums = 64 * min(2048, -(-lat.N // 256))
    assert 0 <= size - 15 * (8 if prec == "f64" else 4) * lat.N - sums <= 4 * 256 + 1024
    q = lat.set_uniaxial(torch.tensor([0.6, 0.0, 0.8], dtype=torch.float64, device="cuda")[:, None].expand(3, lat.N).contiguous(),
                         lat.empty())
    v, F = lat.empty(), lat.empty()
    fp = lqfire.make_fire_params(force_tol=0.0, max_steps=3)
    r = lqfire.MinResult()
    rc = lqfire.lib().lq_minimize_noalloc(lat.h, C.byref(fp), C.c_void_p(q.data_ptr()), C.c_void_p(v.data_ptr()),
                                          C.c_void_p(F.data_ptr()), C.byref(r))
    assert rc == (lqfire.LQ_OK if size <= lqfire.NOALLOC_WORKSPACE_BYTES else lqfire.LQ_ENOMEM)
    lat.close()
