"""The marching kernels: batches, minimizers, stops, resumes and divergence on
lattices above the sizes that step in bricks.
"""
import numpy as np
import pytest

from paper_1911_07045_amd import lqfire, synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

ELASTIC = {"one": {}, "l23": dict(L2=1.16, L3=0.7), "chiral": dict(L2=0.9, L3=1.16, L4=-0.6)}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    lqfire.lib()


def _objects(shape):
    nx, ny, nz = shape
    return [dict(kind="sphere", center=(nx * 0.4, ny * 0.6, nz * 0.5), radius=min(shape) / 6.0 + 0.3, law="rp", W=3.0,
                 dir="normal"),
            dict(kind="wall", axis=2, plane=nz - 1, law="fg", W=0.7)]


def _lattice(shape, prec, elastic, periodic=(True, True, True)):
    lat = lqfire.Lattice(shape, periodic, prec, L1=2.32, **ELASTIC[elastic])
    lat.set_boundaries(_objects(shape))
    return lat


def _dev(a, dtype):
    return torch.from_numpy(np.ascontiguousarray(a)).to(device="cuda", dtype=dtype).contiguous()


def _random_start(lat, seed=5):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    d = torch.randn(3, lat.N, generator=g, device="cuda", dtype=torch.float64)
    return lat.set_uniaxial(d / d.norm(dim=0), lat.empty())


def _fire(shape, prec, elastic, seed=5):
    lat = _lattice(shape, prec, elastic)
    q, v, F = _random_start(lat, seed), lat.empty(), lat.empty()
    lat.fire_init(lqfire.make_fire_params(force_tol=0.0, max_steps=10 ** 6), q, v, F)
    return lat, q, v, F


# precision, members (elastic terms, shape): narrow and wide marching tiles and
# a box that steps in bricks; L2/L3 and chiral members share a batch; the second
# and the last batch hold boxes beyond the cache, whose steps march both ways
BATCHES = [
    ("f64", [("l23", (64, 84, 90)), ("chiral", (64, 80, 90)), ("l23", (61, 96, 90)), ("chiral", (60, 92, 84)), ("l23", (24, 20, 18))]),
    ("f64", [("l23", (64, 132, 140)), ("chiral", (64, 132, 140)), ("l23", (61, 140, 150)), ("chiral", (61, 96, 100)), ("l23", (24, 20, 18))]),
    ("f64", [("one", (64, 84, 80)), ("one", (61, 96, 90)), ("one", (24, 20, 18))]),
    ("f32", [("l23", (64, 80, 84)), ("chiral", (64, 76, 84)), ("l23", (61, 80, 90)), ("chiral", (60, 84, 84)), ("l23", (24, 20, 18))]),
    ("f32", [("l23", (64, 192, 190)), ("chiral", (64, 192, 190)), ("l23", (61, 80, 90)), ("chiral", (60, 84, 84)), ("l23", (24, 20, 18))]),
]


@pytest.mark.parametrize("prec,members", BATCHES, ids=["f64_l23", "f64_l23_large", "f64_one", "f32_l23", "f32_l23_large"])
def test_batch_equals_alone_bitwise(prec, members):
    """A member follows its solo trajectory bit for bit, sums and steering
    included, over calls of odd and even length.  (Sums taken in another order
    differ in the last bit of a total only now and then, hence the many steps.)"""
    alone = []
    for i, (elastic, shape) in enumerate(members):
        print(f"[march] alone {prec} {elastic} {shape}", flush=True)
        lat, *fields = _fire(shape, prec, elastic, seed=5 + i)
        rep = lat.fire_step(403)
        alone.append(([f.clone() for f in fields], rep.as_dict()))
        lat.close()
    b = lqfire.Batch(len(members))
    held = [_fire(shape, prec, elastic, seed=5 + i) for i, (elastic, shape) in enumerate(members)]
    for h in held:
        b.add(h[0])
    print(f"[march] batch {prec}", flush=True)
    for n in (5, 201, 130, 67):
        reps = b.step(n)
    for (lat, *fields), (ref, rep_a), rep in zip(held, alone, reps):
        assert rep.as_dict() == rep_a
        assert all(torch.equal(x, y) for x, y in zip(fields, ref))
    b.close()
    for h in held:
        h[0].close()


# precision, elastic terms, shape: marching tiles of both widths, and boxes of
# up to 256 bricks (controller in one wave), above 256 (in the block) and above
# one brick per thread of a block
STOPS = [("f64", "l23", (64, 84, 90)), ("f64", "one", (61, 96, 90)), ("f64", "chiral", (60, 92, 84)),
         ("f32", "one", (128, 96, 90)), ("f32", "l23", (61, 80, 90)), ("f32", "one", (24, 20, 18)),
         ("f64", "l23", (44, 40, 40)), ("f32", "one", (66, 64, 64))]


def _start(prec, elastic, shape, method, tol=0.0, cap=10 ** 6):
    lat = _lattice(shape, prec, elastic)
    q, v, F = _random_start(lat), lat.zeros(), lat.empty()
    if method == "fire":
        lat.fire_init(lqfire.make_fire_params(force_tol=tol, max_steps=cap), q, v, F)
    else:
        mu = 0.8 if method == "nesterov" else 0.0
        lat.descent_init(lqfire.make_descent_params(method, 2e-3, mu, force_tol=tol, max_steps=cap), q, v, F)
    return lat, q, v, F


@pytest.mark.parametrize("method", ["fire", "gd", "nesterov"])
@pytest.mark.parametrize("prec,elastic,shape", STOPS)
def test_stop_inside_a_call(prec, elastic, shape, method):
    """A run that stops inside one call, by its tolerance or its step limit,
    has the state and report of the same run taken one step per call; the
    kernels after the stop, and later calls, change nothing."""
    print(f"[march] stop {prec} {elastic} {shape} {method}", flush=True)
    lat, *_ = _start(prec, elastic, shape, method)
    tol = lat.fire_step(40).maxF * (1.0 + 1e-12)  # reached after 40 steps at the latest
    lat.close()
    for tol, cap in ((tol, 10 ** 6), (0.0, 17), (0.0, 18)):
        out = []
        for n in (90, 1):
            lat, *fields = _start(prec, elastic, shape, method, tol, cap)
            rep = lat.fire_step(n)
            while n == 1 and rep.status == lqfire.RUNNING and rep.step < 90:
                rep = lat.fire_step(1)
            state = [f.clone() for f in fields]
            for more in (3, 0, 30):
                assert lat.fire_step(more).as_dict() == rep.as_dict()
            assert all(torch.equal(a, b) for a, b in zip(state, fields))
            out.append((rep.as_dict(), state))
            lat.close()
        assert out[0][0] == out[1][0]
        assert all(torch.equal(a, b) for a, b in zip(out[0][1], out[1][1]))
        rep = out[0][0]
        assert (rep["status"] == lqfire.CONVERGED and 0 < rep["step"] <= 40) if tol else \
            (rep["status"] == lqfire.MAX_STEPS and rep["step"] == cap)
