"""The two families of step kernels against the oracle, at the sizes where
each could go wrong: bricks (small lattices) around whole and partial bricks,
on periodic and open boxes; marching tiles just above the sizes that bricks
serve, on narrow and wide tiles, alone and in batches.

Tolerances as elsewhere: FP64 forces differ from the oracle's by the rounding
of some 30 summed terms (1e-12 relative), along a few FIRE steps by 1e-10; one
FP32 force evaluation by 30 roundings of 2^-24 (1e-5 relative; test inputs of
order one); the F that a fused step leaves equals the force kernel's bit for
bit, since both evaluate one site the same way.
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


def _objects(shape, periodic):
    nx, ny, nz = shape
    if min(shape) < 5:
        return [], []
    objs = [dict(kind="sphere", center=(nx * 0.4, ny * 0.6, nz * 0.5), radius=min(shape) / 4.0 + 0.3, law="rp", W=3.0,
                 dir="normal"),
            dict(kind="wall", axis=2, plane=nz - 1, law="fg", W=0.7)]
    return objs, [dict(site=nx * ny + 1, law="nd", W=0.4, n0=(1.0, 2.0, 2.0))]


def _lattice(shape, periodic, prec, elastic, objs, recs):
    lat = lqfire.Lattice(shape, periodic, prec, L1=2.32, **ELASTIC[elastic])
    if objs or recs:
        lat.set_boundaries(objs, recs)
    return lat


def _dev(a, dtype):
    return torch.from_numpy(np.ascontiguousarray(a)).to(device="cuda", dtype=dtype).contiguous()


def _check(ora, shape, periodic, elastic, steps=4):
    print(f"[kinds] {shape} {periodic} {elastic}", flush=True)
    objs, recs = _objects(shape, periodic)
    p = ora.Problem(shape, periodic, L1=2.32, objects=objs, site_records=recs, **ELASTIC[elastic])
    q = synth.random_field(11, p.N).reshape(p.field_shape)
    F_ora = p.forces(q)
    scale = np.abs(F_ora).max()
    lat = _lattice(shape, periodic, "f64", elastic, objs, recs)
    F = lat.compute_forces(_dev(q, torch.float64)).cpu().numpy()
    assert np.abs(F - F_ora).max() <= 1e-12 * scale
    # a few fused steps
    q0 = p.uniaxial(synth.random_directors(3, p.N))
    prm = ora.fire_params(force_tol=0.0, max_steps=10 ** 6)
    st, qo, vo, Fo = p.fire_init(prm, q0)
    p.fire_steps(prm, st, qo, vo, Fo, steps)
    qd, v, F = _dev(q0, torch.float64), lat.empty(), lat.empty()
    lat.fire_init(lqfire.make_fire_params(force_tol=0.0, max_steps=10 ** 6), qd, v, F)
    rep = lat.fire_step(steps)
    assert rep.step == st.step and rep.dt == pytest.approx(st.dt, rel=1e-15)
    assert np.abs(F.cpu().numpy() - Fo).max() <= 1e-10 * np.abs(Fo).max()
    assert np.abs(qd.cpu().numpy() - qo).max() <= 1e-12
    lat.close()


def _check_f32(ora, shape, periodic, elastic):
    print(f"[kinds] f32 {shape} {periodic} {elastic}", flush=True)
    objs, recs = _objects(shape, periodic)
    p = ora.Problem(shape, periodic, L1=2.32, objects=objs, site_records=recs, **ELASTIC[elastic])
    q32 = synth.random_field(11, p.N).reshape(p.field_shape).astype(np.float32)
    F_ora = p.forces(q32.astype(np.float64))
    lat = _lattice(shape, periodic, "f32", elastic, objs, recs)
    F = lat.compute_forces(_dev(q32, torch.float32)).cpu().numpy()
    assert np.abs(F - F_ora).max() <= 1e-5 * np.abs(F_ora).max()
    q, v, F = _dev(p.uniaxial(synth.random_directors(3, p.N)), torch.float32), lat.empty(), lat.empty()
    lat.fire_init(lqfire.make_fire_params(force_tol=0.0, max_steps=10 ** 6), q, v, F)
    lat.fire_step(3)
    assert torch.equal(F, lat.compute_forces(q))
    lat.close()


BRICKS = [((16, 8, 4), (True, True, True)), ((17, 9, 5), (True, True, True)), ((15, 7, 3), (False, True, False)),
          ((3, 3, 3), (True, True, True)), ((33, 16, 13), (True, False, True)), ((32, 24, 8), (False, False, False)),
          ((5, 41, 6), (True, True, False))]


@pytest.mark.parametrize("elastic", sorted(ELASTIC))
@pytest.mark.parametrize("shape,periodic", BRICKS)
def test_bricks(ora, shape, periodic, elastic):
    _check(ora, shape, periodic, elastic)
    _check_f32(ora, shape, periodic, elastic)


# just above the sizes that bricks serve: narrow tiles, then wide ones
# (rows of whole half lines, with the state in the cache or beyond it, and ragged ones)
MARCH64 = [("one", (61, 142, 120)), ("one", (64, 100, 80)), ("one", (129, 150, 81)), ("one", (136, 150, 81)), ("l23", (61, 100, 100)), ("l23", (65, 120, 120)),
           ("chiral", (61, 100, 80)), ("chiral", (65, 100, 105))]
MARCH32 = [("one", (100, 142, 120)), ("one", (128, 96, 90)), ("one", (129, 140, 120)), ("one", (144, 140, 120)), ("l23", (61, 80, 81)), ("l23", (65, 95, 93)),
           ("chiral", (61, 80, 81)), ("chiral", (65, 95, 93))]


@pytest.mark.parametrize("elastic,shape", MARCH64)
def test_marching_tiles_fp64(ora, elastic, shape):
    _check(ora, shape, (True, True, False), elastic)


@pytest.mark.parametrize("elastic,shape", MARCH32)
def test_marching_tiles_fp32(ora, elastic, shape):
    _check_f32(ora, shape, (True, False, True), elastic)


@pytest.mark.parametrize("elastic", ["one", "l23"])
def test_batch_of_all_kinds_equals_alone(elastic):
    """Members in bricks, on narrow and on wide marching tiles go in launches
    of their own; each follows its solo trajectory bit for bit."""
    shapes = [(20, 17, 9), (100, 142, 120) if elastic == "one" else (61, 80, 81),
              (129, 140, 120) if elastic == "one" else (65, 95, 93), (24, 24, 24)]

    def bound(shape):
        objs, recs = _objects(shape, (True,) * 3)
        lat = _lattice(shape, (True,) * 3, "f32", elastic, objs, recs)
        q = lat.set_uniaxial(_dev(synth.random_directors(5, lat.N), torch.float64), lat.empty())
        v, F = lat.empty(), lat.empty()
        lat.fire_init(lqfire.make_fire_params(force_tol=0.0, max_steps=10 ** 6), q, v, F)
        return lat, q, v, F

    alone = []
    for shape in shapes:
        lat, *fields = bound(shape)
        rep = lat.fire_step(9)
        alone.append(([f.clone() for f in fields], rep.as_dict()))
        lat.close()
    b = lqfire.Batch(len(shapes))
    held = [bound(s) for s in shapes]
    for h in held:
        b.add(h[0])
    b.step(5)
    reps = b.step(4)
    for (lat, *fields), (ref, rep_a), rep in zip(held, alone, reps):
        assert all(torch.equal(x, y) for x, y in zip(fields, ref))
        assert rep.as_dict() == rep_a
    b.close()


@pytest.mark.parametrize("shape", [(20, 17, 9), (129, 140, 120)])
def test_unaligned_buffers_equal_aligned(shape):
    """State buffers that start inside a 16-byte piece take the finalize's
    scalar form; results are the same bit for bit."""
    out = []
    for shift in (0, 1):
        lat = lqfire.Lattice(shape, prec="f32")
        n = 5 * lat.N
        q, v, F = [torch.empty(n + 4, dtype=torch.float32, device="cuda")[shift:shift + n].view(lat.field_shape)
                   for _ in range(3)]
        lat.set_uniaxial(_dev(synth.random_directors(5, lat.N), torch.float64), q)
        lat.fire_init(lqfire.make_fire_params(force_tol=0.0, max_steps=10 ** 6), q, v, F)
        lat.fire_step(3)
        rep = lat.fire_step(4)
        out.append(([t.clone() for t in (q, v, F)], rep.as_dict()))
        lat.close()
    assert all(torch.equal(a, b) for a, b in zip(out[0][0], out[1][0])) and out[0][1] == out[1][1]
