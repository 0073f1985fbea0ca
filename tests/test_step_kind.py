"""Host checks of the step kernels' choice (lq_step_kind; no GPU): small boxes
step in bricks, larger ones on narrow or wide marching tiles, and the boxes of
the GPU tests step in the kernels that those tests are about.
"""
import ctypes as C

import pytest

import test_gpu_march
import test_gpu_step_kinds
from paper_1911_07045_amd import lqfire

ELASTIC = {"one": {}, "l23": dict(L2=1.16, L3=0.7), "chiral": dict(L2=0.9, L3=1.16, L4=-0.6)}


def kind(shape, prec, elastic, periodic=(True, True, True)):
    return lqfire.step_kind(shape, periodic, prec, L1=2.32, **ELASTIC[elastic])


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("elastic", sorted(ELASTIC))
def test_kinds_of_boxes(prec, elastic):
    for shape in ((3, 3, 3), (16, 16, 16), (32, 32, 32), (64, 64, 64), (40, 30, 9)):
        assert kind(shape, prec, elastic) == "bricks"
    for shape in ((128, 128, 128), (256, 256, 256), (230, 187, 141)):
        assert kind(shape, prec, elastic) == "wide"
    for shape in ((31, 400, 300), (3, 3, 20000)):  # the second leaves most of its bricks' sites empty
        assert kind(shape, prec, elastic) == "narrow"
    # once a cube marches, larger ones do
    kinds = [kind((n, n, n), prec, elastic) for n in range(3, 140)]
    first = kinds.index("wide" if "narrow" not in kinds else "narrow")
    assert "bricks" not in kinds[first:] and set(kinds[:first]) == {"bricks"}


def test_boxes_of_the_gpu_tests():
    for prec, boxes in (("f64", test_gpu_step_kinds.MARCH64), ("f32", test_gpu_step_kinds.MARCH32)):
        got = {(elastic, kind(shape, prec, elastic)) for elastic, shape in boxes}
        assert got == {(e, k) for e in ELASTIC for k in ("narrow", "wide")}
    for shape, periodic in test_gpu_step_kinds.BRICKS:
        for elastic in ELASTIC:
            assert {kind(shape, p, elastic, periodic) for p in ("f32", "f64")} == {"bricks"}
    for prec, members in test_gpu_march.BATCHES:
        got = {(elastic, kind(shape, prec, elastic)) for elastic, shape in members}
        terms = {e for e, _ in members}
        assert got >= {(e, k) for e in terms for k in ("narrow", "wide")} and "bricks" in {k for _, k in got}
    got = {(prec, kind(shape, prec, elastic)) for prec, elastic, shape in test_gpu_march.STOPS}
    assert got == {(p, k) for p in ("f32", "f64") for k in ("narrow", "wide", "bricks")}
    got = {(prec, elastic, kind(shape, prec, elastic, periodic)) for prec, elastic, shape, periodic in test_gpu_march.BOXES}
    assert got == {(p, e, k) for p in ("f32", "f64") for e in ELASTIC for k in ("narrow", "wide")}
    bricks = [(prec, elastic, shape) for prec, elastic, shape, _ in test_gpu_march.BRICKS]
    bricks += [(prec, elastic, shape) for prec, members in test_gpu_march.BRICK_BATCHES for elastic, shape in members]
    assert {kind(shape, prec, elastic) for prec, elastic, shape in bricks} == {"bricks"}
    got = [kind(shape, prec, elastic) for prec, elastic, shape in test_gpu_march.RESUMES]
    assert got == ["wide"] * 5 + ["bricks"]


def test_bad_arguments():
    with pytest.raises(lqfire.LQError) as e:
        lqfire.step_kind((0, 16, 16))
    assert e.value.code == lqfire.LQ_EINVAL
    p = lqfire.make_params((16, 16, 16))
    assert lqfire.lib().lq_step_kind(C.byref(p), None) == lqfire.LQ_EINVAL
    assert lqfire.lib().lq_step_kind(None, C.byref(C.c_int32())) == lqfire.LQ_EINVAL
