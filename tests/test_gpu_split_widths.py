"""Lane widths of the global-memory lightweight products: 4 or 8 bytes for an env with an inverse of its own
(8 beyond 8192 vertices; FP64 always 8), 16 for envs that share one.  A column's sum does not depend on the
width, so an env gives the same bits alone as next to a twin.  Budgets 1 to 3 end on either of the two
multiplier buffers."""
import numpy as np
import pytest

from paper_2604_17513_amd import scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,n,budget", [("fp32", 17, 3), ("fp32", 33, 2), ("fp32", 91, 1), ("fp64", 24, 3)])
def test_alone_and_with_a_twin_give_the_same_bits(prec, n, budget):
    from paper_2604_17513_amd import flash as F
    kw = dict(precision=F.FLASH_FP64 if prec == "fp64" else F.FLASH_FP32, max_contacts=n * n + 8, inner_tol=1e-300,
              contact_metric=F.FLASH_METRIC_LIGHTWEIGHT, global_contact_solve=1)
    out = []
    for copies in (1, 2):
        sc = scenes.cloth_fold(copies, n=n)
        sc.params.max_inner_iterations = budget
        b = F.from_scene(sc, twin_chunk=1, **kw)
        b.step(2)
        x = b.split(b.get_state()[0])
        out.append((x, b.contacts(0), b.stats()[0]["inner_iterations"]))
        if copies == 2:
            assert np.array_equal(x[0], x[1])
    (xa, ca, ia), (xb, cb, ib) = out
    assert len(ca["vertex"]) > 0 and ia == ib > 0
    assert np.array_equal(xa[0], xb[0]) and np.array_equal(ca["lambda"], cb["lambda"])


@pytest.mark.parametrize("copies,prec", [(5, "fp32"), (11, "fp32"), (40, "fp32"), (40, "fp64")])
def test_default_chunks_give_the_bits_of_single_envs(copies, prec):
    """Chunks by default (of 4, of 8, and of 16 with a partial last one in FP32) against one env per workgroup:
    the matrix-core products keep the vector order, also where the envs' contact rows part (one sheet starts
    above the table)."""
    from paper_2604_17513_amd import flash as F
    n = 72 if copies == 40 else 100 if copies == 5 else 84
    kw = dict(precision=F.FLASH_FP64 if prec == "fp64" else F.FLASH_FP32, max_contacts=n * n + 8, inner_tol=1e-300,
              contact_metric=F.FLASH_METRIC_LIGHTWEIGHT, global_contact_solve=1)
    for part in (False, True):
        out = []
        for chunk in (0, 1):
            sc = scenes.cloth_fold(copies, n=n)
            sc.params.max_inner_iterations = 2
            if part:
                sc.x0[1] = sc.x0[1] + np.array([0.0, 0.02, 0.0])
            b = F.from_scene(sc, twin_chunk=chunk, **kw)
            b.step(1)
            out.append((b.get_state(), [b.stats()[e]["contacts"] for e in range(copies)]))
        (sa, ca), (sb, cb) = out
        assert ca == cb and (len(set(ca)) > 1) == part
        assert np.array_equal(sa[0], sb[0]) and np.array_equal(sa[1], sb[1])
