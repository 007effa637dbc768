"""Irregular-voxel kernel (one element per lane, 42 voxels per workgroup) against
the oracle's operator, at the sizes where its lists can go wrong: fewer voxels
than a workgroup takes, a last workgroup of a few voxels, voxels whose elements
are all cut, and voxels that are irregular without a cut element (interface
through nodes, several materials).  Element by element: FP64 1e-12, FP32 2e-5
relative to the largest force (the step-level bars), with and without macro
strain and average stress, and the voxel stress."""

import numpy as np
import pytest

import microstructure as ms
from oracle.system import System
from oracle.xfem import Discretization

pytestmark = pytest.mark.gpu

LAME = np.array([[0.5769231, 0.3846154], [27.77778, 41.66667], [4.0, 4.0]])


def _slab(n, x0, x1):
    """Layer x0 <= x < x1 of material 1 (interfaces at x0 and x1, voxel units)."""
    x = np.arange(n[0] * n[1] * n[2]) % n[0]
    d = np.minimum(np.abs(x - x0), np.abs(x - x1))
    inside = (x >= x0) & (x < x1)
    return np.where(inside, -d, d).astype(float), inside.astype(np.int32)


def _cell(name):
    if name == "dot":                       # one small sphere: fewer than 42 irregular voxels
        n = (8, 6, 8)
        L, ph = ms.spheres_levelset(n, [np.array([4.13, 2.93, 4.21])], [0.9])
    elif name == "slab128":                 # 2 x 64 irregular voxels: three workgroups of 42 and one of 2
        n = (12, 8, 8)
        L, ph = _slab(n, 3.4, 8.7)
    elif name == "nodes":                   # interfaces through the nodes: voxels of two materials, none cut
        n = (12, 6, 4)
        L, ph = _slab(n, 3.0, 8.0)
    else:                                   # tilted layers: every element of many voxels is cut
        n = (16, 12, 12)
        i = np.arange(n[0] * n[1] * n[2])
        x, y, z = i % n[0], (i // n[0]) % n[1], i // (n[0] * n[1])
        L = 1.1 * np.sin(2 * np.pi * (x / n[0] * 3 + y / n[1] * 2 + z / n[2]) + 0.3)
        ph = np.where(L < 0, 1 + (x > 8), 0).astype(np.int32)
    return n, L, ph


def _rel(a, b):
    return np.abs(a - b).max() / max(np.abs(b).max(), 1e-300)


@pytest.mark.parametrize("name", ["dot", "slab128", "nodes", "tilted"])
def test_irregular_voxels_match_oracle(name):
    from paper_2601_02172_amd import Problem
    n, L, ph = _cell(name)
    ln = [float(v) for v in n]
    d = Discretization(n, tuple(ln), L, ph, LAME, keep_qp=False)
    rng = np.random.default_rng(5)
    x, E = rng.standard_normal(d.ndof), rng.standard_normal(6)
    S = System(d)
    y0 = S.apply(x)
    y1 = y0 - S.rhs(E)
    avg = S.average_stress(x, E)
    with Problem(n, ln, L, ph, LAME) as p:
        assert p.nX == d.nX
        for prec, tol in (("fp64", 1e-12), ("fp32", 2e-5)):
            a, _ = p.apply_operator(x, precision=prec, with_stress=False)
            b, s = p.apply_operator(x, macro_strain=E, precision=prec)
            assert _rel(a, y0) < tol and _rel(b, y1) < tol, prec
            assert _rel(s, avg) < tol, prec
        vs = p.voxel_stress(x, macro_strain=E)
        np.testing.assert_allclose(vs.mean(axis=1), avg, rtol=0, atol=1e-12 * np.abs(vs).max())
