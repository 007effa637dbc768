"""Green operator, element by element, at the compile-time line lengths that
test_gpu_fft_lengths.py leaves out (64, 128 and 256 on every axis, 32 along y
and 96 along z; 64^3 has the xy-plane kernels and the two-stage z pass in both
precisions), in every FFT variant, at the bounds of that file.  A CPU test
asserts that the two lists of shapes together hold every compile-time length on
every axis."""

import os
import re

import numpy as np
import pytest

import microstructure as ms
from oracle.green import GreenOperator
from oracle.xfem import Discretization
from test_gpu_fft_lengths import LAME, SHAPES as OTHER_SHAPES, _rel

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHAPES = [(64, 64, 64), (12, 32, 18), (18, 64, 12), (64, 12, 18), (12, 16, 96), (128, 12, 4), (12, 128, 4),
          (4, 12, 128), (256, 12, 4), (12, 256, 4), (4, 12, 256)]


def _compile_time_lengths():
    src = open(os.path.join(ROOT, "paper_2601_02172_amd", "csrc", "fft.hip")).read()
    m = re.search(r"#define FFT_LENGTHS\(F\) \\\n(.*)\n", src)
    return sorted(int(v) for v in re.findall(r"F\((\d+)\)", m.group(1)))


def test_every_compile_time_length_is_covered_on_every_axis():
    lengths = _compile_time_lengths()
    assert len(lengths) == 18 and lengths[0] == 12 and lengths[-1] == 256
    for axis in range(3):
        have = {n[axis] for n in SHAPES + OTHER_SHAPES}
        assert not set(lengths) - have, (axis, sorted(set(lengths) - have))


@pytest.mark.gpu
@pytest.mark.parametrize("n", SHAPES, ids=lambda n: "x".join(map(str, n)))
def test_green_operator_at_the_other_lengths(n):
    from paper_2601_02172_amd import Problem
    L, ph = ms.spheres_levelset(n, [0.5 * np.array(n) + 0.13], [min(0.4 * min(n), 5.0)])
    ln = [float(v) for v in n]
    d = Discretization(n, tuple(ln), L, ph, LAME, keep_qp=False)
    f = np.random.default_rng(31).standard_normal(d.ndof)
    y = GreenOperator(n).apply(f, d.nX)
    r2 = float(f @ y)
    tol = max(1e-12, 12.0 * 2.0 ** -53 / (2.0 * np.sin(np.pi / max(n)) ** 2))
    for variant in range(4):
        with Problem(n, ln, L, ph, LAME, fft_variant=variant) as p:
            for prec, t in (("fp64", tol), ("fp32", 2e-5)):
                a, ra = p.apply_precond(f, precision=prec)
                assert _rel(a, y) < t, (variant, prec)
                assert abs(ra - r2) < t * abs(r2), (variant, prec)
