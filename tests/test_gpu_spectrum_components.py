"""The velocity spectrum of a field whose components differ by many orders of magnitude: one large
component in the shells below 4 and one of amplitude 1e-8 alone in shell n/2 - 1.

The energy of that shell is the small component's.  Transformed by itself, as a real field is, its
rounding error is relative to its own size, and the large component adds its own rounding squared:
with amplitudes of rounding below 1e-15 of the large one that is 1e-30 against 1e-16.  The bar, 1e-12
of the shell's energy, leaves both two orders; a transform in which the large component's rounding
reaches the small one's amplitudes misses it (1e-15 / 1e-8).
"""
import math

import numpy as np
import pytest

import synthetic
from gpu_util import dev, make
from paper_2401_06841_amd import dg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,p", [((24, 24, 24), 1), ((16, 12, 20), 1), ((18, 15, 10), 2), ((16, 9, 6), 3), ((40, 3, 5), 5)])
def test_uniform_flow_is_exact(shape, p):
    """v = (1, 2, 2) everywhere: every sum of the transform is a whole number, and the energy of shell 0
    is 4.5 to the bit when nothing but the squared point count divides it."""
    print(f"spectrum of a uniform flow {shape} p={p}", flush=True)
    ctx = make(*shape, 1, 0)
    u = ctx.empty_state()
    u.zero_()
    for v, x in enumerate((1.0, 1.0, 2.0, 2.0)):
        u[v, 0] = x
    e = dg.dg_velocity_spectrum(ctx, u, p)
    assert e[0] == 4.5 and np.abs(e[1:]).max() < 1e-28


@pytest.mark.parametrize("big", [0, 1, 2])
@pytest.mark.parametrize("small", [1, 2])       # axes after the large one
@pytest.mark.parametrize("n,p,k", [(24, 1, 1), (25, 1, 3), (20, 3, 2), (20, 2, 1), (12, 5, 3)])
def test_small_component_beside_a_large_one(n, p, k, big, small):
    print(f"spectrum components n={n} p={p} k={k} big={big} small=+{small}", flush=True)
    small = (big + small) % 3
    rng = np.random.default_rng(7)
    nb, e, K0 = synthetic.nbasis(k), 1e-8, n // 2 - 1
    z, y, x = np.meshgrid(*[np.arange(n)] * 3, indexing="ij")
    f = 0.0
    for _ in range(6):
        q = rng.integers(-1, 2, 3)
        f = f + rng.uniform(0.5, 1.0) * np.cos(2 * math.pi * (q[0] * x + q[1] * y + q[2] * z) / n + rng.uniform(0, 6))
    u = np.zeros((4, nb, n ** 3))
    u[0, 0] = 1.0
    u[1 + big, 0] = f.ravel()
    u[1 + small, 0] = (e * (np.cos(2 * math.pi * K0 * x / n + 0.3) + np.cos(2 * math.pi * K0 * y / n + 0.4))).ravel()
    ctx = make(n, n, n, k, 0)
    got = dg.dg_velocity_spectrum(ctx, dev(u, ctx), p)
    # a cell's value stands at p points: the amplitude of wave number K0 is that of the cells' times
    # (1/p) |sum_s exp(-2 pi i K0 s / (n p))|
    a = abs(np.exp(-2j * math.pi * K0 * np.arange(p) / (n * p)).sum()) / p
    ref = 0.5 * e * e * a * a
    assert abs(got[K0] - ref) < 1e-12 * ref
