"""GPU tests of the two-launch step on crystals that take the brick step by
default ("fused" = 0 keeps them on it): records of systems with several groups
of 256 tiles, whose sums are work items of their own, against the FP64 oracle.

Bounds: a handful of steps accumulate a few rounding errors per spin component
(2^-53 and 2^-24); m and E are means and sums of such terms.  The reference's
sums are numpy's pairwise ones over the oracle's spins (the oracle adds site
after site, and after 262,144 sites that alone is off by 5e-12).
"""
import numpy as np
import pytest

import oracle
import paper_1310_6143_amd as sl
from spin_systems import sc_reference
from spin_systems.lattice import simple_cubic
from tests.gpu_util import max_angle

pytestmark = pytest.mark.gpu


def _two_launch(w, prec, **options):
    g = sl.from_workload(w, precision=prec, check_symmetry=False)
    g.set_option("fused", 0)
    for key, value in options.items():
        g.set_option(key, value)
    assert g.get_option("brick_active") == 0 and g.get_option("fused_active") == 0
    return g


def _sc(dims):
    lat = simple_cubic(dims, (True, True, True))
    n = lat.n
    w = sc_reference(L=5)
    w.lattice, w.temperature, w.H = lat, 300.0, np.array([0.3, -0.2, 0.5])
    w.mu_s, w.k_u = np.full(n, w.mu_s[0]), np.full(n, w.k_u[0])
    w.easy_axis = np.tile([0.6, 0.0, 0.8], (n, 1))
    S = np.random.default_rng(n).standard_normal((n, 3)) + [0.0, 0.0, 2.0]
    w.S0 = S / np.linalg.norm(S, axis=1, keepdims=True)
    return w


def _records(w, dims, steps):
    """m and E after every step of the oracle, and its last spins."""
    S, sys_, m, E = w.S0.copy(), oracle.System(w), [], []
    e, mu, ku, J = w.easy_axis[0], w.mu_s[0], w.k_u[0], float(w.J[0])
    for k in range(steps):
        sys_.integrate(S, k, 1)
        m.append(S.mean(axis=0))
        c = S.reshape(dims[2], dims[1], dims[0], 3)
        links = sum((c * np.roll(c, 1, axis=a)).sum(axis=-1) for a in range(3))     # each once
        E.append(-J * links.sum() - ku * ((S @ e) ** 2).sum() - mu * (S @ w.H).sum())
    return S, np.array(m), np.array(E)


# tiles of 512 sites: one group; 256 and 257 tiles; 512, which just fill the
# chip in FP64; three groups with a remainder
@pytest.mark.parametrize("dims", [(16, 16, 16), (64, 64, 32), (64, 64, 33), (64, 64, 64), (64, 64, 73)])
def test_records_of_several_tile_groups(dims):
    w = _sc(dims)
    S_ref, m_ref, E_ref = _records(w, dims, 5)
    for prec, bound in ((sl.FP64, 1e-12), (sl.FP32, 2e-5)):
        first = None
        for remap in (1, 0, 2):
            with _two_launch(w, prec, tile_sites=512, xcd_remap=remap) as g:
                parts = [g.integrate(k) for k in (1, 2, 2)]
                m, E = np.concatenate([p[0] for p in parts]), np.concatenate([p[1] for p in parts])
                S = g.get_spins()
            assert max_angle(S, S_ref) < bound
            assert np.abs(m - m_ref).max() < bound
            assert (np.abs(E - E_ref) / np.abs(E_ref)).max() < bound
            if first is None:
                first = (S, m, E)
            assert all(np.array_equal(a, b) for a, b in zip(first, (S, m, E)))
