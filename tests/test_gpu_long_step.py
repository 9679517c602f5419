"""GPU parity of the long-range step (tiles of 8 x 8 x 4 cells, links up to
four cells away) against the FP64 oracle: lattices of the fewest cells an axis
may have, tiles cut on every axis, short and full reach, links on one axis
only, and rows it must leave to the wide form.

Bounds: 20 steps accumulate a few dozen rounding errors per spin component and
the sums of a few hundred links (2^-53 and 2^-24): well below 1e-12 and 2e-5.
"""
import numpy as np
import pytest

import oracle
import paper_1310_6143_amd as sl
from spin_systems import sc_reference
from spin_systems.lattice import Lattice
from tests.gpu_util import max_angle

pytestmark = pytest.mark.gpu


def _workload(dims, keep, drop_site=None):
    """Periodic sc lattice with every link (dx, dy, dz) that keep() accepts,
    typed by squared length (at most 16 types, cyclic)."""
    nx, ny, nz = dims
    n = nx * ny * nz
    i = np.arange(n)
    x, y, z = i % nx, i // nx % ny, i // (nx * ny)
    R = 5
    offs = [(dx, dy, dz) for dz in range(-R, R + 1) for dy in range(-R, R + 1) for dx in range(-R, R + 1)
            if (dx, dy, dz) != (0, 0, 0) and keep(dx, dy, dz)]
    col = np.stack([(x + dx) % nx + nx * ((y + dy) % ny + ny * ((z + dz) % nz)) for dx, dy, dz in offs], axis=1)
    typ = np.tile(np.array([(dx * dx + dy * dy + dz * dz) % 16 for dx, dy, dz in offs], dtype=np.uint8), (n, 1))
    order = np.argsort(col, axis=1)
    col, typ = np.take_along_axis(col, order, 1), np.take_along_axis(typ, order, 1)
    mask = np.ones(col.shape, dtype=bool)
    if drop_site is not None:      # one link and its reverse removed
        j = col[drop_site, 0]
        mask[drop_site, 0] = False
        mask[j, np.nonzero(col[j] == drop_site)[0][0]] = False
    lat = Lattice("sc long", np.stack([x, y, z], axis=1).astype(float),
                  np.concatenate([[0], np.cumsum(mask.sum(1))]).astype(np.int64), col[mask].astype(np.int32), typ[mask])
    w = sc_reference(L=5)
    w.lattice, w.temperature, w.H = lat, 300.0, np.array([0.3, -0.2, 0.5])
    w.J = 6.0e-21 * np.exp(-0.3 * np.arange(16)) * np.where(np.arange(16) % 5 == 4, -1.0, 1.0)
    w.mu_s, w.k_u = np.full(n, w.mu_s[0]), np.full(n, w.k_u[0])
    w.easy_axis = np.tile([0.6, 0.0, 0.8], (n, 1))
    S = np.random.default_rng(n).standard_normal((n, 3)) + [0.0, 0.0, 2.0]
    w.S0 = S / np.linalg.norm(S, axis=1, keepdims=True)
    return w


def _sphere(r2):
    return lambda dx, dy, dz: dx * dx + dy * dy + dz * dz <= r2


CASES = [((9, 9, 9), _sphere(20), None, 1), ((10, 17, 13), _sphere(20), None, 1), ((16, 8 + 1, 12), _sphere(6), None, 1),
         ((11, 24, 9), lambda dx, dy, dz: max(abs(dx), abs(dy), abs(dz)) <= 2, None, 1),
         ((12, 10, 9), lambda dx, dy, dz: abs(dx) <= 4 and abs(dy) <= 1 and abs(dz) <= 3, None, 1),
         ((11, 12, 13), _sphere(25), None, 0),          # five cells away
         ((10, 11, 12), _sphere(9), 321, 0)]            # one link missing


@pytest.mark.parametrize("dims,keep,drop,active", CASES)
def test_long_range_step_matches_oracle(dims, keep, drop, active):
    w = _workload(dims, keep, drop)
    S_ref = w.S0.copy()
    m_ref, E_ref = oracle.System(w).integrate(S_ref, 0, 20)
    for prec, bound in ((sl.FP64, 1e-12), (sl.FP32, 2e-5)):
        with sl.from_workload(w, precision=prec) as g:
            assert g.get_option("brick_active") == active
            m1, E1 = g.integrate(7)
            m2, E2 = g.integrate(13)
            assert max_angle(g.get_spins(), S_ref) < bound
            assert np.abs(np.concatenate([m1, m2]) - m_ref).max() < bound
            assert (np.abs(np.concatenate([E1, E2]) - E_ref) / np.abs(E_ref)).max() < bound
            if active:     # new couplings reach the step's own table
                g.set_conditions(300.0, (0.0, 0.0, 0.0))
                g.set_option("fused", 0)
                assert g.get_option("brick_active") == 0
                g.integrate(1)


def test_new_moments_reach_the_steps_own_couplings():
    """The step's table holds J / mu_ref: set_materials with another uniform
    moment on a running system has to rebuild it.  Continued against an oracle
    that continues with the new moment, and against the two-launch step."""
    w = _workload((10, 9, 13), _sphere(20))
    S_ref = w.S0.copy()
    oracle.System(w).integrate(S_ref, 0, 6)
    v = _workload((10, 9, 13), _sphere(20))
    v.mu_s, v.k_u = 0.6 * w.mu_s, 2.0 * w.k_u
    m_ref, E_ref = oracle.System(v).integrate(S_ref, 6, 9)
    for prec, bound in ((sl.FP64, 1e-12), (sl.FP32, 2e-5)):
        for fused in (1, 0):
            with sl.from_workload(w, precision=prec) as g:
                g.set_option("fused", fused)
                g.integrate(6)
                g.set_materials(v.mu_s[:1], v.k_u[:1], v.easy_axis[:1], per_site=0)
                assert g.get_option("brick_active") == fused
                m, E = g.integrate(9)
                assert max_angle(g.get_spins(), S_ref) < bound
                assert np.abs(m - m_ref).max() < bound
                assert (np.abs(E - E_ref) / np.abs(E_ref)).max() < bound


@pytest.mark.parametrize("fused", [1, 0])
@pytest.mark.parametrize("prec", [sl.FP32, sl.FP64])
def test_non_finite_spins_are_reported(prec, fused):
    """A field too large for the arithmetic drives the spins to NaN: the step
    that writes them reports it, at the call's end or at the next call."""
    w = _workload((9, 9, 9), _sphere(20))
    w.temperature, w.H = 0.0, np.array([1e300, 0.0, 0.0])
    with sl.from_workload(w, precision=prec) as g:
        g.set_option("fused", fused)
        assert g.get_option("brick_active") == fused
        g.integrate_dev(3)
        assert g.get_option("numeric_fault") == 1
        g.set_spins(w.S0)
        assert g.get_option("numeric_fault") == 0
        with pytest.raises(sl.SllgError) as e:
            g.integrate(2, record=False)
        assert e.value.name == "SLLG_E_NUMERIC"
        g.set_spins(w.S0)
        g.set_conditions(0.0, (0.0, 0.0, 1.0))
        g.integrate_dev(3)
        assert g.get_option("numeric_fault") == 0


def test_monte_carlo_records_of_the_steps_tiles():
    """Monte Carlo records take the step's measuring launch: a whole chain
    with m and E against the oracle."""
    w = _workload((10, 9, 13), _sphere(20))
    w.temperature = 900.0
    S_ref = w.S0.copy()
    m_ref, E_ref, acc_ref = oracle.System(w).mc(S_ref, 0, 6)
    for fused in (1, 0):
        with sl.from_workload(w, precision=sl.FP64) as g:
            g.set_option("fused", fused)
            m, E, acc = g.mc(6)
            assert np.array_equal(acc, acc_ref) and max_angle(g.get_spins(), S_ref) < 1e-12
            assert np.abs(m - m_ref).max() < 1e-12 and (np.abs(E - E_ref) / np.abs(E_ref)).max() < 1e-12
