"""GPU tests of the two-launch step on crystals that take the brick step by
default ("fused" = 0 keeps them on it): records of systems with several groups
of 256 tiles, whose sums are work items of their own, and whole runs against
the FP64 oracle; and what must not change a bit: tile order, tile size, LDS
window, row format, chunks, graphs and XCD mapping.  The wide form of
long-range rows likewise, which takes the long-range step by default.

Bounds: a handful of steps accumulate a few rounding errors per spin component
(2^-53 and 2^-24); m and E are means and sums of such terms.  The reference's
sums are numpy's pairwise ones over the oracle's spins (the oracle adds site
after site, and after 262,144 sites that alone is off by 5e-12).
"""
import numpy as np
import pytest

import oracle
import paper_1310_6143_amd as sl
from spin_systems import bcc_block, bcc_film, long_range_sc, sc_reference
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


def _warm(w, T=300.0):
    w.temperature, w.H = T, np.array([0.2, -0.1, 0.5])
    return w


SYSTEMS = [lambda: _warm(sc_reference(L=12, seed=2)), lambda: _warm(bcc_film(nx=12, ny=10, nz=5, seed=3)),
           lambda: _warm(bcc_block(cells=10, n_steps=100))]


@pytest.mark.parametrize("make", SYSTEMS)
def test_two_launch_step_matches_oracle(make):
    w = make()
    S_ref = w.S0.copy()
    m_ref, E_ref = oracle.System(w).integrate(S_ref, 0, 150)
    with _two_launch(w, sl.FP64) as g:
        m, E = g.integrate(150)
        assert max_angle(g.get_spins(), S_ref) < 1e-12
        assert np.abs(m - m_ref).max() < 1e-12 and (np.abs(E - E_ref) / np.abs(E_ref)).max() < 1e-12
    with _two_launch(w, sl.FP32) as g:
        m, E = g.integrate(40)
        assert np.abs(m - m_ref[:40]).max() < 2e-5 and (np.abs(E - E_ref[:40]) / np.abs(E_ref[:40])).max() < 2e-5


def _runs(w, prec, variants, steps=60, fmt=None):
    out = []
    for options in variants:
        options = dict(options)
        stencil = options.pop("stencil", 1)
        g = sl.from_workload(w, precision=prec, check_symmetry=False, stencil=stencil)
        with g:
            g.set_option("fused", 0)
            for key, value in options.items():
                g.set_option(key, value)
            assert g.get_option("brick_active") == 0 and g.get_option("fused_active") == 0
            if fmt is not None:
                assert g.get_option("neighbour_format") == (fmt if stencil else 0)
            parts = [g.integrate(k) for k in (steps - steps // 3, steps // 3)]
            out.append((g.get_spins(), np.concatenate([p[0] for p in parts]), np.concatenate([p[1] for p in parts])))
    return out


@pytest.mark.parametrize("prec", [sl.FP32, sl.FP64])
def test_launch_shapes_give_the_same_bits(prec):
    """Tile order and group, XCD mapping, graphs, launch grid, LDS window and
    row format only reorder the work or change where a term is read."""
    variants = [{}, {"tile_order": 0}, {"tile_group": 1}, {"tile_group": 3}, {"xcd_remap": 0}, {"xcd_remap": 2},
                {"graph_steps": 0}, {"graph_steps": 16}, {"grid_scale_pct": 50}, {"lds_window": 0}, {"stencil": 0},
                {"stencil": 0, "lds_window": 0}]
    for w in (_warm(bcc_block(cells=24, n_steps=100)), _warm(bcc_film(nx=20, ny=14, nz=7))):
        res = _runs(w, prec, variants, fmt=1)
        for options, other in zip(variants[1:], res[1:]):
            assert all(np.array_equal(a, b) for a, b in zip(res[0], other)), options


@pytest.mark.parametrize("prec,largest", [(sl.FP32, 2048), (sl.FP64, 1024)])
def test_tile_size_moves_records_only_at_rounding(prec, largest):
    res = _runs(_warm(bcc_block(cells=24, n_steps=100)), prec, [{"tile_sites": t} for t in (0, 512, largest)])
    for S, m, E in res[1:]:
        assert np.array_equal(S, res[0][0])
        assert np.allclose(m, res[0][1], rtol=0, atol=1e-13) and np.allclose(E, res[0][2], rtol=1e-13, atol=0)


def _long(L=12):
    w = _warm(long_range_sc(L=L, r_cut=4.5))
    S = np.random.default_rng(L).standard_normal((w.n, 3)) * 0.3 + [0.0, 0.0, 1.0]
    w.S0 = S / np.linalg.norm(S, axis=1, keepdims=True)
    return w


@pytest.mark.parametrize("prec", [sl.FP32, sl.FP64])
def test_wide_rows_match_oracle_in_every_form(prec):
    """388 links per site: the wide stencil and the SELL form, near links from
    the LDS window or every link from memory, give the same bits, and the
    oracle's trajectory to rounding."""
    w = _long()
    S_ref = w.S0.copy()
    m_ref, E_ref = oracle.System(w).integrate(S_ref, 0, 60)
    variants = [{}, {"lds_window": 0}, {"stencil": 0}, {"stencil": 0, "lds_window": 0}]
    res = _runs(w, prec, variants, fmt=2)
    bound = 1e-12 if prec == sl.FP64 else 2e-5
    for options, (S, m, E) in zip(variants, res):
        assert max_angle(S, S_ref) < bound, options
        assert np.abs(m - m_ref).max() < bound and (np.abs(E - E_ref) / np.abs(E_ref)).max() < bound, options
    for a, b in ((0, 1), (2, 3)):
        assert all(np.array_equal(x, y) for x, y in zip(res[a], res[b])), variants[b]


@pytest.mark.parametrize("fused", [0, 1])
def test_long_range_steps_at_full_size(fused):
    """64^3 spins, 388 links a site: the wide two-launch step and the
    long-range step, every site after 3 steps."""
    w = _long(64)
    S_ref = w.S0.copy()
    oracle.System(w).integrate(S_ref, 0, 3, record=False)
    for prec, bound in ((sl.FP64, 1e-14), (sl.FP32, 5e-6)):
        with sl.from_workload(w, precision=prec, check_symmetry=False) as g:
            g.set_option("fused", fused)
            assert g.get_option("brick_active") == fused and g.get_option("neighbour_format") == 2
            g.integrate(3, record=False)
            assert max_angle(g.get_spins(), S_ref) <= bound
