"""GPU parity of the brick step (one launch per Heun step on small crystals)
against the FP64 oracle, at the edges of its bricks: lattices of one brick,
of bricks cut on every axis, of the fewest cells an axis may have, and with
an open surface inside a brick.

Bounds: 40 steps accumulate at most a few dozen rounding errors per spin
component (2^-53 and 2^-24), well below 1e-12 and 2e-5; m and E are sums of
such terms.
"""
import numpy as np
import pytest

import oracle
import paper_1310_6143_amd as sl
from spin_systems import bcc_block, bcc_film, sc_reference
from spin_systems.lattice import bcc, simple_cubic
from tests.gpu_util import max_angle

pytestmark = pytest.mark.gpu

# simple cubic bricks are 8 x 8 x 4 cells, bcc ones 8 x 4 x 4
CASES = [("sc", (5, 5, 5)), ("sc open", (8, 8, 4)), ("sc", (9, 7, 6)), ("sc", (17, 5, 13)), ("sc open", (9, 8, 1)),
         ("sc open", (7, 16, 5)), ("bcc8", (8, 8, 8)), ("bcc8", (9, 5, 6)), ("bcc8 open", (5, 9, 2)),
         ("bcc8 open", (16, 6, 7)), ("bcc14", (8, 8, 8)), ("bcc14", (5, 5, 5)), ("bcc14", (11, 7, 9)),
         ("bcc14 open", (9, 6, 5))]


def _workload(kind, dims):
    per = (True, True, "open" not in kind)
    if kind.startswith("sc"):
        w, lat = sc_reference(L=5), simple_cubic(dims, per)
    else:
        second = "14" in kind
        w = bcc_block(cells=5) if second else bcc_film(nx=5, ny=5, nz=5)
        lat = bcc(dims, per, second_neighbours=second)
    n = lat.n
    w.lattice, w.temperature, w.H = lat, 300.0, np.array([0.3, -0.2, 0.5])
    w.mu_s, w.k_u = np.full(n, w.mu_s[0]), np.full(n, w.k_u[0])
    w.easy_axis = np.tile([0.6, 0.0, 0.8], (n, 1))
    S = np.random.default_rng(n).standard_normal((n, 3)) + [0.0, 0.0, 2.0]
    w.S0 = S / np.linalg.norm(S, axis=1, keepdims=True)
    return w


@pytest.mark.parametrize("kind,dims", CASES)
def test_brick_step_matches_oracle(kind, dims):
    w = _workload(kind, dims)
    S_ref = w.S0.copy()
    m_ref, E_ref = oracle.System(w).integrate(S_ref, 0, 40)
    for prec, bound in ((sl.FP64, 1e-12), (sl.FP32, 2e-5)):
        with sl.from_workload(w, precision=prec) as g:
            assert g.get_option("brick_active") == 1 and g.get_option("fused_active") == 0
            m1, E1 = g.integrate(13)
            m2, E2 = g.integrate(27)
            S = g.get_spins()
            assert max_angle(S, S_ref) < bound
            assert np.abs(np.concatenate([m1, m2]) - m_ref).max() < bound
            assert (np.abs(np.concatenate([E1, E2]) - E_ref) / np.abs(E_ref)).max() < bound
        # the two-launch step: the same bits, records summed in another order
        with sl.from_workload(w, precision=prec) as g:
            g.set_option("fused", 0)
            assert g.get_option("brick_active") == 0
            m, E = g.integrate(40)
            assert np.array_equal(S, g.get_spins())
            assert np.abs(np.concatenate([m1, m2]) - m).max() < 1e-13
            assert (np.abs(np.concatenate([E1, E2]) - E) / np.abs(E)).max() < 1e-12


def test_brick_needs_five_cells_on_periodic_axes():
    for dims, on in (((4, 8, 8), 0), ((8, 8, 4), 0), ((5, 8, 5), 1)):
        w = _workload("bcc8", dims)
        with sl.from_workload(w, precision=sl.FP64) as g:
            assert g.get_option("brick_active") == on


def test_brick_chunks_graphs_and_mapping_bitwise():
    """The spins do not depend on how the steps are launched, nor do the
    records (sums over the same bricks in the same order)."""
    w = _workload("bcc8 open", (20, 13, 9))
    out = []
    for graph, remap, calls in ((64, 1, (200,)), (0, 0, (200,)), (16, 2, (7, 130, 63))):
        with sl.from_workload(w, precision=sl.FP32) as g:
            g.set_option("graph_steps", graph)
            g.set_option("xcd_remap", remap)
            parts = [g.integrate(c) for c in calls]
            out.append((g.get_spins(), np.concatenate([p[0] for p in parts]), np.concatenate([p[1] for p in parts])))
    for other in out[1:]:
        assert all(np.array_equal(a, b) for a, b in zip(out[0], other))
