"""GPU test of reading large states back: the staged path starts at 2^20
reals and works in pieces of 4 MiB; sizes just below and at its start, a
whole number of pieces, and remainders."""
import numpy as np
import pytest

import paper_1310_6143_amd as sl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [sl.FP32, sl.FP64])
@pytest.mark.parametrize("n", [349525, 349526, 524288, 1048576, 1048577])
def test_large_states_read_back_exactly(n, prec):
    rng = np.random.default_rng(n)
    S = np.zeros((n, 3))                      # signed axis vectors: exact in both precisions
    S[np.arange(n), rng.integers(0, 3, n)] = rng.choice([-1.0, 1.0], n)
    with sl.SpinSystem(n, precision=prec) as s:
        s.set_neighbours(np.zeros(n + 1, dtype=np.int64), np.zeros(0, dtype=np.int32), None, [0.0])
        s.set_materials(1e-23, 0.0, [0.0, 0.0, 1.0])
        s.set_integrator(0.1, 1.76e11, 1e-16)
        s.set_spins(S)
        s.integrate_dev(0)                    # onto the device
        assert np.array_equal(s.get_spins(), S)
        assert np.array_equal(s.get_spins(), S)


@pytest.mark.parametrize("prec", [sl.FP32, sl.FP64])
@pytest.mark.parametrize("n", [349526, 699050, 699051])
def test_first_and_later_reads_agree(prec, n):
    """From 2^20 reals the second read of a system is staged, from 2^21 the
    first one too: sizes on both sides of the second line, read three times
    with a changed state in between."""
    S = np.zeros((n, 3))
    S[np.arange(n), np.arange(n) % 3] = np.where(np.arange(n) % 5 < 2, -1.0, 1.0)
    with sl.SpinSystem(n, precision=prec) as s:
        s.set_neighbours(np.zeros(n + 1, dtype=np.int64), np.zeros(0, dtype=np.int32), None, [0.0])
        s.set_materials(1e-23, 0.0, [0.0, 0.0, 1.0])
        s.set_integrator(0.1, 1.76e11, 1e-16)
        s.set_spins(S)
        s.integrate_dev(0)
        for k in range(3):
            assert np.array_equal(s.get_spins(), S), k
            S = np.roll(S, 1, axis=1)
            s.set_spins(S)
