"""Cells whose hydrogen is all ionised or all molecular after one chemistry
update: the update clamps the number density to the cell's hydrogen and divides
by n_u again, so rho_H2 + rho_H+ ends a unit in the last place above rho in some
of them.  Heating and cooling of such cells is finite and takes n_H as zero."""
import numpy as np
import pytest

import oracle


def ionised(n):
    """Hot atomic gas that one update ionises fully: rho, T, x_H2, x_H+ of n cells."""
    rng = np.random.default_rng(91)
    return rng.uniform(0.2, 5.0, n), rng.uniform(2.5e4, 1e5, n), rng.uniform(0.0, 1e-3, n), rng.uniform(1e-2, 0.3, n)


def molecular(n):
    """Dense cold gas that one update turns fully molecular."""
    rng = np.random.default_rng(92)
    return rng.uniform(0.2, 5.0, n), rng.uniform(50.0, 300.0, n), rng.uniform(0.5, 0.9, n), np.zeros(n)


def full_state(P, cells):
    """Conserved state of a row of these cells at rest, and the energy of each."""
    rho, T, x2, xp = cells
    U = np.zeros((11, 1, 1, len(rho)))
    U[0, 0, 0], U[9, 0, 0], U[10, 0, 0] = rho, x2 * rho, xp * rho
    for c in range(len(rho)):
        g = oracle.gamma_cell(P, rho[c], x2[c] * rho[c], xp[c] * rho[c])
        U[5, 0, 0, c] = T[c] * rho[c] * (1.0 - 0.5 * x2[c] + xp[c]) / (P.T_unit * (g - 1.0))
    U[4] = U[5]
    return U


# (network, cells, n_u, dt): dt long enough that the update reaches its clamp
CASES = [(True, ionised, 5.0, 1e-3), (False, molecular, 1e12, 1.0)]


@pytest.mark.parametrize("network, cells, n_u, dt", CASES)
def test_cooling_of_full_cells(network, cells, n_u, dt):
    n = 2000
    units = (n_u,) + tuple(oracle.default_units()[1:])
    P = oracle.make_params((1, 1, n), units=units, cooling=True, ionisation=network)
    U = full_state(P, cells(n))
    oracle.clamp_h2(P, U)
    oracle.chemistry(P, U, dt)
    rest = U[0] - U[9] - U[10]
    assert np.abs(rest).max() <= 4e-16 * U[0].max()     # all cells are full
    assert (rest < 0).sum() > 10                        # some by one unit too much
    oracle.cooling(P, U, dt)
    assert np.isfinite(U).all()
