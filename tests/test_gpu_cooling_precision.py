"""Rounding of the cooling of reaction 2 in cold gas, against the formulas in
extended precision.  Its two limits are powers of ten with exponents of up to
24 in magnitude.  Such an exponent rounds to a unit of 3.6e-15 two or three
times on its way, 1e-15 rms each, so its power cannot be known better than
ln(10) sqrt(3) 1e-15 = 4e-15 rms; the bound is one and a half times that."""
import numpy as np
import pytest

from paper_1608_08748_amd import binding

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    torch.cuda.set_device(0)


def _gain_minus_loss(T, nH, nH2):
    """The appendix heating and cooling of reactions 1-4 (each constant as FP64 holds it)."""
    L = np.longdouble
    log, exp, log10 = np.log, np.exp, np.log10
    n = nH + nH2
    x = log10(T / 10000)
    t2 = T / 100
    k1 = L(3e-17) * np.sqrt(t2) / (1 + L(0.4) * np.sqrt(t2) + L(0.2) * t2 + L(0.08) * t2 * t2)
    ncr = L(10) ** (4 - L(0.416) * x - L(0.327) * x * x)
    g1 = L(7.2e-12) * k1 * n * nH / (1 + ncr / n)
    g4 = L(6.4e-13) * L(3.3) * L(1.7e-11) * nH2
    assert (T < 1087).all()
    lh = L(10) ** (-L(19.24) + L(0.474) * x - L(1.247) * x * x)
    ll = (nH2 ** L(0.77) + L(1.2) * nH ** L(0.77)) * L(10) ** (-L(22.9) - L(0.553) * x - L(1.148) * x * x)
    l2 = nH2 * lh / (1 + lh / ll)

    def lnf(t):
        a = 1 + 1 / (L(8.617333262e-5) * t)
        return log(t) / 2 + log(a) - a

    ln_ll = log(L(8.18e-13)) + log(n) + log(L(6.29e-15) * L(1.38)) + lnf(T) - lnf(L(4500))
    ln_lh = log(L(1.1e-13)) - 6744 / T
    l3 = nH2 * exp(ln_lh) / (1 + exp(ln_lh - ln_ll))
    return g1 + g4 - l2 - l3


@pytest.mark.skipif(np.finfo(np.longdouble).eps > 1e-18, reason="no extended precision here")
def test_cooling_of_cold_gas():
    L = np.longdouble
    nu, Tu, tu = 1e4, binding.DEFAULT_UNITS[1], binding.DEFAULT_UNITS[2]
    shape, n = (4, 32, 32), 4096
    T = np.linspace(600.0, 1050.0, n)
    U = np.zeros((binding.NFIELDS, n))
    U[0], U[9] = 1.0, 0.98
    U[5] = T * (1.0 - 0.49) / (Tu * (5.0 / 3.0 - 1.0))
    U[4] = U[5]
    box = binding.Box(shape, units=(nu, Tu, tu), chemistry=False, cooling=True)
    e = U[5].astype(L)
    h2 = U[9].astype(L)
    Te = L(Tu) * (L(5.0 / 3.0) - 1) * e / (1 - h2 / 2)
    rate = _gain_minus_loss(Te, L(nu) * (1 - h2), L(nu) * h2 / 2) * L(tu) / (L(nu) * L(1.380649e-16) * L(Tu))
    assert (rate < 0).all()
    rel = []
    for dt in 0.5 * np.quantile(np.asarray(-e / rate, dtype=float), [0.02, 0.3, 0.7]):
        box.set_state(U.reshape((binding.NFIELDS,) + shape))
        box.debug_stage(binding.STAGE_TAIL, float(dt))
        got = box.get_state()[5].reshape(n)
        de = rate * L(float(dt))
        some = (de < -0.05 * e) & (de > -0.8 * e)
        assert some.sum() > 200
        rel.append(np.asarray(((got - e) - de) / de, dtype=float)[some])
    rel = np.concatenate(rel)
    print("cooling: rms %.2e max %.2e of %d cells" % (np.sqrt((rel ** 2).mean()), np.abs(rel).max(), len(rel)))
    assert np.sqrt((rel ** 2).mean()) <= 6e-15


def test_cooling_where_the_limits_underflow():
    # reaction 2's limits leave the normal range together between 1e-12 and
    # 1e-11 K; their quotient is finite there as elsewhere
    import oracle
    shape, n = (4, 16, 16), 1024
    T = np.geomspace(3e-13, 1e-9, n)
    U = np.zeros((binding.NFIELDS, n))
    U[0], U[9] = 1.0, 0.3
    U[5] = T * (1.0 - 0.15) / (binding.DEFAULT_UNITS[1] * (5.0 / 3.0 - 1.0))
    U[4] = U[5]
    U = U.reshape((binding.NFIELDS,) + shape)
    P = oracle.make_params(shape, chemistry=False, cooling=True)
    V = U.copy()
    oracle.cooling(P, V, 1e-6)
    box = binding.Box(shape, chemistry=False, cooling=True)
    box.set_state(U)
    box.debug_stage(binding.STAGE_TAIL, 1e-6)
    e, want = box.get_state()[5], V[5]
    there = np.isfinite(want)
    assert there.sum() > n // 2
    assert (np.abs(e - want)[there] <= 1e-12 * np.abs(want)[there]).all()
