"""The Gaussian sweep kernel with its threshold table in LDS (L <= 10), on several
tiles per workgroup (split 4) and on one (split 8, where a wave may have no sites),
against the oracle: part-filled last tiles and workgroups, more tiles than the resident workgroups take at once,
inverse temperatures at which every threshold is 2^32, shares its upper half with
most others, or is 0 (the draws that only the exact threshold decides: one in
2^16), and a copy step whose sources lie in one, several and many old tiles.
Spins, energy words and family labels must be equal, bit for bit."""
import numpy as np
import pytest

import oracle
import pa_inputs

pytestmark = pytest.mark.gpu

MODELS = {"gauss16": ("couplings_gauss16", "GaussPopulation"),
          "gauss": ("couplings_gauss", "GaussRealPopulation")}


@pytest.fixture(scope="module")
def pam():
    import paper_1711_02146_amd as m

    yield m
    m.pa_autotune_reset()


def pair(pam, model, L, R, seed, layout):
    couplings, population = MODELS[model]
    J = getattr(pa_inputs, couplings)(L, 31 + L)
    return (pam.Population(L, R, J, seed, layout=layout, model=model),
            getattr(oracle, population)(L, J, R, seed))


def assert_state(g, o):
    s, u, f = g.export_state()
    assert s.shape[0] == o.R_tilde
    np.testing.assert_array_equal(s.reshape(-1), o.spins)
    np.testing.assert_array_equal(np.asarray(u).astype(o.U.dtype), o.U)
    np.testing.assert_array_equal(f, o.fam)


@pytest.mark.parametrize("model", ["gauss16", "gauss"])
@pytest.mark.parametrize("split", [4, 8])
@pytest.mark.parametrize("L", [4, 6, 8, 10])
@pytest.mark.parametrize("beta", [0.0, 1e-17, 1e-6, 0.7, 30.0])
def test_forms_and_thresholds(pam, model, L, split, beta):
    R = 64 * 3 + 7
    pam.pa_autotune_set(L, R, split, layout="bitpack64", model=model)
    g, o = pair(pam, model, L, R, 5 * L, "bitpack64")
    g.sweep(beta, 2)
    o.sweep(beta, 2)
    assert_state(g, o)
    pam.pa_autotune_reset()
    g.close()


# tiles past those that the resident workgroups take at once, and sizes on either
# side of the default rule
@pytest.mark.parametrize("model", ["gauss16", "gauss"])
@pytest.mark.parametrize("layout", ["int8", "bitpack64"])
@pytest.mark.parametrize("L,R", [(4, 64 * 899), (4, 64 * 4097 + 1), (6, 64 * 1098 + 1), (6, 64 * 2049),
                                 (8, 64 * 1027 + 63), (8, 64 * 1600), (10, 64 * 256),
                                 (10, 64 * 257 + 5), (10, 64 * 513 + 1), (10, 64 * 770)])
def test_sizes(pam, model, layout, L, R):
    pam.pa_autotune_reset()
    g, o = pair(pam, model, L, R, 77 + L, layout)
    g.sweep(0.3, 1)
    o.sweep(0.3, 1)
    g.resample(0.35)
    o.resample(0.35)
    g.sweep(0.35, 1)
    o.sweep(0.35, 1)
    assert_state(g, o)
    g.close()


@pytest.mark.parametrize("model", ["gauss16", "gauss"])
@pytest.mark.parametrize("L,dbeta", [(6, 0.05), (6, 1.0), (10, 0.1), (10, 1.0)])
def test_copy_step_spread(pam, model, L, dbeta):
    R = 5000
    pam.pa_autotune_set(L, R, 4, layout="bitpack64", model=model)
    g, o = pair(pam, model, L, R, 9 * L + 1, "bitpack64")
    g.resample(dbeta)
    o.resample(dbeta)
    pam.pa_autotune_set(L, o.R_tilde, 4, layout="bitpack64", model=model)
    g.sweep(dbeta, 1)
    o.sweep(dbeta, 1)
    assert_state(g, o)
    pam.pa_autotune_reset()
    g.close()
