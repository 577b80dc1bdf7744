"""pa_choose_beta on the GPU against the oracle's bisection where the search has
little to go by: culling targets from small to nearly everything, populations of
one to a few replicas, equal energies, ranges that end before the crossing."""
import pytest

import oracle
import pa_inputs

pytestmark = pytest.mark.gpu

MODELS = {"pm": ("couplings_pm", "Population", {}),
          "gauss16": ("couplings_gauss16", "GaussPopulation", {"model": "gauss16"}),
          "gauss": ("couplings_gauss", "GaussRealPopulation", {"model": "gauss"})}


@pytest.mark.parametrize("model", ["pm", "gauss16", "gauss"])
@pytest.mark.parametrize("R,target,beta_max", [(1, 0.1, 5.0), (2, 0.3, 5.0), (3, 0.02, 40.0),
                                               (65, 0.5, 5.0), (700, 0.95, 5.0), (700, 0.01, 5.0),
                                               (3000, 0.1, 0.004), (3000, 0.1, 1e-9),
                                               (20011, 0.1, 5.0)])
def test_choose_beta(model, R, target, beta_max):
    import paper_1711_02146_amd as pam

    L = 6
    couplings, population, kw = MODELS[model]
    J = getattr(pa_inputs, couplings)(L, 3)
    g = pam.Population(L, R, J, 11, **kw)
    o = getattr(oracle, population)(L, J, R, 11)
    assert g.choose_beta(target, beta_max) == o.choose_beta(target, beta_max)
    g.sweep(0.4, 3)
    o.sweep(0.4, 3)
    assert g.choose_beta(target, beta_max) == o.choose_beta(target, beta_max)
    g.close()
