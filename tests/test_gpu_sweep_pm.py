"""The +-J sweep kernel against the oracle where its forms and branches change:
workgroups with several tiles (L <= 8) with a part-filled last workgroup and a
part-filled last tile, one tile on four and on eight waves with full, part and
single-group chunks, the pass at inverse temperatures where an energy-raising
move has a threshold of 2^32, a threshold of 0 for every move, and a copy step
whose sources lie in one, several and many old tiles.  Spins, energy words and
family labels must be equal, bit for bit."""
import numpy as np
import pytest

import oracle
import pa_inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pam():
    import paper_1711_02146_amd as m

    yield m
    m.pa_autotune_reset()


def pair(pam, L, R, seed, layout):
    J = pa_inputs.couplings_pm(L, 31 + L)
    return pam.Population(L, R, J, seed, layout=layout), oracle.Population(L, J, R, seed)


def assert_state(g, o):
    s, u, f = g.export_state()
    assert s.shape[0] == o.R_tilde
    np.testing.assert_array_equal(s.reshape(-1), o.spins)
    np.testing.assert_array_equal(u.astype(np.int32), o.U)
    np.testing.assert_array_equal(f, o.fam)


# sizes on either side of the packed form's workgroups: 4 tiles at L = 4 and 6
# (from 1500 tiles), 2 at L = 8 (from 3200)
@pytest.mark.parametrize("layout", ["int8", "bitpack64"])
@pytest.mark.parametrize("L,R", [(4, 1), (4, 64 * 5 + 1), (4, 64 * 600 + 3), (6, 64 * 1499),
                                 (6, 64 * 1501 + 33), (8, 64 * 3199 + 1), (8, 64 * 3201 + 1)])
def test_packed_forms(pam, layout, L, R):
    pam.pa_autotune_reset()
    g, o = pair(pam, L, R, 77 + R, layout)
    for b in (0.3, 0.6):
        g.resample(b)
        o.resample(b)
        g.sweep(b, 1)
        o.sweep(b, 1)
    assert_state(g, o)
    g.close()


@pytest.mark.parametrize("split", [4, 8])
@pytest.mark.parametrize("L", [4, 6, 8, 10, 12, 14, 16])
@pytest.mark.parametrize("beta", [0.0, 1e-17, 3e-17, 0.7, 20.0])
def test_forms_and_thresholds(pam, L, split, beta):
    R = 70
    pam.pa_autotune_set(L, R, split)
    g, o = pair(pam, L, R, 5 * L, "bitpack64")
    g.sweep(beta, 2)
    o.sweep(beta, 2)
    assert_state(g, o)
    pam.pa_autotune_reset()
    g.close()


@pytest.mark.parametrize("layout", ["int8", "bitpack64"])
@pytest.mark.parametrize("L,dbeta", [(4, 0.05), (4, 1.0), (6, 0.4), (8, 0.25), (10, 0.3), (10, 1.5)])
def test_copy_step_spread(pam, layout, L, dbeta):
    """dbeta from a few per cent culled to a handful of survivors: the 64
    sources of a new tile lie in two, several or very many old tiles."""
    R = 5000
    g, o = pair(pam, L, R, 9 * L + 1, layout)
    g.resample(dbeta)
    o.resample(dbeta)
    g.sweep(dbeta, 1)
    o.sweep(dbeta, 1)
    assert_state(g, o)
    g.close()


@pytest.mark.parametrize("layout", ["int8", "bitpack64"])
@pytest.mark.parametrize("split", [4, 8])
@pytest.mark.parametrize("L", [4, 6, 8, 10, 12, 14, 16])
def test_infinite_temperature(pam, L, split, layout):
    """beta = 0, where every move is taken: odd and even numbers of sweeps, with
    and without a pending copy step, then sweeps with draws."""
    R = 70
    pam.pa_autotune_set(L, R, split, layout=layout)
    g, o = pair(pam, L, R, 3 * L, layout)
    for resample, beta, n in ((None, 0.0, 1), (None, 0.0, 2), (0.4, 0.0, 3), (None, 0.5, 1)):
        for p in (g, o):
            if resample is not None:
                p.resample(resample)
            p.sweep(beta, n)
        assert_state(g, o)
    pam.pa_autotune_reset()
    g.close()


def test_infinite_temperature_is_not_slower(pam):
    """Ten sweeps at beta = 0 take no longer than ten with draws (through the pass
    that serves any threshold they took three to five times as long)."""
    import time

    import torch

    s = torch.cuda.Stream()
    g = pam.Population(8, 20000, pa_inputs.couplings_pm(8, 1), 1, layout="bitpack64", stream=s)

    def ms(beta):
        best = 1e9
        for _ in range(6):
            s.synchronize()
            t0 = time.perf_counter()
            for _ in range(10):
                g.sweep(beta, 10)
            s.synchronize()
            best = min(best, 1e3 * (time.perf_counter() - t0))
        return best

    with_draws = ms(0.7)
    assert ms(0.0) < 1.2 * with_draws
    g.close()


# the packed kernels of L = 6 (a tile per wave) and 8 (two waves per tile) at their own
# sizes, with a part-filled last workgroup and last tile; L = 4 packs at any size
@pytest.mark.parametrize("layout", ["int8", "bitpack64"])
@pytest.mark.parametrize("L,R,few", [(4, 64 * 9 + 5, 2.0), (6, 64 * 1501 + 33, 1.2),
                                     (8, 64 * 3201 + 1, 0.8)])
def test_packed_forms_every_branch(pam, layout, L, R, few):
    """A threshold of 2^32 for every move (beta = 0, odd and even numbers of sweeps) and
    for some (1e-17), the largest below 2^32 (3e-17), a copy step to a handful of
    survivors (sources spread over many old tiles) and all thresholds 0 (beta = 20)."""
    pam.pa_autotune_set(L, R, 4, layout=layout)
    g, o = pair(pam, L, R, 41 + L, layout)
    for resample, beta, n in ((None, 0.0, 1), (None, 0.0, 2), (None, 1e-17, 1), (None, 3e-17, 1),
                              (few, few, 1), (None, 20.0, 1)):
        for p in (g, o):
            if resample is not None:
                p.resample(resample)
            p.sweep(beta, n)
        assert_state(g, o)
    pam.pa_autotune_reset()
    g.close()
