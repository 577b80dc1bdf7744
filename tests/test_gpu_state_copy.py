"""pa_import_state and pa_export_state convert on the device through the
population's other buffer: sizes below one staged piece, with a part-filled last
tile and over several pieces, both layouts.  Spins come back as they went in, the
energies are those of the spins, the untouched slots of the last tile are zero for
later sweeps, and a state with a value other than +1 and -1 is refused and changes
nothing."""
import numpy as np
import pytest

import oracle
import pa_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout", ["int8", "bitpack64"])
@pytest.mark.parametrize("L", [4, 6, 16])
@pytest.mark.parametrize("R,held", [(1, 1), (40, 33), (200, 200), (1500, 1153), (1500, 0)])
def test_round_trip(layout, L, R, held):
    import paper_1711_02146_amd as pam

    rng = np.random.default_rng(L * R + held)
    N = L ** 3
    J = pa_inputs.couplings_pm(L, 7)
    g = pam.Population(L, R, J, 3, layout=layout)
    spins = rng.choice(np.array([-1, 1], np.int8), (held, N))
    fam = np.sort(rng.integers(0, R, held)).astype(np.uint32)
    g.import_state(spins, fam, 5, 1, 0.25, 0.5)
    s, u, f = g.export_state()
    np.testing.assert_array_equal(s, spins)
    np.testing.assert_array_equal(f, fam)
    if held:
        bad = spins.copy()
        for at, value in ((0, 0), (-1, 2), (-1, -128), (-1, 127)):
            bad.reshape(-1)[at] = value
            with pytest.raises(Exception):
                g.import_state(bad, fam, 9, 2, 0.5, 0.0)
            bad.reshape(-1)[at] = spins.reshape(-1)[at]
        np.testing.assert_array_equal(g.export_state()[0], spins)
        o = oracle.Population(L, J, R, 3)
        o.spins, o.fam, o.R_tilde, o.t = spins.reshape(-1).copy(), fam.copy(), held, 5
        o.U = u.astype(np.int32)
        g.sweep(0.4, 1)
        o.sweep(0.4, 1)
        s, u, f = g.export_state()
        np.testing.assert_array_equal(s.reshape(-1), o.spins)
        np.testing.assert_array_equal(u.astype(np.int32), o.U)
    g.close()
