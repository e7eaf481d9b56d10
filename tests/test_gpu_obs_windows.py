"""The one-thread-per-event observables take a 256-event window per block up to
262144 events and windows of 192 or 256 per wave beyond: an event's values do
not depend on which (nor on its neighbours), and every event is counted once."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("massive", [False, True])
def test_events_do_not_depend_on_the_window(massive):
    import paper_2403_08692_amd as P

    ctx = P.Context()
    kw = dict(seed=12, ecm=91.2, t_cut=1.0, max_partons=64, mass_c=1.5 if massive else 0.0,
              mass_b=4.8 if massive else 0.0)
    ref = ctx.generate(100_003, **kw)
    for n in (262_144, 262_145, 393_217, 1_048_577):
        print(f"case windows n={n} massive={massive}", flush=True)
        got = ctx.generate(n, **kw)
        for key in ("sum_i", "sum_d"):
            np.testing.assert_array_equal(got[key][:, :100_003], ref[key])
        assert got["n_done"] == n
        w = got["sum_d"][0]
        # column 2 of a cell counts its entries; every histogram has each event once
        np.testing.assert_array_equal(got["hist"][:7, :, 2].sum(axis=1), np.full(7, float(n)))
        np.testing.assert_allclose(got["hist"][:7, :, 0].sum(axis=1), w.sum(), rtol=1e-10)
    ctx.close()
