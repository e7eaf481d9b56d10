"""The initial-state shower gives an event 16 to 2 lanes, by the number of
events.  Whichever it is, an event has the same bits: requests on either side
of each step against the first events of the largest, also where records
overflow and where final states outgrow a lane group's registers."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2403_08692_amd as P

    c = P.Context()
    yield c
    c.close()


@pytest.mark.parametrize("cap,tcut", [(64, 0.3), (64, 1.0), (6, 1.0), (3, 1.0)])
def test_events_do_not_depend_on_the_lanes(ctx, cap, tcut):
    kw = dict(seed=17, max_partons=cap, t_cut=tcut, records=True)
    full = ctx.generate_isr(131_073, **kw)
    if tcut < 1.0:
        assert full["sum_i"][0].max() > 2 + 16  # more than sixteen final-state partons
    for n in (1, 17, 4096, 4097, 32_768, 32_769, 131_072):
        print(f"case lanes n={n} cap={cap} tcut={tcut}", flush=True)
        g = ctx.generate_isr(n, **kw)
        np.testing.assert_array_equal(g["sum_i"], full["sum_i"][:, :n])
        np.testing.assert_array_equal(g["hash"], full["hash"][:n])
        np.testing.assert_array_equal(g["sum_d"], full["sum_d"][:, :n])
        m = int(g["rec_offsets"][-1])
        for k in ("rec_p", "rec_pid", "rec_col", "rec_acol"):
            np.testing.assert_array_equal(g[k], full[k][:m])
        assert g["hist"][:4, :, 2].sum(1).tolist() == [g["n_done"]] * 4
