"""Requests that finish in one epoch are measured by one set of launches: a
burst of requests (small and large, fixed-point, per-event energies, record
capacities below the lane groups and above 512 partons) gives each the bits of
the same request generated alone.  A massive request among them has the whole
epoch showered by the massive kernels, whose rounding of massless events
differs: there the events' decisions, counts and histories are compared."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2403_08692_amd as P

    c = P.Context()
    yield c
    c.close()


def _requests(massive):
    rng = np.random.default_rng(7)
    r = [dict(n_events=n, seed=k, ecm=91.2, t_cut=1.0, max_partons=64) for k, n in enumerate((1, 255, 256, 257, 40_001))]
    r += [dict(n_events=9_001, seed=20, ecm=200.0, t_cut=0.5, max_partons=128, fixed_hist=True),
          dict(n_events=3_000, seed=21, ecm=91.2, t_cut=1.0, max_partons=64, t_over=10.0,
               **(dict(mass_c=1.5, mass_b=4.8) if massive else {})),
          dict(n_events=2_000, seed=22, ecm=35.0, t_cut=2.0, max_partons=8),
          dict(n_events=700, seed=23, ecm=500.0, t_cut=0.5, max_partons=600),
          dict(n_events=5_000, seed=24, max_partons=128, cycle_limit=30, ecm_per_event=rng.uniform(10, 500, 5_000),
               tcut_per_event=rng.uniform(0.5, 4, 5_000))]
    return r


@pytest.mark.parametrize("rounds,massive", [(1, False), (3, False), (1, True)])
def test_burst_equals_alone(ctx, rounds, massive):
    reqs = _requests(massive) * rounds
    print(f"case burst of {len(reqs)} massive={massive}", flush=True)
    tickets = [ctx.submit(summary=True, **r) for r in reqs]
    got = [ctx.wait(t) for t in tickets]
    for r, g in zip(reqs, got):
        alone = ctx.generate(summary=True, **r)
        np.testing.assert_array_equal(g["sum_i"], alone["sum_i"])
        np.testing.assert_array_equal(g["hash"], alone["hash"])
        assert g["n_done"] == alone["n_done"]
        if massive:
            continue
        np.testing.assert_array_equal(g["sum_d"], alone["sum_d"])
        if r.get("fixed_hist"):
            np.testing.assert_array_equal(g["hist"], alone["hist"])
        else:  # sums of n positive weights in another order: at most n ulp
            np.testing.assert_allclose(g["hist"], alone["hist"], rtol=r["n_events"] * 2.0 ** -52,
                                       atol=0 if "t_over" not in r else 1e-6)
