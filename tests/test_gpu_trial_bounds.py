"""The flattened kernels rank a cycle's trials by single-precision bounds and
compare exactly where those do not prove the order (a few cycles in 10^6);
the one-lane mapping compares every trial exactly.  Enough cycles for tens of
such cases of each kind: both mappings give the same winners (the hash chains
every emission's kernel, splitter and spectator) and, for massless events, the
same bits throughout (the mappings round a massive emission's kinematics
differently in a few events in 10^4)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2403_08692_amd as P

    c = P.Context()
    was = c.get_tuning()
    yield c
    c.set_tuning(**{k: v for k, v in was.items() if k != "from_cache"})
    c.close()


@pytest.mark.parametrize("persistent", [False, True])
@pytest.mark.parametrize("n,ecm,tcut,cap,massive", [
    (600_000, 91.2, 1.0, 64, False),
    (120_000, 500.0, 0.25, 128, False),
    (120_000, 500.0, 0.25, 256, False),
    (300_000, 200.0, 0.5, 64, True),
    (120_000, 200.0, 0.5, 128, True),
])
def test_bounds_pick_the_exact_winner(ctx, persistent, n, ecm, tcut, cap, massive):
    kw = dict(seed=77, ecm=ecm, t_cut=tcut, max_partons=cap, persistent=persistent,
              mass_c=1.5 if massive else 0.0, mass_b=4.8 if massive else 0.0)
    got = []
    for mapping in (0, 1):
        ctx.set_tuning(mapping=mapping, plain_mapping=mapping)
        print(f"case bounds n={n} ecm={ecm} cap={cap} massive={massive} persistent={persistent} mapping={mapping}",
              flush=True)
        got.append(ctx.generate(n, **kw))
    for key in ("sum_i", "hash") if massive else ("sum_i", "hash", "sum_d"):
        np.testing.assert_array_equal(got[0][key], got[1][key])
