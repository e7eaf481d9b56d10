"""The flattened kernels spread a small launch's events over every resident
wave (1 to 64 events per wave).  An event is a pure function of its name, so
its summary has the same bits whatever the number of events beside it: the
first events of a launch with 64 events per wave against the same events in
launches on either side of each step of the split."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2403_08692_amd as P

    c = P.Context()
    yield c
    c.close()


def _same(a, b, n):
    np.testing.assert_array_equal(a["sum_i"][:, :n], b["sum_i"][:, :n])
    np.testing.assert_array_equal(a["hash"][:n], b["hash"][:n])
    np.testing.assert_array_equal(a["sum_d"][:, :n], b["sum_d"][:, :n])


@pytest.mark.parametrize("persistent", [False, True])
@pytest.mark.parametrize("ecm,tcut,cap,massive,full,sizes", [
    (91.2, 1.0, 64, False, 262_200, (1, 17, 4096, 4097, 8193, 65_537, 131_073, 258_049)),
    (200.0, 0.5, 128, False, 229_500, (2, 3584, 3585, 7169)),
    (200.0, 0.5, 256, False, 180_300, (2816, 2817, 30_000)),
    (91.2, 1.0, 64, True, 70_000, (1, 1024, 1025, 64_513)),
])
def test_events_do_not_depend_on_the_split(ctx, persistent, ecm, tcut, cap, massive, full, sizes):
    kw = dict(seed=5, ecm=ecm, t_cut=tcut, max_partons=cap, t_over=10.0, persistent=persistent,
              mass_c=1.5 if massive else 0.0, mass_b=4.8 if massive else 0.0)
    ref = ctx.generate(full, **kw)
    for n in sizes:
        print(f"case split n={n} of {full} ecm={ecm} cap={cap} massive={massive} persistent={persistent}", flush=True)
        _same(ctx.generate(n, **kw), ref, n)


def test_full_waves_past_the_item_list(ctx):
    # long showers, 64 events per wave (one wave per compute unit): a cycle
    # has more items and stale partons than the LDS list holds, against the
    # same events a few to a wave
    kw = dict(seed=8, ecm=500.0, t_cut=0.05, max_partons=256, persistent=True)
    n = 256 * 64
    few = ctx.generate(n, **kw)
    assert few["sum_i"][0].mean() * 64 > 1500
    was = ctx.get_tuning()
    try:
        ctx.set_tuning(waves_per_cu=1)
        print("case full waves past the item list", flush=True)
        full = ctx.generate(n, **kw)
    finally:
        ctx.set_tuning(**{k: v for k, v in was.items() if k != "from_cache"})
    _same(full, few, n)
