"""Each layout of the flattened kernels with 64 events in every wave against
the same events in launches that spread a few to a wave: an event's summary has
the same bits in both.  The full launch has 64 events for each of the sixteen
blocks per compute unit that any of the kernels reaches, so it stays full
whatever the rule of the split; the small ones hold 1, 2, ... to a wave under
any rule between four and sixteen blocks per compute unit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

KEYS = ("sum_i", "hash", "sum_d")


@pytest.fixture(scope="module")
def ctx():
    import paper_2403_08692_amd as P

    with P.Context(0) as c:
        yield c


@pytest.mark.parametrize("persistent", [False, True])
@pytest.mark.parametrize("cap,massive", [(64, False), (128, False), (256, False), (64, True), (128, True), (256, True)])
def test_full_waves_equal_sparse_ones(ctx, persistent, cap, massive):
    import torch

    cus = torch.cuda.get_device_properties(0).multi_processor_count
    kw = dict(seed=6, ecm=200.0 if cap > 64 else 91.2, t_cut=0.5 if cap > 64 else 1.0, max_partons=cap, t_over=10.0,
              persistent=persistent, mass_c=1.5 if massive else 0.0, mass_b=4.8 if massive else 0.0)
    full = 64 * 16 * cus + 3
    print(f"case full waves cap={cap} massive={massive} persistent={persistent} n={full}", flush=True)
    ref = ctx.generate(full, **kw)
    for n in (1, 4 * cus, 12 * cus, 12 * cus + 1, 16 * cus + 1, 48 * cus + 1, 160 * cus + 1, 640 * cus + 1):
        print(f"case sparse waves cap={cap} massive={massive} persistent={persistent} n={n}", flush=True)
        got = ctx.generate(n, **kw)
        for k in KEYS:
            np.testing.assert_array_equal(got[k], ref[k][..., :n])
