"""Records gathered by 128 consecutive events per block, below 32 MiB straight
into the result's pinned block and above through device memory: an event's
record is the same whatever the size of the call, and follows its summary."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", ["plain", "batched", "isr"])
def test_records_do_not_depend_on_the_call(form):
    import paper_2403_08692_amd as P

    ctx = P.Context()

    def call(n):
        print(f"case gather form={form} n={n}", flush=True)
        if form == "isr":
            return ctx.generate_isr(n, seed=4, records=True)
        return ctx.generate(n, seed=4, records=True, persistent=form == "batched")

    ref = call(400_001)  # above the direct path's bound
    keys = ("rec_p", "rec_pid", "rec_col", "rec_acol")
    assert sum(np.asarray(ref[k]).nbytes for k in keys) > 32 << 20
    for n in (1, 127, 128, 129, 257, 20_000):
        got = call(n)
        off = np.asarray(got["rec_offsets"])
        np.testing.assert_array_equal(off, np.asarray(ref["rec_offsets"])[: n + 1])
        np.testing.assert_array_equal(np.diff(off.astype(np.int64)), got["sum_i"][0])
        for k in keys:
            np.testing.assert_array_equal(got[k], np.asarray(ref[k])[: len(got[k])])
            assert len(got[k]) == off[-1]
    ctx.close()
