"""Without records, the initial-state kernel writes its summaries straight into
the result's pinned block; with records they pass through device memory.  Same
bits either way, at the sizes around a wave's events for each split (16, 8, 4
and 2 lanes per event), with earlier results still held."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_direct_summaries_have_the_same_bits():
    import paper_2403_08692_amd as P

    ctx = P.Context()
    held = []
    for n in (1, 4, 5, 63, 4096, 4097, 32_769, 131_073):
        print(f"case isr direct n={n}", flush=True)
        direct = ctx.generate_isr(n, seed=3, first_event=n)
        through = ctx.generate_isr(n, seed=3, first_event=n, records=True)
        held.append((direct, through))
    for direct, through in held:
        for key in ("sum_d", "sum_i", "hash"):
            np.testing.assert_array_equal(direct[key], through[key])
        np.testing.assert_allclose(direct["hist"], through["hist"], rtol=1e-9, atol=0)
        assert direct["n_done"] == through["n_done"] and direct["total_cycles"] == through["total_cycles"]
    ctx.close()
