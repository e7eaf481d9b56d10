"""Results on the host live in pinned blocks that later calls use again: arrays
of one result keep their values while other calls run, in any order of their
going, past the context, from several threads, beyond the blocks' bound, and a
request processed in pieces gives the arrays of the same request in one."""
import gc
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

KEYS = ("sum_d", "sum_i", "hash", "rec_offsets", "rec_p", "rec_pid", "rec_col", "rec_acol")


def _copy(r):
    return {k: np.array(r[k]) for k in KEYS if k in r}


def _same(r, ref):
    for k, v in ref.items():
        np.testing.assert_array_equal(r[k], v)


def test_results_outlive_later_calls_and_the_context():
    import paper_2403_08692_amd as P

    ctx = P.Context(0)
    held = []
    for k, n in enumerate((1, 100, 5003, 30_011, 30_011, 5003)):
        r = ctx.generate(n, seed=k, records=True, persistent=k % 2 == 1)
        held.append((r, _copy(r)))
        if k == 3:
            del held[1]  # its blocks go back and are used again
            gc.collect()
    col = held[-1][0]["sum_d"][3]  # a view of a view keeps the result
    want = col.copy()
    ctx.close()
    for r, ref in held:
        _same(r, ref)
    held.clear()
    del r
    gc.collect()
    np.testing.assert_array_equal(col, want)
    col += 1.0  # the caller's to write
    assert (col == want + 1.0).all()


def test_more_results_than_the_blocks_hold():
    import paper_2403_08692_amd as P

    # 10^6 events: 116 MB of summaries each, twelve at once exceed 1 GiB
    with P.Context(0) as ctx:
        a = ctx.generate_isr(1_000_000, seed=1)
        ref = _copy(a)
        held = [ctx.generate_isr(1_000_000, seed=1) for _ in range(11)]
        for r in held:
            _same(r, ref)


def test_threads_share_a_context():
    import paper_2403_08692_amd as P

    with P.Context(0) as ctx:
        want = {s: _copy(ctx.generate(4000, seed=s)) for s in range(4)}
        bad = []

        def work(s):
            for _ in range(6):
                r = ctx.generate(4000, seed=s)
                if any(not np.array_equal(r[k], v) for k, v in want[s].items()):
                    bad.append(s)

        th = [threading.Thread(target=work, args=(s,)) for s in range(4)]
        [t.start() for t in th]
        [t.join() for t in th]
        assert not bad


@pytest.mark.parametrize("call", ["plain", "batched", "isr"])
def test_pieces_equal_one_piece(call):
    import paper_2403_08692_amd as P

    def run(ctx):
        if call == "isr":
            return ctx.generate_isr(20_000, seed=2, records=True)
        return ctx.generate(20_000, seed=2, records=True, persistent=call == "batched")

    with P.Context(0) as ctx:
        ref = run(ctx)
    # a budget for a third or so of the events at a time
    budget = {"plain": 80 << 20, "batched": 1350 << 20, "isr": 40 << 20}[call]
    with P.Context(0, mem_budget_bytes=budget) as ctx:
        _same(run(ctx), {k: ref[k] for k in KEYS})
