"""A worker that is forked from a program holding results reads them: arrays
that view pinned memory of the library, which the driver does not map into
forked children, have the same values there."""
import multiprocessing

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

KEYS = ("sum_d", "sum_i", "hash", "rec_offsets", "rec_p", "rec_pid", "rec_col", "rec_acol")


def _worker(results, out):
    out.send([[np.array(r[k]) for k in KEYS if k in r] for r in results])
    results[0]["sum_d"][0] = -1.0  # the worker's own
    out.close()


def test_forked_worker_reads_results():
    import paper_2403_08692_amd as P

    fork = multiprocessing.get_context("fork")
    with P.Context(0) as ctx:
        print("case forked worker", flush=True)
        results = [ctx.generate(20_011, seed=3, records=True), ctx.generate_isr(100_003, seed=4)]
        for _ in range(2):
            rx, tx = fork.Pipe(False)
            w = fork.Process(target=_worker, args=(results, tx))
            w.start()
            tx.close()
            got = rx.recv()
            w.join(60)
            assert w.exitcode == 0
            for r, arrays in zip(results, got):
                for k, a in zip((k for k in KEYS if k in r), arrays):
                    np.testing.assert_array_equal(r[k], a)
        again = ctx.generate(20_011, seed=3, records=True)  # the device still serves the parent
        for k in KEYS:
            np.testing.assert_array_equal(again[k], results[0][k])
