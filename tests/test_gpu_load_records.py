"""Caller-supplied starts are checked and laid out on the device: each kind of
fault is refused with the message of the first faulty event, wherever it sits
among valid ones; what is valid (also closed loops, self-closed gluons, starts
that begin inside longer arrays and a long record) comes back
parton for parton when the cutoff leaves no phase space."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2403_08692_amd as P

    c = P.Context()
    yield c
    c.close()


def _pair(axis=2):
    p = np.zeros((2, 4))
    p[:, 0] = 10.0
    p[0, 1 + axis], p[1, 1 + axis] = 10.0, -10.0
    return p, [2, -2], [7, 0], [0, 7]


def _pack(ev):
    off = np.cumsum([0] + [len(x[1]) for x in ev]).astype(np.uint64)
    return (off, np.concatenate([x[0] for x in ev]), np.concatenate([x[1] for x in ev]).astype(np.int8),
            np.concatenate([x[2] for x in ev]).astype(np.uint16), np.concatenate([x[3] for x in ev]).astype(np.uint16))


def _faulty(kind):
    p, pid, col, acol = _pair()
    if kind == "flavour":
        pid = [6, -2]
    elif kind == "quark anticolour":
        acol = [7, 7]
    elif kind == "gluon colour":
        pid, col, acol = [21, -2], [7, 0], [0, 7]
    elif kind == "label":
        col, acol = [2049, 0], [0, 2049]
    elif kind == "open line":
        acol = [0, 8]
    elif kind == "line used twice":
        p, pid, col, acol = np.vstack([p, p]) / 2, [1, -1, 1, -1], [7, 0, 7, 0], [0, 7, 0, 7]
    elif kind == "energy":
        p = -p
    elif kind == "nan energy":
        p = p.copy()
        p[1, 0] = np.nan
    elif kind == "one parton":
        p, pid, col, acol = p[:1], pid[:1], col[:1], acol[:1]
    elif kind == "too many partons":
        p, pid, col, acol = np.vstack([p] * 40), pid * 40, col * 40, acol * 40
    return p, pid, col, acol


@pytest.mark.parametrize("at", [0, 37, 299])
@pytest.mark.parametrize("kind,message", [
    ("flavour", "parton 0: bad flavour/colour"), ("quark anticolour", "parton 0: bad flavour/colour"),
    ("gluon colour", "parton 0: bad flavour/colour"), ("label", "parton 0: bad flavour/colour"),
    ("open line", "colour line 7 is not closed once"), ("line used twice", "colour line 7 is not closed once"),
    ("energy", "total energy must be > 0"), ("nan energy", "total energy must be > 0"),
    ("one parton", "parton count must be in 2..max_partons"),
    ("too many partons", "parton count must be in 2..max_partons"),
])
def test_faults_are_refused(ctx, kind, message, at):
    import paper_2403_08692_amd as P

    ev = [_pair(k % 3) for k in range(300)]
    ev[at] = _faulty(kind)
    if at < 290:
        ev[290] = _faulty("open line")  # a later fault is not the one reported
    print(f"case refused start {kind} at {at}", flush=True)
    with pytest.raises(P.VshError) as ei:
        ctx.shower_records(*_pack(ev), t_cut=1.0, max_partons=64)
    assert ei.value.code == -1
    assert f"event {at}" in str(ei.value) and message in str(ei.value)


@pytest.mark.parametrize("n", [1, 15, 16, 17, 4099])
def test_valid_starts_come_back(ctx, n):
    ev = [_pair(k % 3) for k in range(n)]
    p, pid, col, acol = _pair()
    ev[n // 2] = (p, [21, 21], [3, 4], [4, 3])  # a closed loop
    if n > 4:  # self-closed gluons beside a pair
        ev[n // 3] = (np.vstack([p, p]), [1, -1, 21, 21], [7, 0, 9, 5], [0, 7, 9, 5])
    off, p, pid, col, acol = _pack(ev)
    # the arrays may hold more than the request's events
    pad = 5
    P4, PI, C, A = np.vstack([np.full((pad, 4), np.nan), p]), np.r_[[99] * pad, pid], np.r_[[9] * pad, col], np.r_[[9] * pad, acol]
    print(f"case valid starts n={n}", flush=True)
    g = ctx.shower_records(off + np.uint64(pad), P4, PI, C, A, t_cut=1e4, max_partons=4)
    np.testing.assert_array_equal(g["rec_offsets"], off)
    np.testing.assert_array_equal(g["rec_p"], p)
    np.testing.assert_array_equal(g["rec_pid"], pid)
    np.testing.assert_array_equal(g["rec_col"], col)
    np.testing.assert_array_equal(g["rec_acol"], acol)
    assert g["n_done"] == n and (g["sum_d"][0] == 1.0).all() and (g["sum_d"][[1, 9]] == 0.0).all()
    assert (g["sum_i"][4] == 0).all()


def test_long_record(ctx):
    # one chain of 512 partons: quark, 1022 gluons, antiquark (scaled so
    # that the cutoff leaves no phase space)
    n = 512
    rng = np.random.default_rng(4)
    v = rng.normal(size=(n // 2, 3))
    v = np.vstack([v, -v])
    p = np.column_stack([np.linalg.norm(v, axis=1), v])
    pid, col, acol = [1] + [21] * (n - 2) + [-1], list(range(1, n)) + [0], [0] + list(range(1, n))
    print("case long record", flush=True)
    g = ctx.shower_records(*_pack([(p, pid, col, acol)]), t_cut=1e8, max_partons=n)
    np.testing.assert_array_equal(g["rec_p"], p)
    np.testing.assert_array_equal(g["rec_acol"], np.array(acol, np.uint16))
    assert g["sum_i"][0, 0] == n and g["sum_i"][2, 0] == 1
