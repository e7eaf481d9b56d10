"""Timed cases of the shower engine: the calls that a user of this library makes.

Each case is one call (serving: one burst of requests) through the public entry
points of ``paper_2403_08692_amd``, over the range of sizes, energies, options
and forms of ``workloads.py``, the tests and the benchmark.  ``listed()`` is a
fixed set, ``draw(rng)`` one more case of the same ranges, ``prepare`` what a
program has in hand before the call, ``run`` the call, ``work`` the bytes and
operations it cannot do without and ``exact`` the values that plain NumPy gives
in 64 bits.

An event is named by (seed, event id, sqrt(s), t_C, capacity, options), so the
seed of a case is the request's Philox seed: another seed gives other events.
"""
import math
import random

import numpy as np
import torch

import paper_2403_08692_amd as P
from paper_2403_08692_amd import workloads


def _case(call, n, **kw):
    """A case with the defaults of the calls filled in: call is the entry
    point; form, cap, summary, records, fixed, t_over, cycle_limit, massive and
    mixed are the request's options."""
    c = dict(call=call, n=n, ecm=91.2, tcut=1.0, cap=64, form="plain", summary=True, records=False, fixed=False,
             t_over=0.0, cycle_limit=0, massive=False, mixed=False)
    c.update(kw)
    return c


def listed():
    return [
        # a few events at a time (a notebook, an event display, the smallest
        # requests of the serving trace): launches and latency
        _case("generate", 100, name="lep_100"),
        # the small LEP workload with its event records, as an analysis reads it
        _case("generate", 1000, records=True, name="lep_1e3_records"),
        # a caller that cannot allocate (graph capture, a serving loop of its
        # own), with the weighted veto; a ragged count
        _case("into_static", 5003, t_over=10.0, name="static_5003"),
        # a mid-sized sample at a higher energy, batched, with reproducible
        # histograms, results on the host
        _case("generate", 30011, ecm=200.0, tcut=0.5, cap=128, form="batched", fixed=True, name="batched_30k_fixed"),
        # q g qbar starts from the caller's own generator, records back
        _case("shower_records", 20011, records=True, name="records_20k"),
        # Drell-Yan events with the initial-state shower, summaries on the host
        _case("generate_isr", 200003, name="isr_200k"),
        # charm and bottom masses, results left on the device
        _case("into", 250007, massive=True, name="massive_250k"),
        # the headline sample: 10^6 LEP events per call, in both forms
        _case("into", 1000000, name="lep_1e6_plain"),
        _case("into", 1000000, form="batched", name="lep_1e6_batched"),
        # every event with its own sqrt(s) and t_C (device arrays), ragged count
        _case("into", 3000017, cap=128, form="batched", mixed=True, name="mixed_3e6_batched"),
        # long showers: 500 GeV down to t_C = 0.25
        _case("into", 1000000, ecm=500.0, tcut=0.25, cap=256, name="stress_1e6_plain"),
        # a burst of 32 requests of the serving trace, waited for together
        _case("serve", 32, cap=128, summary=False, name="serving_32"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    call = rng.choice(["generate", "generate", "into", "into", "into_static", "shower_records", "generate_isr", "serve"])
    ecm = rng.choice(list(workloads.SERVING_ENERGIES))
    tcut = rng.choice(list(workloads.SERVING_CUTOFFS))
    if call == "serve":
        return _case(call, rng.randint(4, 40), cap=128, summary=rng.random() < 0.3)
    if call == "generate_isr":
        return _case(call, _log_int(rng, 50, 300000), tcut=tcut, records=rng.random() < 0.2)
    if call == "shower_records":
        return _case(call, _log_int(rng, 30, 30000), ecm=max(ecm, 35.0), tcut=tcut, records=True,
                     massive=rng.random() < 0.2)
    cap = 64 if ecm < 150.0 else rng.choice([128, 256])
    opts = dict(ecm=ecm, tcut=tcut, cap=cap, fixed=rng.random() < 0.3, massive=rng.random() < 0.25)
    if rng.random() < 0.2:
        opts.update(t_over=10.0)
    if rng.random() < 0.2:
        opts.update(cycle_limit=rng.randint(20, 80))
    if call == "into_static":
        return _case(call, _log_int(rng, 30, 5000 if cap == 64 else (2500 if cap == 128 else 1200)), **opts)
    form = rng.choice(["plain", "batched"])
    if call == "generate":
        return _case(call, _log_int(rng, 30, 100000), form=form, records=rng.random() < 0.25, **opts)
    if rng.random() < 0.35:
        opts.update(mixed=True, cap=128)
    return _case(call, _log_int(rng, 1000, 1000000), form=form, **opts)


# --- the program's side -----------------------------------------------------

_ctx = None


def _context():
    """One context per device and process, as the library's users keep it."""
    global _ctx
    if _ctx is None:
        _ctx = P.Context(0)
    return _ctx


def _masses(case):
    return (1.5, 4.8) if case["massive"] else (0.0, 0.0)


def _mixed(case, seed):
    return workloads.mixed_energies(seed, case["n"])


def _qgq(n, ecm, seed):
    """Massless q g qbar events (CSR): x1, x2 uniform over the Dalitz triangle
    away from its edges, random orientation, random light flavour."""
    rng = np.random.Generator(np.random.PCG64(seed))
    x1, x2 = 0.5 + 0.45 * rng.random(n), 0.5 + 0.45 * rng.random(n)
    low = x1 + x2 < 1.05  # x3 = 2 - x1 - x2 at most 0.95
    x1, x2 = np.where(low, 1.45 - x1, x1), np.where(low, 1.45 - x2, x2)
    x3 = 2.0 - x1 - x2
    c12 = 1.0 - 2.0 * (x1 + x2 - 1.0) / (x1 * x2)
    s12 = np.sqrt(np.maximum(0.0, 1.0 - c12 * c12))
    ct, ph, ps = 2.0 * rng.random(n) - 1.0, 2.0 * np.pi * rng.random(n), 2.0 * np.pi * rng.random(n)
    st = np.sqrt(1.0 - ct * ct)
    a = np.stack([st * np.cos(ph), st * np.sin(ph), ct], 1)
    u = np.stack([ct * np.cos(ph), ct * np.sin(ph), -st], 1)
    v = np.cross(a, u)
    b = np.cos(ps)[:, None] * u + np.sin(ps)[:, None] * v
    p1 = (x1 * ecm / 2)[:, None] * a
    p2 = (x2 * ecm / 2)[:, None] * (c12[:, None] * a + s12[:, None] * b)
    p = np.empty((n, 3, 4))
    p[:, 0, 1:], p[:, 1, 1:], p[:, 2, 1:] = p1, -(p1 + p2), p2
    p[:, 0, 0], p[:, 1, 0], p[:, 2, 0] = x1 * ecm / 2, x3 * ecm / 2, x2 * ecm / 2
    f = rng.integers(1, 4, n)
    pid = np.stack([f, np.full(n, 21), -f], 1).astype(np.int8)
    col = np.tile(np.array([1, 2, 0], np.uint16), (n, 1))
    acol = np.tile(np.array([0, 1, 2], np.uint16), (n, 1))
    return (np.arange(n + 1, dtype=np.uint64) * 3, np.ascontiguousarray(p.reshape(3 * n, 4)), pid.ravel(), col.ravel(),
            acol.ravel())


_RECORDS = dict(rec_p=np.float64, rec_pid=np.int8, rec_col=np.uint16, rec_acol=np.uint16)


def _event_store(n):
    """The arrays into which the program reads its event records: room for 24
    partons per event on average (LEP has 5, the highest energy drawn 12)."""
    return {k: np.zeros((24 * n, 4) if k == "rec_p" else 24 * n, t) for k, t in _RECORDS.items()}


def prepare(case, seed):
    s = dict(case=case, seed=seed, ctx=_context())
    n, call = case["n"], case["call"]
    if case["records"]:
        s["store"] = _event_store(n)
    if call in ("into", "into_static"):
        dev = "cuda:0"
        ecm = tcut = None
        if case["mixed"]:
            s["ecm"], s["tcut"] = (torch.from_numpy(a).to(dev) for a in _mixed(case, seed))
            ecm, tcut = s["ecm"].data_ptr(), s["tcut"].data_ptr()
        flags = P.VSH_SUMMARY | P.VSH_INPUTS_ON_DEVICE
        flags |= P.VSH_FORM_PERSISTENT if case["form"] == "batched" else P.VSH_FORM_PLAIN
        flags |= P.VSH_HIST_FIXEDPOINT if case["fixed"] else 0
        mc, mb = _masses(case)
        s["req"], _ = P.make_request(n, seed=seed, ecm=case["ecm"], t_cut=case["tcut"], max_partons=case["cap"],
                                     flags=flags, ecm_per_event=ecm, tcut_per_event=tcut,
                                     cycle_limit=case["cycle_limit"], t_over=case["t_over"], mass_c=mc, mass_b=mb)
        if call == "into":
            s["ws_bytes"] = s["ctx"].workspace_size(s["req"])
            s["ws"] = torch.empty(s["ws_bytes"], dtype=torch.uint8, device=dev)
        s["hist"] = torch.zeros(P.HIST_DOUBLES, dtype=torch.float64, device=dev)
        s["sum_d"] = torch.empty((P.NSUM_D, n), dtype=torch.float64, device=dev)
        s["sum_i"] = torch.empty((P.NSUM_I, n), dtype=torch.int32, device=dev)
        s["hash"] = torch.empty(n, dtype=torch.int64, device=dev)
    elif call == "shower_records":
        s["starts"] = _qgq(n, case["ecm"], seed)
    elif call == "generate" and case["mixed"]:
        s["ecm"], s["tcut"] = _mixed(case, seed)
    elif call == "serve":
        # n requests of the trace (sizes 10^2 .. 10^5), their seeds from ours
        s["trace"] = workloads.serving_trace(n, master_seed=seed).requests
    return s


def _summaries(sum_d, sum_i, h):
    """The summary fields: those that the matrix element alone fixes by
    themselves (weight, cos(theta), azimuth), then the observables."""
    return dict(weight=sum_d[0], cos_theta=sum_d[1], phi=sum_d[9], observables=sum_d[2:9], ints=sum_i, hash=h)


_COUNTS = ("n_events", "n_done", "n_overflow", "n_nonfinite", "n_conservation", "n_cycle_limit", "total_cycles",
           "total_trials", "total_ends", "total_emissions", "max_cycles")


def _host(r, store=None):
    """What a call that returns host results gave, its timings left out; the
    event records go into the program's store."""
    out = dict(counts=np.array([r[k] for k in _COUNTS], np.int64), sums=np.array([r["sum_w"], r["sum_w2"]]),
               hist=r["hist"])
    if "sum_d" in r:
        out.update(_summaries(r["sum_d"], r["sum_i"], r["hash"].view(np.int64)))
    if "rec_p" in r:
        for k in _RECORDS:
            store[k][:len(r[k])] = r[k]
        out.update(rec_offsets=r["rec_offsets"].view(np.int64), rec_p=store["rec_p"], rec_pid=store["rec_pid"],
                   rec_col=store["rec_col"].view(np.int16), rec_acol=store["rec_acol"].view(np.int16))
    return out


def run(s):
    case, ctx, seed, call = s["case"], s["ctx"], s["seed"], s["case"]["call"]
    mc, mb = _masses(case)
    if call in ("into", "into_static"):
        stream = torch.cuda.current_stream().cuda_stream
        s["hist"].zero_()
        outs = (s["hist"].data_ptr(), s["sum_d"].data_ptr(), s["sum_i"].data_ptr(), s["hash"].data_ptr())
        if call == "into":
            ctx.generate_into(s["req"], stream, s["ws"].data_ptr(), s["ws_bytes"], *outs)
        else:
            ctx.generate_into_static(s["req"], stream, *outs)
        return dict(hist=s["hist"], **_summaries(s["sum_d"], s["sum_i"], s["hash"]))
    if call == "generate":
        return _host(ctx.generate(case["n"], seed=seed, ecm=case["ecm"], t_cut=case["tcut"], max_partons=case["cap"],
                                  summary=case["summary"], records=case["records"],
                                  persistent=case["form"] == "batched", ecm_per_event=s.get("ecm"),
                                  tcut_per_event=s.get("tcut"), cycle_limit=case["cycle_limit"],
                                  t_over=case["t_over"], mass_c=mc, mass_b=mb, fixed_hist=case["fixed"]), s.get("store"))
    if call == "generate_isr":
        return _host(ctx.generate_isr(case["n"], sqrt_s_hadron=1960.0, q=case["ecm"], t_cut=case["tcut"], seed=seed,
                                      max_partons=case["cap"], summary=case["summary"], records=case["records"]),
                     s.get("store"))
    if call == "shower_records":
        return _host(ctx.shower_records(*s["starts"], seed=seed, t_cut=case["tcut"], max_partons=case["cap"],
                                        records=case["records"], mass_c=mc, mass_b=mb), s["store"])
    tickets = [ctx.submit(r.n_events, seed=r.seed + seed, ecm=r.ecm, t_cut=r.tcut, max_partons=r.cap,
                          summary=case["summary"]) for r in s["trace"]]
    got = [_host(ctx.wait(t)) for t in tickets]
    return {k: (np.stack if k in ("counts", "sums", "hist") else np.concatenate)(
        [g[k] for g in got], **({} if k in ("counts", "sums", "hist") else {"axis": -1})) for k in got[0]}


# --- what a call cannot do without ------------------------------------------

def _event_flops(ecm, tcut):
    """FP64 operations of one event, about: 2 x 16.7 k issue slots at LEP
    (trials, decisions, emissions), growing with the number of cycles times
    the number of dipole ends, which follow ln(s / t_C) (30.9 cycles of 4 ends
    at LEP, 141 of 15 at 500 GeV and t_C = 0.25)."""
    span = max(1.0, math.log(max(ecm * ecm / tcut, math.e)))
    return 33400.0 * (span / 9.02) ** 5.7


def work(case):
    n = case["n"]
    hist = P.HIST_DOUBLES * 8
    if case["call"] == "serve":  # the trace's mean request
        n, hist = n * 14400, n * hist
    per = 116.0 if case["summary"] else 0.0
    flops = _event_flops(case["ecm"], case["tcut"])
    if case["mixed"]:
        per += 16.0
    partons = 2.0 + max(0.0, 0.35 * (math.log(max(case["ecm"] ** 2 / case["tcut"], math.e)) - 0.8))
    if case["records"]:
        per += 8.0 + 37.0 * partons
    if case["call"] == "shower_records":
        per += 8.0 + 37.0 * 3
    if case["call"] == "generate_isr":  # two lines per cycle, 61 cycles
        flops = 2.0 * 61 * 250
    return {"bytes": n * per + hist, "flops": n * flops}


# --- plain NumPy in 64 bits -------------------------------------------------

def _philox(c0, c1, c2, c3, seed):
    """Philox4x32-10 (Salmon et al., SC'11) over arrays of counter words."""
    m = np.uint64(0xFFFFFFFF)
    c = [np.asarray(a, np.uint64) for a in (c0, c1, c2, c3)]
    k0, k1 = seed & 0xFFFFFFFF, (seed >> 32) & 0xFFFFFFFF
    for _ in range(10):
        a, b = np.uint64(0xD2511F53) * c[0], np.uint64(0xCD9E8D57) * c[2]
        c = [(b >> np.uint64(32)) ^ c[1] ^ np.uint64(k0), b & m, (a >> np.uint64(32)) ^ c[3] ^ np.uint64(k1), a & m]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return c


def _unit(hi, lo):
    m = ((hi >> np.uint64(12)) << np.uint64(32)) | lo
    return (2.0 * m.astype(np.float64) + 1.0) * 2.0 ** -53


def _me_draws(n, seed):
    ids = np.arange(n, dtype=np.uint64)
    zero, me = np.zeros(n, np.uint64), np.uint64(1 << 24)
    lo, hi = ids & np.uint64(0xFFFFFFFF), ids >> np.uint64(32)
    return _philox(lo, hi, zero, zero + me, seed), _philox(lo, hi, zero, zero + me + np.uint64(1), seed)


def _me_weight(f, s, c, m2, n_open):
    """LO e+e- -> q qbar through photon and Z, weight in pb (quark mass^2 m2)."""
    mz, gz, mw = 91.1876, 2.4952, 80.385
    sw2 = 1.0 - (mw / mz) ** 2
    kappa = 1.0 / (4.0 * sw2 * (1.0 - sw2))
    den = (s - mz * mz) ** 2 + gz * gz * mz * mz
    chi1, chi2 = kappa * s * (s - mz * mz) / den, kappa * kappa * s * s / den
    ae, ve = -0.5, -0.5 + 2.0 * sw2
    up = (f == 2) | (f == 4)
    qf, af = np.where(up, 2.0 / 3.0, -1.0 / 3.0), np.where(up, 0.5, -0.5)
    vf = af - 2.0 * qf * sw2
    beta2 = 1.0 - 4.0 * m2 / s
    vector = qf * qf - 2.0 * qf * ve * vf * chi1 + (ae * ae + ve * ve) * vf * vf * chi2
    axial = (ae * ae + ve * ve) * af * af * chi2
    inter = -4.0 * qf * ae * af * chi1 + 8.0 * ae * af * ve * vf * chi2
    me = vector * (2.0 - beta2 * (1.0 - c * c)) + axial * beta2 * (1.0 + c * c) + inter * np.sqrt(beta2) * c
    e2 = 4.0 * np.pi / 128.802
    return n_open * np.sqrt(beta2) * e2 * e2 * 3.0 * me / (16.0 * np.pi * s) * 0.389379656e9


def exact(case, seed):
    """The fields that closed forms of the draws fix: weight, cos(theta) and
    azimuth of the matrix element (initial-state shower: the weight).  What
    the shower decides emission by emission has no closed form: None."""
    n, call = case["n"], case["call"]
    if call in ("shower_records", "serve"):
        return None
    a, b = _me_draws(n, seed)
    if call == "generate_isr":
        Y, tau = math.log(1960.0 / case["ecm"]), (case["ecm"] / 1960.0) ** 2
        y = -Y + 2.0 * Y * _unit(a[2], a[3])
        w = np.full(n, 10.0 * 2.0 * Y * tau)
        for x in (math.sqrt(tau) * np.exp(y), math.sqrt(tau) * np.exp(-y)):
            w *= 63.0 / 128.0 / np.sqrt(x) * (1.0 - x) ** 3
        return dict(weight=w)
    ecm = _mixed(case, seed)[0] if case["mixed"] else np.full(n, case["ecm"])
    masses = np.array([0.0, 0.0, 0.0, 0.0, *_masses(case)])
    is_open = 4.0 * masses[1:, None] ** 2 < ecm * ecm  # [flavour - 1][event]
    n_open = is_open.sum(0)
    idx = ((a[0] * n_open.astype(np.uint64)) >> np.uint64(32)).astype(np.int64)
    f = 1 + idx  # masses grow with the flavour: the open ones come first
    c = 2.0 * _unit(a[2], a[3]) - 1.0
    phi = 2.0 * np.pi * _unit(b[0], b[1])
    out = dict(cos_theta=c, phi=phi)
    if case["t_over"] == 0.0:  # else the weighted veto's factors multiply it
        out["weight"] = _me_weight(f, ecm * ecm, c, masses[f] ** 2, n_open)
    return out
