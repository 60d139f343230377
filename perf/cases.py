"""The work that a program has this library do, as cases to time.

A case is one call (or, for a window of arrivals, one short sequence of calls)
of the public Python binding on device buffers that the program owns.  Kinds:

  chain      resident chain over all cohorts of a descriptor, one launch
  one        resident chain of a single cohort of a descriptor, cohorts in turn
  floor      no-decision floor over all cohorts (a replay of known decisions)
  roundtrip  host round trip over all cohorts
  window     a window of arrivals from the compactor to the chain's effects:
             batches, cohorts, a handle for them, the gather of the sessions'
             state from a device-resident store, the chain

Each pass continues the chains of the state: step0 advances by T.  Outputs are
whole numbers and bit-exact by the definition of the transition.
"""
import functools
import math
import random

import numpy as np
import torch

from paper_2608_12123_amd import rc_cohort as rc
from paper_2608_12123_amd import workload as wk

ZIPF_S = 1.1
WINDOW_K = 32            # safe-suffix threshold of the window's routes
WINDOW_LATENCY_NS = 25_000
WINDOW_CAPACITY = 4096
ONE_COHORTS = 1000       # cohorts of the descriptor whose cohorts run one at a time


def _case(name, kind, sessions, words, routes, mode, p, steps, sizes, ld_pad=0):
    c = {"kind": kind, "sessions": sessions, "words": words, "routes": routes, "mode": mode, "p": p,
         "steps": steps, "sizes": sizes, "ld_pad": ld_pad}
    return dict(c, name=name) if name else c


def listed():
    return [
        # Latency of the smallest call: one control event of a 32-session
        # cohort (the benchmark's tiny workload).
        _case("one32_step", "one", 32, 8, 4, "mod", 0.5, 1, "32"),
        # A 64-session cohort over an observation-free horizon of 8 steps
        # (the benchmark's k64 workload): still a latency-bound call.
        _case("one64_t8", "one", 64, 16, 16, "mod", 0.5, 8, "64"),
        # One full cohort, long horizon, skewed routes (the k256 workload).
        _case("one256_t32", "one", 256, 32, 64, "zipf", 0.3, 32, "256"),
        # The same shape with every cohort of the descriptor in one launch:
        # a busy server's batch of full cohorts.
        _case("all256_t32", "chain", 256_000, 32, 64, "zipf", 0.3, 32, "256"),
        # The throughput workload of the benchmark: 391 cohorts, the last
        # partial.
        _case("chain_100k", "chain", 100_000, 32, 256, "mod", 0.5, 16, "256"),
        # One step of the same sessions: outcomes come from outside after
        # every step (tool results), so nothing can be chained.
        _case("step_100k", "chain", 100_000, 32, 256, "mod", 0.5, 1, "256"),
        # The largest workload of the benchmark: a million sessions in
        # variable cohorts formed from Poisson arrivals, widest state, most
        # routes.
        _case("chain_1m", "chain", 1_000_000, 64, 1024, "zipf", 0.05, 16, "formed"),
        # A mid-size launch in which nothing is round: cohorts of any size,
        # 13 words, 23 routes, 7 steps, padded leading dimension.
        _case("ragged_w13", "chain", 30_011, 13, 23, "mod", 0.3, 7, "any", 53),
        # Wide state and many routes, again with ragged cohorts and an odd
        # word count: the masks of all routes do not fit on chip.
        _case("ragged_w48", "chain", 60_007, 48, 1000, "mod", 0.5, 24, "any"),
        # Replay of recorded decisions of the throughput workload.
        _case("floor_100k", "floor", 100_000, 32, 256, "mod", 0.5, 16, "256"),
        # A program that has to look at every decision on the host.
        _case("roundtrip_100k", "roundtrip", 100_000, 32, 256, "mod", 0.5, 16, "256"),
        # Two launch deadlines' worth of arrivals, formed, fed and run.
        _case("window_20k", "window", 20_000, 64, 1024, "zipf", 0.05, 16, "formed"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["chain"] * 8 + ["one"] * 3 + ["floor", "roundtrip", "roundtrip", "window"])
    words = rng.choice([rng.randint(4, 64), rng.randint(4, 64), rng.choice([4, 8, 16, 32, 64])])
    mode = rng.choice(["mod", "zipf"])
    routes = _log_int(rng, 1, 1024)
    p = rng.choice([0.05, 0.3, 0.5, round(rng.uniform(0.0, 1.0), 3)])
    steps = _log_int(rng, 1, 48)
    sizes = rng.choice(["any", "formed", "32", "64", "128", "256", str(rng.randint(1, 256))])
    if kind == "one":
        if sizes in ("any", "formed"):
            sizes = str(rng.randint(1, 256))
        return _case(None, kind, int(sizes), words, routes, mode, p, steps, sizes)
    if kind == "window":
        return _case(None, kind, _log_int(rng, 2_000, 20_000), words, max(routes, 16), "zipf", p,
                     min(steps, 16), "formed")
    # at most the bytes of the largest listed case
    most = 9e8 / (8 * words + 8 + 24 * steps)
    if kind == "roundtrip":
        steps, most = min(steps, 16), 100_000
    sessions = _log_int(rng, 32, min(1_000_000, most))
    return _case(None, kind, sessions, words, routes, mode, p, steps, sizes, rng.choice([0, 0, rng.randint(1, 200)]))


def _cdf(case):
    return wk.zipf_cdf(case["routes"], ZIPF_S) if case["mode"] == "zipf" else None


@functools.lru_cache(maxsize=None)
def _arrivals(n, routes):
    """Release times and routes of n Poisson arrivals (the same for every
    seed, so that a case's shapes are its own)."""
    t = wk.poisson_arrivals_ns(n, wk.ARRIVAL_RATE_PER_S, n, routes, wk.A_ARRIVAL)
    o = wk.uniform_u32(n, n, routes, wk.A_ARRIVAL_OUTCOME)
    return t, wk.route_of_outcomes_cdf(o, wk.zipf_cdf(routes, ZIPF_S)).astype(np.uint32)


@functools.lru_cache(maxsize=None)
def _layout(sessions, routes, sizes):
    """Cohort sizes of a descriptor (and the route every cohort starts from,
    where the former grouped arrivals by route)."""
    if sizes == "formed":
        t, r = _arrivals(sessions, routes)
        order, info = wk.form_cohorts(t, r.astype(np.int64), wk.DEADLINE_NS)
        return info["sizes_array"], r[order]
    if sizes == "any":
        rng, out, left = random.Random(sessions), [], sessions
        while left:
            out.append(min(left, rng.randint(1, 256)))
            left -= out[-1]
        return np.asarray(out), None
    k = int(sizes)
    return np.asarray([k] * (sessions // k) + ([sessions % k] if sessions % k else [])), None


def _offsets(sizes):
    return np.concatenate([[0], np.cumsum(sizes)]).astype(np.uint32)


def _outcomes_on(route, cdf, rng):
    """Outcomes drawn uniformly among those of each session's route."""
    lo = np.concatenate([[0], cdf]).astype(np.int64)
    hi = np.concatenate([cdf, [1 << 32]]).astype(np.int64)
    lo, hi = lo[route], hi[route]
    return (lo + (rng.random(route.size) * (hi - lo)).astype(np.int64)).astype(np.uint32)


def _words(shape, g):
    return torch.randint(-(1 << 31), 1 << 31, shape, dtype=torch.int32, device="cuda", generator=g)


def _as_device(u32):
    return torch.from_numpy(u32.view(np.int32)).cuda()


def prepare(case, seed):
    rng = np.random.default_rng(seed)
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    table = rng.integers(0, 1 << 32, size=(case["routes"], 16), dtype=np.uint32)
    spec = {"n_words": case["words"], "n_routes": case["routes"], "table": table,
            "route_mode": rc.RC_ROUTE_CDF if case["mode"] == "zipf" else rc.RC_ROUTE_MOD,
            "route_cdf": _cdf(case), "decide_thr": wk.threshold_from_p(case["p"]),
            "max_steps": case["steps"]}
    st = {"case": case, "step": 0, "next": 0}
    if case["kind"] == "window":
        n = case["sessions"]
        times, route = _arrivals(n, case["routes"])
        st.update(spec=spec, times=times, route=route,
                  k=np.full(case["routes"], WINDOW_K, dtype=np.uint32),
                  state=_words((case["words"], n), g),
                  outcome=_as_device(_outcomes_on(route, spec["route_cdf"], rng)))
        return st
    n = case["sessions"] * (ONE_COHORTS if case["kind"] == "one" else 1)
    sizes, route = _layout(n, case["routes"], case["sizes"])
    co = rc.Cohort(cohort_offsets=_offsets(sizes), ld=n + case["ld_pad"], **spec)
    co.t["state"].copy_(_words((case["words"], co.ld), g))
    co.t["outcome"].copy_(_words((co.ld,), g))
    if route is not None and case["mode"] == "zipf":
        co.t["outcome"][:n] = _as_device(_outcomes_on(route, spec["route_cdf"], rng))
    if case["kind"] == "floor":
        bits = torch.rand((case["steps"], (co.ld + 31) // 32, 32), device="cuda", generator=g) < case["p"]
        weight = torch.arange(32, device="cuda", dtype=torch.int64)
        st["bits"] = (bits.to(torch.int64) << weight).sum(-1).to(torch.int32).contiguous()
    st["co"] = co
    return st


def _run_window(st):
    case = st["case"]
    res, batch, _ = rc.rc_online_compact(release_ns=st["times"], route=st["route"], k_of_route=st["k"],
                                       delta_ns=wk.DEADLINE_NS, latency_ns=WINDOW_LATENCY_NS,
                                       capacity=WINDOW_CAPACITY, witness=True)
    order, offsets = rc.rc_cohorts_from_batches(batch, res["n_batches"])
    co = rc.Cohort(cohort_offsets=offsets, **st["spec"])
    index = torch.from_numpy(order.astype(np.int64)).cuda()
    torch.index_select(st["state"], 1, index, out=co.t["state"])
    torch.index_select(st["outcome"], 0, index, out=co.t["outcome"])
    co.run_chain(st["step"], case["steps"])
    st["step"] += case["steps"]
    torch.cuda.synchronize()  # the handle goes away only after its work
    out = co.t
    co.close()
    return out


def run(st):
    case = st["case"]
    if case["kind"] == "window":
        return _run_window(st)
    co, T, step = st["co"], case["steps"], st["step"]
    st["step"] = (step + T) & 0xFFFFFFFF
    if case["kind"] == "chain":
        co.run_chain(step, T)
    elif case["kind"] == "roundtrip":
        co.run_chain(step, T, rc.RC_MODE_HOST_ROUNDTRIP)
    elif case["kind"] == "floor":
        rc.rc_cohort_run_floor(co.handle, co.buffers, st["bits"].data_ptr(), T, 0, co.n_cohorts)
    else:
        c = st["next"]
        st["next"] = (c + 1) % co.n_cohorts
        co.run_chain(step, T, cohort_begin=c, cohort_end=c + 1)
    return co.t


def work(case):
    """State and outcome read and written once per chain (once per step where
    the host looks at every step), 24 bytes per effect, the counts."""
    n, W, T = case["sessions"], case["words"], case["steps"]
    if case["kind"] == "window":
        # every session's state once from the store to the handle's buffers too
        return {"bytes": 16.0 * W * n + 24.0 * n * T, "flops": 0.0}
    cohorts = 1 if case["kind"] == "one" else len(_layout(n, case["routes"], case["sizes"])[0])
    passes = T if case["kind"] == "roundtrip" else 1
    bits = n * T / 8.0 if case["kind"] == "floor" else 0.0
    return {"bytes": (8.0 * W + 8.0) * n * passes + 24.0 * n * T + 4.0 * cohorts * T + bits, "flops": 0.0}


def tolerance(case):
    return "exact"
