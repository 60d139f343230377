"""The table-image chain (the masks of all routes do not fit on chip) where
its split can go wrong, bit-exact against the oracle (needs an MI355X): word
counts around the 16-word bands, chains around the 4-step chunks, launches of
fewer and of more bins than the device holds workgroups (so that a workgroup
takes several), both bin classes, ragged cohort ranges, and the no-decision
floor.
"""
import numpy as np
import pytest

import oracle
from paper_2608_12123_amd import rc_cohort as rc
from paper_2608_12123_amd import workload as wk

pytestmark = pytest.mark.gpu

KEYS = ("state", "outcome", "eff_sid", "eff_tool", "eff_payload", "n_taken")


@pytest.fixture(scope="module")
def orc():
    oracle.build(force=False)
    return oracle.load()


def inputs(W, R, mode, T, sessions, seed):
    rng = np.random.default_rng(seed)
    sizes = []
    while sum(sizes) < sessions:
        sizes.append(int(rng.choice([1, 31, 32, 63, 64, 65, 100, 128, 129, 192, 255, 256])))
    return wk.make_custom(n_words=W, n_routes=R, route_mode=mode, decide_thr=19661, cohort_sizes=sizes,
                          n_steps=T, seed_key=seed, ld=sum(sizes) + 5)


def assert_same(got, want, what):
    for k in KEYS:
        assert np.array_equal(got[k], want[k]), "%s: %s differs at %d places" % (
            what, k, int((got[k] != want[k]).sum()))


@pytest.mark.parametrize("W,R,mode,T,sessions", [
    (17, 1024, wk.ROUTE_CDF, 5, 2_000),      # two bands, one word in the second; chunk of 4 + 1
    (32, 600, wk.ROUTE_MOD, 4, 300),         # two whole bands, one whole chunk
    (33, 1024, wk.ROUTE_MOD, 3, 90_000),     # three bands, a chunk cut short, several bins a workgroup
    (48, 777, wk.ROUTE_CDF, 9, 200_000),     # three or more bins for some workgroups
    (49, 1023, wk.ROUTE_MOD, 1, 150_000),    # one step
    (64, 1024, wk.ROUTE_CDF, 8, 80_000),
    (63, 300, wk.ROUTE_MOD, 17, 700),
])
def test_table_chain(orc, W, R, mode, T, sessions):
    inp = inputs(W, R, mode, T, sessions, W * 31 + T)
    print("table W=%d R=%d mode=%d T=%d N=%d C=%d" % (W, R, mode, T, inp.n_sessions, inp.n_cohorts), flush=True)
    want = orc.run_inputs(inp, n_steps=T)
    co = rc.Cohort.from_inputs(inp, max_steps=T)
    try:
        co.run_chain(0, T)
        assert_same(co.download(T), want, "whole")
    finally:
        co.close()
    co = rc.Cohort.from_inputs(inp, max_steps=T)
    try:
        cuts = [0, 1, inp.n_cohorts // 3, inp.n_cohorts // 3 + 1, inp.n_cohorts]
        for a, b in zip(cuts, cuts[1:]):
            co.run_chain(0, T, cohort_begin=a, cohort_end=b)
        assert_same(co.download(T), want, "ranges")
    finally:
        co.close()


@pytest.mark.parametrize("W,R,T,sessions", [(33, 1024, 9, 90_000), (64, 900, 3, 1_000), (20, 1000, 16, 500)])
def test_table_floor(orc, W, R, T, sessions):
    inp = inputs(W, R, wk.ROUTE_CDF, T, sessions, W + T)
    print("table floor W=%d R=%d T=%d N=%d" % (W, R, T, inp.n_sessions), flush=True)
    rng = np.random.default_rng(T)
    bits = rng.integers(0, 1 << 32, size=(T, (inp.ld + 31) // 32), dtype=np.uint32)
    want = orc.run_inputs(inp, n_steps=T, decisions=bits)
    co = rc.Cohort.from_inputs(inp, max_steps=T)
    try:
        co.run_floor(bits, T)
        assert_same(co.download(T), want, "floor")
    finally:
        co.close()
