"""A handle's device memory (needs an MI355X): one allocation whose parts hold
the plan, the table, the image, the host round trip's slots and its counters.
Shapes whose parts are as small or as odd as they get, handles that take over
memory that others have left, and several handles alive at once: both
mechanisms against the oracle, right after create.
"""
import numpy as np
import pytest

import oracle
from paper_2608_12123_amd import rc_cohort as rc
from paper_2608_12123_amd import workload as wk

pytestmark = pytest.mark.gpu

KEYS = ("state", "outcome", "eff_sid", "eff_tool", "eff_payload", "n_taken")
T = 3

# (words, routes, route mode, cohort sizes)
SHAPES = [
    (4, 1, wk.ROUTE_MOD, [1]),
    (4, 2, wk.ROUTE_CDF, [63]),
    (9, 3, wk.ROUTE_MOD, [64, 65, 1]),
    (16, 1024, wk.ROUTE_CDF, [1] * 300),
    (32, 7, wk.ROUTE_CDF, [256, 255, 129, 64, 31]),
    (17, 1000, wk.ROUTE_CDF, [33] * 9),
    (64, 1023, wk.ROUTE_MOD, [256] * 3 + [5]),
]


def check(orc, co, inp, mode, what):
    co.upload(inp.state, inp.outcome)
    co.run_chain(0, T, mode)
    got, want = co.download(T), orc.run_inputs(inp, n_steps=T)
    for k in KEYS:
        assert np.array_equal(got[k], want[k]), (what, k)


def test_handles_in_turn_and_together():
    oracle.build(force=False)
    orc = oracle.load()
    inputs = [wk.make_custom(n_words=W, n_routes=R, route_mode=mode, decide_thr=32768, cohort_sizes=sizes, n_steps=T,
                             seed_key=900 + i) for i, (W, R, mode, sizes) in enumerate(SHAPES)]
    modes = (rc.RC_MODE_HOST_ROUNDTRIP, rc.RC_MODE_RESIDENT)
    for turn in range(2):  # each handle in memory of the one before it
        for i, inp in enumerate(inputs):
            print("handle in turn", turn, SHAPES[i][:3], flush=True)
            co = rc.Cohort.from_inputs(inp, max_steps=T)
            try:
                for mode in modes:
                    check(orc, co, inp, mode, (turn, i, mode))
            finally:
                co.close()
    alive = [rc.Cohort.from_inputs(inp, max_steps=T) for inp in inputs]
    try:
        for mode in modes * 2:
            for i, (co, inp) in enumerate(zip(alive, inputs)):
                print("handles together", mode, SHAPES[i][:3], flush=True)
                check(orc, co, inp, mode, ("together", i, mode))
    finally:
        for co in alive:
            co.close()
