"""The two-track kernel and what feeds it at the edges of their ranges: every
slot against the oracle (indices and flags bit-exact, parameters within 1e-5
relative) or, where a test says so, bit for bit."""
import numpy as np
import pytest

import lfgen
import oracle
from parity import PARAM_KEYS, W, compare, oracle_parallel, run_gpu, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _built():
    oracle.build()


@pytest.mark.parametrize("odd,exp", [(49, 122), (117, 121), (227, 120)])
def test_subnormal_quotients(odd, exp):
    """Tolerances near the largest binary32 number: every chi2 is a subnormal
    quotient, many of them halfway between two subnormal numbers, and the
    quality their sum.  All modes and the oracle agree in every bit (each
    divides with correct rounding, and sums of subnormals are exact)."""
    tol = float(odd) * 2.0 ** exp
    params = {"T_x": tol, "T_y": tol, "T_uv_scale": 0.0, "T_uv_floor": tol}
    ev = lfgen.generate("nominal", n_events=41, seed=90)
    ref = oracle_parallel(ev, params)
    q = ref["Q"][ref["found"] == 1]
    assert ((q > 0) & (q < 1.1754944e-38)).sum() > 1000
    for mode in ("plain", "batched", "persistent"):
        say(f"[gpu] subnormal quotients mode={mode} tolerance={tol}")
        got = run_gpu(ev, mode, params)
        compare(ref, got, label=mode)
        for k in PARAM_KEYS:
            assert np.array_equal(ref[k].view(np.uint32), got[k].view(np.uint32)), (mode, k)
