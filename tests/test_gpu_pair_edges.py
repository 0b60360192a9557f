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


def _device(ev):
    """The batch's arrays and result slots in device memory."""
    import torch
    from paper_2402_14670_amd import lf
    src = {k: torch.from_numpy(getattr(ev, k).view(np.int32) if k.endswith("off") else getattr(ev, k)).cuda()
           for k in lf._IN_FIELDS}
    out = {k: torch.zeros((ev.n_tracks, 12) if k == "hit_idx" else ev.n_tracks, device="cuda",
                          dtype=torch.uint8 if k in ("found", "n_hits") else
                          torch.int32 if k == "hit_idx" else torch.float32) for k in lf._OUT_FIELDS}
    return src, out


def _noalloc(ctx, src, out, mode):
    import torch
    from paper_2402_14670_amd import lf
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    lf.lf_find_tracks_noalloc(ctx, src, out, mode, s.cuda_stream)
    s.synchronize()
    return {k: v.cpu().numpy() for k, v in out.items()}


@pytest.mark.parametrize("mode", ["batched", "persistent"])
def test_noalloc_with_fewer_tracks_than_the_offsets(mode):
    """Offsets that count more tracks than the call does (and than the fixed
    scratch holds): the call's own tracks are found, nothing past them is
    written."""
    import torch
    from paper_2402_14670_amd import lf
    ev = lfgen.generate("nominal", n_events=3, seed=91)
    ref = oracle_parallel(ev)
    src, out = _device(ev)
    off = ev.trk_off.copy()
    off[-1] = (1 << 22) + 300000
    src["trk_off"] = torch.from_numpy(off.view(np.int32)).cuda()
    ctx = lf.lf_create(W)
    try:
        say(f"[gpu] noalloc, offsets past the tracks, mode={mode}")
        compare(ref, _noalloc(ctx, src, out, mode), label=mode)
    finally:
        lf.lf_destroy(ctx)


@pytest.mark.parametrize("budget", [0, 1 << 33], ids=["indexed", "budget"])
def test_upload_of_millions_of_events(budget):
    """2,900,000 events, nearly all empty: more than one launch of the event
    kernel can hold; the events with hits and tracks stand at the ends of its
    slices."""
    from paper_2402_14670_amd import lf
    E = 2_900_000
    at = np.array([0, (1 << 20) - 1, 1 << 20, (1 << 21) - 1, 1 << 21, E - 1])
    some = lfgen.generate("nominal", n_events=len(at), seed=92)
    ref = oracle_parallel(some)
    # buckets and tracks per event of the long batch, from those of the short one
    nh, nt = np.zeros((E, 24), np.int64), np.zeros(E, np.int64)
    nh[at] = np.diff(some.hit_off.astype(np.int64)).reshape(-1, 24)
    nt[at] = np.diff(some.trk_off.astype(np.int64))
    ev = lfgen.Events(**{**some.__dict__, "n_events": E,
                         "hit_off": np.concatenate([[0], np.cumsum(nh.ravel())]).astype(np.uint32),
                         "trk_off": np.concatenate([[0], np.cumsum(nt)]).astype(np.uint32)})
    assert ev.n_events == E and ev.n_tracks == some.n_tracks
    ctx = lf.lf_create(W, None, budget)
    try:
        say(f"[gpu] upload of {E} events budget={budget}")
        bid = lf.lf_upload_events(ctx, ev)
        for mode in ("batched", "persistent"):
            lf.lf_poison_tracks(ctx, bid)
            lf.lf_find_tracks(ctx, bid, mode)
            compare(ref, lf.lf_copy_tracks(ctx, bid), label=mode)
    finally:
        lf.lf_destroy(ctx)
