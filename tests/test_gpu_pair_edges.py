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


def _with_long_buckets(ev, lengths, odd):
    """The first event's listed buckets made as long as given by random hits;
    odd: the hit of each of them (first, middle, last or none) that is off the
    bucket's z and slope."""
    rng = np.random.default_rng(93)
    arr = {k: getattr(ev, k) for k in ("hit_x", "hit_z", "hit_dxdy", "hit_pid")}
    off = ev.hit_off.astype(np.int64)
    for b, n in lengths.items():
        f, l = int(off[b]), int(off[b + 1])
        x = np.sort(np.concatenate([arr["hit_x"][f:l], rng.uniform(-3000, 3000, n - (l - f)).astype(np.float32)]))
        z, d = np.full(n, arr["hit_z"][f]), np.full(n, arr["hit_dxdy"][f])
        if odd is not None:
            i = {"first": 0, "middle": n // 2, "last": n - 1}[odd]
            z[i] += np.float32(2.0)
            d[i] += np.float32(0.01)
        new = dict(hit_x=x, hit_z=z, hit_dxdy=d, hit_pid=np.full(n, -1, np.int32))
        arr = {k: np.concatenate([v[:f], new[k], v[l:]]) for k, v in arr.items()}
        off[b + 1:] += n - (l - f)
    return lfgen.Events(**{**ev.__dict__, **arr, "hit_off": off.astype(np.uint32)})


# a block of the event kernel takes six buckets: one, two and six long ones of
# a block, some of every block, at the edges of a round, of a piece and of the
# index
LONG = [{0: 2048}, {5: 2049}, {3: 3072, 4: 2305}, {b: 2100 + 64 * b for b in range(6)},
        {0: 65535, 7: 65536, 13: 2047, 23: 4097}, {b: 2500 for b in range(24)}]


@pytest.mark.parametrize("odd", [None, "first", "middle", "last"])
@pytest.mark.parametrize("lengths", LONG, ids=lambda v: "_".join(str(n) for n in list(v.values())[:4]))
def test_long_buckets(lengths, odd):
    """Buckets that the whole block shares, with and without the index, beside
    events whose buckets are short."""
    from paper_2402_14670_amd import lf
    ev = _with_long_buckets(lfgen.generate("nominal", n_events=3, seed=94), lengths, odd)
    ref = oracle_parallel(ev)
    for budget in (0, 1 << 30):
        ctx = lf.lf_create(W, None, budget)
        try:
            say(f"[gpu] long buckets {lengths} odd={odd} budget={budget}")
            bid = lf.lf_upload_events(ctx, ev)
            for mode in ("plain", "batched"):
                lf.lf_poison_tracks(ctx, bid)
                lf.lf_find_tracks(ctx, bid, mode)
                compare(ref, lf.lf_copy_tracks(ctx, bid), label=f"{mode} budget={budget}")
        finally:
            lf.lf_destroy(ctx)


@pytest.mark.parametrize("budget", [0, 1 << 30])
def test_refused_upload_waits_for_its_own_stream_only(budget):
    """A batch with a bad value is refused while another stream still works,
    and the block that it took serves the next upload."""
    import torch
    from paper_2402_14670_amd import lf
    ev = lfgen.generate("nominal", n_events=5, seed=95)
    bad = lfgen.Events(**{**ev.__dict__, "trk_tx": ev.trk_tx.copy()})
    bad.trk_tx[-1] = np.inf
    ctx = lf.lf_create(W, None, budget)
    busy, mine, done = torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.Event()
    try:
        lf.lf_release_batch(ctx, lf.lf_upload_events(ctx, ev, mine.cuda_stream))
        torch.cuda.synchronize()
        with torch.cuda.stream(busy):
            torch.cuda._sleep(500_000_000)   # a quarter of a second
            done.record(busy)
        with pytest.raises(lf.LFError) as e:
            lf.lf_upload_events(ctx, bad, mine.cuda_stream)
        assert not done.query()
        assert e.value.code == lf.LF_ERR_INVALID and "non-finite track state" in str(e.value)
        busy.synchronize()
        bid = lf.lf_upload_events(ctx, ev)
        lf.lf_find_tracks(ctx, bid)
        compare(oracle_parallel(ev), lf.lf_fetch_tracks(ctx, bid), label="after a refusal")
    finally:
        lf.lf_destroy(ctx)


def _jitter(ev, seed):
    rng = np.random.default_rng(seed)
    return lfgen.Events(**{**ev.__dict__, "hit_z": ev.hit_z + rng.uniform(-1.5, 1.5, ev.n_hits).astype(np.float32),
                           "hit_dxdy": ev.hit_dxdy * (1 + rng.uniform(-0.02, 0.02, ev.n_hits)).astype(np.float32)})


@pytest.mark.parametrize("params", [
    {}, {"n_hits_window": 64, "n_triplets": 32}, {"velo_only": 1}, {"velo_only": 1, "n_hits_window": 32},
    {"seed_fp16": 1}, {"seed_fp16": 1, "n_hits_window": 64}],
    ids=["default", "w64", "velo_only", "velo_only_w32", "fp16", "fp16_w64"])
def test_one_track_kernels(params):
    """A context with a device budget has no search indexes: the one-track
    batched and persistent kernels, for every kind of input, on the planes and
    off them, with each number of wavefronts per block."""
    from paper_2402_14670_amd import lf
    base = lfgen.generate("uneven", n_events=14, seed=96)
    ev = lfgen.concat([base, _jitter(lfgen.generate("nominal", n_events=5, seed=97), 98)])
    ref = oracle_parallel(ev, params)
    ctx = lf.lf_create(W, params, 1 << 30)
    try:
        bid = lf.lf_upload_events(ctx, ev)
        for waves in (1, 2, 4):
            lf.lf_set_exec(ctx, waves_per_block=waves)
            for mode in ("batched", "persistent", "persistent"):
                say(f"[gpu] one-track kernels {params} waves={waves} mode={mode}")
                lf.lf_poison_tracks(ctx, bid)
                lf.lf_find_tracks(ctx, bid, mode)
                compare(ref, lf.lf_copy_tracks(ctx, bid), label=f"{mode}/{waves}")
    finally:
        lf.lf_destroy(ctx)


@pytest.mark.parametrize("n_events", [8191, 8192, 8193])
def test_noalloc_at_the_end_of_the_fixed_indexes(n_events):
    """The fixed scratch holds the search indexes of 8,192 events; longer calls
    go without.  Every slot, both modes, after a call of the other kind."""
    from paper_2402_14670_amd import lf
    small = lfgen.generate("single", n_events=600, seed=99)
    ev = lfgen.select_events(small, np.arange(n_events) % 600)
    ref = oracle_parallel(ev)
    ctx = lf.lf_create(W)
    try:
        src, out = _device(ev)
        few, few_out = _device(small)
        for mode in ("batched", "persistent"):
            say(f"[gpu] noalloc {n_events} events mode={mode}")
            _noalloc(ctx, few, few_out, mode)
            compare(ref, _noalloc(ctx, src, out, mode), label=f"{n_events}/{mode}")
    finally:
        lf.lf_destroy(ctx)
