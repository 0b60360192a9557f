"""The two-tracks-per-wavefront kernel: every slot against the oracle at the
edges of its lists, windows and event flags.  Indices and flags bit-exact,
parameters within 1e-5 relative (the same expressions in the same order on both
sides)."""
import numpy as np
import pytest

import lfgen
import oracle
from parity import W, compare, oracle_parallel, run_gpu, say

pytestmark = pytest.mark.gpu
MIN = 4096


@pytest.fixture(scope="module", autouse=True)
def _built():
    oracle.build()


def _check(ev, label, params=None, world=None, modes=("batched", "persistent")):
    assert ev.n_tracks >= MIN
    ref = oracle_parallel(ev, params, world)
    for mode in modes:
        say(f"[gpu] pair {label}: mode={mode} events={ev.n_events} tracks={ev.n_tracks} params={params}")
        st = compare(ref, run_gpu(ev, mode, params, world=world), label=f"{label}/{mode}")
        say(f"    found={st['found']} bit-exact params {st['bit_exact_params']}/{st['params']}")


def _jitter(ev, z_mm, slope_rel, seed):
    rng = np.random.default_rng(seed)
    return lfgen.Events(**{**ev.__dict__,
                           "hit_z": ev.hit_z + rng.uniform(-z_mm, z_mm, ev.n_hits).astype(np.float32),
                           "hit_dxdy": ev.hit_dxdy * (1 + rng.uniform(-slope_rel, slope_rel, ev.n_hits)).astype(np.float32)})


def _cut_tracks(ev, n):
    """The batch without its last tracks: n left."""
    off = np.minimum(ev.trk_off, n).astype(np.uint32)
    cut = {k: getattr(ev, k)[:n] for k in ("trk_x", "trk_y", "trk_tx", "trk_ty", "trk_qop", "trk_pid")}
    return lfgen.Events(**{**ev.__dict__, "trk_off": off, **cut})


@pytest.mark.parametrize("n_tracks", [1, 2, 3, 63, 64, 65, MIN - 1, MIN, MIN + 1])
def test_slot_counts(n_tracks):
    ev = _cut_tracks(lfgen.generate("nominal", n_events=21, seed=50), n_tracks)
    ref = oracle_parallel(ev)
    for mode in ("batched", "persistent"):
        for exec_cfg in ({"waves_per_block": 1, "items_per_grab": 1}, {"waves_per_block": 4, "items_per_grab": 5}):
            say(f"[gpu] pair slots={n_tracks} mode={mode} exec={exec_cfg}")
            compare(ref, run_gpu(ev, mode, None, exec_cfg), label=f"slots {n_tracks}/{mode}")


@pytest.mark.parametrize("waves,items", [(1, 1), (1, 3), (2, 4), (4, 16)])
def test_persistent_chunks(waves, items):
    """One block per compute unit: large chunks, then small ones; odd track
    counts, and launches that find the queue words as the last one left them."""
    from paper_2402_14670_amd import lf
    for n in (4199, 4200, 2049, 513):
        ev = _cut_tracks(lfgen.generate("nominal", n_events=21, seed=58), n)
        ref = oracle_parallel(ev)
        say(f"[gpu] persistent chunks n={n} waves={waves} items={items}")
        ctx = lf.lf_create(W)
        bid = lf.lf_upload_events(ctx, ev)
        lf.lf_set_exec(ctx, waves_per_block=waves)
        lf.lf_set_exec(ctx, items_per_grab=items, blocks_per_cu=1)
        for launch in range(3):
            lf.lf_poison_tracks(ctx, bid)
            lf.lf_find_tracks(ctx, bid, "persistent")
            compare(ref, lf.lf_copy_tracks(ctx, bid), label=f"chunks {n}/{waves}/{items} launch {launch}")
        lf.lf_destroy(ctx)


@pytest.mark.parametrize("window,triplets", [(1, 1), (8, 16), (31, 17), (32, 32), (33, 12), (64, 16), (64, 32)])
def test_window_and_list_lengths(window, triplets):
    ev = lfgen.generate("nominal", n_events=21, seed=51)
    params = {"n_hits_window": window, "n_triplets": triplets}
    _check(ev, f"w{window} t{triplets}", params)
    _check(_jitter(ev, 1.5, 0.02, 52), f"w{window} t{triplets} per-hit z and slope", params)


def test_dense_events_and_long_pair_queues():
    """Full windows; then filters so loose that every pair of a track passes
    and its queue is filled many times over."""
    ev = lfgen.generate("stress", n_events=9, seed=53)
    _check(ev, "stress")
    loose = {"magtol_min": 3000.0, "magtol_max": 3000.0, "T_triplet": 50.0}
    small = lfgen.generate("nominal", n_events=21, seed=54)
    _check(small, "loose filters", loose)
    _check(small, "loose filters, 64 hits", {**loose, "n_hits_window": 64, "n_triplets": 32})
    _check(_jitter(small, 3.0, 0.05, 55), "loose filters, per-hit z and slope", loose)


def test_event_kinds_side_by_side():
    """Events on the layer planes, shifted off them bucket by bucket, jittered
    in z, in slope or in both, without hits and without tracks, alternating so
    that wavefronts hold tracks of two kinds; odd track counts everywhere."""
    parts = []
    base = lfgen.generate("uneven", n_events=36, seed=56)
    for e in range(base.n_events):
        ev = lfgen.select_events(base, [e])
        ev = _cut_tracks(ev, ev.n_tracks - (ev.n_tracks + 1) % 2 if ev.n_tracks else 0)
        kind = e % 6
        if kind == 1:
            ev = lfgen.Events(**{**ev.__dict__, "hit_z": ev.hit_z + np.float32(2.5)})
        elif kind == 2:
            ev = _jitter(ev, 1.5, 0.02, e)
        elif kind == 3:
            ev = _jitter(ev, 0.0, 0.02, e)
        elif kind == 4:
            ev = _jitter(ev, 40.0, 0.0, e)
        elif kind == 5 and e > 20:
            z = np.zeros(0, np.float32)
            ev = lfgen.Events(**{**ev.__dict__, "hit_off": np.zeros(25, np.uint32), "hit_x": z, "hit_z": z,
                                 "hit_dxdy": z, "hit_pid": np.zeros(0, np.int32)})
        parts.append(ev)
    _check(lfgen.concat(parts), "event kinds")


@pytest.mark.parametrize("spread", ["one_x", "two_x", "tiny", "far"])
def test_bucket_index_of_odd_ranges(spread):
    """Buckets whose x range is nothing, one step, subnormal, or has a far
    outlier (most hits in one cell of the search index)."""
    ev = lfgen.generate("nominal", n_events=21, seed=57)
    hx = ev.hit_x.copy()
    for b in range(24 * ev.n_events):
        f, n = int(ev.hit_off[b]), int(ev.hit_off[b + 1])
        if n - f < 4 or b % 5:
            continue
        v = hx[f:n]
        if spread == "one_x":
            v[:] = v[len(v) // 2]
        elif spread == "two_x":
            v[:] = v[len(v) // 2]
            v[len(v) // 2:] = np.nextafter(v[0], np.float32(np.inf))
        elif spread == "tiny":
            v[:] = np.float32(0.0)
            v[-1] = np.float32(1e-42)
        else:
            v[-1] = np.float32(3e30)
            v[0] = np.float32(-1e9)
    ev = lfgen.Events(**{**ev.__dict__, "hit_x": hx})
    _check(ev, f"index {spread}")
    _check(_jitter(ev, 1.5, 0.02, 58), f"index {spread}, per-hit z and slope")


def test_bucket_longer_than_the_index():
    """A bucket of 70,000 hits, which the 16-bit search index cannot hold."""
    ev = lfgen.generate("nominal", n_events=21, seed=59)
    b, n = 24 * 7 + 8, 70000
    f, l = int(ev.hit_off[b]), int(ev.hit_off[b + 1])
    rng = np.random.default_rng(60)
    x = np.sort(np.concatenate([ev.hit_x[f:l], rng.uniform(-3000, 3000, n - (l - f)).astype(np.float32)]))
    off = ev.hit_off.astype(np.int64)
    off[b + 1:] += n - (l - f)

    def put(a, mid):
        return np.concatenate([a[:f], mid, a[l:]])
    big = lfgen.Events(**{**ev.__dict__, "hit_off": off.astype(np.uint32), "hit_x": put(ev.hit_x, x),
                          "hit_z": put(ev.hit_z, np.full(n, ev.hit_z[f])),
                          "hit_dxdy": put(ev.hit_dxdy, np.full(n, ev.hit_dxdy[f])),
                          "hit_pid": put(ev.hit_pid, np.full(n, -1, np.int32))})
    _check(big, "70,000-hit bucket")
    _check(_jitter(big, 1.5, 0.02, 61), "70,000-hit bucket, per-hit z and slope", modes=("batched",))


@pytest.mark.parametrize("field", ["toy", "paper"])
def test_geometries(field):
    """Both field forms, both polarities, a cubic term; planes too close for
    the bracket (the context then runs one track per wavefront)."""
    ev = lfgen.generate("nominal", field=field, n_events=21, seed=62)
    w = lfgen.world(field)
    worlds = [w, dict(w, polarity=-1), dict(w, dRatio=-3.0e-4), dict(w, z_mag=w["z"][0] + 0.5)]
    for k, world in enumerate(worlds):
        _check(ev, f"{field} world {k}", None, world, modes=("batched",))
        _check(_jitter(ev, 1.5, 0.02, 63), f"{field} world {k}, per-hit z and slope", None, world, modes=("batched",))


def test_equal_hits_and_ties():
    """Every hit doubled or tripled: plateaus of equal distances in the middle
    window, the extensions and the top-n order."""
    ev = lfgen.generate("nominal", n_events=21, seed=64)
    rep = np.random.default_rng(65).integers(1, 4, ev.n_hits)
    cum = np.concatenate([[0], np.cumsum(rep)])
    dup = lfgen.Events(**{**ev.__dict__, "hit_off": cum[ev.hit_off.astype(np.int64)].astype(np.uint32),
                          **{k: np.repeat(getattr(ev, k), rep) for k in ("hit_x", "hit_z", "hit_dxdy", "hit_pid")}})
    _check(dup, "doubled hits")
    _check(dup, "doubled hits, 64 per window", {"n_hits_window": 64, "n_triplets": 32})
    # slopes that differ within the equal hits: moved hits out of x order
    _check(_jitter(dup, 0.0, 0.1, 66), "doubled hits, slopes", {"n_hits_window": 64})


@pytest.mark.parametrize("window,triplets", [(64, 20), (32, 12), (8, 32), (50, 3)])
def test_velo_only_input(window, triplets):
    """One track per wavefront, a half for each side: list and window lengths,
    the pool cut across the sides, per-hit z and slopes, shifted planes, the
    paper-form field, and filters so loose that the pair queues overflow."""
    ev = lfgen.generate("nominal", n_events=21, seed=74)
    params = {"velo_only": 1, "n_hits_window": window, "n_triplets": triplets}
    _check(ev, f"no-UT w{window} t{triplets}", params)
    _check(_jitter(ev, 1.5, 0.02, 75), f"no-UT w{window} t{triplets} per-hit z and slope", params)
    shifted = lfgen.Events(**{**ev.__dict__, "hit_z": ev.hit_z + np.float32(1.5)})
    _check(shifted, "no-UT shifted planes", params, modes=("batched",))
    _check(ev, "no-UT loose filters", {**params, "magtol_min": 3000.0, "magtol_max": 3000.0, "T_triplet": 50.0},
           modes=("batched",))
    paper = lfgen.generate("nominal", field="paper", n_events=21, seed=76)
    _check(paper, "no-UT paper field", params, lfgen.world("paper"), modes=("batched",))


def test_velo_only_dense_and_tied():
    ev = lfgen.generate("stress", n_events=9, seed=77)
    _check(ev, "no-UT stress", {"velo_only": 1})
    rep = np.random.default_rng(78).integers(1, 4, ev.n_hits)
    cum = np.concatenate([[0], np.cumsum(rep)])
    dup = lfgen.Events(**{**ev.__dict__, "hit_off": cum[ev.hit_off.astype(np.int64)].astype(np.uint32),
                          **{k: np.repeat(getattr(ev, k), rep) for k in ("hit_x", "hit_z", "hit_dxdy", "hit_pid")}})
    _check(dup, "no-UT doubled hits", {"velo_only": 1}, modes=("batched",))


@pytest.mark.parametrize("extra", [
    {}, {"n_hits_window": 64, "n_triplets": 32}, {"n_hits_window": 8, "n_triplets": 3},
    {"magtol_min": 3000.0, "magtol_max": 3000.0, "T_triplet": 50.0}, {"magtol_max": 1e5, "magtol_txscale": 50.0},
    {"magtol_txscale": -20.0, "magtol_min": 0.5}, {"p_charge_cut": 50000.0, "T_triplet": 1e5},
], ids=["default", "w64_t32", "w8_t3", "loose", "tolerance_past_binary16", "falling_tolerance", "charge_filter_loose_cut"])
def test_binary16_seeding(extra):
    """The pairs that the bracket leaves out are those that the binary16 filter
    rejects, whatever its constants; sets whose windows hold one z off the
    planes, and sets with mixed z, which stay binary32."""
    params = {"seed_fp16": 1, **extra}
    ev = lfgen.generate("nominal", n_events=21, seed=80)
    _check(ev, f"binary16 {extra}", params)
    shifted = lfgen.Events(**{**ev.__dict__, "hit_z": ev.hit_z + np.float32(1.5)})
    _check(shifted, f"binary16 shifted {extra}", params, modes=("batched",))
    rng = np.random.default_rng(81)
    some = np.isin(ev.hit_z, np.array([lfgen.LAYER_Z[l] for l in (0, 11)], np.float32)) & (rng.random(ev.n_hits) < 0.02)
    hz = (ev.hit_z + np.where(some, rng.uniform(-3.0, 3.0, ev.n_hits), 0.0)).astype(np.float32)
    _check(lfgen.Events(**{**ev.__dict__, "hit_z": hz}), f"binary16 mixed {extra}", params, modes=("batched",))
    _check(lfgen.generate("nominal", field="paper", n_events=21, seed=82), f"binary16 paper {extra}", params,
           lfgen.world("paper"), modes=("batched",))


def test_binary16_dense_events():
    _check(lfgen.generate("stress", n_events=9, seed=83), "binary16 stress", {"seed_fp16": 1})


def test_noalloc_and_budget_contexts():
    """The caller's device buffers, and a context with a device budget (its
    batches carry no search index), against the plain upload path."""
    import torch
    from paper_2402_14670_amd import lf
    ev = lfgen.concat([lfgen.generate("uneven", n_events=12, seed=67),
                       _jitter(lfgen.generate("nominal", n_events=12, seed=68), 1.5, 0.02, 69)])
    ref = oracle_parallel(ev)
    ctx = lf.lf_create(W, None, budget_bytes=1 << 30)
    try:
        say(f"[gpu] pair budget tracks={ev.n_tracks}")
        bid = lf.lf_upload_events(ctx, ev)
        lf.lf_find_tracks(ctx, bid, "batched")
        compare(ref, lf.lf_fetch_tracks(ctx, bid), label="budget")
        dev = {k: torch.from_numpy(getattr(ev, k).view(np.int32) if k.endswith("off") else getattr(ev, k)).cuda()
               for k in lf._IN_FIELDS}
        out = {k: torch.zeros((ev.n_tracks, 12) if k == "hit_idx" else ev.n_tracks, device="cuda",
                              dtype=torch.uint8 if k in ("found", "n_hits") else
                              torch.int32 if k == "hit_idx" else torch.float32) for k in lf._OUT_FIELDS}
        s = torch.cuda.Stream()
        s.wait_stream(torch.cuda.current_stream())
        for mode in ("batched", "persistent", "batched"):
            say(f"[gpu] pair noalloc mode={mode}")
            lf.lf_find_tracks_noalloc(ctx, dev, out, mode, s.cuda_stream)
            s.synchronize()
            compare(ref, {k: v.cpu().numpy() for k, v in out.items()}, label=f"noalloc/{mode}")
    finally:
        lf.lf_destroy(ctx)


def test_served_batches_of_mapped_slots():
    """Serving from a device pool with large batches: slots mapped to pool
    tracks, two per wavefront."""
    from paper_2402_14670_amd import lf
    ev = lfgen.concat([lfgen.generate("uneven", n_events=20, seed=70),
                       _jitter(lfgen.generate("nominal", n_events=5, seed=71), 1.5, 0.02, 72)])
    ref = lf.result_digests(oracle_parallel(ev), ev.trk_off)
    req = np.random.default_rng(73).integers(0, ev.n_events, 1500).astype(np.uint32)
    ctx = lf.lf_create(W)
    try:
        for pool in (0, 1):
            say(f"[gpu] pair serving pool_on_device={pool}")
            dig, lat, st = lf.lf_serve_run(ctx, ev, req, np.zeros(len(req)),
                                           {"pool_on_device": pool, "max_batch_events": 200, "verify_results": 1})
            assert np.array_equal(dig, ref[req]) and st["result_mismatches"] == 0
    finally:
        lf.lf_destroy(ctx)


@pytest.mark.parametrize("budget", [0, 1 << 20, 1 << 30])
def test_invalid_values_refused_while_the_batch_is_sent(budget):
    """A bad value is reported whatever else is wrong with the batch (here: its
    size), and the context goes on."""
    from paper_2402_14670_amd import lf
    ev = lfgen.generate("nominal", n_events=21, seed=59)
    small = lfgen.generate("single", n_events=2, seed=60)
    ctx = lf.lf_create(W, None, budget)
    for k, i in (("hit_x", ev.n_hits - 1), ("hit_dxdy", 0), ("trk_tx", ev.n_tracks - 1)):
        a = getattr(ev, k).copy()
        a[i] = np.nan
        with pytest.raises(lf.LFError) as e:
            lf.lf_upload_events(ctx, lfgen.Events(**{**ev.__dict__, k: a}))
        assert e.value.code == lf.LF_ERR_INVALID and "non-finite" in str(e.value)
    bid = lf.lf_upload_events(ctx, small)
    lf.lf_find_tracks(ctx, bid)
    compare(oracle_parallel(small), lf.lf_fetch_tracks(ctx, bid, small.n_tracks), label="after refusals")
    lf.lf_destroy(ctx)
