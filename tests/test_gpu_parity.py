"""HIP path vs the FP64 oracle, through the C ABI (needs an MI355X).

Bars (per output):
  * currents: per-pixel relative L2 error e_p = ||I_gpu - I_orc||_2 / max(||I_orc||_2, 10 e-) <= 1e-4;
  * integer / index work (sample-point counts, Philox words, pixel sets, hand-traced packets): bit-exact;
  * packets: tick and ADC code bit-exact, except where the oracle flags a decision within the FP32 error margin
    (ADC value near an LSB boundary, or the pixel's timeline after a near-threshold decision);
  * charge report: FP64 sums within the FP32 accumulation error.
"""
import dataclasses
import json
import os
import time

import numpy as np
import pytest

from paper_2212_09807_amd import workloads as W

pytestmark = pytest.mark.gpu

GOLD = os.path.join(os.path.dirname(__file__), "golden")
TOL_WAVE = 1e-4
EPS_REL, EPS_ABS = 2e-6, 0.1      # decision margin (electrons) within which FP32 and FP64 may legitimately differ


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "GPU tests need a visible MI355X"
    return t


@pytest.fixture(scope="module")
def lt(torch):
    from paper_2212_09807_amd import ltsim
    ltsim.lib()
    return ltsim


def per_pixel_errors(g, o):
    num = np.sqrt(((g - o) ** 2).sum(axis=1))
    den = np.maximum(np.sqrt((o ** 2).sum(axis=1)), 10.0)
    return num / den


def run_gpu(lt, w, ev=0, mode=0, table=None, slices=1, rt=0, shift=False, matrix=False):
    ctx = lt.Context.from_workload(w, table=table, reduce_mode=mode)
    ctx.set_induce_slices(slices)
    ctx.set_ticks_per_thread(rt)
    ctx.set_lane_exchange(shift)
    ctx.set_matrix_cores(matrix)
    segs = lt.to_device(w.events[ev])
    r = ctx.simulate(segs, event_id=w.event_ids[ev])
    h = r.host()
    return ctx, h


def gpu_packets_by_pixel(h):
    out = {}
    for p, t, a, f in zip(h["pkt_pixel"], h["pkt_tick"], h["pkt_adc"], h["pkt_flags"]):
        out.setdefault(int(p), []).append((int(t), int(a), int(f)))
    return out


def near_edge_pixels(w, uv):
    """Pixels whose table reach holds a bin where a Monte Carlo draw landed within FP32 reach of a bin edge."""
    ro, tb = w.readout, w.table
    out = set()
    for u, v in uv:
        for ix in range(max(0, (u - tb.b_x) // ro.n_sub - 1), min(ro.n_x, (u + tb.b_x) // ro.n_sub + 2)):
            for iy in range(max(0, (v - tb.b_y) // ro.n_sub - 1), min(ro.n_y, (v + tb.b_y) // ro.n_sub + 2)):
                uc, vc = ix * ro.n_sub + ro.n_sub // 2, iy * ro.n_sub + ro.n_sub // 2
                if -tb.b_x <= u - uc < tb.b_x and -tb.b_y <= v - vc < tb.b_y:
                    out.add(iy * ro.n_x + ix)
    return out


def compare_packets(h, pixels, orc_pk, ufrom, uncertain_pixels=()):
    """Return (compared, flagged, mismatches) over the oracle's pixels.  A pixel in `uncertain_pixels` whose
    packets differ counts as flagged (its current may legitimately differ by a draw landing across a bin edge)."""
    gb = gpu_packets_by_pixel(h)
    compared = flagged = 0
    bad = []
    for q, p in enumerate(pixels):
        ot, oa, of = orc_pk[q]
        uf = int(ufrom[q])
        if int(p) in uncertain_pixels:
            g = gb.get(int(p), [])
            if [(int(t), int(a)) for t, a in zip(ot, oa)] != [(x[0], x[1]) for x in g]:
                flagged += len(ot)
                continue
        g = gb.get(int(p), [])
        gt = np.array([x[0] for x in g], np.int64)
        ga = np.array([x[1] for x in g], np.int64)
        osel, gsel = ot < uf, gt < uf
        flagged += int((~osel).sum())
        if osel.sum() != gsel.sum() or np.any(ot[osel] != gt[gsel]):
            bad.append((int(p), "ticks", ot[osel].tolist(), gt[gsel].tolist()))
            continue
        chk = (of[osel] & 1) == 0
        flagged += int((~chk).sum())
        compared += int(chk.sum())
        if np.any(oa[osel][chk] != ga[gsel][chk]):
            bad.append((int(p), "adc", oa[osel].tolist(), ga[gsel].tolist()))
    return compared, flagged, bad


def check_event(lt, orc, w, ev=0, mode=0, table=None, slices=1, rt=0, shift=False, matrix=False):
    ctx, h = run_gpu(lt, w, ev, mode, table, slices, rt, shift, matrix)
    segs = w.events[ev]
    r = orc.simulate(w, ev, table=table, eps_rel=EPS_REL, eps_abs=EPS_ABS)
    opix = r["pixels"]
    gpix = h["pixel_id"]
    # every pixel the oracle reaches is active on the GPU; GPU-only pixels carry no current at all
    assert np.all(np.diff(gpix) > 0)
    pos = np.searchsorted(gpix, opix)
    assert np.all(pos < len(gpix)) and np.array_equal(gpix[pos], opix)
    extra = np.setdiff1d(np.arange(len(gpix)), pos)
    assert np.all(h["current"][extra] == 0.0)
    e = per_pixel_errors(h["current"][pos].astype(np.float64), r["wave"])
    assert e.max() <= TOL_WAVE, (e.max(), opix[np.argmax(e)])
    # FP64 report
    rep_g = h["report"][0]
    rep_o = r["report"]
    assert rep_g[0] == pytest.approx(rep_o["q_after_quench"], rel=2e-6)
    assert rep_g[1] == pytest.approx(rep_o["q_collected"], rel=2e-6)
    scale = rep_o["q_collected"]
    assert rep_g[2] == pytest.approx(rep_o["q_induced"], abs=1e-5 * scale)
    assert rep_g[3] == pytest.approx(rep_o["q_clipped"], abs=1e-5 * scale)
    assert rep_g[4] == pytest.approx(rep_o["q_offgrid"], abs=1e-5 * scale)
    unc = near_edge_pixels(w, r["mc_near_edges"]) if w.physics.mc_draws > 0 else ()
    cmp_, flg, bad = compare_packets(h, opix, r["packets"], r["uncertain_from"], unc)
    assert not bad, bad[:5]
    return h, r, e, (cmp_, flg)


# ----------------------------------------------------------------------------------------------- Philox / stages

def test_philox_known_answers_and_oracle(lt, orc, torch):
    rows = [list(map(lambda x: int(x, 16), l.split())) for l in open(os.path.join(GOLD, "philox4x32_10_kat.txt"))
            if l.strip() and not l.startswith("#")]
    for v in rows:
        ctr = torch.tensor(np.array(v[:4], np.uint32).view(np.int32)[None], device="cuda")
        out = lt.philox(ctr, v[4], v[5]).cpu().numpy().view(np.uint32)[0]
        assert out.tolist() == v[6:]
    rng = np.random.default_rng(3)
    ctr = rng.integers(0, 2 ** 32, size=(4096, 4), dtype=np.uint64).astype(np.uint32)
    k0, k1 = 0x12345678, 0x9ABCDEF0
    out = lt.philox(torch.tensor(ctr.view(np.int32), device="cuda"), k0, k1).cpu().numpy().view(np.uint32)
    for i in range(0, 4096, 97):
        assert out[i].tolist() == orc.philox4x32_10(ctr[i], [k0, k1]).tolist()


@pytest.mark.parametrize("cfg,model", [(1, 0), (2, 0), (2, 1)])
def test_quench_drift_stage(lt, orc, torch, cfg, model):
    w = W.make_workload(cfg)
    w.physics.recomb_model = model
    ctx = lt.Context.from_workload(w)
    f, i = ctx.stage_quench_drift(lt.to_device(w.events[0]))
    f, i = f.cpu().numpy().astype(np.float64), i.cpu().numpy()
    o = orc.quench_drift(w.physics, w.events[0])
    assert np.array_equal(i[:, 0], o["n_points"])                    # integer decided in FP32 on both sides
    assert np.array_equal(i[:, 1], o["flags"])
    for k, name in enumerate(("q_r", "q_a", "t_drift", "sigma_t", "sigma_time", "dedx")):
        np.testing.assert_allclose(f[:, k], o[name], rtol=2e-6, atol=1e-12, err_msg=name)


@pytest.mark.parametrize("cfg", [1, 2])
def test_charge_cells(lt, orc, torch, cfg):
    w = W.make_workload(cfg)
    if cfg == 2:
        w.events[0] = w.events[0].subset(np.arange(0, 20000, 500))
    ctx = lt.Context.from_workload(w)
    ctx.simulate(lt.to_device(w.events[0]))
    torch.cuda.synchronize()
    for s in range(0, w.events[0].n, max(1, w.events[0].n // 25)):
        (ga0, gna, gu0, gnu, gv0, gnv), gc = ctx.debug_cells(s)
        (oa0, ona, ou0, onu, ov0, onv), oc = orc.segment_cells(w.physics, w.readout, w.events[0], s)
        big = np.zeros((max(ga0 + gna, oa0 + ona) - min(ga0, oa0), max(gu0 + gnu, ou0 + onu) - min(gu0, ou0),
                        max(gv0 + gnv, ov0 + onv) - min(gv0, ov0)))
        A, U, V = min(ga0, oa0), min(gu0, ou0), min(gv0, ov0)
        g = big.copy()
        g[ga0 - A:ga0 - A + gna, gu0 - U:gu0 - U + gnu, gv0 - V:gv0 - V + gnv] = gc
        big[oa0 - A:oa0 - A + ona, ou0 - U:ou0 - U + onu, ov0 - V:ov0 - V + onv] = oc
        assert np.abs(g - big).max() <= 2e-6 * big.sum(), s
        assert g.sum() == pytest.approx(big.sum(), rel=2e-6)


# ----------------------------------------------------------------------------------------------- whole events

@pytest.mark.parametrize("mode,slices", [(0, 8), (0, 1), (1, 1), (2, 1)])
def test_cfg1_event_parity(lt, orc, torch, mode, slices):
    h, r, e, (cmp_, flg) = check_event(lt, orc, W.make_workload(1), mode=mode, slices=slices)
    print(f"cfg1 mode={mode} slices={slices}: pixels {len(r['pixels'])} max e_p {e.max():.2e} p99 {np.percentile(e, 99):.2e} "
          f"packets compared {cmp_} flagged {flg}")
    assert cmp_ > 50


def _ragged_workload(seed=7):
    """Several tiles' worth of pixels in a non-square grid, a tick count that is not a multiple of 4, segments
    leaving the grid, arriving before tick 0 and after the window, one zero-length deposit and one segment that
    crosses the anode plane."""
    rng = np.random.default_rng(seed)
    w = W.config(1)
    w.readout = W.Readout(n_x=23, n_y=17, n_ticks=777)
    parts = []
    for _ in range(6):
        p0 = np.array([rng.uniform(-1.0, 11.0), rng.uniform(-1.0, 8.5), rng.uniform(0.2, 12.0)])
        d = W.isotropic(rng)
        n = 30
        s = np.arange(n + 1) / n * rng.uniform(1.0, 6.0)
        pts = p0[None] + s[:, None] * d[None]
        pts[:, 2] = np.abs(pts[:, 2]) + 0.05
        L = np.linalg.norm(np.diff(pts, axis=0), axis=1)
        t0 = rng.uniform(-5.0, 30.0)
        parts.append(W.make_segments(pts[:-1], pts[1:], W.mip_dedx(rng, n) * L, t0=t0, t1=t0))
    parts.append(W.make_segments([[4.0, 3.0, 2.0]], [[4.0, 3.0, 2.0]], [0.02], t0=[1.0], t1=[1.0], dedx=[3.0]))
    parts.append(W.make_segments([[5.0, 4.0, -0.05]], [[5.05, 4.02, 0.07]], [0.05], t0=[2.0], t1=[2.0]))
    segs = W.Segments.concat(parts)
    segs.dedx = np.where(np.isnan(segs.dedx), np.float32(0.0), segs.dedx).astype(np.float32)
    w.events, w.event_ids = [segs], [77]
    return w


@pytest.mark.parametrize("mode,slices", [(0, 8), (0, 3), (1, 1), (2, 1)])
def test_ragged_multi_tile_parity(lt, orc, torch, mode, slices):
    h, r, e, _ = check_event(lt, orc, _ragged_workload(), mode=mode, slices=slices)
    assert r["report"]["q_clipped"] != 0.0 and r["report"]["q_offgrid"] > 0.0


def _max_window_workload():
    """The largest tick window the library accepts (8000 ticks) with a table longer than one 2048-tick pass of the
    per-pair kernel (T_R = 2300), steep segments whose charge boxes span ~200 ticks, a vertical track whose summed
    column series needs several pieces, a late track and one crossing the end of the window."""
    rng = np.random.default_rng(5)
    w = W.config(1)
    w.readout = W.Readout(n_x=12, n_y=10, n_ticks=8000)
    w.table = W.TableShape(2300, 10, 10)
    parts = []
    zs = np.linspace(2.0, 20.0, 7)                      # vertical track: 6 segments of 3 cm at one (x, y)
    a = np.stack([np.full(6, 2.13), np.full(6, 2.21), zs[:-1]], 1)
    b = np.stack([np.full(6, 2.13), np.full(6, 2.21), zs[1:]], 1)
    parts.append(W.make_segments(a, b, 2.1 * 3.0 * np.ones(6), t0=np.zeros(6), t1=np.zeros(6)))
    for t0, z0 in ((600.0, 4.0), (780.0, 6.0)):         # inclined tracks, late and at the window's end
        p0 = np.array([rng.uniform(0.5, 4.5), rng.uniform(0.5, 3.5), z0])
        d = np.array([0.5, 0.3, 0.8]) / np.linalg.norm([0.5, 0.3, 0.8])
        n = 12
        pts = p0[None] + (np.arange(n + 1) / n * 3.0)[:, None] * d[None]
        L = np.linalg.norm(np.diff(pts, axis=0), axis=1)
        parts.append(W.make_segments(pts[:-1], pts[1:], W.mip_dedx(rng, n) * L, t0=np.full(n, t0),
                                     t1=np.full(n, t0)))
    segs = W.Segments.concat(parts)
    w.events, w.event_ids = [segs], [123]
    return w


def _stacked_tracks_workload():
    """Two parallel 20-segment tracks over the same pixels at 5 and 15 cm of drift (about 600 ticks apart), plus a
    third one crossing both at 10 cm: the sub-pixel columns under them hold charge in separate tick ranges, which the
    summed induction must cut into separate pieces (a column's span is far longer than its segments' charge)."""
    rng = np.random.default_rng(21)
    w = W.config(1)
    parts = []
    for z, (x0, x1), (y0, y1) in ((5.0, (8.0, 20.0), (12.0, 12.3)), (15.0, (8.0, 20.0), (12.0, 12.3)),
                                  (10.0, (14.0, 14.4), (6.0, 18.0))):
        n = 20
        s = np.arange(n + 1) / n
        pts = np.stack([x0 + s * (x1 - x0), y0 + s * (y1 - y0), np.full(n + 1, z)], 1)
        L = np.linalg.norm(np.diff(pts, axis=0), axis=1)
        parts.append(W.make_segments(pts[:-1], pts[1:], W.mip_dedx(rng, n) * L, t0=np.zeros(n), t1=np.zeros(n)))
    w.events, w.event_ids = [W.Segments.concat(parts)], [31]
    return w


@pytest.mark.parametrize("mode", [0, 2])
def test_stacked_drift_separated_tracks_parity(lt, orc, torch, mode):
    h, r, e, (cmp_, flg) = check_event(lt, orc, _stacked_tracks_workload(), mode=mode)
    print(f"stacked tracks mode={mode}: pixels {len(r['pixels'])} max e_p {e.max():.2e} packets compared {cmp_}")
    assert cmp_ > 20


def test_stacked_tracks_summed_batch_equals_single(lt, torch):
    """The gap-cut summed columns are batch-invariant: a batch of the stacked event with a shifted copy gives each
    event's single-call currents bit for bit."""
    w = _stacked_tracks_workload()
    evs = [w.events[0], w.events[0].shifted(dt=2.5)]
    ctx = lt.Context.from_workload(w, reduce_mode=2)
    singles = [ctx.simulate(lt.to_device(s), event_id=i).host() for s, i in zip(evs, (31, 32))]
    offs = np.r_[0, np.cumsum([s.n for s in evs])]
    b = ctx.simulate_batch(lt.to_device(W.Segments.concat(evs)), offs, [31, 32]).host()
    po = b["event_pixel_offsets"]
    for e, s in enumerate(singles):
        assert np.array_equal(b["pixel_id"][po[e]:po[e + 1]], s["pixel_id"])
        assert np.array_equal(b["current"][po[e]:po[e + 1]], s["current"])


def _drift_parallel_track_workload():
    """A track along the drift direction (10 cm of drift at almost fixed x and y, 834 segments of 120 um) plus a short
    one beside it: each sub-pixel column under the long track holds several hundred segments whose charge forms one
    interval of ~625 ticks, cut into several pieces; the column sort, the interval scan and the summed charges take
    their long-list paths there (more than 64 and more than 256 segments per column)."""
    rng = np.random.default_rng(47)
    w = W.config(1)
    parts = []
    for (x0, x1), (y0, y1), (z0, z1), n in (((15.30, 15.34), (15.10, 15.13), (4.0, 14.0), 834),
                                            ((17.0, 17.6), (15.1, 15.2), (6.0, 6.05), 6)):
        s = np.arange(n + 1) / n
        pts = np.stack([x0 + s * (x1 - x0), y0 + s * (y1 - y0), z0 + s * (z1 - z0)], 1)
        L = np.linalg.norm(np.diff(pts, axis=0), axis=1)
        parts.append(W.make_segments(pts[:-1], pts[1:], W.mip_dedx(rng, n) * L, t0=np.zeros(n), t1=np.zeros(n)))
    w.events, w.event_ids = [W.Segments.concat(parts)], [33]
    return w


@pytest.mark.parametrize("mode,rt", [(0, 0), (2, 0), (2, 8)])
def test_drift_parallel_track_parity(lt, orc, torch, mode, rt):
    h, r, e, (cmp_, flg) = check_event(lt, orc, _drift_parallel_track_workload(), mode=mode, rt=rt)
    print(f"drift-parallel track mode={mode} rt={rt}: pixels {len(r['pixels'])} max e_p {e.max():.2e} "
          f"packets compared {cmp_}")
    assert cmp_ > 20


def test_calls_on_two_streams_do_not_race(lt, torch):
    """Consecutive calls on one context given different streams, with no host synchronisation between their
    device work, give the results of separate synchronised calls (each call waits for the previous one's work on
    the shared scratch pool)."""
    w = W.make_workload(1, n_events=2)
    w.events[1] = w.events[1].shifted(dt=4.0)
    ctx = lt.Context.from_workload(w)
    d = [lt.to_device(s) for s in w.events]
    ref = [ctx.simulate(x, event_id=i).host() for x, i in zip(d, w.event_ids)]
    outs = [ctx._alloc(ref[k]["counts"][0], ref[k]["counts"][0] * w.electronics.max_packets, 1, False)
            for k in range(2)]
    torch.cuda.synchronize()
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    for rep in range(3):
        for k, st in ((0, s1), (1, s2)):
            ctx.simulate(d[k], event_id=w.event_ids[k], stream=st, out=outs[k])
        torch.cuda.synchronize()
        for k in range(2):
            g = outs[k].host()
            assert np.array_equal(g["pixel_id"], ref[k]["pixel_id"]), (rep, k)
            assert np.array_equal(g["current"], ref[k]["current"]), (rep, k)
            assert np.array_equal(g["pkt_tick"], ref[k]["pkt_tick"]), (rep, k)


def test_host_allocation_failure_returns_oom(lt, torch):
    """A host allocation that fails inside a call comes back as LTS_ERR_OOM (no exception crosses the ABI), and the
    context and a server keep working: the failed server batch fails only its own tickets."""
    w = W.make_workload(1, n_events=2)
    table = W.response_table(w.table, w.readout, w.physics.v_drift)
    ctx = lt.Context.from_workload(w, table=table)
    lt.fail_host_alloc(0)
    try:
        with pytest.raises(lt.LtsimError) as ei:
            ctx._check(lt.lib().lts_set_response(ctx._h, np.ascontiguousarray(table).ctypes.data_as(
                __import__("ctypes").c_void_p), *table.shape))
        assert ei.value.status == 3
    finally:
        lt.fail_host_alloc(-1)
    h = ctx.simulate(lt.to_device(w.events[0]), event_id=w.event_ids[0]).host()      # still usable
    assert h["counts"][0] > 0
    srv = lt.Server(ctx, n_lanes=1, max_batch_events=1)
    try:
        lt.fail_host_alloc(0)                       # the next allocation point: the submission's copy
        with pytest.raises(lt.LtsimError) as ei:
            srv.submit(w.events[0], w.event_ids[0])
        assert ei.value.status == 3
        lt.fail_host_alloc(1)                       # the submission passes, the lane's batch set-up fails
        t0 = srv.submit(w.events[0], w.event_ids[0])
        with pytest.raises(lt.LtsimError) as ei:
            srv.wait(t0, 60.0)
        assert ei.value.status == 3
        lt.fail_host_alloc(-1)
        t1 = srv.submit(w.events[1], w.event_ids[1])
        g = srv.wait(t1, 60.0)
        assert g["status"] == 0 and len(g["pixel_id"]) > 0
        srv.release(t0)
        srv.release(t1)
    finally:
        lt.fail_host_alloc(-1)
        srv.stop()


@pytest.mark.parametrize("mode,rt,shift", [(0, 0, False), (0, 8, False), (0, 0, True), (1, 0, False), (2, 0, False),
                                           (2, 8, False), (2, 0, True)])
def test_max_window_long_table_parity(lt, orc, torch, mode, rt, shift):
    w = _max_window_workload()
    h, r, e, (cmp_, flg) = check_event(lt, orc, w, mode=mode, rt=rt, shift=shift)
    print(f"max window mode={mode} rt={rt} shift={shift}: pixels {len(r['pixels'])}, max e_p {e.max():.2e}, "
          f"packets compared {cmp_}")
    assert r["report"]["q_clipped"] != 0.0 and cmp_ > 0


@pytest.mark.parametrize("mode,matrix", [(0, False), (2, False), (0, True)])
def test_cfg2_full_size_sampled_pixels(lt, orc, torch, mode, matrix):
    """The module-scale event at full size, in the launch configurations the benchmark times; the oracle
    recomputes a sample of pixels one by one."""
    w = W.make_workload(2)
    ctx, h = run_gpu(lt, w, mode=mode, matrix=matrix)
    gpix, cur = h["pixel_id"], h["current"]
    tot = np.abs(cur).sum(axis=1)
    rng = np.random.default_rng(11)
    pick = np.unique(np.r_[np.argsort(tot)[-4:], rng.choice(len(gpix), 4, replace=False)])
    o_wave, _ = orc.waveforms(w.physics, w.readout, W.response_table(w.table, w.readout, w.physics.v_drift),
                              w.events[0], gpix[pick])
    e = per_pixel_errors(cur[pick].astype(np.float64), o_wave)
    print("cfg2 sampled e_p:", e)
    assert e.max() <= TOL_WAVE
    qd = orc.quench_drift(w.physics, w.events[0])
    rep = h["report"][0]
    assert rep[0] == pytest.approx(qd["q_r"].sum(), rel=2e-6)
    assert rep[1] == pytest.approx(qd["q_a"].sum(), rel=2e-6)
    # conservation at full size: collected = induced in window + clipped + off-grid
    assert rep[2] + rep[3] + rep[4] == pytest.approx(rep[1], rel=2e-5)
    pk, _, uf = orc.electronics(w.electronics, w.readout, w.event_ids[0], gpix[pick], o_wave, EPS_REL, EPS_ABS,
                                with_uncertain=True)
    _, _, bad = compare_packets(h, gpix[pick], pk, uf)
    assert not bad


@pytest.mark.parametrize("mode", [0, 2])
def test_large_spill_tile_sampled_pixels(lt, orc, torch, mode):
    """One tile of the large spill (halo replicas included, 5000 ticks, full reset/discriminator/sample noise), in
    the launch configuration of the large-spill benchmark; the oracle recomputes a sample of pixels one by one."""
    w = W.make_workload(5)
    ev = sorted(range(len(w.events)), key=lambda i: w.events[i].n)[2]        # a cosmic-dominated tile, ~14k segments
    ctx, h = run_gpu(lt, w, ev=ev, mode=mode)
    gpix, cur = h["pixel_id"], h["current"]
    tot = np.abs(cur).sum(axis=1)
    rng = np.random.default_rng(5)
    pick = np.unique(np.r_[np.argsort(tot)[-3:], rng.choice(len(gpix), 3, replace=False)])
    o_wave, _ = orc.waveforms(w.physics, w.readout, W.response_table(w.table, w.readout, w.physics.v_drift),
                              w.events[ev], gpix[pick])
    e = per_pixel_errors(cur[pick].astype(np.float64), o_wave)
    print(f"large-spill tile {ev} ({w.events[ev].n} segments) sampled e_p:", e)
    assert e.max() <= TOL_WAVE
    qd = orc.quench_drift(w.physics, w.events[ev])
    rep = h["report"][0]
    assert rep[1] == pytest.approx(qd["q_a"].sum(), rel=2e-6)
    assert rep[2] + rep[3] + rep[4] == pytest.approx(rep[1], rel=2e-5)
    pk, _, uf = orc.electronics(w.electronics, w.readout, w.event_ids[ev], gpix[pick], o_wave, EPS_REL, EPS_ABS,
                                with_uncertain=True)
    cmp_, flg, bad = compare_packets(h, gpix[pick], pk, uf)
    print(f"large-spill tile packets: compared {cmp_} flagged {flg}")
    assert not bad and cmp_ > 0


def test_summed_kernels_reproducible_and_agree(lt, torch):
    """Summed induction on a spill-mix event whose pixels have long runs of same-bin pieces (merged records up to
    the 248-tick cap): the 256-tick kernel gives bit-identical currents call after call, and agrees with the
    512-tick kernel to FP32 summation order."""
    w = W.make_workload(3, n_events=8)
    ev, eid = w.events[2], w.event_ids[2]
    runs = {}
    for rt in (0, 0, 8):
        ctx = lt.Context.from_workload(w, reduce_mode=2)
        ctx.set_ticks_per_thread(rt)
        runs.setdefault(rt, []).append(ctx.simulate(lt.to_device(ev), event_id=eid).host())
        ctx.close()
    a, b, c = runs[0][0], runs[0][1], runs[8][0]
    assert np.array_equal(a["pixel_id"], b["pixel_id"]) and np.array_equal(a["current"], b["current"])
    assert np.array_equal(a["pixel_id"], c["pixel_id"])
    e = per_pixel_errors(a["current"].astype(np.float64), c["current"].astype(np.float64))
    print(f"summed 256 vs 512 kernel: max e_p {e.max():.2e}")
    assert e.max() <= 1e-5


def test_sorted_and_atomic_agree(lt, torch):
    w = W.make_workload(1)
    _, a = run_gpu(lt, w, mode=0)
    _, b = run_gpu(lt, w, mode=1)
    _, c = run_gpu(lt, w, mode=0, slices=1)
    assert np.array_equal(a["pixel_id"], b["pixel_id"]) and np.array_equal(a["pixel_id"], c["pixel_id"])
    assert per_pixel_errors(b["current"].astype(np.float64), a["current"].astype(np.float64)).max() < 1e-5
    assert per_pixel_errors(c["current"].astype(np.float64), a["current"].astype(np.float64)).max() < 1e-5
    # the sorted reduction is deterministic: a second run is bit-identical
    _, a2 = run_gpu(lt, w, mode=0)
    assert np.array_equal(a["current"], a2["current"])


# ----------------------------------------------------------------------------------------------- edge cases

@pytest.mark.parametrize("off", [(0,), (3,), (7,), (0, 1, 4, 7), tuple(range(8))])
def test_atomic_segments_off_the_readout(lt, orc, torch, off):
    """Atomic mode with segments that reach no pixel at the start, in the middle and at the end of a block of eight, in
    neighbouring pairs and as whole blocks: the currents of the others, and no work for them (the call takes milliseconds;
    a walk over a rectangle that they do not have would take seconds)."""
    w = W.make_workload(1)
    segs = w.events[0].subset(np.arange(0, 48))
    away = (np.arange(48) // 8 % 2 == 0) & np.isin(np.arange(48) % 8, off)      # (every other block)
    for c in ("x0", "x1"):
        getattr(segs, c)[away] += np.float32(500.0)
    w.events = [segs]
    h, r, e, _ = check_event(lt, orc, w, mode=1)
    assert len(r["pixels"]) > 50
    ctx = lt.Context.from_workload(w, reduce_mode=1)
    d = lt.to_device(segs)
    out = ctx.simulate(d, event_id=w.event_ids[0])
    torch.cuda.synchronize()
    t = time.perf_counter()
    ctx.simulate(d, event_id=w.event_ids[0], out=out)
    torch.cuda.synchronize()
    t = time.perf_counter() - t
    print(f"off {off}: {len(r['pixels'])} pixels, max e_p {e.max():.2e}, {t * 1e3:.2f} ms")
    assert t < 0.2


def test_empty_event(lt, torch):
    w = W.make_workload(1)
    w.events = [w.events[0].subset(np.arange(0))]
    ctx = lt.Context.from_workload(w)
    h = ctx.simulate(lt.to_device(w.events[0])).host()
    assert h["counts"][0] == 0 and h["counts"][1] == 0 and np.all(h["report"] == 0.0)


def test_invalid_inputs_and_capacity(lt, torch):
    w = W.make_workload(1)
    ctx = lt.Context.from_workload(w)
    bad = w.events[0].subset(np.arange(5))
    bad.x0 = bad.x0.copy()
    bad.x0[2] = np.nan
    with pytest.raises(lt.LtsimError) as ei:
        ctx.simulate(lt.to_device(bad))
    assert ei.value.status == 1
    zl = W.make_segments([[1.0, 1.0, 1.0]], [[1.0, 1.0, 1.0]], [0.01])
    with pytest.raises(lt.LtsimError) as ei:
        ctx.simulate(lt.to_device(zl))
    assert ei.value.status == 1
    long = W.make_segments([[1.0, 1.0, 1.0]], [[1.0, 1.0, 20.0]], [40.0])
    with pytest.raises(lt.LtsimError) as ei:
        ctx.simulate(lt.to_device(long))
    assert ei.value.status == 1
    segs = lt.to_device(w.events[0])
    need = ctx.plan(segs)
    small = ctx._alloc(need["pixels"] - 1, need["packets"], 1, False)
    with pytest.raises(lt.LtsimError) as ei:
        ctx.simulate(segs, out=small)
    assert ei.value.status == 2
    assert int(small.counts[0].item()) == need["pixels"]
    # the context stays usable after recoverable errors
    h = ctx.simulate(segs).host()
    assert h["counts"][0] == need["pixels"]
    # parameter combinations the library does not offer are refused at context creation
    for bad_ph in (dataclasses.replace(w.physics, per_point=1, mc_draws=4), dataclasses.replace(w.physics, per_point=2),
                   dataclasses.replace(w.physics, mc_draws=-1)):
        with pytest.raises(lt.LtsimError) as ei:
            lt.Context(bad_ph, w.readout, w.electronics, W.response_table(w.table, w.readout, w.physics.v_drift))
        assert ei.value.status == 1


# ----------------------------------------------------------------------------------------------- electronics

def test_electronics_hand_traced(lt, orc, torch):
    for c in json.load(open(os.path.join(GOLD, "electronics_traces.json")))["cases"]:
        w = W.config(1)
        w.readout = W.Readout(n_x=4, n_y=4, n_ticks=len(c["current"]))
        w.electronics = W.Electronics(threshold=c["threshold"], hold_ticks=c["hold_ticks"],
                                      min_spacing=c["min_spacing"], q_lsb=c["q_lsb"], pedestal=c["pedestal"],
                                      adc_bits=c["adc_bits"], sigma_unc=0.0, max_packets=16,
                                      reset_period=c.get("reset_period", 0))
        ctx = lt.Context.from_workload(w)
        pix = torch.tensor([5], dtype=torch.int32, device="cuda")
        cur = torch.tensor(np.array(c["current"], np.float32)[None], device="cuda")
        h = ctx.stage_electronics(0, pix, cur).host()
        got = [[int(t), int(a)] for t, a in zip(h["pkt_tick"], h["pkt_adc"])]
        assert got == c["packets"], c["name"]
        assert int(h["counts"][2]) == c["dropped"], c["name"]


@pytest.mark.parametrize("period", [0, 37])
def test_electronics_with_full_noise_vs_oracle(lt, orc, torch, period):
    w = W.config(5)
    w.electronics.reset_period = period
    w.readout = W.Readout(n_x=64, n_y=64, n_ticks=1500)
    rng = np.random.default_rng(9)
    n = 400
    cur = np.zeros((n, 1500))
    for q in range(n):
        for _ in range(rng.integers(1, 5)):
            t0, amp, wid = rng.integers(0, 1400), rng.uniform(200, 3000), rng.uniform(2, 30)
            tt = np.arange(1500)
            cur[q] += amp * np.exp(-0.5 * ((tt - t0) / wid) ** 2)
    cur32 = cur.astype(np.float32)
    pix = np.sort(rng.choice(64 * 64, n, replace=False)).astype(np.int32)
    ctx = lt.Context.from_workload(w)
    h = ctx.stage_electronics(123, torch.tensor(pix, device="cuda"), torch.tensor(cur32, device="cuda")).host()
    pk, st, uf = orc.electronics(w.electronics, w.readout, 123, pix, cur32.astype(np.float64), EPS_REL, EPS_ABS,
                                 with_uncertain=True)
    cmp_, flg, bad = compare_packets(h, pix, pk, uf)
    print(f"noise electronics: compared {cmp_} flagged {flg}")
    assert not bad, bad[:3]
    assert cmp_ > 500 and flg <= 0.01 * (cmp_ + flg)


@pytest.mark.parametrize("period,hold,spacing", [(64, 0, 0), (1, 0, 0), (5, 70, 3), (128, 16, 11),
                                                 (0, 2**31 - 1, 11), (0, 16, 2**31 - 1)])
def test_electronics_walk_edges_vs_oracle(lt, orc, torch, period, hold, spacing):
    """Resets on chunk edges and on every tick, samples at the crossing tick, holds that skip several resets, and
    holds or spacings beyond every tick; 1000 ticks end in a partial 40-tick chunk."""
    w = W.config(5)
    w.electronics.reset_period, w.electronics.hold_ticks, w.electronics.min_spacing = period, hold, spacing
    nt = 1000
    w.readout = W.Readout(n_x=32, n_y=32, n_ticks=nt)
    rng = np.random.default_rng(11 + period)
    n = 200
    tt = np.arange(nt)
    cur = np.zeros((n, nt))
    for q in range(n):
        for _ in range(rng.integers(1, 6)):
            t0, amp, wid = rng.integers(0, nt), rng.uniform(200, 6000), rng.uniform(0.5, 20)
            cur[q] += amp * np.exp(-0.5 * ((tt - t0) / wid) ** 2)
    cur32 = cur.astype(np.float32)
    pix = np.sort(rng.choice(32 * 32, n, replace=False)).astype(np.int32)
    ctx = lt.Context.from_workload(w)
    h = ctx.stage_electronics(77, torch.tensor(pix, device="cuda"), torch.tensor(cur32, device="cuda")).host()
    pk, st, uf = orc.electronics(w.electronics, w.readout, 77, pix, cur32.astype(np.float64), EPS_REL, EPS_ABS,
                                 with_uncertain=True)
    cmp_, flg, bad = compare_packets(h, pix, pk, uf)
    print(f"walk edges {period} {hold} {spacing}: compared {cmp_} flagged {flg} dropped {h['counts'][2]} / {st[0]}")
    assert not bad, bad[:3]
    n_unc = int((uf < nt).sum())
    assert abs(int(h["counts"][2]) - int(st[0])) <= n_unc            # dropped samples
    if hold >= nt:
        assert len(h["pkt_tick"]) == 0 and int(st[0]) > 0
    else:
        assert cmp_ > 20 and flg <= 0.02 * (cmp_ + flg)
    if spacing >= nt:                                                  # one sample per pixel at most
        assert len(np.unique(h["pkt_pixel"])) == len(h["pkt_pixel"])


@pytest.mark.parametrize("n_ticks,period", [(1, 0), (63, 0), (64, 50), (65, 0), (255, 0), (257, 64), (1000, 0), (1000, 300)])
def test_electronics_idle_chunks_vs_oracle(lt, orc, torch, n_ticks, period):
    """Charges that hold still 0.2 to 8 noise widths below the threshold: chunks that need no draw, that their draws
    settle, and that have a crossing, in windows that end within a chunk, a group of four and a loaded word."""
    w = W.config(5)
    w.electronics.reset_period = period
    w.readout = W.Readout(n_x=32, n_y=32, n_ticks=n_ticks)
    el = w.electronics
    rng = np.random.default_rng(n_ticks + period)
    n = 256
    cur = rng.normal(0.0, 0.01, (n, n_ticks)) * el.sigma_disc
    cur[:, 0] += el.threshold - el.sigma_disc * np.linspace(0.2, 8.0, n)
    cur[::3, n_ticks // 2] += 3.0 * el.sigma_disc
    cur[::5, n_ticks - 1] -= 2.0 * el.threshold
    cur32 = cur.astype(np.float32)
    pix = np.arange(n, dtype=np.int32)
    ctx = lt.Context.from_workload(w)
    h = ctx.stage_electronics(9, torch.tensor(pix, device="cuda"), torch.tensor(cur32, device="cuda")).host()
    pk, st, uf = orc.electronics(el, w.readout, 9, pix, cur32.astype(np.float64), EPS_REL, EPS_ABS, with_uncertain=True)
    cmp_, flg, bad = compare_packets(h, pix, pk, uf)
    print(f"idle chunks {n_ticks} {period}: compared {cmp_} flagged {flg} dropped {h['counts'][2]} / {st[0]}")
    assert not bad, bad[:3]
    assert abs(int(h["counts"][2]) - int(st[0])) <= int((uf < n_ticks).sum())
    assert float(h["report"][0][2]) == pytest.approx(float(cur32.astype(np.float64).sum()), rel=1e-12)


# ----------------------------------------------------------------------------------------------- batching

@pytest.mark.parametrize("mode", [0, 2])
def test_batch_equals_single_events(lt, torch, mode):
    w = W.make_workload(1, n_events=3)
    w.events[1] = w.events[1].shifted(dt=3.0)
    ctx = lt.Context.from_workload(w, reduce_mode=mode)
    singles = [ctx.simulate(lt.to_device(s), event_id=i).host() for s, i in zip(w.events, w.event_ids)]
    allsegs = W.Segments.concat(w.events)
    offs = np.r_[0, np.cumsum([s.n for s in w.events])]
    b = ctx.simulate_batch(lt.to_device(allsegs), offs, w.event_ids).host()
    po, ko = b["event_pixel_offsets"], b["event_packet_offsets"]
    for e, s in enumerate(singles):
        assert np.array_equal(b["pixel_id"][po[e]:po[e + 1]], s["pixel_id"])
        assert np.array_equal(b["current"][po[e]:po[e + 1]], s["current"])          # bit-identical (sorted mode)
        assert np.array_equal(b["pkt_tick"][ko[e]:ko[e + 1]], s["pkt_tick"])
        assert np.array_equal(b["pkt_adc"][ko[e]:ko[e + 1]], s["pkt_adc"])
        np.testing.assert_allclose(b["report"][e], s["report"][0], rtol=1e-12, atol=1e-9)


@pytest.mark.parametrize("n,per_point", [(1, 0), (255, 1), (256, 0)])
def test_cells_are_the_same_in_any_workgroup(lt, torch, n, per_point):
    """Charge cells by 1024 threads a segment (few segments) and by 256 (the same events five times in a batch): the same
    currents bit for bit."""
    w = W.make_workload(1, n_events=1)
    w.physics.per_point = per_point
    e = w.events[0]
    part = dataclasses.replace(e, **{f.name: getattr(e, f.name)[:n] for f in dataclasses.fields(e)
                                     if isinstance(getattr(e, f.name), np.ndarray)})
    ctx = lt.Context.from_workload(w)
    one = ctx.simulate(lt.to_device(part), event_id=3).host()
    k = 5 if n > 1 else 300
    b = ctx.simulate_batch(lt.to_device(W.Segments.concat([part] * k)), np.arange(k + 1) * part.n, [3] * k).host()
    po = b["event_pixel_offsets"]
    for i in (0, k - 1):
        assert np.array_equal(b["pixel_id"][po[i]:po[i + 1]], one["pixel_id"])
        assert np.array_equal(b["current"][po[i]:po[i + 1]], one["current"])


@pytest.mark.parametrize("n,draws", [(1, 471), (1, 472), (6, 2)])
def test_draw_counts_in_any_width(lt, orc, torch, n, draws):
    """Hits of 139 points x 471 draws fit in 16 bits (two cells a word), of 472 draws they need not."""
    w = W.make_workload(1, n_events=1)
    w.physics.mc_draws = draws
    e = w.events[0]
    w.events[0] = dataclasses.replace(e, **{f.name: getattr(e, f.name)[:n] for f in dataclasses.fields(e)
                                            if isinstance(getattr(e, f.name), np.ndarray)})
    check_event(lt, orc, w, mode=0)


@pytest.mark.parametrize("n_x,n_y,mode", [(127, 129, 0), (128, 128, 2), (8, 1024, 0), (130, 127, 2)])
def test_pixel_scans_at_their_limits(lt, orc, torch, n_x, n_y, mode):
    """Pixel grids whose counts are scanned by one workgroup in one or two passes (8192 and 16,384 elements) or by tiles."""
    w = _edge_workload(255, 37, 5, 3, 10)
    w.readout = dataclasses.replace(w.readout, n_x=n_x, n_y=n_y)
    check_event(lt, orc, w, mode=mode)


@pytest.mark.parametrize("n_ev", [16, 17])
def test_events_listed_in_the_launch_or_copied(lt, torch, n_ev):
    w = W.make_workload(1, n_events=1)
    e = w.events[0]
    part = dataclasses.replace(e, **{f.name: getattr(e, f.name)[:9] for f in dataclasses.fields(e)
                                     if isinstance(getattr(e, f.name), np.ndarray)})
    ids = [(1 << 40) + 7 * i for i in range(n_ev)]
    ctx = lt.Context.from_workload(w)
    b = ctx.simulate_batch(lt.to_device(W.Segments.concat([part] * n_ev)), np.arange(n_ev + 1) * part.n, ids).host()
    po, ko = b["event_pixel_offsets"], b["event_packet_offsets"]
    for i in (0, n_ev - 1):
        s = ctx.simulate(lt.to_device(part), event_id=ids[i]).host()
        assert np.array_equal(b["pixel_id"][po[i]:po[i + 1]], s["pixel_id"])
        assert np.array_equal(b["current"][po[i]:po[i + 1]], s["current"])
        assert np.array_equal(b["pkt_adc"][ko[i]:ko[i + 1]], s["pkt_adc"])
        assert np.array_equal(b["pkt_tick"][ko[i]:ko[i + 1]], s["pkt_tick"])


def test_pixel_products_are_the_same_in_any_workgroup(lt, torch):
    """An event whose pixels take 512 threads each gives, in a batch with more than 2048 pixels (256 threads each), the
    same currents bit for bit; dense segments, so that a pixel has several groups and stages."""
    w = W.make_workload(2)
    e = w.events[0]
    part = dataclasses.replace(e, **{f.name: getattr(e, f.name)[:300] for f in dataclasses.fields(e)
                                     if isinstance(getattr(e, f.name), np.ndarray)})
    ctx = lt.Context.from_workload(w)
    one = ctx.simulate(lt.to_device(part), event_id=5).host()
    assert len(one["pixel_id"]) <= 2048
    k = 2048 // len(one["pixel_id"]) + 1
    b = ctx.simulate_batch(lt.to_device(W.Segments.concat([part] * k)), np.arange(k + 1) * part.n, [5] * k).host()
    po = b["event_pixel_offsets"]
    for i in (0, k - 1):
        assert np.array_equal(b["pixel_id"][po[i]:po[i + 1]], one["pixel_id"])
        assert np.array_equal(b["current"][po[i]:po[i + 1]], one["current"])


def test_more_records_than_threads_of_a_launch(lt, torch):
    """A batch of 64 spill-mix events has over 2^32 / 8 merged records: its last events are those of single calls."""
    w = W.make_workload(3, n_events=64)
    ctx = lt.Context.from_workload(w, reduce_mode=2)
    offs = np.r_[0, np.cumsum([e.n for e in w.events])]
    dev = {i: lt.to_device(w.events[i]) for i in (40, 63)}
    cap = sum(ctx.plan(lt.to_device(e))["pixels"] for e in w.events)
    out = ctx._alloc(cap, cap * w.electronics.max_packets // 4 + 4096, 64, True)
    b = ctx.simulate_batch(lt.to_device(W.Segments.concat(w.events)), offs, w.event_ids, out=out)
    po = b.event_pixel_offsets.cpu().numpy()
    for i, d in dev.items():
        one = ctx.simulate(d, event_id=w.event_ids[i])
        n = int(po[i + 1] - po[i])
        assert torch.equal(b.pixel_id[po[i]:po[i + 1]], one.pixel_id[:n])
        assert torch.equal(b.current[po[i]:po[i + 1]], one.current[:n])


def test_graph_replay_equals_direct_launches(lt, torch):
    """Calls replayed as HIP graphs (updated in place between events of different sizes, re-instantiated when the
    launch structure changes) give the same results as direct launches, with the program's own GPU work and
    synchronisations between the calls."""
    w = W.make_workload(1, n_events=4)
    for e in range(4):
        w.events[e] = w.events[e].shifted(dt=0.7 * e)
    direct = lt.Context.from_workload(w)
    graph = lt.Context.from_workload(w)
    graph.set_graph(True)
    dev = [lt.to_device(x) for x in w.events]
    ref = [direct.simulate(d, event_id=i).host() for d, i in zip(dev, w.event_ids)]
    scratch = torch.zeros(1 << 20, device="cuda")
    for rep in range(3):
        for d, i, r in zip(dev, w.event_ids, ref):
            g = graph.simulate(d, event_id=i).host()
            scratch.add_(1.0)
            torch.cuda.synchronize()
            for k in ("pixel_id", "current", "pkt_pixel", "pkt_tick", "pkt_adc", "pkt_flags", "counts"):
                assert np.array_equal(g[k], r[k]), (rep, k)
            np.testing.assert_allclose(g["report"], r["report"], rtol=1e-12, atol=1e-9)
    upd, inst = graph.graph_stats()
    print(f"graph: {upd} in-place updates, {inst} instantiations over 12 calls")
    assert upd + inst == 12                                  # every call ran as a graph
    allsegs = W.Segments.concat(w.events)
    offs = np.r_[0, np.cumsum([x.n for x in w.events])]
    bd = direct.simulate_batch(lt.to_device(allsegs), offs, w.event_ids).host()
    bg = graph.simulate_batch(lt.to_device(allsegs), offs, w.event_ids).host()
    for k in ("pixel_id", "current", "pkt_tick", "pkt_adc", "event_pixel_offsets", "event_packet_offsets"):
        assert np.array_equal(bd[k], bg[k]), k
    assert graph.graph_stats()[1] == inst + 1                # the batch's extra offsets kernel: a new instance
    for mode in (1, 2):                                      # atomic (graph), summed (direct launches)
        direct.set_reduce_mode(mode)
        graph.set_reduce_mode(mode)
        a = direct.simulate(dev[0], event_id=w.event_ids[0]).host()
        b = graph.simulate(dev[0], event_id=w.event_ids[0]).host()
        assert np.array_equal(a["pixel_id"], b["pixel_id"])
        np.testing.assert_allclose(b["current"], a["current"], rtol=1e-5, atol=1e-3)


# ----------------------------------------------------------------------------------------------- serving

def test_served_results_equal_alone(lt, torch):
    """Events served in a mix (continuous batching over two lanes) give the same result as each event alone."""
    w = W.make_workload(1, n_events=6)
    for e in range(6):                              # the last event arrives late: samples fall past the window
        w.events[e] = w.events[e].shifted(dt=0.5 * e if e < 5 else 21.5)
    ctx = lt.Context.from_workload(w)
    alone = [ctx.simulate(lt.to_device(s), event_id=i).host() for s, i in zip(w.events, w.event_ids)]
    assert alone[5]["counts"][2] > 0 and alone[0]["counts"][2] == 0
    srv = lt.Server(ctx, n_lanes=2, max_batch_events=4, return_currents=True)
    try:
        tickets = [srv.submit(s, i) for s, i in zip(w.events, w.event_ids)]
        got = [srv.wait(t, 60.0) for t in tickets]
        for t in tickets:
            srv.release(t)
    finally:
        srv.stop()
    assert max(g["batch_events"] for g in got) > 1          # some events really were batched together
    for a, g in zip(alone, got):
        assert g["status"] == 0
        assert np.array_equal(a["pixel_id"], g["pixel_id"])
        assert np.array_equal(a["current"], g["current"])            # deterministic sorted reduction
        assert np.array_equal(a["pkt_tick"], g["pkt_tick"]) and np.array_equal(a["pkt_adc"], g["pkt_adc"])
        assert np.array_equal(a["pkt_flags"], g["pkt_flags"])
        assert np.array_equal(a["counts"], g["counts"])              # per-event dropped / overflow counts
        np.testing.assert_allclose(a["report"][0], g["report"], rtol=1e-12, atol=1e-9)


def test_server_admission_by_device_memory(lt, torch):
    """Memory-based admission on the device: with a budget below one event's footprint every event finishes with
    LTS_ERR_OOM and the server keeps serving; with a budget that holds a few events the lanes halve their batches
    (no batch reaches the 8 events submitted together) and every result equals the event alone."""
    w = W.make_workload(1, n_events=8)
    for e in range(8):
        w.events[e] = w.events[e].shifted(dt=0.3 * e)
    ctx = lt.Context.from_workload(w)
    alone = [ctx.simulate(lt.to_device(s), event_id=i).host() for s, i in zip(w.events, w.event_ids)]
    srv = lt.Server(ctx, n_lanes=2, max_batch_events=8, mem_budget_bytes=2 << 20)        # 1 MiB per lane
    try:
        tickets = [srv.submit(s, i) for s, i in zip(w.events, w.event_ids)]
        for t in tickets:
            with pytest.raises(lt.LtsimError) as ei:
                srv.wait(t, 60.0)
            assert ei.value.status == 3
            srv.release(t)
    finally:
        srv.stop()
    # one event's footprint: table (~0.7 MB), scratch and outputs of a 70x70-pixel, 2000-tick event (a few MB)
    srv = lt.Server(ctx, n_lanes=1, max_batch_events=8, mem_budget_bytes=40 << 20, return_currents=True)
    try:
        tickets = [srv.submit(s, i) for s, i in zip(w.events, w.event_ids)]
        got = [srv.wait(t, 60.0) for t in tickets]
        for t in tickets:
            srv.release(t)
    finally:
        srv.stop()
    sizes = [g["batch_events"] for g in got]
    print(f"admission under a 40 MiB budget: batch sizes {sizes}")
    assert max(sizes) < 8
    for a, g in zip(alone, got):
        assert g["status"] == 0
        for k in ("pixel_id", "current", "pkt_tick", "pkt_adc", "counts"):
            assert np.array_equal(a[k], g[k]), k


def test_server_lanes_share_the_response_table(lt, torch):
    """Eight lanes take less device memory than one copy of the table's columns (45 x 45 x 1950: 28.6 MB of FP32 with their
    padding, 31.6 MB of prefix sums); they keep the table they were made with when the context takes another, or goes."""
    w = W.make_workload(3, n_events=1)
    w.events = [w.events[0].subset(np.arange(300))]
    table = W.response_table(w.table, w.readout, w.physics.v_drift)
    ctx = lt.Context.from_workload(w, table=table)
    d = lt.to_device(w.events[0])
    alone = ctx.simulate(d, event_id=3).host()
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    srv = lt.Server(ctx, n_lanes=8, max_batch_events=1, return_currents=True)
    try:
        used = before - torch.cuda.mem_get_info()[0]
        print(f"eight lanes: {used / 1e6:.1f} MB")
        assert used < 28e6
        import ctypes as C
        other = np.ascontiguousarray(2 * table)
        ctx._check(lt.lib().lts_set_response(ctx._h, other.ctypes.data_as(C.c_void_p), *table.shape))
        twice = ctx.simulate(d, event_id=3).host()
        assert not np.array_equal(twice["current"], alone["current"])
        for _ in range(8):
            g = srv.wait(srv.submit(w.events[0], 3), 60.0)
            for k in ("pixel_id", "current", "pkt_tick", "pkt_adc"):
                assert np.array_equal(alone[k], g[k]), k
    finally:
        srv.stop()


# ----------------------------------------------------------------------------------------------- autotuner

def test_autotune_table_is_accurate_and_applied(lt, torch, tmp_path):
    """The autotuner times its candidates per event-size class, keeps only those within 1e-5 of the sorted
    reference, caches the table, and the library applies the table's entry per call: a batch under the table gives
    the results of a context set to that entry's knobs directly."""
    from paper_2212_09807_amd import autotune as AT
    w = W.make_workload(1)
    cands = [AT.Choice(0, 1, 0), AT.Choice(1, 1, 0), AT.Choice(2, 1, 0), AT.Choice(0, 1, 4)]
    res = AT.autotune(w, sizes=(200,), candidates=cands, events_per_class=4, cache=str(tmp_path / "tune.json"))
    (cls,) = res["classes"]
    assert len(cls["all"]) == 4 and all(r["ms"] > 0 for r in cls["all"])
    assert cls["best"]["max_rel_l2_vs_sorted"] <= 1e-5
    again = AT.autotune(w, sizes=(200,), candidates=cands, events_per_class=4, cache=str(tmp_path / "tune.json"))
    assert again["table"] == res["table"]
    (entry,) = res["table"]
    evs = AT.class_events(w, 200, 3, seed=5)
    offs = np.r_[0, np.cumsum([e.n for e in evs])]
    ids = [11, 12, 13]
    tuned = lt.Context.from_workload(w)
    tuned.set_tuning([entry])
    direct = lt.Context.from_workload(w)
    AT.Choice(*entry[1:]).apply(direct)
    a = tuned.simulate_batch(lt.to_device(W.Segments.concat(evs)), offs, ids).host()
    b = direct.simulate_batch(lt.to_device(W.Segments.concat(evs)), offs, ids).host()
    assert np.array_equal(a["pixel_id"], b["pixel_id"])
    if entry[1] == 1:                       # FP32 atomics: the summation order differs from run to run
        assert per_pixel_errors(a["current"].astype(np.float64), b["current"].astype(np.float64)).max() < 1e-6
    else:
        assert np.array_equal(a["current"], b["current"])
    # a two-entry table: small calls take the first entry, large ones the second
    tuned.set_tuning([[0, 2, 1, 0, 0], [100000, 1, 1, 0, 0]])
    c = tuned.simulate_batch(lt.to_device(W.Segments.concat(evs)), offs, ids).host()
    summed = lt.Context.from_workload(w, reduce_mode=2).simulate_batch(lt.to_device(W.Segments.concat(evs)), offs,
                                                                      ids).host()
    assert np.array_equal(c["current"], summed["current"])
    with pytest.raises(lt.LtsimError):
        tuned.set_tuning([[10, 0, 1, 0, 0], [5, 0, 1, 0, 0]])             # not ascending


def test_disabled_channels_produce_no_packets(lt, torch):
    w = W.make_workload(1)
    ctx = lt.Context.from_workload(w)
    segs = lt.to_device(w.events[0])
    full = ctx.simulate(segs, event_id=w.event_ids[0]).host()
    rng = np.random.default_rng(8)
    mask = rng.random(w.readout.n_x * w.readout.n_y) < 0.078           # Module-0 disabled fraction (Sec. 6)
    ctx.set_channel_mask(mask)
    part = ctx.simulate(segs, event_id=w.event_ids[0]).host()
    assert np.array_equal(full["current"], part["current"])           # currents are still computed
    keep = ~mask[full["pkt_pixel"]]
    assert not mask[part["pkt_pixel"]].any()
    assert np.array_equal(full["pkt_pixel"][keep], part["pkt_pixel"])
    assert np.array_equal(full["pkt_tick"][keep], part["pkt_tick"])
    assert np.array_equal(full["pkt_adc"][keep], part["pkt_adc"])
    ctx.set_channel_mask(None)
    again = ctx.simulate(segs, event_id=w.event_ids[0]).host()
    assert np.array_equal(again["pkt_tick"], full["pkt_tick"])


def test_lane_exchange_is_bit_identical(lt, torch):
    """Sharing table windows across lanes only changes where the values come from: same products, same order."""
    w = W.make_workload(3, n_events=1)
    ctx = lt.Context.from_workload(w)
    d = lt.to_device(w.events[0])
    ctx.set_lane_exchange(True)
    a = ctx.simulate(d, event_id=w.event_ids[0]).host()
    ctx.set_lane_exchange(False)
    b = ctx.simulate(d, event_id=w.event_ids[0]).host()
    assert np.array_equal(a["pixel_id"], b["pixel_id"])
    assert np.array_equal(a["current"], b["current"])
    assert np.array_equal(a["pkt_tick"], b["pkt_tick"]) and np.array_equal(a["pkt_adc"], b["pkt_adc"])


# ----------------------------------------------------------------------------------------------- per-point drift

@pytest.mark.parametrize("mode", [0, 2])
def test_per_point_drift_parity(lt, orc, torch, mode):
    """Lifetime and diffusion at every sample point (with a short lifetime, so the gradient along a segment is
    visible), per-pair and summed induction."""
    w = W.make_workload(1)
    w.physics = dataclasses.replace(w.physics, per_point=1, lifetime=500.0)
    h, r, e, (cmp_, flg) = check_event(lt, orc, w, mode=mode)
    print(f"per-point mode={mode}: pixels {len(r['pixels'])}, max e_p {e.max():.2e}, packets compared {cmp_}")


# ----------------------------------------------------------------------------------------------- Monte Carlo diffusion

@pytest.mark.parametrize("cfg,M,mode", [(1, 1, 0), (1, 16, 0), (1, 16, 2), (1, 64, 1)])
def test_mc_diffusion_parity(lt, orc, torch, cfg, M, mode):
    """The paper's estimator (M Philox-keyed perturbations per point): the device draws the same normals as the
    oracle, so currents meet the same bar; packets are exact except on pixels in reach of a draw that landed within
    FP32 reach of a bin edge (recorded by the oracle)."""
    w = W.make_workload(cfg)
    w.physics = dataclasses.replace(w.physics, mc_draws=M)
    h, r, e, (cmp_, flg) = check_event(lt, orc, w, 0, mode)
    print(f"[mc] cfg{cfg} M={M} mode={mode}: pixels {len(r['pixels'])}, max e_p {e.max():.2e}, packets compared "
          f"{cmp_}, flagged {flg}, near-edge draws {len(r['mc_near_edges'])}")
    # the expectation differs from one Monte Carlo realisation by far more than the bar
    w0 = dataclasses.replace(w.physics, mc_draws=0)
    w.physics = w0
    r0 = orc.simulate(w, 0, pixels=r["pixels"], with_packets=False)
    assert per_pixel_errors(h["current"][np.searchsorted(h["pixel_id"], r["pixels"])].astype(np.float64),
                            r0["wave"]).max() > 10 * TOL_WAVE


def test_mc_diffusion_batch_invariant(lt, torch):
    """Draws are keyed by (event id, segment index in the event): a batch gives each event's single-call result."""
    w = W.make_workload(3, n_events=3)
    w.events = [e.subset(np.arange(0, min(e.n, 3000))) for e in w.events]
    w.physics = dataclasses.replace(w.physics, mc_draws=8)
    ctx = lt.Context.from_workload(w)
    singles = [ctx.simulate(lt.to_device(e), event_id=i).host() for e, i in zip(w.events, w.event_ids)]
    offs = np.r_[0, np.cumsum([e.n for e in w.events])]
    b = ctx.simulate_batch(lt.to_device(W.Segments.concat(w.events)), offs, w.event_ids).host()
    po = b["event_pixel_offsets"]
    for e, s in enumerate(singles):
        assert np.array_equal(b["pixel_id"][po[e]:po[e + 1]], s["pixel_id"])
        assert np.array_equal(b["current"][po[e]:po[e + 1]], s["current"])


# ----------------------------------------------------------------------------------------------- stage hooks

def _stage_workloads():
    w2 = W.make_workload(2)
    w2.events[0] = w2.events[0].subset(np.arange(0, 20000, 97))
    return {"cfg1": W.make_workload(1), "ragged": _ragged_workload(), "cfg2-sub": w2}


@pytest.mark.parametrize("name", ["cfg1", "ragged", "cfg2-sub"])
def test_rasterized_pairs_equal_the_oracle_reach(lt, orc, torch, name):
    """Pair set (exact): for every segment, the pixels paired with it are the pixels whose table reach meets its
    truncated charge box in the oracle; pixel-major, ascending segment within a pixel."""
    w = _stage_workloads()[name]
    segs = w.events[0]
    ctx = lt.Context.from_workload(w)
    sg, px = ctx.stage_rasterize(lt.to_device(segs))
    sg, px = sg.cpu().numpy(), px.cpu().numpy()
    key = px.astype(np.int64) * (segs.n + 1) + sg
    assert np.all(np.diff(key) > 0)
    for s in range(segs.n):
        want = orc.active_pixels(w.physics, w.readout, w.table, segs.subset([s]))
        got = px[sg == s]
        assert np.array_equal(np.sort(got), want), (name, s)
    print(f"{name}: {len(sg)} pairs over {segs.n} segments")


@pytest.mark.parametrize("name", ["cfg1", "ragged", "cfg2-sub"])
def test_materialised_pair_currents_vs_oracle(lt, orc, torch, name):
    """Per-pair currents I_sp (the paper's (segment, pixel, tick) tensor) against the oracle's single-segment
    waveforms, on a sample of segments; e_p <= 1e-4 per pair."""
    w = _stage_workloads()[name]
    segs = w.events[0]
    table = W.response_table(w.table, w.readout, w.physics.v_drift)
    ctx = lt.Context.from_workload(w)
    sg, px, cur = ctx.stage_induce(lt.to_device(segs), event_id=w.event_ids[0])
    sg, px, cur = sg.cpu().numpy(), px.cpu().numpy(), cur.cpu().numpy().astype(np.float64)
    worst = 0.0
    for s in range(0, segs.n, max(1, segs.n // 12)):
        sel = np.flatnonzero(sg == s)
        if len(sel) == 0:
            continue
        o, _ = orc.waveforms(w.physics, w.readout, table, segs.subset([s]), px[sel])
        e = per_pixel_errors(cur[sel], o)
        worst = max(worst, float(e.max()))
        assert e.max() <= TOL_WAVE, (name, s, e.max())
    print(f"{name}: {len(sg)} pairs, worst sampled e_p {worst:.2e}")


@pytest.mark.parametrize("name", ["cfg1", "ragged", "cfg2-sub"])
def test_reduce_of_materialised_pairs_equals_fused_path(lt, torch, name):
    """Materialise-then-sum (the paper's data flow) gives the pixels and currents of the fused sorted path to FP32
    rounding (both Kahan-sum the same per-pair values in the same order)."""
    w = _stage_workloads()[name]
    segs = w.events[0]
    ctx = lt.Context.from_workload(w)
    d = lt.to_device(segs)
    sg, px, cur = ctx.stage_induce(d, event_id=w.event_ids[0])
    pid, red = ctx.stage_reduce(px, cur)
    h = ctx.simulate(d, event_id=w.event_ids[0]).host()
    pid = pid.cpu().numpy()
    assert np.array_equal(pid, h["pixel_id"])
    e = per_pixel_errors(red.cpu().numpy().astype(np.float64), h["current"].astype(np.float64))
    assert e.max() <= 2e-6, (name, e.max())


def test_stage_hooks_capacity_and_order_errors(lt, torch):
    import ctypes as C
    w = W.make_workload(1)
    ctx = lt.Context.from_workload(w)
    d = lt.to_device(w.events[0])
    s = d.struct()
    seg = torch.empty(4, dtype=torch.int32, device="cuda")
    n = C.c_int64(0)
    st = lt.lib().lts_stage_rasterize(ctx._h, C.byref(s), lt._ptr(seg), lt._ptr(seg), 4, C.byref(n),
                                      lt._stream(None))
    assert st == 2 and n.value > 4                                             # LTS_ERR_CAPACITY, need reported
    pix = torch.tensor([3, 5, 4], dtype=torch.int32, device="cuda")            # not grouped in ascending order
    cur = torch.zeros((3, w.readout.n_ticks), dtype=torch.float32, device="cuda")
    with pytest.raises(lt.LtsimError):
        ctx.stage_reduce(pix, cur)
    pid, red = ctx.stage_reduce(pix[:0], cur[:0])
    assert pid.numel() == 0 and red.shape[0] == 0


# ----------------------------------------------------------------------------------------------- matrix cores

@pytest.mark.parametrize("name", ["cfg1", "ragged", "max-window"])
def test_matrix_core_induction_parity(lt, orc, torch, name):
    """The Toeplitz form of the per-pair induction on the FP32 matrix cores meets the same bar against the oracle
    (cfg1 in full, the ragged multi-tile event, the longest window with ~200-tick charge boxes)."""
    w = {"cfg1": W.make_workload, "ragged": _ragged_workload, "max-window": _max_window_workload}[name]
    w = w(1) if name == "cfg1" else w()
    h, r, e, (cmp_, flg) = check_event(lt, orc, w, matrix=True)
    print(f"matrix cores {name}: pixels {len(r['pixels'])} max e_p {e.max():.2e} packets compared {cmp_} flagged {flg}")


def test_matrix_core_module_event_agrees_with_vector_path(lt, torch):
    """Full module-scale event: matrix-core and vector-ALU per-pair paths give the same pixels, and currents within
    the parity bar of each other (the two sum the products in different orders; bipolar currents on non-collecting
    pixels make the relative difference of FP32 sums reach ~1e-5)."""
    w = W.make_workload(2)
    _, a = run_gpu(lt, w)
    _, b = run_gpu(lt, w, matrix=True)
    assert np.array_equal(a["pixel_id"], b["pixel_id"])
    e = per_pixel_errors(b["current"].astype(np.float64), a["current"].astype(np.float64))
    print(f"module event: matrix vs vector max e_p {e.max():.2e}, p99 {np.percentile(e, 99):.2e}")
    assert e.max() <= TOL_WAVE


# ----------------------------------------------------------------------------------------------- tile edges

def _edge_workload(n_ticks, t_r, b_x, b_y, n_sub):
    """Charge at every residue of the start tick mod 8, single-tick to ~250-tick intervals (a drift-parallel track whose
    columns hold several pieces and parts), charge values over four decades, and windows cut at both ends."""
    w = W.config(1)
    w.readout = dataclasses.replace(w.readout, n_x=6, n_y=5, n_ticks=n_ticks, n_sub=n_sub)
    w.table = W.TableShape(t_r, b_x, b_y)
    parts = []
    n = 250
    z = np.linspace(0.4, 4.4, n + 1)
    r = np.stack([np.full(n + 1, 1.31), np.full(n + 1, 1.12), z], 1)
    parts.append(W.make_segments(r[:-1], r[1:], np.full(n, 2.1 * 0.016)))
    for k in range(9):
        p = np.array([0.3 + 0.27 * k, 0.4 + 0.19 * k, 0.02 + 0.3 * k])
        parts.append(W.make_segments(p, p + [0.01, 0.004, 0.002], 10.0 ** (-3 + 0.5 * k), t0=0.1 * k, t1=0.1 * k))
    w.events, w.event_ids = [W.Segments.concat(parts)], [77]
    return w


# A tenth of the parity bar: half-pair products are within 3 x 2^-22 (7e-7) of their values, the cells within ~2e-6.
TOL_EDGE = 1e-5


@pytest.mark.parametrize("n_ticks,t_r,b_x,b_y,n_sub", [(1, 1, 1, 1, 2), (255, 37, 5, 3, 10), (256, 256, 9, 8, 4),
                                                       (769, 200, 17, 10, 10), (1537, 1001, 20, 31, 10)])
def test_summed_matrix_tile_edges(lt, orc, torch, n_ticks, t_r, b_x, b_y, n_sub):
    """Summed induction on the matrix cores where its tiles, units, steps and parts end (ticks and table lengths around
    256 and 768, intervals around 32, 72 and 248, reaches that are no multiple of anything)."""
    h, r, e, _ = check_event(lt, orc, _edge_workload(n_ticks, t_r, b_x, b_y, n_sub), mode=2)
    print(f"summed edges {n_ticks}/{t_r}/{b_x}x{b_y}/{n_sub}: pixels {len(r['pixels'])} max e_p {e.max():.2e}")
    assert e.max() <= TOL_EDGE


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("n_ticks,t_r,b_x,b_y,n_sub", [(1, 1, 1, 1, 2), (130, 17, 2, 9, 4), (255, 37, 5, 3, 10),
                                                       (256, 256, 9, 8, 4), (1537, 1001, 20, 31, 10)])
def test_group_product_edges(lt, orc, torch, mode, n_ticks, t_r, b_x, b_y, n_sub):
    """Per-pair induction as group products where groups, octets, stages and tiles end (more than 16 segments of a pixel,
    groups cut by their span, reaches of 1 to 4 octets, tables and windows around 16 and 32 ticks); pair by pair, the
    materialised form adds up to the same."""
    w = _edge_workload(n_ticks, t_r, b_x, b_y, n_sub)
    h, r, e, _ = check_event(lt, orc, w, mode=mode)
    assert e.max() <= TOL_EDGE
    if mode == 0:
        segs = lt.to_device(w.events[0])
        c = lt.Context.from_workload(w)
        _, pix, cur = c.stage_induce(segs, w.event_ids[0])
        ids, red = c.stage_reduce(pix, cur)
        red, ids = red.cpu().numpy().astype(np.float64), ids.cpu().numpy()
        row = {int(p): k for k, p in enumerate(h["pixel_id"])}
        full = np.asarray(h["current"], np.float64)
        diff = max(np.abs(red[k] - full[row[int(p)]]).max() for k, p in enumerate(ids))
        assert diff <= 2 * TOL_EDGE * np.abs(full).max()
        c.close()


def _bright_and_faint():
    """Two deposits a hundred thousand times weaker than their neighbours in the same pixels, 60 and 90 ticks behind them,
    and a track; charge that only diffusion's tails bring to the outer pixels."""
    w = W.make_workload(1)
    p = np.array([[12.0, 13.0, 3.0], [12.0, 13.0, 3.0], [14.1, 13.4, 6.0], [14.1, 13.4, 6.0]])
    t = [0.0, 6.0, 0.0, 9.0]
    w.events = [W.Segments.concat([W.make_segments(p, p + [0.02, 0.01, 0.005], [2.0, 2e-5, 1.0, 1e-5], t0=t, t1=t),
                                   w.events[0].subset(np.arange(0, 200, 9))])]
    return w


def _hard_table(w, kind):
    """corner: a round reach (zeros in the table's corner); padded: zeros past the pad's third of the reach; units: the
    corner table in other units; wide: columns whose peaks span twelve decades."""
    t = W.response_table(w.table, w.readout, w.physics.v_drift).copy()
    i, j = np.meshgrid(np.arange(w.table.b_x), np.arange(w.table.b_y), indexing="ij")
    if kind in ("corner", "units"):
        t[:, np.hypot(i, j) > 9.5] = 0.0
    if kind == "padded":
        t[:, j >= 6] = 0.0
    if kind == "wide":
        t *= np.float32(10.0) ** -((i + j) * 2 // 3)
    return np.ascontiguousarray(t * np.float32(1e-6) if kind == "units" else t, dtype=np.float32)


def check_faint(lt, orc, mode, rt, kind):
    """The matrix-core currents of every pixel are as near to the oracle as the FP32 vector kernels' of the same mode, each
    relative to its own norm (down to 1e-7 of the brightest pixel's, FP32's resolution of it), and so are the ticks that
    only a weak deposit reaches behind a strong one in its pixel.  The cells' own error is in both; the products may add
    TOL_EDGE, ten times what half pairs and an FP32 sum of some thousand products come to."""
    w = _bright_and_faint()
    table = _hard_table(w, kind)
    (_, a), (_, b) = run_gpu(lt, w, mode=mode, table=table), run_gpu(lt, w, mode=mode, table=table, rt=rt)
    assert np.array_equal(a["pixel_id"], b["pixel_id"])
    o = orc.simulate(w, 0, table=table, with_packets=False)
    row = np.searchsorted(a["pixel_id"], o["pixels"])
    ref, ga, gb = o["wave"], a["current"][row].astype(np.float64), b["current"][row].astype(np.float64)
    norm = np.linalg.norm(ref, axis=1)
    k = norm > 1e-7 * norm.max()
    ea, eb = (np.linalg.norm(g - ref, axis=1)[k] / norm[k] for g in (ga, gb))
    late = 0.0
    for s in (0, 2):                                     # the strong one alone: the ticks behind its last
        alone, _ = orc.waveforms(w.physics, w.readout, table, w.events[0].subset([s]), o["pixels"])
        both, _ = orc.waveforms(w.physics, w.readout, table, w.events[0].subset([s, s + 1]), o["pixels"])
        if kind == "wide":                               # (some of its columns' currents are below any resolution)
            continue
        for q in np.flatnonzero(np.abs(both[:, :]).max(1) > 0.1 * np.abs(both).max()):
            n = np.flatnonzero(alone[q])[-1] + 1
            sl = np.arange(n, np.flatnonzero(both[q])[-1] + 1)
            sl = sl[ref[q, sl] == both[q, sl]]           # (no other segment there)
            if len(sl) >= 20:
                m = np.linalg.norm(ref[q, sl])
                d, dv = (np.linalg.norm(g[q, sl] - ref[q, sl]) / m for g in (ga, gb))
                assert d <= dv + TOL_EDGE, (q, d, dv)
                late = max(late, d)
    print(f"faint mode={mode} {kind}: {k.sum()} pixels, max own error {ea.max():.2e} (vector {eb.max():.2e}), behind {late:.2e}")
    assert np.all(ea <= eb + TOL_EDGE)
    assert late > 0.0 or kind == "wide"


@pytest.mark.parametrize("mode,rt", [(0, 4), (1, 4), (2, 8)])
def test_infinite_charge_stays_in_its_window(lt, torch, mode, rt):
    """A deposit whose charge overflows FP32 leaves no finite current in its own window and changes none outside it: the
    matrix-core currents are finite wherever the vector kernels' are, and the same to rounding there.  (A table of 200
    ticks: its last tile of 16 has padding.)"""
    w = W.make_workload(1)
    p = np.array([[12.0, 13.0, 6.0]])
    segs = w.events[0].subset(np.arange(0, 200, 3))
    w.events = [W.Segments.concat([segs, W.make_segments(p, p + 0.01, 1e36), W.make_segments(p + 0.05, p + 0.06, 0.02)])]
    w.electronics = dataclasses.replace(w.electronics, q_lsb=1e9)
    (_, a), (_, b) = run_gpu(lt, w, mode=mode), run_gpu(lt, w, mode=mode, rt=rt)
    assert np.array_equal(a["pixel_id"], b["pixel_id"])
    fa, fb = np.isfinite(a["current"]), np.isfinite(b["current"])
    print(f"mode {mode}: {(~fa).sum()} values not finite (vector {(~fb).sum()})")
    assert 0 < (~fa).sum() and np.all(fa[fb])
    x, y = np.where(fb, a["current"], 0.0).astype(np.float64), np.where(fb, b["current"], 0.0).astype(np.float64)
    assert per_pixel_errors(x, y).max() <= TOL_EDGE


@pytest.mark.parametrize("mode", [0, 1, 2])
def test_report_adds_up_the_currents_returned(lt, torch, mode):
    """The report's induced charge is the FP64 sum of the currents that the call returns, also where pixels were settled
    (codes one electron wide: many a charge lies near an edge)."""
    w = W.make_workload(1)
    w.electronics = dataclasses.replace(w.electronics, q_lsb=1.0, adc_bits=16)
    _, h = run_gpu(lt, w, mode=mode)
    assert np.count_nonzero(h["pkt_flags"]) > 5
    cur = h["current"].astype(np.float64)
    assert abs(h["report"][0][2] - cur.sum()) <= 1e-13 * np.abs(cur).sum()      # (a quarter million FP64 additions)


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("kind", ["whole", "corner", "padded", "units", "wide"])
def test_faint_currents_of_group_products(lt, orc, torch, mode, kind):
    check_faint(lt, orc, mode, 4, kind)


@pytest.mark.parametrize("kind", ["whole", "corner", "padded", "units", "wide"])
def test_faint_currents_of_summed_records(lt, orc, torch, kind):
    check_faint(lt, orc, 2, 8, kind)


@pytest.mark.parametrize("cfg,ev", [(1, 0), (1, 1), (3, 0)])
def test_packets_do_not_depend_on_the_summing_units(lt, torch, cfg, ev):
    """Decisions that rounding could turn are settled in the vector kernels' summation order: the matrix-core forms give
    the same packets and flags, and a pixel with a flagged packet has the vector kernels' current bit for bit."""
    w = W.make_workload(cfg, n_events=2)
    _, a = run_gpu(lt, w, ev, 0, rt=0)
    _, b = run_gpu(lt, w, ev, 0, rt=4)
    for k in ("pixel_id", "pkt_pixel", "pkt_tick", "pkt_adc", "pkt_flags"):
        assert np.array_equal(a[k], b[k])
    flagged = np.unique(a["pkt_pixel"][(a["pkt_flags"] & 3) != 0])
    rows = np.searchsorted(a["pixel_id"], flagged)
    assert np.array_equal(a["current"][rows], b["current"][rows])
    _, c = run_gpu(lt, w, ev, 1, rt=0)
    assert len(c["pkt_adc"]) == len(a["pkt_adc"])
    print(f"config {cfg} event {ev}: {len(a['pkt_adc'])} packets, {len(flagged)} flagged pixels")


@pytest.mark.parametrize("mode", [0, 1, 2])
def test_settled_pixels_are_the_same_first_and_late_in_the_list(lt, torch, mode):
    """Settled currents are the same bits whether a pixel's rounds are spread over the chip and handed on from workgroup to
    workgroup (the first 64 of a call) or taken one after the other (those beyond): an event alone against six copies of it
    in one call, with codes one electron wide, so that many pixels are settled."""
    w = W.make_workload(1)
    wide = dataclasses.replace(w.electronics, q_lsb=1e9)            # (no code's edge is near)
    w.electronics = dataclasses.replace(w.electronics, q_lsb=1.0, adc_bits=16)
    n = 6
    d, many = lt.to_device(w.events[0]), lt.to_device(W.Segments.concat([w.events[0]] * n))
    ctx = lt.Context.from_workload(w, reduce_mode=mode)
    ctx.set_ticks_per_thread(0)
    one = ctx.simulate(d, event_id=5).host()
    off = np.arange(n + 1) * w.events[0].n
    b = ctx.simulate_batch(many, off, [5] * n).host()
    w.electronics = wide
    rough = lt.Context.from_workload(w, reduce_mode=mode).simulate(d, event_id=5).host()
    settled = np.flatnonzero(np.any(one["current"] != rough["current"], axis=1))
    po, ko = b["event_pixel_offsets"], b["event_packet_offsets"]
    for e in range(n):
        rows = b["current"][po[e]:po[e + 1]]
        if mode != 1:
            assert np.array_equal(rows, one["current"])
        for k in ("pkt_pixel", "pkt_tick", "pkt_adc", "pkt_flags"):
            assert np.array_equal(b[k][ko[e]:ko[e + 1]], one[k])
    if mode != 1:                                                   # (atomic sums differ from call to call)
        print(f"mode {mode}: {len(settled)} settled rows of {len(one['current'])}")
        assert 12 <= len(settled) and n * len(settled) > 64


@pytest.mark.parametrize("cfg,ev", [(1, 0), (1, 1), (3, 0)])
def test_atomic_packets_are_the_sorted_modes(lt, torch, cfg, ev):
    """Decisions near an edge are settled in the sorted order in the atomic mode, too: its packets are the sorted mode's,
    codes and ticks, whatever order the atomics took."""
    w = W.make_workload(cfg, n_events=2)
    _, a = run_gpu(lt, w, ev, 0)
    _, b = run_gpu(lt, w, ev, 1)
    for k in ("pkt_pixel", "pkt_tick", "pkt_adc", "pkt_flags"):
        assert np.array_equal(a[k], b[k]), k
