#!/usr/bin/env python3
"""Benchmark of the differentiable Gaussian-splatting rasterizer on one MI355X.

Headline: mapping iterations per second at 1200x680 with 300,000 Gaussians
(scales log-normal(-4.5, 0.7), 20% near-transparent), full resolution, no
pruning.  One step = render_fwd + L1 colour / 0.5 L1 depth loss + render_bwd
to every Gaussian parameter + an Adam update of the map (applied inside the
backward's per-Gaussian pass, bitwise the update of a separate Adam kernel),
i.e. one mapping iteration of the SLAM back end; inputs are resident in HBM.

Also reported on the same line: the roofline of the dominant kernel (timed
with HIP events on its own stream inside the timed region), a per-stage
breakdown, the as-written variant (gradient pruning with ratio 0.5 after
iteration 30 and a 1-in-4 alpha-based pixel mask), and the CPU oracle timed
on a bounded pixel sample.

Usage: python bench.py [--gpus 1] [--steps K] [--warmup W]
"""
import argparse
import json
import math
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "fwd+bwd iters/s at 1200x680/300k Gaussians; served p50/p99 frame latency"

# Algorithmic FP32 operations per unit of work of the reverse compositing
# (raster_bwd): alpha re-evaluation of a list entry up to the pixel's last
# blended fragment, and the gradient of one blended fragment including the
# ten additions that merge it into its Gaussian.  Counted from the operations
# the method must perform (an FMA counts as two).
FLOP_BWD_PER_ENTRY = 18
FLOP_BWD_PER_BLEND = 65
FLOP_FWD_PER_ENTRY = 18
FLOP_FWD_PER_BLEND = 12
# MI355X vector FP32 peak as published: 256 CUs x 4 SIMDs x 16 lanes x 2 flop
# (FMA) x 2 (packed FP32) x 2.4 GHz.  The kernels are built without packed FP32
# instructions, so the rate they can reach is half of it (reported beside).
PEAK_FP32_PUBLISHED = 157.3
PEAK_FP32_NONPACKED = 256 * 4 * 16 * 2 * 2.4e9 / 1e12
PEAK_HBM_GBS = 8000.0
CLOCK_HZ = 2.4e9                 # peak shader clock (VALU-issue fractions)
SIMDS = 256 * 4
COUNTERS_FILE = os.path.join(ROOT, "profiles", "mapping_1200x680_300k_counters.md")
CSRC = os.path.join(ROOT, "paper_2510_06644_amd", "csrc")


def _code_only(src):
    """Source text without comments and with whitespace runs collapsed: two
    sources that differ only there compile to the same kernels."""
    import re
    src = re.sub(rb"/\*.*?\*/", b" ", src, flags=re.S)
    src = re.sub(rb"//[^\n]*", b" ", src)
    return b" ".join(src.split())


def kernel_hash():
    """Digest of the code (comments aside) of every source the library's
    kernels are compiled from."""
    import hashlib
    h = hashlib.sha256()
    for f in sorted(os.listdir(CSRC)):
        if f.endswith((".hip", ".h")):
            with open(os.path.join(CSRC, f), "rb") as fh:
                h.update(f.encode() + b"\0" + _code_only(fh.read()))
    return h.hexdigest()[:16]


def counter_record():
    """Per-kernel PMC figures (HBM bytes per launch, wave-level VALU
    instructions) from the committed counter summary, if it was taken on the
    current kernel sources (else None)."""
    try:
        text = open(COUNTERS_FILE).read()
    except OSError:
        return None
    start = text.find("```json")
    if start < 0:
        return None
    rec = json.loads(text[start + 7:text.index("```", start + 7)])
    if rec.get("kernel_hash") != kernel_hash():
        return None
    return rec


# Algorithmic HBM bytes per launch of the bandwidth-bound stages, from the
# per-unit figures of the method (n Gaussians, p pairs): projection 56 B of
# parameters in, the 64 B raster record, tile rectangle and count out (152 B);
# the per-chunk histogram reads rectangle and count (20 B); emit 12 B and sort
# 12 B per pair (key written and read, id written); merge 40 B per pair and 40 B
# per Gaussian written (the method's count: the kernel reads 40 B per quadrant of
# a pair that has sums, and a 4-byte flag word per pair); the preprocessing backward with the map's
# Adam update fused 392 B per Gaussian (rectangle 16 and merged 2D gradient 40
# read, 14 parameters read and written with both Adam moments, 24 B each);
# a separate Adam 28 B for each of 14 parameters per Gaussian.  Kernel names
# per stage as the profiler lists them.
HBM_STAGES = {
    "preprocess": (lambda n, p: 152 * n, ("k_preprocess<false, true>",)),
    "bin_count": (lambda n, p: 20 * n, ("k_chunk_hist<true>",)),
    "emit": (lambda n, p: 12 * p, ("k_emit<true>",)),
    "sort": (lambda n, p: 12 * p, ("k_sort_tiles<true>", "k_sort_big_tiles")),
    "merge": (lambda n, p: 40 * p + 40 * n, ("k_merge",)),
    "preprocess_bwd": (lambda n, p: 392 * n, ("k_gauss_bwd<10, true, true, false, false>",)),
    "adam": (lambda n, p: 392 * n, ("k_adam",)),
}
# the raster variants the headline step launches (the statistics forward of
# the work counts is another)
VALU_STAGES = {"raster_fwd": ("k_raster_fwd<false, false, false, true, false>",),
               "raster_bwd": ("k_raster_bwd<10, false, false, false, true, false, 6>",)}


def _kernel_sum(rec, prefixes, field):
    if rec is None:
        return None
    tot, hit = 0.0, False
    for name, k in rec["kernels"].items():
        if name.startswith(prefixes) and k.get(field) is not None:
            tot += k[field]
            hit = True
    return tot if hit else None


def per_kernel(stages_ms, cnt, n, rec):
    """Per stage: live time, algorithmic GB/s against 8 TB/s, PMC traffic
    (bytes per launch, when the counter record matches the kernel sources)
    and, for the raster kernels, the VALU-issue fraction."""
    p = cnt["pairs"]
    out = {}
    for st, (fn, names) in HBM_STAGES.items():
        ms = stages_ms.get(st)
        if not ms:
            continue
        alg = fn(n, p)
        d = {"avg_us": 1000 * ms, "bound": "hbm", "alg_bytes": alg,
             "alg_gbs": alg / (ms * 1e-3) / 1e9, "frac_of_8tbs": alg / (ms * 1e-3) / 8e12}
        t = _kernel_sum(rec, names, "bytes")
        if t is not None:
            d.update(traffic_bytes=t, traffic_gbs=t / (ms * 1e-3) / 1e9,
                     traffic_over_alg=t / alg)
        out[st] = d
    for st, names in VALU_STAGES.items():
        ms = stages_ms.get(st)
        if not ms:
            continue
        d = {"avg_us": 1000 * ms, "bound": "alu"}
        v = _kernel_sum(rec, names, "valu_insts")
        if v is not None:
            d.update(valu_insts=v, valu_issue_frac=v * 4 / (SIMDS * CLOCK_HZ * ms * 1e-3))
        t = _kernel_sum(rec, names, "bytes")
        if t is not None:
            d.update(traffic_bytes=t, traffic_gbs=t / (ms * 1e-3) / 1e9)
        out[st] = d
    return out


# Slot-count roofline of the whole iteration: per stage the larger of its
# algorithmic HBM bytes at 8 TB/s and its algorithmic VALU operations plus
# three extra slots per transcendental (exp, rcp at quarter rate) at
# 1024 SIMDs x 16 lanes x 2.4 GHz.  Per-unit counts: forward 12 VALU + 1 exp
# per list entry visited and 10 per blend; backward 12 + 1 exp per entry up to
# the last blend and 55 + 1 rcp per blended fragment; bytes 152 (projection)
# + 40 (merged 2D gradient written) + 392 (its backward with the fused Adam
# update) per Gaussian, 12 (emit) + 24 (sort) + 40 (merge) per pair, 48 (loss)
# per pixel.
SLOT_RATE = 1024 * 16 * 2.4e9
HBM_BYTES_PER_S = 8e12


def path_roofline(cnt, ms_per_step, bwd_ms, fwd_ms, spec):
    fwd_us = (12 * cnt["visited"] + 10 * cnt["blended"] + 3 * cnt["visited"]) / SLOT_RATE * 1e6
    bwd_us = (12 * cnt["visited_to_last"] + 55 * cnt["blended"]
              + 3 * (cnt["visited_to_last"] + cnt["blended"])) / SLOT_RATE * 1e6
    hbm_bytes = (584 * spec.n + 76 * cnt["pairs"] + 48 * spec.width * spec.height)
    hbm_us = hbm_bytes / HBM_BYTES_PER_S * 1e6
    t_roof = fwd_us + bwd_us + hbm_us
    return {"model": "sum over stages of max(bytes / 8 TB/s, (VALU ops + 3 per exp or rcp) "
                     "/ 39.3T lane-slots/s)",
            "t_roof_us": t_roof, "raster_fwd_us": fwd_us, "raster_bwd_us": bwd_us,
            "hbm_stages_us": hbm_us, "frac": t_roof / (1000.0 * ms_per_step),
            "raster_bwd_frac": bwd_us / (1000.0 * bwd_ms),
            "raster_fwd_frac": fwd_us / (1000.0 * fwd_ms)}


def log(*a):
    print(*a, file=sys.stderr, flush=True)


CALIB_COPY_BYTES = 128 << 22           # the --calib-copy copy: 128 Mi floats


def _short_kernel(name):
    import re
    name = name.replace("rtgs::(anonymous namespace)::", "").replace("void ", "")
    return re.sub(r"\(.*", "", name).strip()


def _pmc_per_kernel(db):
    """{short kernel name: {counter: median per dispatch}} from a rocprofv3
    results database (rows of one dispatch and counter are summed), plus the
    median dispatch duration in ns and the dispatch count."""
    import sqlite3
    import statistics
    from collections import defaultdict
    cur = sqlite3.connect(db).cursor()
    per = defaultdict(lambda: defaultdict(float))
    names, dur = {}, {}
    for disp, kname, cname, val, d in cur.execute(
            "select dispatch_id, kernel_name, counter_name, value, duration "
            "from counters_collection"):
        per[disp][cname] += val
        names[disp] = kname
        dur[disp] = d
    byk = defaultdict(lambda: defaultdict(list))
    for disp, cs in per.items():
        k = _short_kernel(names[disp])
        for c, v in cs.items():
            byk[k][c].append(v)
        byk[k]["duration_ns"].append(dur[disp])
    return {k: {**{c: statistics.median(v) for c, v in cs.items()},
                "dispatches": len(cs["duration_ns"])} for k, cs in byk.items()}


def _copy_counter(db, counter):
    """The counter of the largest copy dispatch of a run (the calibration
    copy of --calib-copy is the largest copy this bench makes)."""
    import sqlite3
    cur = sqlite3.connect(db).cursor()
    return max(v for (v,) in cur.execute(
        "select value from counters_collection where counter_name = ? and "
        "kernel_name like '%copyBuffer%'", (counter,)))


def counter_summary(root):
    """Markdown summary of four counter runs of this bench (FETCH_SIZE,
    WRITE_SIZE, two SQ sets) with the record `counter_record` reads: HBM
    bytes per launch (FETCH_SIZE and WRITE_SIZE in KiB, each scaled by what it
    reads for the --calib-copy copy of known size) and wave-level VALU
    instructions, keyed by the hash of the kernel sources."""
    db = lambda x: os.path.join(root, x, "run_results.db")
    fetch, write = _pmc_per_kernel(db("fetch")), _pmc_per_kernel(db("write"))
    sq, sqw = _pmc_per_kernel(db("sq")), _pmc_per_kernel(db("sqw"))
    cf = _copy_counter(db("fetch"), "FETCH_SIZE") * 1024
    cw = _copy_counter(db("write"), "WRITE_SIZE") * 1024
    sf, sw = CALIB_COPY_BYTES / cf, CALIB_COPY_BYTES / cw
    rec = {"kernel_hash": kernel_hash(),
           "calibration": {"copy_bytes": CALIB_COPY_BYTES, "fetch_counter_bytes": cf,
                           "write_counter_bytes": cw, "fetch_scale": sf, "write_scale": sw},
           "kernels": {}}
    rows = []
    for k in sorted(set(fetch) & set(write) & set(sq)):
        if not k.startswith("k_"):
            continue
        f = fetch[k]["FETCH_SIZE"] * 1024 * sf
        w = write[k]["WRITE_SIZE"] * 1024 * sw
        q = sq[k]
        e = {"fetch_bytes": f, "write_bytes": w, "bytes": f + w,
             "valu_insts": q.get("SQ_INSTS_VALU"), "salu_insts": q.get("SQ_INSTS_SALU"),
             "lds_insts": q.get("SQ_INSTS_LDS"), "trans_insts": q.get("SQ_INSTS_VALU_TRANS_F32"),
             "waves": q.get("SQ_WAVES"), "wave_cycles": q.get("SQ_WAVE_CYCLES"),
             "busy_cycles": q.get("SQ_BUSY_CYCLES"), "cycles": q.get("SQ_CYCLES"),
             "duration_us": fetch[k]["duration_ns"] / 1000.0}
        if k in sqw:
            e.update(wait_any=sqw[k].get("SQ_WAIT_ANY"),
                     wait_inst_lds=sqw[k].get("SQ_WAIT_INST_LDS"),
                     lds_bank_conflict=sqw[k].get("SQ_LDS_BANK_CONFLICT"))
        rec["kernels"][k] = e
        rows.append((k, e))
    rows.sort(key=lambda r: -r[1]["duration_us"])
    out = ["| kernel | us (counter run) | fetch MB | write MB | VALU insts | trans | LDS insts "
           "| waves | wait_any / wave_cycles |", "|---|---:|---:|---:|---:|---:|---:|---:|---:|"]
    for k, e in rows:
        wr = (e.get("wait_any") or 0) / e["wave_cycles"] if e.get("wave_cycles") else None
        out.append(f"| {k} | {e['duration_us']:.1f} | {e['fetch_bytes'] / 1e6:.1f} | "
                   f"{e['write_bytes'] / 1e6:.1f} | {e['valu_insts'] or 0:.0f} | "
                   f"{e['trans_insts'] or 0:.0f} | {e['lds_insts'] or 0:.0f} | "
                   f"{e['waves'] or 0:.0f} | {'' if wr is None else f'{wr:.2f}'} |")
    cal = (f"Calibration (the {CALIB_COPY_BYTES >> 20} MiB copy of --calib-copy): FETCH_SIZE "
           f"reads {cf / 2**20:.1f} MiB (scale {sf:.4f}), WRITE_SIZE {cw / 2**20:.1f} MiB "
           f"(scale {sw:.4f}).")
    return "\n".join(out + ["", cal, "", "```json", json.dumps(rec, indent=1), "```"])


def setup(spec_name="c2", seed_offset=0):
    import torch
    from paper_2510_06644_amd import rtgs, synth
    spec = synth.CONFIGS[spec_name]
    cam = synth.make_camera(spec.width, spec.height)
    sc = synth.make_scene(spec, cam)
    tgt = synth.perturb_scene(sc, spec.seed + 500)
    dev = torch.device("cuda", 0)
    params = [torch.from_numpy(a).to(dev).requires_grad_(True) for a in sc.arrays()]
    target_scene = tuple(torch.from_numpy(a).to(dev) for a in tgt.arrays())
    view = torch.from_numpy(synth.identity_viewmat()).to(dev)
    rc = rtgs.Cam(cam.width, cam.height, cam.fx, cam.fy, cam.cx, cam.cy)
    return spec, cam, sc, params, target_scene, view, rc


def render_target(R, target_scene, view, rc, seed):
    import torch
    st = R.forward(target_scene, view, rc)
    g = torch.Generator(device="cuda").manual_seed(seed)
    tc = st.color + 0.01 * torch.randn(st.color.shape, generator=g, device="cuda")
    td = st.depth + 0.01 * torch.randn(st.depth.shape, generator=g, device="cuda")
    return tc, td


def make_optimizer(params):
    from paper_2510_06644_amd import optim
    return optim.MapAdam(params, eps=1e-15)


def l1_grads(color, depth, tc, td, pixel_mask=None, n_active=None):
    """dL/dC, dL/dD of L = mean|C - C^| / 3 + 0.5 mean|D - D^| over the active
    pixels (Eq. 6 reading), by the library's loss kernel."""
    import torch
    from paper_2510_06644_amd import rtgs
    gc = torch.empty_like(color)
    gd = torch.empty_like(depth)
    rtgs.loss_l1_grad(color, depth, tc, td, gc, gd, pixel_mask=pixel_mask, n_active=n_active)
    return gc, gd


def mapping_step(R, params, view, rc, opt, tc, td, gauss_mask=None, pixel_mask=None,
                 cov3d=False, sample_log2=0, n_active=None, fused=True):
    """One mapping iteration.  Fused: the forward writes the loss gradients
    as it writes the image, and the Adam update runs inside the backward's
    per-Gaussian pass (both bitwise the results of the separate loss and
    adam_step passes); an iteration whose gradients are wanted (cov3d: the
    inputs of gradient pruning) takes the backward and the optimizer apart."""
    scene = tuple(p.detach() for p in params)
    if fused:
        st = R.forward(scene, view, rc, gauss_mask=gauss_mask, pixel_mask=pixel_mask,
                       sample_log2=sample_log2, l1=(tc, td, n_active))
        gc, gd = st.dL_dcolor, st.dL_ddepth
    else:
        st = R.forward(scene, view, rc, gauss_mask=gauss_mask, pixel_mask=pixel_mask,
                       sample_log2=sample_log2)
        gc, gd = l1_grads(st.color, st.depth, tc, td, pixel_mask, n_active)
    if fused and not cov3d:
        g = R.backward(scene, view, rc, st, gc, gd, pose=False, gauss_mask=gauss_mask,
                       pixel_mask=pixel_mask, adam=opt)
        return st, g
    g = R.backward(scene, view, rc, st, gc, gd, pose=False, map_grads=True, cov3d=cov3d,
                   gauss_mask=gauss_mask, pixel_mask=pixel_mask)
    opt.step(R.handle, [g[k] for k in ("means", "log_scales", "quats", "opacity_logits",
                                        "colors")])
    return st, g


def work_counts(R, params, view, rc):
    """Per-pixel work counts of one forward (fragments blended, list entries
    visited up to the stop, entries up to the last blended) and pair count."""
    import torch
    from paper_2510_06644_amd import rtgs
    n = params[0].shape[0]
    h, w = rc.height, rc.width
    cap = max(R.cap, 1 << 16)
    ws = torch.empty(rtgs.rtgs_workspace_size(n, w, h, cap), dtype=torch.uint8, device="cuda")
    out = dict(scene=tuple(p.detach() for p in params), viewmat=view, cam=rc,
               color=torch.empty(3, h, w, device="cuda"), depth=torch.empty(h, w, device="cuda"),
               alpha=torch.empty(h, w, device="cuda"),
               stats=torch.zeros(3, h, w, dtype=torch.int32, device="cuda"))
    rtgs.render_fwd_batched(R.handle, [out], ws, cap, flags=rtgs.RTGS_FWD_STATS)
    code, pairs, _ = rtgs.rtgs_query(R.handle, True)
    assert code == rtgs.RTGS_OK, "capacity"
    s = out["stats"].to(torch.int64).sum((1, 2)).cpu().numpy()
    return {"blended": int(s[0]), "visited": int(s[1]), "visited_to_last": int(s[2]),
            "pairs": int(pairs)}


def timed_loop(R, params, view, rc, opt, tc, td, steps, profile_stages=None, **kw):
    """steps mapping iterations between two synchronisations; an event is
    recorded on the stream between iterations, so per-iteration times come
    without extra syncs.  Returns (mean ms, host wall ms per step, stage
    profile, per-iteration ms list)."""
    import torch
    from paper_2510_06644_amd import rtgs
    if profile_stages:
        rtgs.rtgs_profile_enable(R.handle, profile_stages)
    torch.cuda.synchronize()
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(steps + 1)]
    t0 = time.perf_counter()
    ev[0].record()
    for i in range(steps):
        mapping_step(R, params, view, rc, opt, tc, td, **kw)
        ev[i + 1].record()
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    prof = {}
    if profile_stages:
        prof = rtgs.rtgs_profile_read(R.handle)
        rtgs.rtgs_profile_enable(R.handle, [])
    R.verify()
    per = [ev[i].elapsed_time(ev[i + 1]) for i in range(steps)]
    return ev[0].elapsed_time(ev[-1]) / steps, wall / steps, prof, per


def iter_stats(per):
    """Median and p90 of per-iteration times; the median over iterations 2
    onward (the first timed iteration follows the warm-up)."""
    a = np.asarray(per)
    tail = a[1:] if len(a) > 1 else a
    return {"median_ms": float(np.median(a)), "p90_ms": float(np.percentile(a, 90)),
            "min_ms": float(a.min()), "max_ms": float(a.max()),
            "median_ms_iters_2_on": float(np.median(tail)),
            "median_iters_per_s_iters_2_on": 1000.0 / float(np.median(tail))}


def as_written_variant(R, params, view, rc, opt, tc, td, iters=60):
    """60 iterations: full frame for iteration 1, then a 1-in-4 alpha-based
    pixel mask from iteration 1's final transmittance (rendered with one sample
    per 2x2 block); gradient pruning (ratio 0.5) after iteration 30, the mask
    kept for the remaining iterations."""
    import torch
    from paper_2510_06644_amd import rtgs
    n = params[0].shape[0]
    h, w = rc.height, rc.width
    pmask = torch.empty(h, w, dtype=torch.uint8, device="cuda")
    gmask = torch.zeros(n, dtype=torch.uint8, device="cuda")
    newmask = torch.empty_like(gmask)
    n_masked = torch.zeros(1, dtype=torch.int32, device="cuda")
    n_act = torch.zeros(1, dtype=torch.int32, device="cuda")
    # warm-up of the masked path (first use of its kernels)
    st, g = mapping_step(R, params, view, rc, opt, tc, td, cov3d=True)
    rtgs.downsample_mask(st.final_T, 2, pmask, n_act)
    mapping_step(R, params, view, rc, opt, tc, td, pixel_mask=pmask, sample_log2=2,
                 n_active=n_act)
    rtgs.prune_by_grad(R.handle, g["means"], g["cov3d"], st.visible, gmask, 0.8, 0.5, newmask,
                       n_masked)
    mapping_step(R, params, view, rc, opt, tc, td, gauss_mask=newmask, pixel_mask=pmask,
                 sample_log2=2, n_active=n_act)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    e0 = torch.cuda.Event(enable_timing=True)
    e1 = torch.cuda.Event(enable_timing=True)
    e0.record()
    st, _ = mapping_step(R, params, view, rc, opt, tc, td)
    rtgs.downsample_mask(st.final_T, 2, pmask, n_act)
    use_gmask = None
    for it in range(2, iters + 1):
        st, g = mapping_step(R, params, view, rc, opt, tc, td, gauss_mask=use_gmask,
                             pixel_mask=pmask, cov3d=(it == 30), sample_log2=2,
                             n_active=n_act)
        if it == 30:
            rtgs.prune_by_grad(R.handle, g["means"], g["cov3d"], st.visible, gmask, 0.8, 0.5,
                               newmask, n_masked)
            use_gmask = newmask
    e1.record()
    torch.cuda.synchronize()
    R.verify()
    return {"iters": iters, "ms_per_iter": e0.elapsed_time(e1) / iters,
            "iters_per_s": 1000.0 * iters / e0.elapsed_time(e1),
            "wall_ms_per_iter": 1000 * (time.perf_counter() - t0) / iters,
            "pruned": int(n_masked.item()), "active_pixels": int(n_act.item())}


def lane_efficiency(work, prev, w, h):
    """Mean over waves of (mean / max) of the entries each lane walked, for
    the quadrant assignment and for the assignment sorted by `prev` (the
    previous forward's per-pixel work); tiles of 16 x 16, waves of 64."""
    tw, th = (w + 15) // 16, (h + 15) // 16
    pad = lambda a: np.pad(a.astype(np.int64), ((0, th * 16 - h), (0, tw * 16 - w)))
    cur = pad(work).reshape(th, 16, tw, 16).transpose(0, 2, 1, 3).reshape(-1, 256)
    old = pad(prev).reshape(th, 16, tw, 16).transpose(0, 2, 1, 3).reshape(-1, 256)
    sy, sx = np.divmod(np.arange(256), 16)
    quad = (sy // 8) * 2 + sx // 8
    def eff(groups):
        out = []
        for q in range(4):
            vals = np.where(groups == q, cur, -1)
            mx = vals.max(1)
            cnt = (groups == q).sum(1)
            mean = np.where(groups == q, cur, 0).sum(1) / np.maximum(cnt, 1)
            ok = mx > 0
            out.append(mean[ok] / mx[ok])
        return float(np.concatenate(out).mean())
    key = old * 256 + np.arange(256)[None, :]
    rank = np.argsort(np.argsort(key, axis=1), axis=1)
    return {"quadrants": eff(np.broadcast_to(quad, cur.shape)), "by_previous_work": eff(rank // 64)}


def lane_balance_run(iters=20):
    """The mapping iteration (1200x680 / 300k) and the tracking iteration
    (640x480 / 100k, pose only) with lanes assigned by the previous
    iteration's work (RTGS_FWD_BALANCE_LANES) against the quadrant
    assignment: raster kernel times (HIP events) and lane efficiency."""
    import torch
    from paper_2510_06644_amd import rtgs, synth
    out = {}
    for name in ("c2", "c1"):
        spec = synth.CONFIGS[name]
        cam = synth.make_camera(spec.width, spec.height)
        sc = synth.make_scene(spec, cam)
        scene = tuple(torch.from_numpy(a).cuda() for a in sc.arrays())
        rc = rtgs.Cam(cam.width, cam.height, cam.fx, cam.fy, cam.cx, cam.cy)
        R = rtgs.Renderer(0, check="deferred")
        view = torch.eye(3, 4, dtype=torch.float32, device="cuda").contiguous()
        tc, td = render_target(R, scene, view, rc, spec.seed)
        h, w = cam.height, cam.width
        bufs = [torch.zeros(h, w, dtype=torch.uint16, device="cuda") for _ in range(2)]
        res = {}
        for mode in ("quadrants", "balanced", "quadrants", "balanced"):
            bal = mode == "balanced"
            rtgs.rtgs_profile_enable(R.handle, ["raster_fwd", "raster_bwd"])
            torch.cuda.synchronize()
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for it in range(iters):
                kw = dict(balance=True, lane_work=bufs[it % 2] if it else None,
                          lane_work_out=bufs[(it + 1) % 2]) if bal else {}
                st = R.forward(scene, view, rc, **kw)
                gc, gd = l1_grads(st.color, st.depth, tc, td)
                R.backward(scene, view, rc, st, gc, gd, pose=name == "c1",
                           map_grads=name == "c2")
            e1.record()
            torch.cuda.synchronize()
            prof = rtgs.rtgs_profile_read(R.handle)
            rtgs.rtgs_profile_enable(R.handle, [])
            R.verify()
            res[mode] = {"ms_per_iter": e0.elapsed_time(e1) / iters,
                         "raster_fwd_us": 1000 * prof["raster_fwd"][0] / prof["raster_fwd"][1],
                         "raster_bwd_us": 1000 * prof["raster_bwd"][0] / prof["raster_bwd"][1]}
        work = bufs[iters % 2].cpu().numpy()
        prev = bufs[(iters + 1) % 2].cpu().numpy()
        res["lane_efficiency"] = lane_efficiency(work, prev, w, h)
        out[f"{w}x{h}_{spec.n // 1000}k_{'mapping' if name == 'c2' else 'tracking'}"] = res
    return out


def state_policy_run(iters=10):
    """Forward + backward to the map at 1200x680 with 300k and 500k
    Gaussians under the three state policies of the backward: the saved
    per-pixel state (final T and last position), the state recomputed by a
    second forward pass, and the saved fragments (each blended fragment's
    alpha, the per-fragment state of the paper's R&B buffer): raster times
    (HIP events), iteration time and workspace bytes."""
    import torch
    from paper_2510_06644_amd import rtgs, synth
    out = {}
    for name in ("c2", "c3"):
        spec = synth.CONFIGS[name]
        cam = synth.make_camera(spec.width, spec.height)
        sc = synth.make_scene(spec, cam)
        scene = tuple(torch.from_numpy(a).cuda() for a in sc.arrays())
        rc = rtgs.Cam(cam.width, cam.height, cam.fx, cam.fy, cam.cx, cam.cy)
        R = rtgs.Renderer(0, check="deferred")
        view = torch.eye(3, 4, dtype=torch.float32, device="cuda").contiguous()
        tc, td = render_target(R, scene, view, rc, spec.seed)
        res = {}
        for pol in ("saved_state", "recompute", "saved_fragments", "saved_state"):
            kw = {"save_state": pol != "recompute", "save_fragments": pol == "saved_fragments"}
            st = R.forward(scene, view, rc, **kw)          # warm-up, sizes the workspace
            torch.cuda.synchronize()
            rtgs.rtgs_profile_enable(R.handle, ["raster_fwd", "raster_bwd"])
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(iters):
                st = R.forward(scene, view, rc, **kw)
                gc, gd = l1_grads(st.color, st.depth, tc, td)
                R.backward(scene, view, rc, st, gc, gd, pose=False, map_grads=True)
            e1.record()
            torch.cuda.synchronize()
            prof = rtgs.rtgs_profile_read(R.handle)
            rtgs.rtgs_profile_enable(R.handle, [])
            R.verify()
            fwd = prof["raster_fwd"]
            res[pol] = {"ms_per_iter": e0.elapsed_time(e1) / iters,
                        "raster_fwd_us_per_launch": 1000 * fwd[0] / fwd[1],
                        "raster_fwd_launches_per_iter": fwd[1] / iters,
                        "raster_bwd_us": 1000 * prof["raster_bwd"][0] / prof["raster_bwd"][1],
                        "workspace_bytes": st.ws.numel() * st.ws.element_size(),
                        "pair_capacity": st.cap}
            del st
            torch.cuda.empty_cache()
        out[f"{cam.width}x{cam.height}_{spec.n // 1000}k"] = res
    return out


def tracking_run(iters=40, lr_rho=1e-3, lr_phi=1e-3, reuse_lists=False, mask_prune=False):
    """Tracking at 640x480 with 100k Gaussians: the map frozen, the camera
    starting 2 cm / 1 degree off the pose its target frame was rendered
    from; each iteration is render_fwd (which also writes the loss gradient),
    render_bwd to the pose only and pose_update (Adam on xi, then
    T <- Exp(-step) T).
    reuse_lists: iterations after the first reuse its tile lists and depth
    order (projection only; Sec. 3, Observation 6).
    mask_prune: the mask-prune schedule of Sec. 4.1 (prune.MaskPruneTracker:
    windows of one full iteration and K masked iterations on its lists, the
    masked Gaussians removed at the next full iteration)."""
    import torch
    from paper_2510_06644_amd import pose, rtgs, synth
    spec = synth.CONFIGS["c1"]
    cam = synth.make_camera(spec.width, spec.height)
    sc = synth.make_scene(spec, cam)
    scene = tuple(torch.from_numpy(a).cuda() for a in sc.arrays())
    rc = rtgs.Cam(cam.width, cam.height, cam.fx, cam.fy, cam.cx, cam.cy)
    R = rtgs.Renderer(0, check="deferred")
    eye = torch.eye(3, 4, dtype=torch.float32, device="cuda").contiguous()
    tc, td = render_target(R, scene, eye, rc, spec.seed)
    xi0 = torch.tensor(synth.pose_offset(51, 0.02, 1.0), dtype=torch.float64, device="cuda")
    start = pose.apply_left(xi0, eye).contiguous()

    def err(vm):
        v = vm.double().cpu()
        t = float(v[:, 3].norm()) * 100.0
        c = float(((v[:, :3].trace() - 1.0) / 2.0).clamp(-1.0, 1.0))
        return {"t_cm": t, "r_deg": float(np.degrees(np.arccos(c)))}

    tracker = [None]

    def run(view, n):
        m = torch.zeros(6, device="cuda")
        v = torch.zeros(6, device="cuda")
        first = None
        if mask_prune:
            from paper_2510_06644_amd import prune
            tr = tracker[0] = prune.MaskPruneTracker(R, scene, rc)
            for it in range(1, n + 1):
                g = tr.iteration(view, lambda st: l1_grads(st.color, st.depth, tc, td))
                rtgs.pose_update([(view, g, m, v, lr_rho, lr_phi, it)])
            return
        for it in range(1, n + 1):
            # the forward also writes the loss gradient (as the mapping step's)
            st = R.forward(scene, view, rc, reuse_lists_of=first, l1=(tc, td, None))
            if reuse_lists and first is None:
                first = st
            g = R.backward(scene, view, rc, st, st.dL_dcolor, st.dL_ddepth, pose=True,
                           map_grads=False)
            rtgs.pose_update([(view, g["pose"], m, v, lr_rho, lr_phi, it)])

    run(start.clone(), 3)                      # warm-up (first launches)
    view = start.clone()
    torch.cuda.synchronize()
    e0 = torch.cuda.Event(enable_timing=True)
    e1 = torch.cuda.Event(enable_timing=True)
    e0.record()
    run(view, iters)
    e1.record()
    torch.cuda.synchronize()
    R.verify()
    ms = e0.elapsed_time(e1) / iters
    out = {"workload": "640x480_100k_tracking", "reuse_lists": reuse_lists, "iters": iters,
           "ms_per_iter": ms, "iters_per_s": 1000.0 / ms, "pose_err_start": err(start),
           "pose_err_end": err(view)}
    if mask_prune:
        tr = tracker[0]
        out.update(mask_prune=True, gaussians_end=tr.n, full_iters=tr.full_iters,
                   masked_iters=tr.masked_iters,
                   windows=[[k, r] for k, r in tr.sched.windows])
    return out


def _cpu_model():
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                return line.split(":", 1)[1].strip()
    except OSError:
        pass
    import platform
    return platform.processor() or "unknown"


def cpu_baseline(c2_sample=448, c1_sample=256, c0_reps=10, seed=5):
    """The float64 oracle timed on the host: c0 (128x128, 2,000 Gaussians)
    full frame fwd + bwd to every parameter and the pose, 10 times on all
    threads and once on one thread; c1 (640x480, 100k) and c2 (1200x680,
    300k, the benchmark's workload) on a random sample of pixels against all
    Gaussians, scaled by pixel count to a full frame.  The headline value is
    c2's."""
    import torch
    import oracle
    from paper_2510_06644_amd import synth

    def frame(name):
        spec = synth.CONFIGS[name]
        cam = synth.make_camera(spec.width, spec.height)
        ocam = (cam.width, cam.height) + tuple(float(np.float32(v))
                                               for v in (cam.fx, cam.fy, cam.cx, cam.cy))
        return spec, cam, synth.make_scene(spec, cam), ocam

    def sampled(name, sample):
        spec, cam, sc, ocam = frame(name)
        rng = np.random.default_rng(seed)
        pix = np.sort(rng.choice(cam.width * cam.height, sample, replace=False))
        gc, gd, _ = synth.upstream_grads(sample, 1, seed)
        t0 = time.perf_counter()
        oracle.render_with_grads(sc.arrays(), synth.identity_viewmat(), ocam, gc.reshape(3, -1),
                                 gd.reshape(-1), pixels=pix, chunk=16)
        dt = time.perf_counter() - t0
        full = dt * cam.width * cam.height / sample
        return {"iters_per_s": 1.0 / full, "seconds": dt,
                "sample": f"{sample} random pixels of {cam.width}x{cam.height} against all "
                          f"{spec.n} Gaussians, scaled by pixel count"}

    threads = torch.get_num_threads()
    spec, cam, sc, ocam = frame("c0")
    gc, gd, _ = synth.upstream_grads(cam.width, cam.height, seed)
    times = []
    for _ in range(c0_reps):
        t0 = time.perf_counter()
        oracle.render_with_grads(sc.arrays(), synth.identity_viewmat(), ocam, gc, gd)
        times.append(time.perf_counter() - t0)
    torch.set_num_threads(1)
    try:
        t0 = time.perf_counter()
        oracle.render_with_grads(sc.arrays(), synth.identity_viewmat(), ocam, gc, gd)
        single = time.perf_counter() - t0
    finally:
        torch.set_num_threads(threads)
    c1 = sampled("c1", c1_sample)
    c2 = sampled("c2", c2_sample)
    return {"value": c2["iters_per_s"], "unit": "iters/s", "cores": threads, "kind": "oracle",
            "sample": c2["sample"] + " (1200x680 / 300k, fwd + bwd in float64, "
                      f"{c2['seconds']:.1f} s)",
            "seconds": c2["seconds"],
            "host": {"cpu_model": _cpu_model(), "os_cpu_count": os.cpu_count(),
                     "torch_threads": threads},
            "c0_full_frame": {"reps": c0_reps, "median_s": float(np.median(times)),
                              "iters_per_s": 1.0 / float(np.median(times)),
                              "single_thread_s": single,
                              "single_thread_iters_per_s": 1.0 / single},
            "c1_sampled": c1, "c2_sampled": c2}


def _served(mode, b, s):
    return {"mode": mode, "trace_s": b["trace_s"], "frames_measured": b["frames_measured"],
            "p50_ms": b["p50_ms"], "p99_ms": b["p99_ms"],
            "per_class_p99_ms": {k: v["p99_ms"] for k, v in b["per_class"].items()},
            "iters_per_s": b["iters_per_s"], "map_jobs": b["map_jobs"],
            "one_at_a_time": {"trace_s": s["trace_s"], "frames_measured": s["frames_measured"],
                              "p50_ms": s["p50_ms"], "p99_ms": s["p99_ms"],
                              "iters_per_s": s["iters_per_s"], "map_jobs": s["map_jobs"]}}


def serving_run(seconds, warmup_s, downsample, mode, seed=4242, rate=30.0, async_mapping=False,
                map_every=1, prune=False, prune_ratio=0.1, max_map_batch=16,
                overlap_frames=False):
    """The 16-session serving mix on a Poisson trace (rate Hz per session)."""
    from paper_2510_06644_amd import serving
    specs = serving.serving_mix()
    ex = serving.GpuExecutor(0, prune=prune, prune_ratio=prune_ratio)
    cfg = serving.ServeConfig(mode=mode, downsample=downsample, async_mapping=async_mapping,
                              map_every=map_every, max_map_batch=max_map_batch,
                              overlap_frames=overlap_frames)
    eng = serving.Engine(specs, ex, cfg)
    eng.preopen()
    ex.warmup(specs, iters=1)
    trace = serving.poisson_trace(len(specs), rate, seconds, seed)
    rep = eng.run(trace, warmup_s=warmup_s)
    rep["sessions"] = len(specs)
    ex.verify()
    rep["mode"] = mode
    rep["downsample"] = downsample
    rep["trace_s"] = seconds
    rep["overflows"] = ex.overflows
    rep["prune"] = prune
    rep["overlap_frames"] = overlap_frames
    rep["map_every"] = map_every
    # release this run's maps before the next run allocates its own
    import gc
    import torch
    del eng, ex
    gc.collect()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    return rep


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=60)
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-variant", action="store_true")
    ap.add_argument("--cpu-sample", type=int, default=448,
                    help="pixels of the 1200x680 frame the CPU oracle evaluates")
    ap.add_argument("--calib-copy", action="store_true",
                    help="end with a 512 MiB device copy (scales PMC byte counters)")
    ap.add_argument("--no-tracking", action="store_true",
                    help="skip the tracking lines (profiler runs of the mapping step)")
    ap.add_argument("--serve-seconds", type=float, default=30.0,
                    help="length of the batched serving traces, the first 2 s not reported "
                         "(0 disables the serving runs)")
    ap.add_argument("--serve-baseline-seconds", type=float, default=10.0,
                    help="length of the one-item-at-a-time serving traces")
    ap.add_argument("--counter-record", metavar="DIR",
                    help="print the counter summary (markdown with the JSON record this "
                         "bench reads) of the rocprofv3 results under DIR/{fetch,write,sq,"
                         "sqw}/run_results.db, and exit")
    args = ap.parse_args()
    if args.counter_record:
        print(counter_summary(args.counter_record))
        return
    if args.gpus != 1:
        print(f"bench.py measures one GPU: this path has no multi-GPU mode "
              f"(--gpus {args.gpus} requested).", file=sys.stderr)
        sys.exit(2)
    import torch
    from paper_2510_06644_amd import rtgs
    if not torch.cuda.is_available():
        print("bench.py needs a GPU", file=sys.stderr)
        sys.exit(1)

    spec, cam, sc, params, target_scene, view, rc = setup("c2")
    R = rtgs.Renderer(0, check="deferred")
    tc, td = render_target(R, target_scene, view, rc, spec.seed)
    R.verify()
    opt = make_optimizer(params)
    log("warmup")
    for _ in range(args.warmup):
        mapping_step(R, params, view, rc, opt, tc, td)
    torch.cuda.synchronize()
    try:
        R.verify()
    except rtgs.RtgsError:
        for _ in range(2):
            mapping_step(R, params, view, rc, opt, tc, td)
        R.verify()
    counts0 = work_counts(R, params, view, rc)
    log(f"counts {counts0}")

    log("timed")
    ms, wall_ms, prof, per_iter = timed_loop(R, params, view, rc, opt, tc, td, args.steps,
                                             profile_stages=["raster_bwd"])
    counts1 = work_counts(R, params, view, rc)
    cnt = {k: 0.5 * (counts0[k] + counts1[k]) for k in counts0}
    bwd_ms = prof["raster_bwd"][0] / prof["raster_bwd"][1]
    flops = FLOP_BWD_PER_ENTRY * cnt["visited_to_last"] + FLOP_BWD_PER_BLEND * cnt["blended"]
    achieved = flops / (bwd_ms * 1e-3) / 1e12
    rec = counter_record()
    khash = kernel_hash()
    bwd_bytes = _kernel_sum(rec, VALU_STAGES["raster_bwd"], "bytes")
    roof = {"kernel": "raster_bwd", "bound": "alu", "achieved": achieved,
            "peak": PEAK_FP32_PUBLISHED, "unit": "TFLOP/s", "frac": achieved / PEAK_FP32_PUBLISHED,
            "traffic": bwd_bytes,
            "frac_vs_nonpacked": achieved / PEAK_FP32_NONPACKED,
            "peak_nonpacked": PEAK_FP32_NONPACKED,
            "avg_ms": bwd_ms, "launches": prof["raster_bwd"][1], "flops_per_launch": flops,
            "kernel_hash": khash, "counters_match": rec is not None}
    log("stage breakdown")
    _, _, stages, _ = timed_loop(R, params, view, rc, opt, tc, td, 10,
                                 profile_stages=list(rtgs.STAGES))
    stages_ms = {k: v[0] / v[1] for k, v in stages.items()}
    fwd_ms = stages_ms.get("raster_fwd", float("nan"))
    fwd_flops = FLOP_FWD_PER_ENTRY * cnt["visited"] + FLOP_FWD_PER_BLEND * cnt["blended"]
    kernels = per_kernel(stages_ms, cnt, spec.n, rec)

    variant = None
    if not args.no_variant:
        log("as-written variant")
        spec2, cam2, sc2, params2, tscene2, view2, rc2 = setup("c2")
        R2 = rtgs.Renderer(0, check="deferred")
        tc2, td2 = render_target(R2, tscene2, view2, rc2, spec2.seed)
        R2.verify()
        opt2 = make_optimizer(params2)
        for _ in range(3):
            mapping_step(R2, params2, view2, rc2, opt2, tc2, td2)
        R2.cap = R.cap
        variant = as_written_variant(R2, params2, view2, rc2, opt2, tc2, td2)
    balance = policies = None
    if not args.no_variant:
        log("lanes assigned by previous work")
        balance = lane_balance_run()
        log("backward state policies")
        policies = state_policy_run()
    tracking = tracking_reuse = tracking_prune = None
    if not args.no_tracking:
        log("tracking 640x480 / 100k")
        tracking = tracking_run()
        tracking_reuse = tracking_run(reuse_lists=True)
        tracking_prune = tracking_run(mask_prune=True)
    serve = None
    if args.serve_seconds > 0:
        serve = {}
        secs, base_secs = args.serve_seconds, args.serve_baseline_seconds
        warm = min(2.0, secs / 4)
        # reading 1 (the paper's algorithm as served): downsampling of
        # non-keyframes (Sec. 4.2), pruning per tracked frame (Sec. 4.1), keyframe
        # mapping as background jobs; a frame's latency is the time to its pose.
        # Batched with overlapping frames, then the same trace one item at a time.
        for mode, length in (("batched", secs), ("serial", base_secs)):
            log(f"serving {mode}: pruning, downsampling, background mapping ({length:.0f} s)")
            serve[f"rtgs_{mode}"] = serving_run(length, min(warm, length / 4), True, mode,
                                                async_mapping=True, map_every=4, prune=True,
                                                overlap_frames=mode == "batched")
        # reading 2 (plain): a keyframe's 20 mapping iterations run in line, so
        # its latency includes them; downsampled non-keyframes, no pruning
        for mode, length in (("batched", secs), ("serial", base_secs)):
            log(f"serving {mode}: mapping in line ({length:.0f} s)")
            serve[f"inline_{mode}"] = serving_run(length, min(warm, length / 4), True, mode)
    cpu = None
    if not args.no_cpu_baseline:
        log("cpu baseline")
        cpu = cpu_baseline(c2_sample=args.cpu_sample)
    line = {
        "metric": METRIC,
        "value": 1000.0 / ms,
        "unit": "iters/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",
        "data": "synthetic",
        "config": {"workload": spec.name, "width": cam.width, "height": cam.height,
                   "gaussians": spec.n, "step": "render_fwd + L1 loss (fused into the forward) + render_bwd "
                   "(all map parameters) + Adam (fused into the backward)", "pixels": "full resolution", "prune": False},
        "roofline": roof,
        "path_roofline": path_roofline(cnt, ms, bwd_ms, fwd_ms, spec),
        "raster_fwd_roofline": {"bound": "alu", "avg_ms": fwd_ms,
                                "achieved": fwd_flops / (fwd_ms * 1e-3) / 1e12,
                                "peak": PEAK_FP32_PUBLISHED, "unit": "TFLOP/s",
                                "frac": fwd_flops / (fwd_ms * 1e-3) / 1e12 / PEAK_FP32_PUBLISHED,
                                "frac_vs_nonpacked":
                                    fwd_flops / (fwd_ms * 1e-3) / 1e12 / PEAK_FP32_NONPACKED},
        "iteration_ms": iter_stats(per_iter),
        "kernels": kernels,
        "stages_ms": stages_ms,
        "work": cnt,
        "host_wall_ms_per_step": 1000.0 * wall_ms,
        "as_written": variant,
        "lane_balance": balance,
        "state_policies": policies,
        "tracking": tracking,
        "tracking_reuse_lists": tracking_reuse,
        "tracking_mask_prune": tracking_prune,
        "serving": serve,
        "served_latency": None if not serve else {
            "sessions": 16, "rate_hz_per_session": 30.0,
            "reading_1": _served("batched: pruning + downsampling, background keyframe "
                                 "mapping, overlapping frames; latency to the pose",
                                 serve["rtgs_batched"], serve["rtgs_serial"]),
            "reading_2": _served("batched: downsampling, keyframe mapping in line; latency "
                                 "includes a keyframe's mapping", serve["inline_batched"],
                                 serve["inline_serial"])},
        "cpu_baseline": cpu,
    }
    print(json.dumps(line), flush=True)
    if args.calib_copy:
        src = torch.ones(128 << 20, dtype=torch.float32, device="cuda")
        dst = torch.empty_like(src)
        torch.cuda.synchronize()
        dst.copy_(src)
        torch.cuda.synchronize()
    _reap_children()


def _reap_children():
    """Leave no process behind: end any child process this run started
    (none is expected)."""
    try:
        import psutil
    except ImportError:
        return
    kids = psutil.Process().children(recursive=True)
    for k in kids:
        log(f"ending child process {k.pid} ({' '.join(k.cmdline()[:3])})")
        k.terminate()
    psutil.wait_procs(kids, timeout=5)


if __name__ == "__main__":
    main()
