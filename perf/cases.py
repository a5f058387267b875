"""The work that users of the rasterizer have it do, as cases to be timed and checked.

A case names one call or one short sequence of calls of the public entry points, as a SLAM
program makes them: a differentiable render through autograd, a plain render, a tracking
iteration (also on reused tile lists, also on a downsampled frame), a mapping iteration with
the map update inside the backward or apart, the end of a pruning window, and the batched
launches of the serving engine.  Sizes are those of the workloads in
``paper_2510_06644_amd.synth`` and ``serving`` (128x128 / 2k up to 1200x680 / 500k and the
16-session mix's classes) and ragged ones between them.

Scenes follow the recipe of ``synth.make_scene`` (centres uniform in the frustum, volume-uniform
depth on [0.5, 5] m, log-normal scales, a share near-transparent for the large frames), drawn on
the device from the seed.  Targets are smooth colour and depth images plus sensor noise; they do
not depend on the rasterizer.

``exact`` composites the same frames in float64 with plain torch, tile by tile, and takes
gradients by automatic differentiation.
"""
import math

import torch

from paper_2510_06644_amd import autograd, optim, rtgs

DEV = torch.device("cuda" if torch.cuda.is_available() else "cpu")
PIX_MAX = 1200 * 680
N_MAX = 500_000


# ---------------------------------------------------------------------------------- cases
def listed():
    return [
        # the smallest call: a differentiable render of a thumbnail, per-call latency and
        # launches; the default policy checks the pair capacity after every forward
        dict(name="autograd_128x128_2k", kind="autograd", w=128, h=128, n=2_000, state="save"),
        # odd sizes, nothing kept per pixel: the backward composites the frame again first
        dict(name="autograd_recompute_333x251_7k", kind="autograd", w=333, h=251, n=7_001,
             state="recompute"),
        # a view of the map without gradients (display, keyframe evaluation)
        dict(name="render_320x240_20k", kind="render", w=320, h=240, n=20_000),
        # one tracking iteration: forward with the loss gradient, pose gradient, pose update
        dict(name="track_640x480_100k", kind="track", w=640, h=480, n=100_000, iters=1),
        # four tracking iterations of one frame, the last three on the first one's tile lists
        dict(name="track_reuse_640x480_100k", kind="track", w=640, h=480, n=100_000, iters=4),
        # tracking a non-keyframe downsampled 1 in 4 (mask from the last final transmittance)
        dict(name="track_1in4_1200x680_500k", kind="down", w=1200, h=680, n=500_000, j=2),
        # a mapping iteration of a small map on a ragged frame
        dict(name="map_727x405_61k", kind="map", w=727, h=405, n=61_003),
        # the mapping iteration that the benchmark times (Adam inside the backward)
        dict(name="map_1200x680_300k", kind="map", w=1200, h=680, n=300_000),
        # a keyframe's scoring iteration: loss pass, every gradient there is (map, pose and
        # covariance), and the map update as a call of its own
        dict(name="score_1200x680_500k", kind="score", w=1200, h=680, n=500_000),
        # the end of a pruning window: select, count the changed tiles, remove for good
        dict(name="prune_500k", kind="prune", n=500_000, ratio=0.1),
        # one batched tracking iteration of the serving engine, the three frame classes of the
        # 16-session mix twice each, every second frame downsampled 1 in 4
        dict(name="serve_track_6", kind="serve_track", sessions=6, scale=1.0),
        # one batched iteration of three keyframe map jobs, one of each class
        dict(name="serve_map_3", kind="serve_map", sessions=3, scale=1.0),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _frame(rng, px_lo=96 * 96, px_hi=PIX_MAX):
    """A frame of any size in the range, ragged, landscape to square."""
    px = _log_uniform(rng, px_lo, px_hi)
    aspect = rng.uniform(1.0, 1.8)
    w = max(64, min(1200, int(math.sqrt(px * aspect))))
    h = max(48, min(680, int(px / w)))
    return w, h


def _count(rng, w, h, most=N_MAX):
    """Gaussians of a frame: about 0.1 to 0.6 a pixel, as in the workloads."""
    return max(500, min(most, int(w * h * _log_uniform(rng, 0.1, 0.6))))


def draw(rng):
    kind = rng.choice(["autograd", "render", "track", "reuse", "down", "map", "score", "prune",
                       "serve_track", "serve_map"])
    if kind == "prune":
        return dict(kind="prune", n=int(_log_uniform(rng, 2_000, N_MAX)),
                    ratio=round(rng.uniform(0.02, 0.5), 3))
    if kind.startswith("serve"):
        return dict(kind=kind, sessions=rng.randint(2, 6 if kind == "serve_track" else 3),
                    scale=round(rng.uniform(0.25, 0.98), 3))
    w, h = _frame(rng, px_hi=640 * 480) if kind in ("autograd", "reuse") else _frame(rng)
    n = _count(rng, w, h)
    if kind == "autograd":
        return dict(kind=kind, w=w, h=h, n=n, state=rng.choice(["save", "recompute"]))
    if kind in ("track", "reuse"):
        return dict(kind="track", w=w, h=h, n=n, iters=1 if kind == "track" else 4)
    if kind == "down":
        return dict(kind=kind, w=w, h=h, n=n, j=rng.choice([2, 3, 4]))
    return dict(kind=kind, w=w, h=h, n=n)


# ---------------------------------------------------------------------------------- inputs
def _gen(seed, salt=0):
    return torch.Generator(device=DEV).manual_seed((seed * 1_000_003 + salt * 7919 + 12345) % (1 << 62))


def _camera(w, h):
    f = 0.8 * w
    return rtgs.Cam(w, h, f, f, w / 2.0, h / 2.0)


def _scene(w, h, n, g):
    """Centres uniform in the frustum, volume-uniform depth; the large frames' scales are finer
    and spread wider and a fifth of their Gaussians is near-transparent."""
    f64 = dict(dtype=torch.float64, device=DEV, generator=g)
    big = w * h > 640 * 480
    cam = _camera(w, h)
    z = (0.5 ** 3 + (5.0 ** 3 - 0.5 ** 3) * torch.rand(n, **f64)) ** (1.0 / 3.0)
    x = (torch.rand(n, **f64) * w - cam.cx) * z / cam.fx
    y = (torch.rand(n, **f64) * h - cam.cy) * z / cam.fy
    means = torch.stack([x, y, z], 1)
    scales = torch.randn(n, 3, **f64) * (0.7 if big else 0.5) + (-4.5 if big else -4.0)
    q = torch.randn(n, 4, **f64)
    q = q / q.norm(dim=1, keepdim=True)
    eta = torch.randn(n, **f64)
    if big:
        faint = torch.rand(n, **f64) < 0.2
        p = 0.005 + 0.045 * torch.rand(n, **f64)
        eta = torch.where(faint, torch.log(p) - torch.log1p(-p), eta)
    colors = torch.rand(n, 3, **f64)
    return tuple(t.to(torch.float32).contiguous() for t in (means, scales, q, eta, colors))


def _view(g, trans=0.02, rot=0.0175):
    """A camera a step of a slow trajectory away from the identity pose, float32 [3, 4]."""
    f64 = dict(dtype=torch.float64, device=DEV, generator=g)
    a, d = torch.randn(3, **f64), torch.randn(3, **f64)
    a, d = a / a.norm() * rot, d / d.norm() * trans
    return torch.cat([_rot(a), d[:, None]], 1).to(torch.float32).contiguous()


def _rot(phi):
    """Rotation matrix of a rotation vector (float64)."""
    zero = torch.zeros((), dtype=phi.dtype, device=phi.device)
    k = torch.stack([zero, -phi[2], phi[1], phi[2], zero, -phi[0], -phi[1], phi[0], zero]).reshape(3, 3)
    return torch.linalg.matrix_exp(k)


def _target(w, h, g):
    """A frame to be matched: smooth colour and depth plus sensor noise."""
    f32 = dict(dtype=torch.float32, device=DEV, generator=g)
    low = torch.rand(1, 4, 12, 20, **f32)
    img = torch.nn.functional.interpolate(low, size=(h, w), mode="bilinear", align_corners=False)[0]
    img = img + 0.01 * torch.randn(4, h, w, **f32)
    return (0.2 + 0.6 * img[:3]).contiguous(), (0.5 + 3.0 * img[3]).contiguous()


def _inputs(w, h, n, seed, salt=0):
    g = _gen(seed, salt)
    return dict(cam=_camera(w, h), scene=_scene(w, h, n, g), view=_view(g), target=_target(w, h, g), g=g)


def _upstream(w, h, g):
    f32 = dict(dtype=torch.float32, device=DEV, generator=g)
    return torch.randn(3, h, w, **f32), torch.randn(h, w, **f32), torch.randn(h, w, **f32)


def _last_T(w, h, g):
    """A final transmittance image of an earlier frame: mostly covered, some free."""
    return (1e-4 + torch.rand(h, w, dtype=torch.float32, device=DEV, generator=g) ** 4).contiguous()


def _classes(case):
    """(width, height, Gaussians, downsampled) of each session of a serving batch."""
    base = [(320, 240, 20_000), (640, 480, 100_000), (1200, 680, 500_000)]
    s = case["scale"]
    out = []
    for k in range(case["sessions"]):
        w, h, n = base[k % 3]
        out.append((max(64, int(w * s)), max(48, int(h * s)), int(n * s * s), 2 if k % 2 else 0))
    return out


def _prune_inputs(case, seed):
    """Gradients of a tracking iteration at the map (three in ten Gaussians carry one, spread
    over decades), visibility, and the window's tile rectangles before and after."""
    n, g = case["n"], _gen(seed, 3)
    f32 = dict(dtype=torch.float32, device=DEV, generator=g)
    live = torch.rand(n, **f32) < 0.3
    mag = torch.exp(2.0 * torch.randn(n, **f32) - 8.0) * live
    gm = mag[:, None] * torch.randn(n, 3, **f32)
    gc = 4.0 * mag[:, None] * torch.randn(n, 6, **f32)
    vis = (torch.randperm(n, device=DEV, generator=g) < int(0.9 * n)).to(torch.uint8)
    r0 = torch.floor(torch.rand(n, 2, **f32) * torch.tensor([75.0, 43.0], device=DEV))
    ext = torch.floor(torch.rand(n, 2, **f32) ** 4 * 12.0)
    ref = torch.cat([r0, r0 + ext], 1).to(torch.int32)
    ref[vis == 0] = torch.tensor([0, 0, -1, -1], dtype=torch.int32, device=DEV)
    move = torch.floor(torch.rand(n, 4, **f32) * 1.1).to(torch.int32)
    cur = torch.where(vis[:, None] != 0, ref + move, ref).contiguous()
    rows = _scene(1200, 680, n, g)
    moments = [1e-3 * torch.randn(t.shape, **f32) for t in rows] + \
              [1e-6 * torch.rand(t.shape, **f32) for t in rows]
    return gm.contiguous(), gc.contiguous(), vis, ref.contiguous(), cur, list(rows) + moments


LRS = tuple(0.01 * x for x in optim.MAP_LRS)   # late in a decayed schedule: the map hardly moves


# ---------------------------------------------------------------------------------- prepare
def _renderer(s, check="deferred"):
    """A renderer whose pair capacity a first frame has settled, as a running program's has."""
    R = rtgs.Renderer(DEV.index or 0, check=check, pairs_per_gaussian=16.0)
    if check == "deferred":
        while True:
            R.forward(s["scene"], s["view"], s["cam"])
            try:
                R.verify()
                break
            except rtgs.RtgsError:
                pass
    return R


def prepare(case, seed):
    kind = case["kind"]
    if kind == "prune":
        gm, gc, vis, ref, cur, rows = _prune_inputs(case, seed)
        n = case["n"]
        taken = int(math.floor(float(torch.tensor(case["ratio"], dtype=torch.float32)) * int(vis.sum())))
        return dict(case=case, h=rtgs.Handle(DEV.index or 0), gm=gm, gc=gc, vis=vis, ref=ref, cur=cur,
                    rows=rows + [cur], keep=n - taken)
    if kind.startswith("serve"):
        return _prepare_serve(case, seed)
    w, h, n = case["w"], case["h"], case["n"]
    s = _inputs(w, h, n, seed)
    s["case"] = case
    if kind == "autograd":
        s["up"] = _upstream(w, h, s["g"])
        s["leaves"] = [t.clone().requires_grad_(True) for t in s["scene"]]
        s["vm"] = s["view"].clone().requires_grad_(True)
        s["R"] = _renderer(s, check="every")
        return s
    s["R"] = _renderer(s)
    if kind in ("map", "score"):
        s["opt"] = optim.MapAdam([t.clone() for t in s["scene"]], lrs=LRS, eps=1e-15)
        s["params"] = tuple(s["opt"].params)
    if kind == "down":
        s["last_T"] = _last_T(w, h, s["g"])
    return s


def _prepare_serve(case, seed):
    """Resident maps, output buffers and call records of a serving batch."""
    handle = rtgs.Handle(DEV.index or 0)
    track = case["kind"] == "serve_track"
    cls = _classes(case)
    k = len(cls)
    start = torch.zeros(k, 24, dtype=torch.float32, device=DEV)      # pose, two Adam moments
    live = torch.zeros_like(start)
    gpose = torch.zeros(k, 6, dtype=torch.float32, device=DEV)
    outs, items, poses, opts, hold = [], [], [], [], []
    for i, (w, h, n, j) in enumerate(cls):
        s = _inputs(w, h, n, seed, salt=17 * (i + 1))
        start[i, :12] = s["view"].reshape(-1)
        o = dict(color=torch.empty(3, h, w, device=DEV), depth=torch.empty(h, w, device=DEV),
                 alpha=torch.empty(h, w, device=DEV), final_T=torch.empty(h, w, device=DEV),
                 last_idx=torch.empty(h, w, dtype=torch.int32, device=DEV))
        gc, gd = torch.empty(3, h, w, device=DEV), torch.empty(h, w, device=DEV)
        it = dict(viewmat=live[i, :12].view(3, 4), cam=s["cam"], dL_dcolor=gc, dL_ddepth=gd,
                  visible=torch.empty(n, dtype=torch.uint8, device=DEV), **o)
        cnt = None
        if track:
            it["scene"] = s["scene"]
            it["g_pose6"] = gpose[i]
            if j:
                mask = torch.empty(h, w, dtype=torch.uint8, device=DEV)
                cnt = torch.zeros(1, dtype=torch.int32, device=DEV)
                rtgs.downsample_mask(_last_T(w, h, s["g"]), j, mask, cnt)
                it.update(pixel_mask=mask, sample_log2=j)
            poses.append(rtgs.pose_item(it["viewmat"], gpose[i], live[i, 12:18], live[i, 18:24], 1e-3, 3e-3))
        else:
            opt = optim.MapAdam([t.clone() for t in s["scene"]], lrs=LRS, eps=1e-15)
            it["scene"] = tuple(opt.params)
            it["adam"] = opt.fused()
            opts.append(opt)
        it["l1"] = rtgs.l1_loss(s["target"][0], s["target"][1], gc, gd, cnt, 1.0, 0.5)
        items.append(rtgs.session_struct(it))
        hold.append((it, s["target"], cnt))
        outs.append(o)
    cap = sum(16 * n + 4 * ((w + 15) // 16) * ((h + 15) // 16) for w, h, n, _ in cls)
    live.copy_(start)
    return dict(case=case, handle=handle, cls=cls, start=start, live=live, gpose=gpose, outs=outs,
                arr=(rtgs.CSession * k)(*items), poses=(rtgs.CPoseItem * k)(*poses) if track else None,
                opts=opts, items=hold, cap=cap)


# ---------------------------------------------------------------------------------- run
def run(s):
    return globals()["_run_" + s["case"]["kind"]](s)


def _run_autograd(s):
    for t in s["leaves"] + [s["vm"]]:
        t.grad = None
    c, d, a, vis = autograd.render(*s["leaves"], s["vm"], s["cam"], renderer=s["R"], state=s["case"]["state"])
    torch.autograd.backward([c, d, a], list(s["up"]))
    return dict(color=c, depth=d, alpha=a, visible=vis, grads=[t.grad for t in s["leaves"]], g_view=s["vm"].grad)


def _run_render(s):
    st = s["R"].forward(s["scene"], s["view"], s["cam"], save_state=False)
    return dict(color=st.color, depth=st.depth, alpha=st.alpha, visible=st.visible)


def _run_track(s):
    """A frame's tracking from its start pose, the tile lists of the first iteration kept."""
    R, cam = s["R"], s["cam"]
    tc, td = s["target"]
    view = s["view"].clone()
    mom = torch.zeros(2, 6, device=DEV)
    first = None
    for it in range(1, s["case"]["iters"] + 1):
        st = R.forward(s["scene"], view, cam, reuse_lists_of=first, l1=(tc, td, None))
        first = first or st
        g = R.backward(s["scene"], view, cam, st, st.dL_dcolor, st.dL_ddepth, pose=True, map_grads=False)
        rtgs.pose_update([(view, g["pose"], mom[0], mom[1], 1e-3, 1e-3, it)])
    return dict(color=st.color, depth=st.depth, final_T=st.final_T, last_idx=st.last_idx,
                g_pose=g["pose"], g_view=g["viewmat"], view=view)


def _run_down(s):
    R, cam, j = s["R"], s["cam"], s["case"]["j"]
    tc, td = s["target"]
    view = s["view"].clone()
    mom = torch.zeros(2, 6, device=DEV)
    mask = torch.empty(cam.height, cam.width, dtype=torch.uint8, device=DEV)
    cnt = torch.zeros(1, dtype=torch.int32, device=DEV)
    rtgs.downsample_mask(s["last_T"], j, mask, cnt)
    st = R.forward(s["scene"], view, cam, pixel_mask=mask, sample_log2=j, l1=(tc, td, cnt))
    g = R.backward(s["scene"], view, cam, st, st.dL_dcolor, st.dL_ddepth, pose=True, map_grads=False, pixel_mask=mask)
    rtgs.pose_update([(view, g["pose"], mom[0], mom[1], 1e-3, 1e-3, 1)])
    return dict(mask=mask, count=cnt, color=st.color, depth=st.depth, final_T=st.final_T,
                g_pose=g["pose"], view=view)


def _run_map(s):
    R, cam, (tc, td) = s["R"], s["cam"], s["target"]
    st = R.forward(s["params"], s["view"], cam, l1=(tc, td, None))
    R.backward(s["params"], s["view"], cam, st, st.dL_dcolor, st.dL_ddepth, pose=False, adam=s["opt"])
    return dict(color=st.color, depth=st.depth, final_T=st.final_T, last_idx=st.last_idx,
                params=list(s["params"]), m=s["opt"].exp_avg, v=s["opt"].exp_avg_sq)


MAP_KEYS = ("means", "log_scales", "quats", "opacity_logits", "colors")


def _run_score(s):
    R, cam, (tc, td) = s["R"], s["cam"], s["target"]
    st = R.forward(s["params"], s["view"], cam)
    gc, gd = torch.empty_like(st.color), torch.empty_like(st.depth)
    rtgs.loss_l1_grad(st.color, st.depth, tc, td, gc, gd)
    g = R.backward(s["params"], s["view"], cam, st, gc, gd, pose=True, map_grads=True, cov3d=True)
    s["opt"].step(R.handle, [g[k] for k in MAP_KEYS])
    return dict(color=st.color, depth=st.depth, final_T=st.final_T, grads=[g[k] for k in MAP_KEYS],
                g_cov=g["cov3d"], g_pose=g["pose"], params=list(s["params"]), m=s["opt"].exp_avg, v=s["opt"].exp_avg_sq)


def _run_prune(s):
    n, keep = s["case"]["n"], s["keep"]
    mask = torch.empty(n, dtype=torch.uint8, device=DEV)
    count = torch.empty(1, dtype=torch.int32, device=DEV)
    kept = torch.empty(1, dtype=torch.int32, device=DEV)
    change = torch.empty(2, dtype=torch.int64, device=DEV)
    rtgs.prune_by_grad(s["h"], s["gm"], s["gc"], s["vis"], None, 0.8, s["case"]["ratio"], mask, count)
    rtgs.tile_pair_change(s["ref"], s["cur"], None, change)
    outs = [torch.empty((keep,) + tuple(t.shape[1:]), dtype=t.dtype, device=DEV) for t in s["rows"]]
    rtgs.compact_by_mask(mask, list(zip(s["rows"], outs)), kept)
    return dict(mask=mask, count=count, kept=kept, change=change, rows=outs)


def _batch_ws(s):
    cls = s["cls"]
    return torch.empty(rtgs.rtgs_workspace_size_batched([c[2] for c in cls], [c[0] for c in cls],
                                                        [c[1] for c in cls], s["cap"]), dtype=torch.uint8, device=DEV)


def _run_serve_track(s):
    """Every frame's first tracking iteration, from its own start pose."""
    k, st = len(s["cls"]), rtgs.stream_ptr()
    s["live"].copy_(s["start"])
    ws = _batch_ws(s)
    rtgs.render_fwd_batched_c(s["handle"], s["arr"], k, ws, s["cap"], rtgs.RTGS_FWD_SAVE_STATE, st)
    rtgs.render_bwd_batched_c(s["handle"], s["arr"], k, ws, s["cap"], rtgs.RTGS_GRAD_POSE, st)
    rtgs.pose_update_c(s["poses"], k, 0.9, 0.999, 1e-8, st)
    return dict(images=[[o["color"], o["depth"], o["final_T"], o["last_idx"]] for o in s["outs"]],
                g_pose=s["gpose"], view=s["live"][:, :12])


def _run_serve_map(s):
    k, st = len(s["cls"]), rtgs.stream_ptr()
    ws = _batch_ws(s)
    for opt, (it, _, _) in zip(s["opts"], s["items"]):
        it["adam"].step = opt.t + 1
    rtgs.render_fwd_batched_c(s["handle"], s["arr"], k, ws, s["cap"], rtgs.RTGS_FWD_SAVE_STATE, st)
    rtgs.render_bwd_batched_c(s["handle"], s["arr"], k, ws, s["cap"], rtgs.RTGS_GRAD_MAP | rtgs.RTGS_GRAD_ADAM, st)
    for opt in s["opts"]:
        opt.t += 1
    return dict(images=[[o["color"], o["depth"]] for o in s["outs"]],
                maps=[[list(o.params), o.exp_avg, o.exp_avg_sq] for o in s["opts"]])


# ---------------------------------------------------------------------------------- work
# A pixel's list entries and blended fragments up to its stop, as the work counters of the
# 1200x680 / 300k frame give them (191 visited, 74 blended at 0.37 Gaussians a pixel; other
# frames in proportion to their density until the stop saturates them at about that), and the
# operations of one: alpha 18, blend 12, reverse 65 (an FMA is two).
def _fragments(w, h, n, j=0):
    px = w * h / 2 ** j
    dense = min(1.0, n / (w * h) / 0.33)
    return 191 * dense * px, 74 * dense * px


def _frame_work(w, h, n, j=0, back="none", loss=True):
    px, (seen, hit) = w * h, _fragments(w, h, n, j)
    b = 56 * n + n + 28 * px                       # map, visibility, five image planes
    f = 18 * seen + 12 * hit + 250 * n
    if loss:
        b += 32 * px                               # target in, loss gradient out
        f += 12 * px
    if back != "none":
        b += 56 * n + 24 * px                      # map, saved state and upstream gradient
        f += 18 * seen + 65 * hit + 600 * n
    if back == "map":
        b += 56 * n
    elif back == "score":
        b += (56 + 24) * n
    elif back == "adam":
        b += 56 * 5 * n                            # both moments in and out, parameters out
        f += 14 * 12 * n
    return b, f


def work(case):
    kind = case["kind"]
    if kind == "prune":
        n, r = case["n"], case["ratio"]
        b = (36 + 1 + 1) * n + 32 * n + (168 + 16) * n * (2 - r)
        return {"bytes": b, "flops": 30 * n}
    if kind.startswith("serve"):
        parts = [_frame_work(w, h, n, j if kind == "serve_track" else 0, "pose" if kind == "serve_track" else "adam")
                 for w, h, n, j in _classes(case)]
        return {"bytes": sum(p[0] for p in parts), "flops": sum(p[1] for p in parts)}
    w, h, n = case["w"], case["h"], case["n"]
    back = dict(autograd="map", render="none", track="pose", down="pose", map="adam", score="score")[kind]
    b, f = _frame_work(w, h, n, case.get("j", 0), back, loss=kind not in ("autograd", "render"))
    if kind == "autograd" and case["state"] == "recompute":
        f += 18 * _fragments(w, h, n)[0] + 12 * _fragments(w, h, n)[1]
    if kind == "score":
        a = 56 * 7 * n
        b, f = b + a, f + 14 * 12 * n
    if kind == "down":
        b += 5 * w * h
    k = case.get("iters", 1)
    return {"bytes": b * k, "flops": f * k}


# ---------------------------------------------------------------------------------- exact
def _project(P, vm, cam):
    """First-order projection in float64: pixel centre, 2D covariance, depth, opacity."""
    means, ls, q, eta, _ = P
    f = [float(torch.tensor(x, dtype=torch.float32)) for x in (cam.fx, cam.fy, cam.cx, cam.cy)]
    p = means @ vm[:, :3].T + vm[:, 3]
    x, y, z = p.unbind(1)
    w, a, b, c = (q / q.norm(dim=1, keepdim=True)).unbind(1)
    rot = torch.stack([1 - 2 * (b * b + c * c), 2 * (a * b - w * c), 2 * (a * c + w * b),
                       2 * (a * b + w * c), 1 - 2 * (a * a + c * c), 2 * (b * c - w * a),
                       2 * (a * c - w * b), 2 * (b * c + w * a), 1 - 2 * (a * a + b * b)], 1).reshape(-1, 3, 3)
    m = rot * torch.exp(ls)[:, None, :]
    lx, ly = 1.3 * 0.5 * cam.width / f[0], 1.3 * 0.5 * cam.height / f[1]
    tx, ty = torch.clamp(x / z, -lx, lx), torch.clamp(y / z, -ly, ly)
    r0 = (f[0] / z)[:, None] * vm[0, :3] - (f[0] * tx / z)[:, None] * vm[2, :3]
    r1 = (f[1] / z)[:, None] * vm[1, :3] - (f[1] * ty / z)[:, None] * vm[2, :3]
    return f, x, y, z, m, r0, r1, torch.sigmoid(eta)


def _splat(P, vm, cam, dsig=None):
    """Rows (u, v, a, b, c, o, r, g, b, z) of the Gaussians, and who is drawn.  dsig: a zero
    offset of the world covariance, whose gradient is the covariance gradient."""
    f, x, y, z, m, r0, r1, o = _project(P, vm, cam)
    with torch.no_grad():
        ok = (z > 0.2) & (255.0 * o >= 1.0)
    zs = torch.where(ok, z, torch.ones_like(z))
    if dsig is None:
        a0, a1 = (r0[:, None, :] @ m)[:, 0], (r1[:, None, :] @ m)[:, 0]
        sxx, sxy, syy = (a0 * a0).sum(1) + 0.3, (a0 * a1).sum(1), (a1 * a1).sum(1) + 0.3
    else:
        sig = m @ m.transpose(1, 2) + dsig
        s0, s1 = (sig @ r0[:, :, None])[..., 0], (sig @ r1[:, :, None])[..., 0]
        sxx, sxy, syy = (r0 * s0).sum(1) + 0.3, (r0 * s1).sum(1), (r1 * s1).sum(1) + 0.3
    det = sxx * syy - sxy * sxy
    rows = torch.stack([f[0] * x / zs + f[2], f[1] * y / zs + f[3], syy / det, -sxy / det, sxx / det, o,
                        *P[4].unbind(1), z], 1)
    return rows, ok, sxx, syy


def _pairs(rows, ok, sxx, syy, w, h):
    """(tile, Gaussian) pairs by tile and depth: the padded bounding boxes on 16x16 tiles."""
    with torch.no_grad():
        t = 2.0 * torch.log(torch.clamp(255.0 * rows[:, 5], min=1.0))
        ex, ey = torch.sqrt(t * sxx), torch.sqrt(t * syy)
        u, v = rows[:, 0], rows[:, 1]
        lo_x, hi_x = torch.floor(u - ex - 1.5), torch.ceil(u + ex + 0.5)
        lo_y, hi_y = torch.floor(v - ey - 1.5), torch.ceil(v + ey + 0.5)
        ok = ok & (hi_x >= 0) & (lo_x <= w - 1) & (hi_y >= 0) & (lo_y <= h - 1)
        ids = torch.nonzero(ok)[:, 0]
        ids = ids[torch.argsort(rows[ids, 9].to(torch.float32), stable=True)]
        x0, x1 = (lo_x[ids].clamp(0, w - 1).long() >> 4), (hi_x[ids].clamp(0, w - 1).long() >> 4)
        y0, y1 = (lo_y[ids].clamp(0, h - 1).long() >> 4), (hi_y[ids].clamp(0, h - 1).long() >> 4)
        nx = x1 - x0 + 1
        cnt = nx * (y1 - y0 + 1)
        rep = torch.repeat_interleave(torch.arange(ids.numel(), device=ids.device), cnt)
        k = torch.arange(rep.numel(), device=ids.device) - (torch.cumsum(cnt, 0) - cnt)[rep]
        tile = (y0[rep] + k // nx[rep]) * ((w + 15) // 16) + x0[rep] + k % nx[rep]
        order = torch.argsort(tile, stable=True)
        n_tiles = ((w + 15) // 16) * ((h + 15) // 16)
        return ids[rep[order]], torch.bincount(tile, minlength=n_tiles), ok


def _composite(rows, gids, counts, w, h, mask, grad_of):
    """Front-to-back compositing over padded groups of tiles; grad_of(C, D, T, pixels), if
    given, returns the upstream gradients of a group's pixels, which go back to rows."""
    dev, tx = rows.device, (w + 15) // 16
    start = torch.cumsum(counts, 0) - counts
    color, depth, trans = (torch.zeros(k, h * w, dtype=torch.float64, device=dev) for k in (3, 1, 1))
    trans += 1.0
    order = torch.argsort(counts, descending=True)
    lens = counts[order].tolist()
    g_rows = torch.zeros_like(rows) if grad_of else None
    leaf = rows.detach()
    i = 0
    while i < len(lens) and lens[i] > 0:
        length = lens[i]
        many = max(1, min(len(lens) - i, 12_000_000 // (256 * length)))
        tiles = order[i:i + many]
        i += many
        at = torch.arange(length, device=dev)
        real = at[None] < counts[tiles][:, None]
        idx = gids[(start[tiles][:, None] + at[None]).clamp(max=gids.numel() - 1)]
        R = leaf[idx]
        if grad_of:
            R.requires_grad_(True)
        p = torch.arange(256, device=dev)
        px = (tiles % tx)[:, None] * 16 + (p % 16)[None]
        py = (tiles // tx)[:, None] * 16 + (p // 16)[None]
        inside = (px < w) & (py < h)
        pix = (py * w + px).clamp(max=h * w - 1)
        if mask is not None:
            inside = inside & mask.reshape(-1)[pix]
        with torch.set_grad_enabled(bool(grad_of)):
            dx = R[:, :, 0, None] - (px[:, None] + 0.5)
            dy = R[:, :, 1, None] - (py[:, None] + 0.5)
            power = -0.5 * (R[:, :, 2, None] * dx * dx + R[:, :, 4, None] * dy * dy) - R[:, :, 3, None] * dx * dy
            alpha = torch.clamp(R[:, :, 5, None] * torch.exp(power), max=0.99)
            with torch.no_grad():
                hit = (alpha >= 1.0 / 255.0) & real[:, :, None] & inside[:, None]
                run = torch.exp(torch.cumsum(torch.log1p(-alpha * hit), 1))
                hit = hit & (run >= 1e-4)
            alpha = alpha * hit
            leave = torch.log1p(-alpha)
            after = torch.cumsum(leave, 1)
            wgt = alpha * torch.exp(after - leave)
            C = [(wgt * R[:, :, k, None]).sum(1) for k in (6, 7, 8)]
            D = (wgt * R[:, :, 9, None]).sum(1)
            T = torch.exp(after[:, -1])
        sel, where = inside, pix[inside]
        for k in range(3):
            color[k, where] = C[k].detach()[sel]
        depth[0, where] = D.detach()[sel]
        trans[0, where] = T.detach()[sel]
        if grad_of:
            gc, gd, ga = grad_of(C, D, pix)
            loss = sum((c * g * sel).sum() for c, g in zip(C, gc)) + (D * gd * sel).sum()
            if ga is not None:
                loss = loss + ((1.0 - T) * ga * sel).sum()
            (gr,) = torch.autograd.grad(loss, R)
            g_rows.index_add_(0, idx.reshape(-1), (gr * real[:, :, None]).reshape(-1, gr.shape[-1]))
    return color.reshape(3, h, w), depth.reshape(h, w), trans.reshape(h, w), g_rows


def _l1_of(target, n_active, w_color=1.0, w_depth=0.5):
    tc, td = target[0].double().reshape(3, -1), target[1].double().reshape(-1)

    def grad_of(C, D, pix):
        gc = [w_color / (3.0 * n_active) * torch.sign(C[k].detach() - tc[k][pix]) for k in range(3)]
        return gc, w_depth / n_active * torch.sign(D.detach() - td[pix]), None
    return grad_of


def _upstream_of(up):
    gc, gd, ga = up[0].double().reshape(3, -1), up[1].double().reshape(-1), up[2].double().reshape(-1)
    return lambda C, D, pix: ([gc[k][pix] for k in range(3)], gd[pix], ga[pix])


def _frame64(scene, view, cam, mask=None, grad_of=None, lists=None, cov=False):
    """One frame in float64: images, and the gradients of map, view matrix and covariance."""
    P = [t.double().clone().requires_grad_(bool(grad_of)) for t in scene]
    vm = view.double().clone().requires_grad_(bool(grad_of))
    dsig = torch.zeros(P[0].shape[0], 3, 3, dtype=torch.float64, device=P[0].device, requires_grad=True) if cov else None
    with torch.set_grad_enabled(bool(grad_of)):
        rows, ok, sxx, syy = _splat(P, vm, cam, dsig)
    if lists is None:
        lists = _pairs(rows.detach(), ok, sxx.detach(), syy.detach(), cam.width, cam.height)[:2]
    c, d, t, g = _composite(rows, lists[0], lists[1], cam.width, cam.height, mask, grad_of)
    out = dict(color=c, depth=d, T=t, lists=lists)
    if grad_of:
        want = P + [vm] + ([dsig] if cov else [])
        got = torch.autograd.grad(rows, want, g, allow_unused=True)
        out["grads"], out["g_view"] = list(got[:5]), got[5]
        if cov:
            s = 0.5 * (got[6] + got[6].transpose(1, 2))
            out["g_cov"] = torch.stack([s[:, 0, 0], s[:, 0, 1], s[:, 0, 2], s[:, 1, 1], s[:, 1, 2], s[:, 2, 2]], 1)
        v = vm.detach()
        gw, gt = out["g_view"][:, :3], out["g_view"][:, 3]
        a = gw @ v[:, :3].T + gt[:, None] * v[:, 3][None]
        out["g_pose"] = torch.cat([gt, torch.stack([a[2, 1] - a[1, 2], a[0, 2] - a[2, 0], a[1, 0] - a[0, 1]])])
    return out


def _pose_step(view, g, m, v, lr, it):
    """Adam on the left tangent, then the retraction, in float64."""
    m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
    step = -lr * (m / (1 - 0.9 ** it)) / (torch.sqrt(v / (1 - 0.999 ** it)) + 1e-8)
    gen = torch.zeros(4, 4, dtype=torch.float64, device=view.device)
    gen[:3, 3] = step[:3]
    gen[0, 1], gen[0, 2], gen[1, 2] = -step[5], step[4], -step[3]
    gen[:3, :3] = gen[:3, :3] - gen[:3, :3].T
    full = torch.cat([view, torch.tensor([[0.0, 0.0, 0.0, 1.0]], dtype=torch.float64, device=view.device)])
    return (torch.linalg.matrix_exp(gen) @ full)[:3], m, v


def _adam_step(P, grads):
    """The first Adam step of every parameter tensor in float64."""
    P = [t.double() for t in P]
    m, v = [0.1 * g for g in grads], [0.001 * g * g for g in grads]
    new = [p - lr * g / (g.abs() + 1e-15) for p, g, lr in zip(P, grads, LRS)]
    return new, m, v


def _mask64(last_T, j):
    """One pixel per block of 2^ceil(j/2) x 2^floor(j/2): the least transmittance, first wins."""
    bw, bh = 1 << ((j + 1) // 2), 1 << (j // 2)
    h, w = last_T.shape
    H, W = -(-h // bh) * bh, -(-w // bw) * bw
    pad = torch.full((H, W), float("inf"), dtype=last_T.dtype, device=last_T.device)
    pad[:h, :w] = last_T
    blocks = pad.reshape(H // bh, bh, W // bw, bw).permute(0, 2, 1, 3).reshape(H // bh, W // bw, bh * bw)
    low = blocks.min(dim=2, keepdim=True).values
    first = (blocks == low).to(torch.uint8).argmax(dim=2)
    hot = torch.nn.functional.one_hot(first, bh * bw).reshape(H // bh, W // bw, bh, bw)
    return hot.permute(0, 2, 1, 3).reshape(H, W)[:h, :w].bool()


def exact(case, seed):
    kind = case["kind"]
    if kind == "prune":
        return None                               # bytes and whole numbers alone
    if kind.startswith("serve"):
        return _exact_serve(case, seed)
    w, h, n = case["w"], case["h"], case["n"]
    s = _inputs(w, h, n, seed)
    cam = s["cam"]
    if kind == "autograd":
        r = _frame64(s["scene"], s["view"], cam, grad_of=_upstream_of(_upstream(w, h, s["g"])))
        return dict(color=r["color"], depth=r["depth"], alpha=1.0 - r["T"], visible=None, grads=r["grads"], g_view=r["g_view"])
    if kind == "render":
        r = _frame64(s["scene"], s["view"], cam)
        return dict(color=r["color"], depth=r["depth"], alpha=1.0 - r["T"], visible=None)
    if kind == "track":
        view, lists = s["view"].double(), None
        m = v = torch.zeros(6, dtype=torch.float64, device=DEV)
        for it in range(1, case["iters"] + 1):
            r = _frame64(s["scene"], view, cam, grad_of=_l1_of(s["target"], w * h), lists=lists)
            lists = r["lists"]
            view, m, v = _pose_step(view, r["g_pose"], m, v, 1e-3, it)
        return dict(color=r["color"], depth=r["depth"], final_T=r["T"], last_idx=None, g_pose=r["g_pose"],
                    g_view=r["g_view"], view=view)
    if kind == "down":
        mask = _mask64(_last_T(w, h, s["g"]), case["j"])
        r = _frame64(s["scene"], s["view"], cam, mask=mask, grad_of=_l1_of(s["target"], int(mask.sum())))
        zero = torch.zeros(6, dtype=torch.float64, device=DEV)
        view = _pose_step(s["view"].double(), r["g_pose"], zero, zero, 1e-3, 1)[0]
        return dict(mask=None, count=None, color=r["color"], depth=r["depth"], final_T=r["T"], g_pose=r["g_pose"], view=view)
    r = _frame64(s["scene"], s["view"], cam, grad_of=_l1_of(s["target"], w * h), cov=kind == "score")
    new, m, v = _adam_step(s["scene"], r["grads"])
    if kind == "map":
        return dict(color=r["color"], depth=r["depth"], final_T=r["T"], last_idx=None, params=new, m=m, v=v)
    return dict(color=r["color"], depth=r["depth"], final_T=r["T"], grads=r["grads"], g_cov=r["g_cov"], g_pose=r["g_pose"],
                params=new, m=m, v=v)


def _exact_serve(case, seed):
    images, poses, views, maps = [], [], [], []
    zero = torch.zeros(6, dtype=torch.float64, device=DEV)
    lr = torch.tensor([1e-3] * 3 + [3e-3] * 3, dtype=torch.float64, device=DEV)
    for i, (w, h, n, j) in enumerate(_classes(case)):
        s = _inputs(w, h, n, seed, salt=17 * (i + 1))
        if case["kind"] == "serve_track":
            mask = _mask64(_last_T(w, h, s["g"]), j) if j else None
            act = int(mask.sum()) if j else w * h
            r = _frame64(s["scene"], s["view"], s["cam"], mask=mask, grad_of=_l1_of(s["target"], act))
            images.append([r["color"], r["depth"], r["T"], None])
            poses.append(r["g_pose"])
            views.append(_pose_step(s["view"].double(), r["g_pose"], zero, zero, lr, 1)[0].reshape(-1))
        else:
            r = _frame64(s["scene"], s["view"], s["cam"], grad_of=_l1_of(s["target"], w * h))
            images.append([r["color"], r["depth"]])
            maps.append(list(_adam_step(s["scene"], r["grads"])))
    if case["kind"] == "serve_track":
        return dict(images=images, g_pose=torch.stack(poses), view=torch.stack(views))
    return dict(images=images, maps=maps)
