"""The work that a user of this framework has it do, as timed cases.

A case is a dict of plain values.  ``prepare`` makes what a training program
holds before the call (seeded inputs, contexts, indices, captured graphs),
``run`` is one pass through the public entry points, ``work`` counts the bytes
and operations the pass cannot do without, and ``exact`` computes its outputs
again with plain torch in 64 bits.  ``listed`` names the cases; ``draw`` takes
others from the same ranges.

Kinds:
  view    render a batch of views, no gradients (evaluation, a viewer)
  train   render and backward through autograd, pose twists included
  joint   one whole iteration: JointStep.run, eager or as a captured graph
  photo   the photometric loss and its image gradient
  track   the track reprojection loss and its gradients through autograd
  ba      one Levenberg-Marquardt step of bundle adjustment
  init    Gaussians from SfM points
  mcmc    relocation of the dead Gaussians, then noise on the means
"""

import math

import numpy as np
import torch

from paper_2603_04847_amd import _lib as L
from paper_2603_04847_amd import splat
from paper_2603_04847_amd.step import PARAM_KEYS, JointStep

DEV = "cuda"
MAX_LISTS = 2 ** 30 - 65536      # the largest list capacity a context takes
FX_PER_W = 300.0 / 256.0         # focal length per pixel of width
# the view sizes of an uneven batch, as shares of the largest view
UNEVEN = (0.4, 0.5, 0.6, 0.64, 0.7731, 0.8, 0.9, 1.0)
TILES = ((16, 16), (16, 8), (8, 8), (32, 16))
DELTA, LAM, NEAR = 1.0, 1e-4, 0.01

_RENDER = dict(views=1, uneven=False, w=256, h=256, n=10_000, sh=0, scene="frustum", tile=0,
               order=0, bg=False)


def _render(kind, **over):
    return dict(_RENDER, kind=kind, **over)


def listed():
    return [
        # the smallest training call: one 256x256 crop, 10k flat-coloured
        # splats, eager autograd; launches and host calls are all of it
        _render("train", name="train_tiny"),
        # a frame of a trained scene at the resolution of the photo sets, for
        # evaluation or a viewer: forward only
        _render("view", name="view_1m", w=1237, h=822, n=1_000_000, sh=3),
        # a batch of eight cameras of unlike resolution around 3M splats whose
        # tile loads differ a hundredfold
        _render("train", name="train_uneven", views=8, uneven=True, w=1600, h=1066, n=3_000_000,
                sh=3, scene="blobs_uneven", order=2),
        # a whole iteration on a small scene, replayed as a captured graph:
        # short dependent kernels back to back
        _render("joint", name="joint_small", n=10_000, scene="blobs", cams=5, points=500,
                max_len=5, graph=True),
        # a whole iteration on an ordinary scene (150 photographs)
        _render("joint", name="joint_150", views=4, w=1237, h=822, n=1_000_000, sh=3,
                scene="blobs", order=1, cams=150, points=100_000, max_len=12, graph=False),
        # a whole iteration on a large scene (1000 photographs, 5M splats):
        # the benchmark's workload
        _render("joint", name="joint_1000", views=4, w=1600, h=1066, n=5_000_000, sh=3,
                scene="blobs", tile=3, cams=1000, points=1_500_000, max_len=30, graph=False),
        # the image loss alone, on odd-sized views, as a trainer with its own
        # renderer settings or an evaluation of SSIM calls it
        dict(name="photo_odd", kind="photo", views=4, uneven=True, w=979, h=545, ssim=0.2),
        # the reprojection term alone through autograd (pose refinement with
        # the Gaussians frozen)
        dict(name="track_150", kind="track", cams=150, points=100_000, max_len=12, w=1237, h=822),
        # bundle adjustment of an ordinary and of a large reconstruction
        dict(name="ba_150", kind="ba", cams=150, points=100_000, max_len=12, w=1237, h=822),
        dict(name="ba_1000", kind="ba", cams=1000, points=1_500_000, max_len=30, w=1600, h=1066),
        # the densification step of a large scene, a fifth of the splats dead
        dict(name="mcmc_5m", kind="mcmc", n=5_000_000, sh=3, dead=0.2),
        # the start of a training run: splats from the SfM points of a large
        # scene
        dict(name="init_1500k", kind="init", n=1_500_000, sh=3, k=4),
    ]


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(("view", "train", "train", "joint", "joint", "photo", "track", "ba", "init",
                       "mcmc"))
    if kind in ("view", "train", "joint"):
        views = rng.choice((1, 1, 2, 3, 4) if kind == "joint" else (1, 1, 2, 4, 6, 8))
        w = rng.randint(160, 1600)
        h = max(120, int(w * rng.uniform(0.56, 0.8)))
        n = log(8_000, min(4_000_000, 18_000_000 // views))
        tile = rng.choice((0, 0, 3, 3, 1, 2))
        if tile in (1, 2):  # the small tiles are for small images
            w, h, n = min(w, 640 + w % 97), min(h, 480 + h % 31), min(n, 400_000)
        c = _render(kind, views=views, uneven=views > 1 and rng.random() < 0.5, w=w, h=h, n=n,
                    sh=rng.choice((0, 1, 2, 3, 3, 3)), tile=tile, order=rng.choice((0, 1, 2)),
                    scene="frustum" if views == 1 and kind != "joint" else
                    rng.choice(("blobs", "blobs", "blobs_uneven")),
                    bg=kind != "joint" and rng.random() < 0.3)
        if kind == "joint":
            cams = log(max(5, views), 1000)
            c.update(cams=cams, points=log(300, 1000 * cams), max_len=rng.randint(3, 30),
                     graph=rng.random() < 0.3)
        return c
    if kind == "photo":
        w = rng.randint(64, 1600)
        return dict(kind=kind, views=rng.choice((1, 2, 4)), uneven=rng.random() < 0.5, w=w,
                    h=max(48, int(w * rng.uniform(0.5, 0.8))), ssim=rng.choice((0.2, 0.2, 1.0)))
    if kind in ("track", "ba"):
        cams = log(5, 1000)
        return dict(kind=kind, cams=cams, points=log(300, 1200 * cams), max_len=rng.randint(3, 30),
                    w=1237, h=822)
    if kind == "init":
        return dict(kind=kind, n=log(1_000, 1_200_000), sh=rng.choice((0, 3)),
                    k=rng.choice((3, 4, 4)))
    return dict(kind="mcmc", n=log(10_000, 4_000_000), sh=rng.choice((0, 2, 3)),
                dead=round(rng.uniform(0.02, 0.3), 3))


# ---------------------------------------------------------------- inputs

class _Draws:
    """One seed's random numbers: large arrays on the GPU, small ones in numpy."""

    def __init__(self, seed):
        self.gen = torch.Generator(DEV).manual_seed(int(seed) % (1 << 62))
        self.np = np.random.Generator(np.random.PCG64(int(seed) % (1 << 62)))

    def normal(self, *shape, mu=0.0, sd=1.0):
        return torch.randn(shape, device=DEV, generator=self.gen).mul_(sd).add_(mu)

    def uniform(self, *shape):
        return torch.rand(shape, device=DEV, generator=self.gen)


def _sizes(case):
    if not case["uneven"]:
        return [(case["w"], case["h"])] * case["views"]
    share = [UNEVEN[(len(UNEVEN) - case["views"] + v) % len(UNEVEN)] for v in range(case["views"])]
    return [(max(32, int(case["w"] * s)), max(32, int(case["h"] * s))) for s in share]


def _look_at(centre, up):
    """World-to-camera [R|t] of a camera at `centre` looking at the origin."""
    f = -centre / np.linalg.norm(centre)
    r = np.cross(f, up)
    r /= np.linalg.norm(r)
    R = np.stack([r, np.cross(f, r), f])
    return np.concatenate([R, -(R @ centre)[:, None]], 1)


def _sphere_cameras(d, sizes):
    vm, intr = [], []
    for w, h in sizes:
        while True:
            c = d.np.normal(size=3)
            c *= 4.0 / np.linalg.norm(c)
            if abs(c[2]) < 3.8:
                break
        vm.append(_look_at(c, np.array([0.0, 0.0, 1.0])).reshape(12))
        intr.append([FX_PER_W * w, FX_PER_W * w, w / 2.0, h / 2.0])
    f = lambda a: torch.tensor(np.array(a), device=DEV, dtype=torch.float32)
    return f(vm), f(intr)


def _blob_points(d, n, dirichlet=0.3, blobs=50):
    c = d.np.normal(size=(blobs, 3))
    c *= 1.5 * d.np.uniform(size=(blobs, 1)) ** (1 / 3) / np.linalg.norm(c, axis=1, keepdims=True)
    sig = np.exp(d.np.uniform(np.log(0.02), np.log(0.4), blobs))
    share = np.cumsum(d.np.dirichlet(np.full(blobs, dirichlet)))
    f = lambda a: torch.tensor(a, device=DEV, dtype=torch.float32)
    of = torch.searchsorted(f(share), d.uniform(n)).clamp_(max=blobs - 1)
    return f(c)[of] + f(sig)[of, None] * d.normal(n, 3)


def _gaussians(d, case, means):
    n, K = means.shape[0], (case["sh"] + 1) ** 2
    small = n <= 20_000  # few splats have to be large to cover the image
    sh = d.normal(K, 3, n, sd=0.1)
    if K == 1:
        sh[0] = (d.uniform(3, n) * 2 - 1) * math.sqrt(math.pi)
    return dict(means=means.t().contiguous(),
                log_scales=d.normal(3, n, mu=-3.0 if small else -4.0, sd=0.5 if small else 0.7),
                quats=d.normal(4, n), opacity_logit=d.normal(n), sh=sh)


def _scene(d, case, sizes):
    """Gaussians and one camera for each size."""
    if case["scene"] == "frustum":
        w, h = sizes[0]
        f = FX_PER_W * w
        R = _look_at(d.np.normal(size=3), np.array([0.0, 0.0, 1.0]))[:, :3]
        t = d.np.normal(size=3)
        z = (8.0 + (216.0 - 8.0) * d.uniform(case["n"])) ** (1 / 3)  # depth 2 to 6
        p = torch.stack([(d.uniform(case["n"]) - 0.5) * w / f * z,
                         (d.uniform(case["n"]) - 0.5) * h / f * z, z], 1)
        tt = lambda a: torch.tensor(a, device=DEV, dtype=torch.float32)
        means = (p - tt(t)) @ tt(R)
        vm = tt(np.concatenate([R, t[:, None]], 1).reshape(1, 12))
        return _gaussians(d, case, means), vm, tt([[f, f, w / 2.0, h / 2.0]])
    means = _blob_points(d, case["n"], 0.05 if case["scene"] == "blobs_uneven" else 0.3)
    g = _gaussians(d, case, means)
    return (g, *_sphere_cameras(d, sizes))


def _images(d, sizes):
    """Smooth images with fine detail, values in [0, 1], views packed."""
    out = []
    for w, h in sizes:
        low = d.uniform(1, 3, 2 + h // 48, 2 + w // 48)
        low = torch.nn.functional.interpolate(low, size=(h, w), mode="bilinear",
                                              align_corners=False)
        x = (low[0].permute(1, 2, 0) + d.normal(h, w, 3, sd=0.05)).clamp_(0.0, 1.0)
        out.append(x.reshape(-1, 3))
    return torch.cat(out).contiguous()


def _tracks(d, case, vm, intr, wh):
    """Track points seen by 2 and more cameras (or, out of every view, by
    none), pixels off by N(0, 1)."""
    C, n = vm.shape[0], case["points"]
    X = _blob_points(d, n)
    M = vm.view(C, 3, 4)
    want = 1 + torch.ceil(torch.log(d.uniform(n).clamp_(min=1e-9)) / math.log(0.7)).clamp_(1, 200)
    want = want.clamp_(max=case["max_len"])
    nc = min(C, 64)
    cams, pts, xys = [], [], []
    for s in range(0, n, 1 << 17):
        x = X[s:s + (1 << 17)]
        m = x.shape[0]
        cand = (d.uniform(m, nc) * C).long().clamp_(max=C - 1) if C > 64 else \
            torch.arange(C, device=DEV).expand(m, C)
        cand = cand.sort(1).values
        T = M[cand]
        p = (T[..., :3] * x[:, None, None, :]).sum(-1) + T[..., 3]
        uv = p[..., :2] / p[..., 2:] * intr[cand][..., :2] + intr[cand][..., 2:]
        see = (p[..., 2] > 0.1) & (uv >= 0).all(-1) & (uv < wh[cand]).all(-1)
        see[:, 1:] &= cand[:, 1:] != cand[:, :-1]
        key = d.uniform(m, nc).masked_fill_(~see, 2.0)
        rank = key.argsort(1).argsort(1)
        take = see & (rank < want[s:s + m, None]) & (see.sum(1, keepdim=True) >= 2)
        i, j = take.nonzero(as_tuple=True)
        cams.append(cand[i, j])
        pts.append(i + s)
        xys.append(uv[i, j])
    cam, pt, xy = torch.cat(cams), torch.cat(pts), torch.cat(xys)
    order = torch.argsort(cam * n + pt)
    xy = xy + d.normal(*xy.shape)
    return dict(X=X.contiguous(), obs_cam=cam[order].int(), obs_pt=pt[order].int(),
                obs_xy=xy[order].contiguous())


def _perturbed(d, vm):
    """Poses moved by about 0.002 rad and 0.005 units."""
    tw = torch.cat([d.normal(vm.shape[0], 3, sd=0.005), d.normal(vm.shape[0], 3, sd=0.002)], 1)
    return _moved(tw.double(), vm.double()).float().contiguous()


def _track_scene(case, seed):
    d = _Draws(seed)
    vm, intr = _sphere_cameras(d, [(case["w"], case["h"])] * case["cams"])
    wh = torch.tensor([[case["w"], case["h"]]] * case["cams"], device=DEV)
    sc = _tracks(d, case, vm, intr, wh)
    sc.update(viewmat=_perturbed(d, vm), intr=intr)
    return d, sc


def _render_inputs(case, seed):
    d = _Draws(seed)
    sizes = _sizes(case)
    params, vm, intr = _scene(d, case, sizes)
    P = sum(w * h for w, h in sizes)
    x = dict(params=params, base=vm, intr=intr, wh=np.array(sizes, np.int32),
             twist=d.normal(len(sizes), 6, sd=0.003), v_rgb=d.normal(P, 3, sd=1.0 / P))
    if case["bg"]:
        x["bg"] = d.uniform(3)
    return x


def _joint_scene(case, seed):
    """The scene dict JointStep takes (host arrays), a batch and its targets."""
    d = _Draws(seed)
    sizes = _sizes(case) + [(case["w"], case["h"])] * (case["cams"] - case["views"])
    params, vm, intr = _scene(d, case, sizes)
    sc = _tracks(d, case, vm, intr, torch.tensor(sizes, device=DEV))
    sc.update(params, viewmat=_perturbed(d, vm), intr=intr)
    targets = _images(d, sizes[:case["views"]])
    sc = {k: v.cpu().numpy() for k, v in sc.items()}
    sc.update(sh_degree=case["sh"], wh=np.array(sizes, np.int32))
    return sc, np.arange(case["views"], dtype=np.int32), targets.cpu().numpy()


# ---------------------------------------------------------------- passes

def _settings(case, **over):
    tw, th = TILES[case["tile"]]
    return L.default_settings(tile_w=tw, tile_h=th, tile_order=case["order"], **over)


def _lists_needed(first, probe):
    """List entries a scene needs: probe(capacity) -> status, as a program
    sizes its context from a first pass."""
    cap = int(min(first, MAX_LISTS))
    while True:
        st = probe(cap)
        if not st["flags"] & L.GS_FLAG_ISECT_OVERFLOW:
            return min(MAX_LISTS, int(st["n_isect_needed"] * 1.15) + 4096)
        if cap == MAX_LISTS:
            raise RuntimeError("the lists of this scene do not fit a context")
        cap = min(MAX_LISTS, max(2 * cap, int(1.2 * st["n_isect_needed"])))


def prepare(case, seed):
    return globals()["_prepare_" + case["kind"]](case, seed)


def run(state):
    return globals()["_run_" + state["kind"]](state)


def _prepare_view(case, seed):
    x = _render_inputs(case, seed)
    s = _settings(case, lazy_lists=1)
    V, n = len(x["wh"]), case["n"]
    tw, th = TILES[case["tile"]]
    tiles = int(sum(-(-int(w) // tw) * -(-int(h) // th) for w, h in x["wh"]))
    vm = torch.empty_like(x["base"])
    L.gs_pose_compose(x["twist"], x["base"], vm)
    cams = L.Cameras(vm, x["intr"], x["wh"])
    g = L.make_gaussians(*(x["params"][k] for k in PARAM_KEYS), case["sh"])

    def context(cap):
        return L.Context(max_pairs=V * n, max_isect=cap, max_tiles=tiles, max_views=V)

    def probe(cap):
        ctx = context(cap)
        L.gs_project(ctx, g, cams, s)
        L.gs_bin_sort(ctx, cams, n, s)
        st = ctx.status()
        ctx.close()
        return st

    cap = _lists_needed(24 * cams.n_pixels + 65536, probe)
    x.update(kind=case["kind"], sh=case["sh"], viewmat=vm,
             splatter=splat.Splatter(context(cap), s, x.get("bg")))
    return x


def _run_view(x):
    return x["splatter"].forward(x["params"], x["sh"], x["viewmat"], x["intr"], x["wh"])[:3]


def _prepare_train(case, seed):
    x = _prepare_view(case, seed)
    for t in (*x["params"].values(), x["twist"]):
        t.requires_grad_(True)
    return x


def _run_train(x):
    rgb = splat.rasterize(x["params"], x["sh"], x["twist"], x["base"], x["intr"], x["wh"],
                          x["splatter"])
    inputs = (*(x["params"][k] for k in PARAM_KEYS), x["twist"])
    return rgb, torch.autograd.grad(rgb, inputs, x["v_rgb"])


def _prepare_joint(case, seed):
    sc, batch, targets = _joint_scene(case, seed)
    P = targets.shape[0]
    js = JointStep(sc, [batch], [targets], settings=_settings(case), max_isect=min(MAX_LISTS, 48 * P))

    def probe(cap):
        if cap != js.ctx.cap.max_isect:
            js.set_capacity(cap)
        js.forward_backward(0)
        return js.ctx.status()

    js.set_capacity(_lists_needed(48 * P, probe))
    # the end of the learning-rate schedule: a pass leaves the scene as it
    # was, however many passes follow
    js.lr = {k: 0.005 * v for k, v in js.lr.items()}
    x = dict(kind="joint", js=js)
    if case["graph"]:
        start = {k: v.clone() for k, v in js._opt_params().items()}
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            js.run(0)
        torch.cuda.current_stream().wait_stream(side)
        torch.cuda.synchronize()
        x["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(x["graph"]):
            js.run(0)
        for k, p in js._opt_params().items():
            p.copy_(start[k])
            js.m[k].zero_()
            js.v[k].zero_()
        js.set_step(0)
    return x


def _run_joint(x):
    js = x["js"]
    if "graph" in x:
        x["graph"].replay()
    else:
        js.run(0)
    return dict(rgb=js.rgb, loss=js.loss, v_twist=js.v_tw, v_X=js.v_X, exp_avg=js.m,
                params=js._opt_params())


def _prepare_photo(case, seed):
    d = _Draws(seed)
    sizes = _sizes(case)
    target = _images(d, sizes)
    rgb = (target + d.normal(*target.shape, sd=0.05)).clamp_(min=0.0)
    one = torch.zeros((len(sizes), 12), device=DEV)
    return dict(kind="photo", ssim=case["ssim"], rgb=rgb, target=target,
                ctx=L.Context(max_pairs=1, max_isect=1, max_tiles=1, max_views=len(sizes)),
                cams=L.Cameras(one, one[:, :4].contiguous(), np.array(sizes, np.int32)),
                v_rgb=torch.empty_like(rgb), loss=torch.zeros(1, device=DEV))


def _run_photo(x):
    x["loss"].zero_()
    L.gs_photo_loss_grad(x["ctx"], x["cams"], x["rgb"], x["target"], x["ssim"], x["v_rgb"],
                         x["loss"])
    return x["loss"], x["v_rgb"]


def _prepare_track(case, seed):
    d, x = _track_scene(case, seed)
    x.update(kind="track", twist=d.normal(case["cams"], 6, sd=0.002).requires_grad_(True),
             ctx=L.Context(max_pairs=1, max_isect=1, max_tiles=1, max_views=1,
                           max_cams=case["cams"]))
    x["X"].requires_grad_(True)
    return x


def _run_track(x):
    loss = splat.track_loss(x["X"], x["twist"], x["viewmat"], x["intr"], x["obs_cam"], x["obs_pt"],
                            x["obs_xy"], x["ctx"], DELTA, LAM)
    return loss, torch.autograd.grad(loss, (x["X"], x["twist"]))


def _prepare_ba(case, seed):
    _, x = _track_scene(case, seed)
    Pt, C = x["X"].shape[0], case["cams"]
    ctx = L.Context(max_pairs=Pt + 1, max_isect=1024, max_tiles=16, max_views=1, max_cams=C)
    x["index"] = L.track_point_index(ctx, x["obs_pt"], Pt, x["obs_cam"], x["obs_xy"])
    torch.cuda.synchronize()
    ctx.close()
    x.update(kind="ba", ba=L.BundleAdjuster(Pt, C), d_twist=torch.empty((C, 6), device=DEV),
             d_X=torch.empty((Pt, 3), device=DEV), stats=torch.zeros(5, device=DEV))
    return x


def _run_ba(x):
    L.gs_ba_lm_step(x["ba"], x["X"], x["viewmat"], x["intr"], x["obs_cam"], x["obs_pt"],
                    x["obs_xy"], x["index"], DELTA, 1e-2, NEAR, 100, 1e-8, x["d_twist"], x["d_X"],
                    x["stats"])
    return x["d_twist"], x["d_X"], x["stats"]


def _prepare_init(case, seed):
    d = _Draws(seed)
    return dict(kind="init", points=_blob_points(d, case["n"]), rgb=d.uniform(case["n"], 3),
                sh=case["sh"], k=case["k"],
                ctx=L.Context(max_pairs=case["n"], max_isect=1024, max_tiles=16, max_views=1))


def _run_init(x):
    return L.gs_init_gaussians(x["ctx"], x["points"], x["rgb"], x["sh"], x["k"])


def _prepare_mcmc(case, seed):
    d = _Draws(seed)
    n = case["n"]
    g = _gaussians(d, case, _blob_points(d, n))
    g["opacity_logit"][d.uniform(n) < case["dead"]] = -9.0
    p = [g[k] for k in PARAM_KEYS]
    return dict(kind="mcmc", sh=case["sh"], params=p, m=[torch.full_like(t, 1e-3) for t in p],
                v=[torch.full_like(t, 1e-6) for t in p], u=d.uniform(n), eta=d.normal(3, n),
                logit=p[3].clone(), scales=p[1].clone(),
                src=torch.empty(n, dtype=torch.int32, device=DEV),
                moved=torch.zeros(1, dtype=torch.int32, device=DEV),
                ctx=L.Context(max_pairs=n, max_isect=1024, max_tiles=16, max_views=1))


def _run_mcmc(x):
    # what the iterations between two relocations do to the splats: some of
    # them die, and the sources grow back
    x["params"][3].copy_(x["logit"])
    x["params"][1].copy_(x["scales"])
    L.gs_mcmc_relocate(x["ctx"], x["params"], x["m"], x["v"], x["sh"], x["u"], src=x["src"],
                       n_relocated=x["moved"])
    means, log_scales, quats, logit, _ = x["params"]
    L.gs_mcmc_noise(means, log_scales, quats, logit, x["eta"], 1e-6)
    return dict(zip(PARAM_KEYS, x["params"])), x["m"], x["v"], x["src"], x["moved"]


# ---------------------------------------------------------------- work

def _obs(case):
    """Observations of a case's tracks: 2 + Geom(0.3) of each, some capped."""
    return case["points"] * min(4.3, case["max_len"] - 0.5)


def work(case):
    """Inputs read once and outputs written once; operations of the steps whose
    number the sizes fix (projection per pair, a chain per pixel or
    observation), not the compositing, which depends on the scene."""
    k = case["kind"]
    if k in ("view", "train", "joint"):
        P = sum(w * h for w, h in _sizes(case))
        V, n, K = case["views"], case["n"], (case["sh"] + 1) ** 2
        gauss = n * (44 + 12 * K)
        bytes_, flops = gauss + 20 * P, V * n * (150 + 6 * K) + 24 * P
        if k == "train":
            bytes_, flops = bytes_ + gauss + 12 * P, 3 * flops
        if k == "joint":
            M = _obs(case)
            bytes_ += 5 * gauss + 24 * P + 28 * M + 7 * 12 * case["points"]
            flops = 3 * flops + 600 * P + n * (11 + 3 * K) * 12 + 120 * M
        return dict(bytes=bytes_, flops=flops)
    if k == "photo":
        P = sum(w * h for w, h in _sizes(case))
        return dict(bytes=36 * P, flops=600 * P)
    if k in ("track", "ba"):
        M, C, n = _obs(case), case["cams"], case["points"]
        if k == "track":
            return dict(bytes=16 * M + 24 * n + 112 * C, flops=120 * M)
        return dict(bytes=16 * M + 28 * n + 88 * C, flops=20 * 200 * M)
    K = (case["sh"] + 1) ** 2
    if k == "init":
        return dict(bytes=case["n"] * (24 + 44 + 12 * K), flops=case["n"] * 1000)
    # the dead are rewritten (parameters and moments), sources read; the noise
    # reads the geometry and writes the means
    row = 44 + 12 * K
    n = case["n"]
    return dict(bytes=n * (8 + 68) + case["dead"] * n * 4 * row, flops=100 * n)


# ------------------------------------------------------- the same in 64 bits

def exact(case, seed):
    f = globals().get("_exact_" + case["kind"])
    return None if f is None else f(case, seed)


def _moved(twist, base):
    """Exp(twist) base of [V,6] left twists and [V,12] poses, in 64 bits."""
    rho, phi = twist[:, :3], twist[:, 3:]
    A = torch.zeros((len(twist), 4, 4), device=twist.device, dtype=torch.float64)
    z = torch.zeros_like(phi[:, 0])
    hat = torch.stack([z, -phi[:, 2], phi[:, 1], phi[:, 2], z, -phi[:, 0], -phi[:, 1], phi[:, 0],
                       z], 1).view(-1, 3, 3)
    A = torch.cat([torch.cat([hat, rho[:, :, None]], 2), A[:, :1]], 1)
    T = base.view(-1, 3, 4)
    E = torch.linalg.matrix_exp(A)
    R = E[:, :3, :3] @ T[:, :, :3]
    t = (E[:, :3, :3] @ T[:, :, 3:]) + E[:, :3, 3:]
    return torch.cat([R, t], 2).reshape(-1, 12)


def _sh_basis(deg, d):
    """Real spherical harmonics (Condon-Shortley phase), m = -l..l, [K, n]."""
    x, y, z = d
    pi = math.pi
    Y = [torch.full_like(x, 0.5 / math.sqrt(pi))]
    if deg > 0:
        a = math.sqrt(3 / (4 * pi))
        Y += [-a * y, a * z, -a * x]
    if deg > 1:
        a = math.sqrt(15 / pi) / 2
        Y += [a * x * y, -a * y * z, math.sqrt(5 / pi) / 4 * (3 * z * z - 1), -a * x * z,
              a / 2 * (x * x - y * y)]
    if deg > 2:
        a, b, c = math.sqrt(35 / (2 * pi)) / 4, math.sqrt(105 / pi) / 2, math.sqrt(21 / (2 * pi)) / 4
        Y += [-a * y * (3 * x * x - y * y), b * x * y * z, -c * y * (5 * z * z - 1),
              math.sqrt(7 / pi) / 4 * z * (5 * z * z - 3), -c * x * (5 * z * z - 1),
              b / 2 * z * (x * x - y * y), -a * x * (x * x - 3 * y * y)]
    return torch.stack(Y)


def _exact_project(p, deg, vm, intr, wh, alpha_min):
    """One view of 64-bit parameters: mean2d [2,n], conic [3,n], opacity,
    colour [3,n], depth, 2D covariance [3,n], the seen ones."""
    T = vm.view(3, 4)
    R, t = T[:, :3], T[:, 3]
    (fx, fy, cx, cy), (W, H) = intr, (float(wh[0]), float(wh[1]))
    c = R @ p["means"] + t[:, None]
    seen = c[2] >= NEAR
    z = torch.where(seen, c[2], torch.ones_like(c[2]))
    x, y = c[0] / z, c[1] / z
    tx = torch.minimum(torch.maximum(x, -(cx / fx + 0.15 * W / fx)), (W - cx) / fx + 0.15 * W / fx)
    ty = torch.minimum(torch.maximum(y, -(cy / fy + 0.15 * H / fy)), (H - cy) / fy + 0.15 * H / fy)
    q = p["quats"] / p["quats"].norm(dim=0)
    w, a, b, e = q
    Q = torch.stack([1 - 2 * (b * b + e * e), 2 * (a * b - w * e), 2 * (a * e + w * b),
                     2 * (a * b + w * e), 1 - 2 * (a * a + e * e), 2 * (b * e - w * a),
                     2 * (a * e - w * b), 2 * (b * e + w * a), 1 - 2 * (a * a + b * b)]).view(3, 3, -1)
    M = (R @ Q.reshape(3, -1)).view(3, 3, -1) * p["log_scales"].exp()[None]
    u = fx / z * (M[0] - tx * M[2])
    v = fy / z * (M[1] - ty * M[2])
    A, B, C = (u * u).sum(0) + 0.3, (u * v).sum(0), (v * v).sum(0) + 0.3
    # |u x v|^2 + 0.3 (|u|^2 + |v|^2) + 0.09: no cancellation for needles
    det = torch.linalg.cross(u, v, dim=0).square().sum(0) + 0.3 * (A + C) - 0.09
    op = torch.sigmoid(p["opacity_logit"])
    d = p["means"] + (R.t() @ t)[:, None]
    Y = _sh_basis(deg, d / d.norm(dim=0))
    rgb = torch.clamp((Y[:, None] * p["sh"]).sum(0) + 0.5, min=0.0)
    return (torch.stack([fx * x + cx, fy * y + cy]), torch.stack([C, -B, A]) / det, op, rgb, c[2],
            torch.stack([A, B, C]), seen & (op > alpha_min))


def _exact_block(g, order, px, py, bg, s):
    """Composite the splats `order` (front to back) over the pixels (px, py)."""
    m2, con, op, col = (g[k][..., order] for k in ("mean2d", "conic", "opacity", "rgb"))
    dx, dy = m2[0] - px[:, None], m2[1] - py[:, None]
    sig = 0.5 * (con[0] * dx * dx + con[2] * dy * dy) + con[1] * dx * dy
    a = torch.clamp(op * torch.exp(-sig), max=s.alpha_max)
    a = torch.where(a >= s.alpha_min, a, torch.zeros_like(a))
    inc = torch.cumprod(1 - a, 1)
    live = (inc >= s.t_min).double()
    exc = torch.cat([torch.ones_like(inc[:, :1]), inc[:, :-1]], 1)
    T = torch.where(live > 0, 1 - a, torch.ones_like(a)).prod(1) if order.numel() else \
        torch.ones_like(px)
    rgb = (a * exc * live) @ col.t()
    return rgb + T[:, None] * bg if bg is not None else rgb, T, live


def _exact_render(params, deg, vm, intr, wh, bg=None, v_rgb=None, v_of=None):
    """Images [P,3] and T [P] of 64-bit leaves; with v_rgb (or v_of(images))
    also backpropagates into the leaves.  Pixel blocks of 32 x 32, each over
    the splats whose alpha >= alpha_min ellipse reaches it, in pieces until
    every pixel has stopped."""
    s = L.default_settings()
    views, images, trans = [], [], []
    grad = v_rgb is not None or v_of is not None
    for v in range(len(wh)):
        out = _exact_project(params, deg, vm[v], intr[v].double(), wh[v], s.alpha_min)
        m2, con, op, rgb, depth, cov, seen = out
        with torch.no_grad():
            r = torch.sqrt(2 * torch.log((op / s.alpha_min).clamp(min=1.0)) * cov[::2]) + 1e-6
            idx = seen.nonzero()[:, 0]
            idx = idx[torch.sort(depth[idx].float(), stable=True).indices]
            lo, hi = (m2 - r)[:, idx], (m2 + r)[:, idx]
        leaf = {k: t.detach().requires_grad_(grad) for k, t in
                zip(("mean2d", "conic", "opacity", "rgb"), (m2, con, op, rgb))}
        views.append(((m2, con, op, rgb), leaf, _blocks(leaf, idx, lo, hi, wh[v], bg, s)))
        img = torch.zeros((int(wh[v][0]) * int(wh[v][1]), 3), device=DEV, dtype=torch.float64)
        T = torch.zeros_like(img[:, 0])
        with torch.no_grad():
            for pix, px, py, order in views[-1][2]:
                img[pix], T[pix], _ = _exact_block(leaf, order, px, py, bg, s)
        images.append(img)
        trans.append(T)
    images, trans = torch.cat(images), torch.cat(trans)
    if not grad:
        return images, trans
    v_rgb = v_of(images) if v_of is not None else v_rgb.double()
    at = 0
    for outs, leaf, blocks in views:
        n = sum(len(b[0]) for b in blocks)
        part, at = v_rgb[at:at + n], at + n
        for pix, px, py, order in blocks:
            if order.numel():
                sub = {k: t.detach()[..., order].requires_grad_(True) for k, t in leaf.items()}
                every = torch.arange(order.numel(), device=DEV)
                img = _exact_block(sub, every, px, py, bg, s)[0]
                img.backward(part[pix])
                for k, t in leaf.items():
                    if t.grad is None:
                        t.grad = torch.zeros_like(t)
                    t.grad.index_add_(-1, order, sub[k].grad)
        torch.autograd.backward(outs, [torch.zeros_like(t) if t.grad is None else t.grad
                                       for t in leaf.values()], retain_graph=True)
    return images, trans


def _blocks(leaf, idx, lo, hi, wh, bg, s, side=32, piece=4096):
    """(pixels, x, y, splats up to the last one a pixel needs) of each block."""
    W, H = int(wh[0]), int(wh[1])
    out = []
    with torch.no_grad():
        for y0 in range(0, H, side):
            y1 = min(H, y0 + side)
            row = ((hi[1] >= y0 + 0.5) & (lo[1] <= y1 - 0.5)).nonzero()[:, 0]
            l, h, i = lo[0, row], hi[0, row], idx[row]
            for x0 in range(0, W, side):
                x1 = min(W, x0 + side)
                order = i[(h >= x0 + 0.5) & (l <= x1 - 0.5)]
                yy, xx = torch.meshgrid(torch.arange(y0, y1, device=DEV),
                                        torch.arange(x0, x1, device=DEV), indexing="ij")
                xx, yy = xx.reshape(-1), yy.reshape(-1)
                px, py = xx.double() + 0.5, yy.double() + 0.5
                if len(order) > piece:
                    T = torch.ones_like(px)
                    for k in range(0, len(order), piece):
                        _, t, live = _exact_block(leaf, order[k:k + piece], px, py, None, s)
                        T = torch.where(T < s.t_min, T, T * torch.where(live[:, -1] > 0, t, t * 0))
                        if bool((T < s.t_min).all()):
                            order = order[:k + piece]
                            break
                out.append((yy * W + xx, px, py, order))
    return out


def _cost(case):
    """Whether the 64-bit renderer is quick enough for a case."""
    P = sum(w * h for w, h in _sizes(case))
    return P * case["n"] <= 1.1e12 and case["scene"] == "frustum" or P * case["n"] <= 2e11


def _leaves(params):
    return {k: v.detach().double().requires_grad_(True) for k, v in params.items()}


def _exact_view(case, seed):
    if not _cost(case):
        return None
    x = _render_inputs(case, seed)
    bg = x["bg"].double() if "bg" in x else None
    vm = _moved(x["twist"].double(), x["base"].double())
    p = {k: v.double() for k, v in x["params"].items()}
    return (*_exact_render(p, case["sh"], vm, x["intr"], x["wh"], bg), None)


def _exact_train(case, seed):
    if not _cost(case):
        return None
    x = _render_inputs(case, seed)
    bg = x["bg"].double() if "bg" in x else None
    p = _leaves(x["params"])
    tw = x["twist"].double().requires_grad_(True)
    vm = _moved(tw, x["base"].double())
    rgb, _ = _exact_render(p, case["sh"], vm, x["intr"], x["wh"], bg, x["v_rgb"])
    return rgb, tuple([p[k].grad for k in PARAM_KEYS] + [tw.grad])


def _exact_photo_loss(rgb, target, wh, lam):
    """The loss of packed views, 64-bit tensors."""
    g = torch.exp(-0.5 * (torch.arange(11, device=DEV, dtype=torch.float64) - 5) ** 2 / 1.5 ** 2)
    g = g / g.sum()
    win = torch.outer(g, g)[None, None]
    loss, at = 0.0, 0
    for W, H in ((int(a), int(b)) for a, b in wh):
        x, y = (t[at:at + W * H].view(H, W, 3).permute(2, 0, 1)[:, None] for t in (rgb, target))
        at += W * H
        blur = lambda t: torch.nn.functional.conv2d(t, win, padding=5)
        mx, my = blur(x), blur(y)
        vx, vy, cv = blur(x * x) - mx * mx, blur(y * y) - my * my, blur(x * y) - mx * my
        c1, c2 = 1e-4, 9e-4
        ssim = (2 * mx * my + c1) * (2 * cv + c2) / ((mx * mx + my * my + c1) * (vx + vy + c2))
        loss = loss + (1 - lam) * (x - y).abs().mean() + lam * (1 - ssim.mean())
    return loss / len(wh)


def _exact_photo(case, seed):
    x = _prepare_photo(case, seed)
    rgb = x["rgb"].double().requires_grad_(True)
    loss = _exact_photo_loss(rgb, x["target"].double(), _sizes(case), case["ssim"])
    loss.backward()
    return loss.detach().view(1), rgb.grad


def _exact_residual(X, T, intr, x):
    """Residuals [M,2] and whether each observation counts."""
    T = T.view(-1, 3, 4)[x["obs_cam"].long()]
    p = (T[..., :3] @ X[x["obs_pt"].long()][..., None])[..., 0] + T[..., 3]
    f = intr[x["obs_cam"].long()]
    return p[:, :2] / p[:, 2:] * f[:, :2] + f[:, 2:] - x["obs_xy"].double(), p[:, 2] >= NEAR, p


def _exact_track_loss(X, T, intr, x):
    r, ok, _ = _exact_residual(X, T, intr, x)
    s = r.square().sum(1)
    rho = torch.where(s <= DELTA ** 2, s, 2 * DELTA * s.clamp(min=1e-30).sqrt() - DELTA ** 2)
    return LAM * rho[ok].sum()


def _exact_track(case, seed):
    x = _prepare_track(case, seed)
    X = x["X"].detach().double().requires_grad_(True)
    tw = x["twist"].detach().double().requires_grad_(True)
    loss = _exact_track_loss(X, _moved(tw, x["viewmat"].double()), x["intr"].double(), x)
    loss.backward()
    return loss.detach(), (X.grad, tw.grad)


def _exact_ba(case, seed):
    """The damped normal equations, points eliminated, solved densely."""
    _, x = _track_scene(case, seed)
    X, T, intr = x["X"].double(), x["viewmat"].double(), x["intr"].double()
    C, Pt = case["cams"], X.shape[0]
    cam, pt = x["obs_cam"].long(), x["obs_pt"].long()
    r, ok, p = _exact_residual(X, T, intr, x)
    s = r.square().sum(1)
    w = torch.where(s <= DELTA ** 2, torch.ones_like(s), DELTA / s.clamp(min=1e-30).sqrt()) * ok
    f, z = intr[cam], p[:, 2]
    o = torch.zeros_like(z)
    Jp = torch.stack([f[:, 0] / z, o, -f[:, 0] * p[:, 0] / z ** 2,
                      o, f[:, 1] / z, -f[:, 1] * p[:, 1] / z ** 2], 1).view(-1, 2, 3)
    hat = torch.stack([o, -z, p[:, 1], z, o, -p[:, 0], -p[:, 1], p[:, 0], o], 1).view(-1, 3, 3)
    Jc = torch.cat([Jp, -Jp @ hat], 2)
    Jx = Jp @ T.view(-1, 3, 4)[cam][..., :3]
    wJc, wJx = w[:, None, None] * Jc, w[:, None, None] * Jx
    add = lambda n, i, t: torch.zeros((n, *t.shape[1:]), device=DEV, dtype=torch.float64).index_add_(0, i, t)
    U, V = add(C, cam, Jc.mT @ wJc), add(Pt, pt, Jx.mT @ wJx)
    gc = add(C, cam, (wJc.mT @ r[..., None])[..., 0])
    gx = add(Pt, pt, (wJx.mT @ r[..., None])[..., 0])
    lm = 1.0 + 1e-2
    for H in (U, V):
        H.diagonal(dim1=1, dim2=2).mul_(lm)
    none = V.diagonal(dim1=1, dim2=2).sum(1) == 0     # points of no observation stay
    V[none] = torch.eye(3, device=DEV, dtype=torch.float64)
    Vi = torch.linalg.inv(V)
    W = wJc.mT @ Jx                                   # [M,6,3]
    WV = W @ Vi[pt]
    S = torch.zeros((C * C, 6, 6), device=DEV, dtype=torch.float64)
    S.index_add_(0, torch.arange(C, device=DEV) * (C + 1), U)
    order = torch.argsort(pt, stable=True)            # observations by point
    count = torch.bincount(pt, minlength=Pt)
    first = torch.cumsum(count, 0) - count
    for k in range(1, int(count.max()) + 1):          # points with k observations
        many = (count == k).nonzero()[:, 0]
        for ids in many.split(max(1, 2_000_000 // (k * k))):
            obs = order[first[ids][:, None] + torch.arange(k, device=DEV)]
            a = obs[:, :, None].expand(-1, k, k).reshape(-1)
            b = obs[:, None, :].expand(-1, k, k).reshape(-1)
            S.index_add_(0, cam[a] * C + cam[b], -(WV[a] @ W[b].mT))
    b = -gc + add(C, cam, (WV @ gx[pt][..., None])[..., 0])
    S = S.view(C, C, 6, 6).permute(0, 2, 1, 3).reshape(6 * C, 6 * C)
    dc = torch.linalg.solve(S, b.reshape(-1)).view(C, 6)
    dX = -(Vi @ (gx + add(Pt, pt, (W.mT @ dc[cam][..., None])[..., 0]))[..., None])[..., 0]
    return dc, dX, None


def _exact_init(case, seed):
    if case["n"] > 400_000:
        return None
    x = _prepare_init(case, seed)
    p, n = x["points"].double(), case["n"]
    dist = []
    for q in p.split(max(1, 200_000_000 // n)):
        d2 = sum((q[:, c, None] - p[None, :, c]).square_() for c in range(3))
        dist.append(d2.topk(case["k"] + 1, dim=1, largest=False).values[:, 1:].sqrt().mean(1))
    scale = torch.cat(dist).clamp_(min=1e-7)
    K = (case["sh"] + 1) ** 2
    sh = torch.zeros((K, 3, n), device=DEV, dtype=torch.float64)
    sh[0] = ((x["rgb"].double() - 0.5) * 2 * math.sqrt(math.pi)).t()
    one = torch.ones(n, device=DEV, dtype=torch.float64)
    return dict(means=p.t().contiguous(), log_scales=scale.log().expand(3, n).contiguous(),
                quats=torch.stack([one, 0 * one, 0 * one, 0 * one]),
                opacity_logit=math.log(0.1 / 0.9) * one, sh=sh)


def _exact_joint(case, seed):
    if not _cost(case):
        return None
    sc, batch, targets = _joint_scene(case, seed)
    t = {k: torch.from_numpy(v).to(DEV) for k, v in sc.items() if isinstance(v, np.ndarray)}
    V, p = case["views"], _leaves({k: t[k] for k in PARAM_KEYS})
    tw = torch.zeros((case["cams"], 6), device=DEV, dtype=torch.float64, requires_grad=True)
    vm = _moved(tw, t["viewmat"].double())
    X = t["X"].double().requires_grad_(True)
    loss_t = _exact_track_loss(X, vm, t["intr"].double(), t)
    loss_t.backward(retain_graph=True)
    target = torch.from_numpy(targets).to(DEV).double()
    found = {}

    def v_of(images):
        x = images.detach().requires_grad_(True)
        found["loss"] = _exact_photo_loss(x, target, sc["wh"][:V], 0.2)
        found["loss"].backward()
        return x.grad

    rgb, _ = _exact_render(p, case["sh"], vm, t["intr"], sc["wh"][:V], v_of=v_of)
    m = {k: 0.1 * v.grad for k, v in p.items()}  # the first moment after one step
    m.update(twist=0.1 * tw.grad, X=0.1 * X.grad)
    return dict(rgb=rgb, loss=torch.stack([found["loss"].detach(), loss_t.detach()]),
                v_twist=tw.grad, v_X=X.grad, exp_avg=m, params={k: None for k in m})
