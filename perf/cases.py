"""Performance cases of the projector library: what a program that uses it
spends its time on, each through a public entry point.

A case is a dict of plain values; its "kind" names the entry point(s):

  drr        project_fwd: DRRs of a volume (rendering, training sets, search)
  drr_grad   project_fwd_grad_pose: pose gradient for a given dL/dl
  ssd        project_fwd_ssd_gauss_newton: one registration step's launch
  fdk        fdk_filter + backproject (FDK weight): a reconstruction
  bp         backproject (plain or FDK weight) of given detector images
  bp_grad    backproject_grad_pose for a given dL/dmu
  fp_fwd     fp_project + fp_project_grad_pose (SF / DD footprints)
  fp_bp      fp_backproject + fp_backproject_grad_pose (SF / DD)
  conv       one layer of the pose-proposal network: forward, weight and
             input gradient (BF16 matrix cores)
  train      one training step of the whole network: forward, backward, Adam

`exact` evaluates the same definitions in plain FP64 torch.
"""
from __future__ import annotations

import math
import types

import torch

import paper_2508_13304_amd as dp
from paper_2508_13304_amd import proposal

F64, F32, BF16 = torch.float64, torch.float32, torch.bfloat16
DEV = "cuda:0"
SAD, SDD, STEP = 1000.0, 1500.0, 0.5


def listed():
    return [
        # the smallest call: one DRR of a 64^3 volume (latency of a single render)
        dict(name="drr_64_1v", kind="drr", nx=64, ny=64, nz=64, h=1.0, nu=128, nv=128, du=1.5,
             views=1, orbit=False, t=5.0, r=5.0),
        # rendering a training phantom's targets: 100 random poses, 256^2
        dict(name="drr_192_100v", kind="drr", nx=192, ny=192, nz=192, h=1.0, nu=256, nv=256, du=1.2,
             views=100, orbit=False, t=30.0, r=20.0),
        # pose gradient of a caller's own loss on a ragged grid around the orbit
        dict(name="drr_grad_ragged_12v", kind="drr_grad", nx=151, ny=133, nz=117, h=0.9, nu=271,
             nv=203, du=0.9, views=12, orbit=True, t=5.0, r=5.0),
        # one registration step: 64 candidate poses, 512^2 from 256^3 (the headline workload)
        dict(name="ssd_256_64v", kind="ssd", nx=256, ny=256, nz=256, h=0.8, nu=512, nv=512, du=0.6,
             views=64, orbit=False, t=10.0, r=10.0),
        # one registration step of a single view of a large volume
        dict(name="ssd_512_1v", kind="ssd", nx=512, ny=512, nz=512, h=0.4, nu=768, nv=768, du=0.4,
             views=1, orbit=False, t=5.0, r=3.0),
        # reconstruction of a full orbit (the reconstruction workload)
        dict(name="fdk_512_360v", kind="fdk", nx=512, ny=512, nz=512, h=0.375, nu=512, nv=384,
             du=0.776, views=360, t=3.0, r=2.0),
        # a small ragged back-projection, plain weight
        dict(name="bp_ragged_30v", kind="bp", nx=97, ny=81, nz=53, h=1.2, nu=149, nv=97, du=1.5,
             views=30, weight=0, t=5.0, r=5.0),
        # motion-compensation gradient of a reconstruction
        dict(name="bp_grad_256_120v", kind="bp_grad", nx=256, ny=256, nz=256, h=0.75, nu=512,
             nv=384, du=0.776, views=120, weight=1, t=3.0, r=2.0),
        # footprint projectors at a step of the projector comparison: separable
        # footprint forward + gradient, distance-driven back-projection + gradient
        dict(name="sf_fwd_256_4v", kind="fp_fwd", fp="sf", nx=256, ny=256, nz=256, h=0.8, nu=384,
             nv=384, du=0.8, views=4, t=5.0, r=3.0),
        dict(name="dd_bp_256_64v", kind="fp_bp", fp="dd", nx=256, ny=256, nz=256, h=0.8, nu=384,
             nv=384, du=0.8, views=64, t=5.0, r=3.0),
        # the third convolution of the proposal network at its training batch
        dict(name="conv_64_128", kind="conv", batch=256, hw=64, ci=64, co=128, stride=2),
        # a whole training step of the proposal network
        dict(name="train_256", kind="train", batch=256, size=256),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed kinds over their ranges, no dearer than the largest listed one."""
    kind = rng.choice(["drr", "drr_grad", "ssd", "fdk", "bp", "bp_grad", "fp_fwd", "fp_bp", "conv", "train"])
    if kind == "conv":
        ci, co = 8 * _logint(rng, 4, 32), 8 * _logint(rng, 4, 32)
        hw = _logint(rng, 7, 128)
        batch = min(256, max(1, (1 << 28) // (hw * hw * ci)))
        return dict(kind=kind, batch=_logint(rng, max(1, batch // 16), batch), hw=hw, ci=ci, co=co,
                    stride=rng.choice([1, 2, 2]))
    if kind == "train":
        return dict(kind=kind, batch=_logint(rng, 16, 256), size=rng.choice([96, 128, 160, 192, 256]))
    big = kind in ("fdk", "bp", "bp_grad")
    n = _logint(rng, 48, 320)
    dims = [max(16, int(n * rng.uniform(0.7, 1.0))) for _ in range(3)]
    vox = dims[0] * dims[1] * dims[2]
    h = round(rng.uniform(150.0, 220.0) / n, 4)
    nu = _logint(rng, max(64, n), min(640, 3 * n))
    nv = max(48, int(nu * rng.uniform(0.6, 1.0)))
    du = round(rng.uniform(300.0, 380.0) / nu, 4)
    most = 360 if big else 64
    if kind in ("fp_fwd", "fp_bp"):
        most = max(1, min(96, int(6e8 / vox)))
    elif kind == "ssd" or kind == "drr_grad":
        most = max(1, min(64, int(2.5e9 / (nu * nv * n))))
    elif kind == "drr":
        most = max(1, min(100, int(4.0e9 / (nu * nv * n))))
    c = dict(kind=kind, nx=dims[0], ny=dims[1], nz=dims[2], h=h, nu=nu, nv=nv, du=du,
             views=_logint(rng, max(1, most // 16), most), t=round(rng.uniform(0, 10), 2),
             r=round(rng.uniform(0, 10), 2))
    if kind in ("drr", "drr_grad", "ssd"):
        c["orbit"] = rng.random() < 0.5
    if kind in ("bp", "bp_grad"):
        c["weight"] = rng.choice([0, 1])
    if kind in ("fp_fwd", "fp_bp"):
        c["fp"] = rng.choice(["sf", "dd"])
    return c


# --------------------------------------------------------------------------
# Inputs
# --------------------------------------------------------------------------

def _geom(c):
    return types.SimpleNamespace(nx=c["nx"], ny=c["ny"], nz=c["nz"], vx=c["h"], vy=c["h"], vz=c["h"],
                                 nu=c["nu"], nv=c["nv"], du=c["du"], dv=c["du"], off_u=0.0, off_v=0.0,
                                 sad=SAD, sdd=SDD, step=STEP)


def _gen(seed):
    return torch.Generator(device="cpu").manual_seed(int(seed))


def _phantom(g, gen, n_ell=16):
    """Additive random ellipsoids (0.01-0.05 / mm) inside a shell of the grid, lightly smoothed."""
    L = [g.nx * g.vx, g.ny * g.vy, g.nz * g.vz]
    ax = [(torch.arange(n, dtype=F32, device=DEV) - (n - 1) / 2) * h
          for n, h in ((g.nx, g.vx), (g.ny, g.vy), (g.nz, g.vz))]
    X, Y, Z = ax[0][None, None, :], ax[1][None, :, None], ax[2][:, None, None]
    shell = lambda s: (X / (s * L[0])) ** 2 + (Y / (s * L[1])) ** 2 + (Z / (s * L[2])) ** 2 <= 1.0
    vol = torch.where(shell(0.45) & ~shell(0.42), 0.08, 0.0).to(F32)
    for _ in range(n_ell):
        p = torch.rand(8, generator=gen).tolist()
        ce = [(p[a] - 0.5) * 0.5 * L[a] for a in range(3)]
        se = [(0.05 + 0.12 * p[3 + a]) * L[a] for a in range(3)]
        cs, sn = math.cos(p[6] * math.pi), math.sin(p[6] * math.pi)
        x, y, z = X - ce[0], Y - ce[1], Z - ce[2]
        q = ((x * cs + y * sn) / se[0]) ** 2 + ((y * cs - x * sn) / se[1]) ** 2 + (z / se[2]) ** 2
        vol += (q <= 1.0) * (0.01 + 0.04 * p[7])
    return torch.nn.functional.avg_pool3d(vol[None, None], 3, stride=1, padding=1)[0, 0].contiguous()


def _images(V, nv, nu, gen, signed=True, blobs=8):
    """Smooth random detector images: sums of separable Gaussian blobs."""
    p = torch.rand((V, blobs, 5), generator=gen).to(DEV)
    bu = torch.exp(-0.5 * ((torch.arange(nu, device=DEV) - nu * (0.1 + 0.8 * p[..., :1])) /
                           (nu * (0.03 + 0.17 * p[..., 1:2]))) ** 2)
    bv = torch.exp(-0.5 * ((torch.arange(nv, device=DEV) - nv * (0.1 + 0.8 * p[..., 2:3])) /
                           (nv * (0.03 + 0.17 * p[..., 3:4]))) ** 2)
    amp = 2 * p[..., 4] - 1 if signed else 0.2 + 0.8 * p[..., 4]
    out = torch.zeros((V, nv, nu), dtype=F32, device=DEV)
    for b in range(blobs):
        out += (amp[:, b, None] * bv[:, b])[:, :, None] * bu[:, b, None, :]
    return out.contiguous()


def _views(c, gen):
    V = c["views"]
    scale = torch.tensor([c["t"]] * 3 + [math.radians(c["r"])] * 3, dtype=F64)
    poses = (2 * torch.rand((V, 6), generator=gen, dtype=F64) - 1) * scale
    angles = torch.zeros(V, dtype=F64)
    if c.get("orbit", True):
        angles = torch.arange(V, dtype=F64) * (2 * math.pi / V) + 0.3
    return angles.to(DEV), poses.to(DEV).contiguous()


def prepare(case, seed):
    c, gen = case, _gen(seed)
    s = types.SimpleNamespace(c=c)
    if c["kind"] == "conv":
        ho = (c["hw"] - 1) // c["stride"] + 1
        s.x = torch.randn((c["batch"], c["hw"], c["hw"], c["ci"]), device=DEV, generator=torch.Generator(DEV).manual_seed(int(seed))).relu().to(BF16)
        s.dz = (torch.randn((c["batch"], ho, ho, c["co"]), device=DEV, generator=torch.Generator(DEV).manual_seed(int(seed) + 1)) * 1e-2).to(BF16)
        row = (9 * c["ci"] + 1 + 7) // 8 * 8  # weights, bias, padding: the network's parameter rows
        W = torch.zeros((c["co"], row))
        W[:, :9 * c["ci"]] = torch.randn((c["co"], 9 * c["ci"]), generator=gen) * math.sqrt(2 / (9 * c["ci"]))
        W[:, 9 * c["ci"]] = 0.1 * torch.randn(c["co"], generator=gen)
        s.W = W.to(DEV)
        s.Wb = s.W.to(BF16)
        s.dw = torch.empty_like(s.W)
        return s
    if c["kind"] == "train":
        s.net = proposal.ProposalNet(size=c["size"], device=DEV, seed=int(seed))
        im = _images(2 * c["batch"], c["size"], c["size"], gen, signed=False)
        s.x = proposal.pair_input(im[:c["batch"]], im[c["batch"]:], c["size"])
        s.labels = (2 * torch.rand((c["batch"], 6), generator=gen) - 1).to(DEV)
        return s
    g = s.g = _geom(c)
    s.angles, s.poses = _views(c, gen)
    V, kind = c["views"], c["kind"]
    if kind in ("drr", "drr_grad", "ssd", "fp_fwd"):
        s.vol = _phantom(g, gen)
    else:
        s.img = _images(V, g.nv, g.nu, gen, signed=kind != "fdk")
    if kind in ("drr_grad", "fp_fwd"):
        s.gl = _images(V, g.nv, g.nu, gen)
    if kind == "ssd":
        s.target = 5.0 * _images(V, g.nv, g.nu, gen, signed=False)
    if kind in ("bp_grad", "fp_bp"):
        s.e = _phantom(g, gen, 8) - _phantom(g, gen, 8)
    ops = {"drr": [dp.OP_FWD], "drr_grad": [dp.OP_FWD_GRAD], "ssd": [dp.OP_FWD_SSD], "fdk": [dp.OP_BP],
           "bp": [dp.OP_BP], "bp_grad": [dp.OP_BP_GRAD], "fp_fwd": [dp.OP_FP_FWD, dp.OP_FP_FWD_GRAD],
           "fp_bp": [dp.OP_FP_BP, dp.OP_FP_BP_GRAD]}[kind]
    # the workspace an iterating program keeps; outputs are allocated by each call
    s.ws = torch.empty(max(dp.workspace_bytes(g, V, op) for op in ops), dtype=torch.uint8, device=DEV)
    return s


def run(s):
    c = s.c
    kind = c["kind"]
    if kind == "conv":
        shape = tuple(s.x.shape)
        y = proposal.conv_fwd(s.x, s.Wb, c["stride"], s.W[:, 9 * c["ci"]], relu=True)
        proposal.conv_wgrad(s.x, s.dz, c["stride"], out=s.dw)
        return {"y": y, "dw": s.dw, "dx": proposal.conv_dgrad_act(s.dz, s.Wb, shape, c["stride"], s.x)}
    if kind == "train":
        out, cache = s.net.forward(s.x, keep=True)
        grads, head = s.net.backward(cache, (2.0 / out.numel()) * (out - s.labels))
        s.net.adam_step(grads, head)
        return {"logits": out, "grad": s.net.G, "params": s.net.P}
    g = s.g
    if kind == "drr":
        return dp.project_fwd(g, s.angles, s.poses, s.vol, ws=s.ws)
    if kind == "drr_grad":
        return dp.project_fwd_grad_pose(g, s.angles, s.poses, s.vol, s.gl, ws=s.ws)
    if kind == "ssd":
        return list(dp.project_fwd_ssd_gauss_newton(g, s.angles, s.poses, s.vol, s.target, ws=s.ws, packed=True))
    if kind == "fdk":
        q = dp.fdk_filter(g, s.img, math.pi / c["views"])
        return {"filtered": q, "vol": dp.backproject(g, s.angles, s.poses, q, dp.W_FDK, ws=s.ws)}
    if kind == "bp":
        return dp.backproject(g, s.angles, s.poses, s.img, c["weight"], ws=s.ws)
    if kind == "bp_grad":
        return dp.backproject_grad_pose(g, s.angles, s.poses, s.img, s.e, c["weight"], ws=s.ws)
    if kind == "fp_fwd":
        return {"proj": dp.fp_project(g, s.angles, s.poses, s.vol, c["fp"], ws=s.ws),
                "grad": dp.fp_project_grad_pose(g, s.angles, s.poses, s.vol, s.gl, c["fp"], ws=s.ws)}
    return {"vol": dp.fp_backproject(g, s.angles, s.poses, s.img, c["fp"], ws=s.ws),
            "grad": dp.fp_backproject_grad_pose(g, s.angles, s.poses, s.img, s.e, c["fp"], ws=s.ws)}


CHANNELS = proposal.CHANNELS


def _layers(size):
    ci, hw, out = 2, size, []
    for co in CHANNELS:
        out.append((ci, co, hw))
        ci, hw = co, (hw - 1) // 2 + 1
    return out, ci * hw * hw


def work(case):
    """What a pass cannot do without: inputs and outputs once, the method's own operations."""
    c = case
    if c["kind"] == "conv":
        ho = (c["hw"] - 1) // c["stride"] + 1
        m, k = c["batch"] * ho * ho, 9 * c["ci"]
        px = c["batch"] * c["hw"] ** 2 * c["ci"]
        return {"bytes": 2.0 * (2 * px + 2 * m * c["co"]) + 8.0 * c["co"] * k, "flops": 6.0 * m * k * c["co"]}
    if c["kind"] == "train":
        layers, feat = _layers(c["size"])
        fl = by = par = 0.0
        for i, (ci, co, hw) in enumerate(layers):
            ho = (hw - 1) // 2 + 1
            fl += (6.0 if i else 4.0) * c["batch"] * ho * ho * 9 * ci * co
            by += 2.0 * c["batch"] * (2 * hw * hw * ci + 3 * ho * ho * co)
            par += co * (9 * ci + 1)
        fl += 6.0 * c["batch"] * 6 * feat
        return {"bytes": by + 30.0 * (par + 6 * feat), "flops": fl}
    V, pix, vox = c["views"], c["views"] * c["nu"] * c["nv"], c["nx"] * c["ny"] * c["nz"]
    per_view = min(vox * c["h"] ** 3 * (SDD / SAD) ** 2 / c["du"] ** 2 / STEP,
                   c["nu"] * c["nv"] * max(c["nx"], c["ny"], c["nz"]) * c["h"] / STEP)
    n, u = per_view * V, float(vox) * V  # ray samples, voxel-view updates
    both = 4.0 * (pix + vox)
    return {"drr": {"bytes": both, "flops": 30 * n}, "drr_grad": {"bytes": both, "flops": 120 * n},
            "ssd": {"bytes": both + 4.0 * pix, "flops": 150 * n},
            "fdk": {"bytes": both + 8.0 * pix, "flops": 25 * u + 2.0 * pix * c["nu"]},
            "bp": {"bytes": both, "flops": 25 * u}, "bp_grad": {"bytes": both, "flops": 90 * u},
            "fp_fwd": {"bytes": 2 * both, "flops": 150 * u},
            "fp_bp": {"bytes": 2 * both, "flops": 150 * u}}[c["kind"]]


# --------------------------------------------------------------------------
# FP64 values
# --------------------------------------------------------------------------

def _rot(gam):
    """R = Rz Ry Rx and its three partial derivatives (3x3 FP64, CPU)."""
    c, s = [math.cos(x) for x in gam], [math.sin(x) for x in gam]
    m = lambda r: torch.tensor(r, dtype=F64)
    X, dX = m([[1, 0, 0], [0, c[0], -s[0]], [0, s[0], c[0]]]), m([[0, 0, 0], [0, -s[0], -c[0]], [0, c[0], -s[0]]])
    Y, dY = m([[c[1], 0, s[1]], [0, 1, 0], [-s[1], 0, c[1]]]), m([[-s[1], 0, c[1]], [0, 0, 0], [-c[1], 0, -s[1]]])
    Z, dZ = m([[c[2], -s[2], 0], [s[2], c[2], 0], [0, 0, 1]]), m([[-s[2], -c[2], 0], [c[2], -s[2], 0], [0, 0, 0]])
    return Z @ Y @ X, (Z @ Y @ dX, Z @ dY @ X, dZ @ Y @ X)


def _view(g, beta, pose):
    cb, sb = math.cos(beta), math.sin(beta)
    R, dR = _rot(pose[3:])
    v = types.SimpleNamespace(R=R, dR=dR, t=torch.tensor(pose[:3], dtype=F64),
                              ew=torch.tensor([-cb, -sb, 0.0], dtype=F64), eu=torch.tensor([-sb, cb, 0.0], dtype=F64),
                              ev=torch.tensor([0.0, 0.0, 1.0], dtype=F64),
                              src=torch.tensor([g.sad * cb, g.sad * sb, 0.0], dtype=F64),
                              cu=0.5 * (g.nu - 1) + g.off_u, cv=0.5 * (g.nv - 1) + g.off_v)
    v.sobj = (R.T @ (v.src - v.t)).tolist()
    return v


def _all_views(g, s):
    return [_view(g, b, p) for b, p in zip(s.angles.tolist(), s.poses.tolist())]


def _voxels(g):
    ax = [(torch.arange(n, dtype=F64, device=DEV) - 0.5 * (n - 1)) * h
          for n, h in ((g.nx, g.vx), (g.ny, g.vy), (g.nz, g.vz))]
    return ax[0][None, None, :], ax[1][None, :, None], ax[2][:, None, None]


def _gradient(g, vol):
    """Central differences per mm of the zero-extended volume."""
    p = torch.nn.functional.pad(vol, (1, 1, 1, 1, 1, 1))
    return ((p[1:-1, 1:-1, 2:] - p[1:-1, 1:-1, :-2]) / (2 * g.vx),
            (p[1:-1, 2:, 1:-1] - p[1:-1, :-2, 1:-1]) / (2 * g.vy),
            (p[2:, 1:-1, 1:-1] - p[:-2, 1:-1, 1:-1]) / (2 * g.vz))


def _march(g, view, field):
    """[nv nu][C]: step * sum of the trilinear samples of field [voxels padded by 1][C] along each ray."""
    dims = torch.tensor([g.nx, g.ny, g.nz], dtype=F64)
    h = torch.tensor([g.vx, g.vy, g.vz], dtype=F64)
    a = ((torch.arange(g.nu, dtype=F64, device=DEV) - view.cu) * g.du)[None, :, None]
    b = ((torch.arange(g.nv, dtype=F64, device=DEV) - view.cv) * g.dv)[:, None, None]
    q = (g.sdd * view.ew.to(DEV) + a * view.eu.to(DEV) + b * view.ev.to(DEV)).reshape(-1, 3)
    u = q / q.norm(dim=1, keepdim=True)
    M = (view.R / h[None, :]).to(DEV)                      # index = (r - t) M + centre
    D = (u @ M) * g.step                                   # index step per sample
    X0 = ((view.src - view.t).to(DEV) @ M + 0.5 * (dims.to(DEV) - 1))[None, :]
    n = dims.to(DEV)
    inv = 1.0 / torch.where(D.abs() < 1e-14, torch.full_like(D, 1e-14), D)
    t0, t1 = (-1.0 - X0) * inv, (n - X0) * inv
    k0 = (torch.minimum(t0, t1).amax(dim=1).floor() - 1).clamp_min(0.0)
    k1 = torch.maximum(t0, t1).amin(dim=1).ceil() + 1
    hit = torch.nonzero(k1 >= k0).flatten()
    C = field.shape[1]
    out = torch.zeros((u.shape[0], C), dtype=F64, device=DEV)
    if hit.numel() == 0:
        return out
    K = int((k1 - k0)[hit].max()) + 1
    px, py = g.nx + 2, g.ny + 2
    per = max(1, (1 << 21) // K)
    ks = torch.arange(K, dtype=F64, device=DEV)
    for r0 in range(0, hit.numel(), per):
        idx = hit[r0:r0 + per]
        k = k0[idx][:, None] + ks[None, :]
        X = [X0[:, c] + k * D[idx, c:c + 1] for c in range(3)]
        ok = torch.ones_like(k, dtype=torch.bool)
        for c in range(3):
            ok &= (X[c] > -1.0) & (X[c] < float(dims[c]))
        fl = [torch.where(ok, x, torch.zeros_like(x)).floor() for x in X]
        w = [[1.0 - (x - f), x - f] for x, f in zip(X, fl)]
        base = ((fl[2] + 1) * py + (fl[1] + 1)) * px + (fl[0] + 1)
        base = base.to(torch.int64)
        acc = torch.zeros((idx.numel(), K, C), dtype=F64, device=DEV) if C > 1 else torch.zeros_like(k)
        for dz in range(2):
            for dy in range(2):
                wyz = torch.where(ok, w[2][dz] * w[1][dy], torch.zeros_like(k))
                for dx in range(2):
                    i = (base + ((dz * py + dy) * px + dx)).reshape(-1)
                    f = field.index_select(0, i) if C > 1 else field[:, 0][i].view_as(k)
                    wt = wyz * w[0][dx]
                    acc += f.view(idx.numel(), K, C) * wt[:, :, None] if C > 1 else f * wt
        out[idx] = g.step * (acc.sum(1) if C > 1 else acc.sum(1, keepdim=True))
    return out


def _padded(chs):
    """[padded voxels][C] from C volumes (one voxel of zero border below, one above)."""
    return torch.stack([torch.nn.functional.pad(ch, (1, 1, 1, 1, 1, 1)).reshape(-1) for ch in chs], dim=1).contiguous()


def _ray_fields(g, vol):
    """mu, its gradient G and p x G (p the voxel centre): what the per-ray pose Jacobian needs."""
    gx, gy, gz = _gradient(g, vol)
    x, y, z = _voxels(g)
    return _padded([vol, gx, gy, gz, y * gz - z * gy, z * gx - x * gz, x * gy - y * gx])


def _ray_jacobian(view, S):
    """[rays][6] from the ray sums of _ray_fields: dl/dt = -R G, dl/dgamma_a = sum G^T (dR_a^T R) p."""
    cols = [-(S[:, 1:4] @ view.R.T.to(DEV))]
    for dR in view.dR:
        O = dR.T @ view.R  # antisymmetric: G^T O p = -o . (p x G)
        o = torch.tensor([float(O[1, 2]), float(O[2, 0]), float(O[0, 1])], dtype=F64, device=DEV)
        cols.append(-(S[:, 4:7] @ o)[:, None])
    return torch.cat(cols, dim=1)


def _contract(view, dLdM):
    """dL/dtheta [6] from dL/dM [3][4] (CPU FP64)."""
    return torch.cat([dLdM[:, 3], torch.stack([(dR * dLdM[:, :3]).sum() for dR in view.dR])])


def _sample_slots(c):
    diag = math.sqrt(c["nx"] ** 2 + c["ny"] ** 2 + c["nz"] ** 2) * c["h"] / STEP
    return c["views"] * c["nu"] * c["nv"] * diag


def _exact_rays(s):
    c, g = s.c, s.g
    vol = s.vol.to(F64)
    views = _all_views(g, s)
    if c["kind"] == "drr":
        f = _padded([vol])
        return torch.stack([_march(g, v, f).view(g.nv, g.nu) for v in views])
    f = _ray_fields(g, vol)
    if c["kind"] == "drr_grad":
        return torch.stack([_ray_jacobian(v, _march(g, v, f)).T @ s.gl[i].reshape(-1).to(F64) for i, v in enumerate(views)])
    pr, lo, gr, he = [], [], [], []
    iu = torch.triu_indices(6, 6, device=DEV)
    for i, v in enumerate(views):
        S = _march(g, v, f)
        J = _ray_jacobian(v, S)
        d = S[:, 0] - s.target[i].reshape(-1).to(F64)
        pr.append(S[:, 0].view(g.nv, g.nu)), lo.append((d * d).sum()), gr.append(2 * (J.T @ d))
        he.append((2 * (J.T @ J))[iu[0], iu[1]])
    return [torch.stack(pr), torch.stack(lo), torch.stack(gr), torch.stack(he)]


def _exact_filter(g, img, scale):
    mag = g.sad / g.sdd
    u = (torch.arange(g.nu, dtype=F64, device=DEV) - (0.5 * (g.nu - 1) + g.off_u)) * g.du * mag
    v = (torch.arange(g.nv, dtype=F64, device=DEV) - (0.5 * (g.nv - 1) + g.off_v)) * g.dv * mag
    tau = g.du * mag
    k = torch.arange(g.nu, device=DEV)
    d = (k[:, None] - k[None, :]).to(F64)
    T = torch.where(d.abs() % 2 == 1, -1.0 / (math.pi ** 2 * d ** 2 * tau ** 2), torch.zeros_like(d))
    T.fill_diagonal_(1.0 / (4 * tau ** 2))
    pw = img.to(F64) * (g.sad / torch.sqrt(g.sad ** 2 + u[None, :] ** 2 + v[:, None] ** 2))
    return (pw.reshape(-1, g.nu) @ T.T).view_as(img) * (scale * tau)


def _project_voxels(g, view, dx=0.0, dy=0.0, dz=0.0):
    """(a, b, w): pixel coordinates and depth of every voxel centre shifted by (dx, dy, dz) mm."""
    x, y, z = _voxels(g)
    R, t = view.R.tolist(), view.t.tolist()
    r = [R[c][0] * (x + dx) + R[c][1] * (y + dy) + R[c][2] * (z + dz) + t[c] for c in range(3)]
    dot = lambda e: e[0] * r[0] + e[1] * r[1] + e[2] * r[2]
    w = dot(view.ew.tolist()) + g.sad
    return (g.sdd / g.du) * dot(view.eu.tolist()) / w + view.cu, (g.sdd / g.dv) * dot(view.ev.tolist()) / w + view.cv, w


def _bilinear(imgs, a, b):
    """Zero-extended bilinear samples of each image at (a, b)."""
    nv, nu = imgs[0].shape
    a, b = a.clamp(-1.5, nu + 0.5), b.clamp(-1.5, nv + 0.5)
    fa, fb = a.floor(), b.floor()
    wa, wb = a - fa, b - fb
    P = [torch.nn.functional.pad(im, (2, 2, 2, 2)).reshape(-1) for im in imgs]
    base = ((fb + 2) * (nu + 4) + fa + 2).to(torch.int64)
    out = []
    for p in P:
        top = p[base] * (1 - wa) + p[base + 1] * wa
        bot = p[base + nu + 4] * (1 - wa) + p[base + nu + 5] * wa
        out.append(top * (1 - wb) + bot * wb)
    return out


def _exact_bp(g, s, img, fdk):
    out = torch.zeros((g.nz, g.ny, g.nx), dtype=F64, device=DEV)
    for i, view in enumerate(_all_views(g, s)):
        a, b, w = _project_voxels(g, view)
        t, = _bilinear([img[i].to(F64)], a, b)
        out += t * (g.sad / w) ** 2 if fdk else t
    return out


def _image_gradient(im):
    p = torch.nn.functional.pad(im, (1, 1, 1, 1))
    return 0.5 * (p[1:-1, 2:] - p[1:-1, :-2]), 0.5 * (p[2:, 1:-1] - p[:-2, 1:-1])


def _bp_contract(g, view, e, la, lb, l, a, b, w, fdk):
    """dL/dtheta of one view: e weights the back-projected image gradient (la, lb) and value l."""
    W = (g.sad / w) ** 2 if fdk else 1.0
    cu = e * W / w * la
    cv = e * W / w * lb
    cw = -(cu * (a - view.cu) + cv * (b - view.cv))
    if fdk:
        cw = cw - 2 * e * W / w * l
    x, y, z = _voxels(g)
    one = torch.ones_like(x)
    M = torch.zeros((3, 4), dtype=F64)
    for f, ax, sc in ((cu, view.eu, g.sdd / g.du), (cv, view.ev, g.sdd / g.dv), (cw, view.ew, 1.0)):
        m = torch.tensor([float((f * p).sum()) for p in (x, y, z, one)], dtype=F64)
        M += sc * ax[:, None] * m[None, :]
    return _contract(view, M)


def _exact_bp_grad(g, s, fdk):
    e, out = s.e.to(F64), []
    for i, view in enumerate(_all_views(g, s)):
        im = s.img[i].to(F64)
        a, b, w = _project_voxels(g, view)
        l, la, lb = _bilinear([im, *_image_gradient(im)], a, b)
        out.append(_bp_contract(g, view, e, la, lb, l, a, b, w, fdk))
    return torch.stack(out)


def _footprints(g, view, kind):
    """Yields (pixel index, weight) of every voxel's footprint, one window offset at a time."""
    so = view.sobj
    x, y, z = _voxels(g)
    dom = 0 if abs(so[0]) >= abs(so[1]) else 1
    if kind == "sf":
        t = torch.stack([_project_voxels(g, view, sx * g.vx / 2, sy * g.vy / 2)[0]
                         for sx in (-1, 1) for sy in (-1, 1)]).sort(dim=0).values
    else:
        sh = [(0.0, sg * g.vy / 2) if dom == 0 else (sg * g.vx / 2, 0.0) for sg in (-1, 1)]
        q = torch.stack([_project_voxels(g, view, *d)[0] for d in sh]).sort(dim=0).values
        t = q[[0, 0, 1, 1]]
    bb = torch.stack([_project_voxels(g, view, dz=sg * g.vz / 2)[1] for sg in (-1, 1)]).sort(dim=0).values
    d = [(x - so[0]).abs(), (y - so[1]).abs(), (z - so[2]).abs()]
    n = torch.sqrt(d[0] ** 2 + d[1] ** 2 + d[2] ** 2)
    hs = (g.vx, g.vy, g.vz)
    if kind == "sf":
        L = torch.stack([(hs[c] * n / d[c]).expand(g.nz, g.ny, g.nx) for c in range(3)]).amin(dim=0)
    else:
        L = hs[dom] * n / d[dom]

    def cdf(v):
        e1, e2 = t[1] - t[0], t[3] - t[2]
        r = torch.minimum(torch.maximum(v, t[0]), t[1]) - t[0]
        f = t[3] - torch.minimum(torch.maximum(v, t[2]), t[3])
        s_ = torch.where(e1 > 0, r * r / (2 * e1), torch.zeros_like(r))
        s_ = s_ + torch.minimum(torch.maximum(v, t[1]), t[2]) - t[1]
        return s_ + torch.where(e2 > 0, (e2 * e2 - f * f) / (2 * e2), torch.zeros_like(f))

    a0, b0 = (t[0] - 0.5).floor() + 1, (bb[0] - 0.5).floor() + 1
    na = int(((t[3] + 0.5).ceil() - 1 - a0).max()) + 1
    nb = int(((bb[1] + 0.5).ceil() - 1 - b0).max()) + 1
    for da in range(na):
        a = a0 + da
        wa = L * (cdf(a + 0.5) - cdf(a - 0.5))
        for db in range(nb):
            b = b0 + db
            wb = (torch.minimum(b + 0.5, bb[1]) - torch.maximum(b - 0.5, bb[0])).clamp_min(0.0)
            ok = (a >= 0) & (a < g.nu) & (b >= 0) & (b < g.nv)
            yield torch.where(ok, b * g.nu + a, torch.zeros_like(a)).to(torch.int64), torch.where(ok, wa * wb, torch.zeros_like(wa))


def _exact_fp(s):
    c, g = s.c, s.g
    views = _all_views(g, s)
    grads = []
    if c["kind"] == "fp_fwd":
        vol = s.vol.to(F64)
        G = _gradient(g, vol)
        x, y, z = _voxels(g)
        proj = torch.zeros((len(views), g.nv * g.nu), dtype=F64, device=DEV)
        for i, v in enumerate(views):
            gl = s.gl[i].reshape(-1).to(F64)
            sj = torch.zeros_like(vol)
            for idx, w in _footprints(g, v, c["fp"]):
                proj[i].index_add_(0, idx.reshape(-1), (w * vol).reshape(-1))
                sj += w * gl[idx]
            m = [sj * q for q in G]
            S = torch.stack([torch.zeros((), dtype=F64, device=DEV)] + [q.sum() for q in m] +
                            [(y * m[2] - z * m[1]).sum(), (z * m[0] - x * m[2]).sum(), (x * m[1] - y * m[0]).sum()])
            grads.append(_ray_jacobian(v, S[None, :])[0])
        return {"proj": proj.view(len(views), g.nv, g.nu), "grad": torch.stack(grads)}
    e = s.e.to(F64)
    out = torch.zeros_like(e)
    for i, v in enumerate(views):
        im = s.img[i].to(F64)
        la, lb = [q.reshape(-1) for q in _image_gradient(im)]
        flat = im.reshape(-1)
        da, db = torch.zeros_like(e), torch.zeros_like(e)
        for idx, w in _footprints(g, v, c["fp"]):
            out += w * flat[idx]
            da += w * la[idx]
            db += w * lb[idx]
        a, b, w = _project_voxels(g, v)
        grads.append(_bp_contract(g, v, e, da, db, None, a, b, w, False))
    return {"vol": out, "grad": torch.stack(grads).to(DEV)}


def _im2col(x, stride):
    """[N Ho Wo][9 C] of an NHWC tensor, column order (ky, kx, c)."""
    N, H, W, C = x.shape
    ho, wo = (H - 1) // stride + 1, (W - 1) // stride + 1
    p = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1))
    return torch.cat([p[:, ky:ky + (ho - 1) * stride + 1:stride, kx:kx + (wo - 1) * stride + 1:stride]
                      for ky in range(3) for kx in range(3)], dim=3).reshape(N * ho * wo, 9 * C)


def _col2im(dcol, shape, stride):
    N, H, W, C = shape
    ho, wo = (H - 1) // stride + 1, (W - 1) // stride + 1
    p = torch.zeros((N, H + 2, W + 2, C), dtype=F64, device=DEV)
    d = dcol.view(N, ho, wo, 9, C)
    for t in range(9):
        ky, kx = divmod(t, 3)
        p[:, ky:ky + (ho - 1) * stride + 1:stride, kx:kx + (wo - 1) * stride + 1:stride] += d[:, :, :, t]
    return p[:, 1:H + 1, 1:W + 1]


def _exact_conv(s):
    c = s.c
    K = 9 * c["ci"]
    ys, dxs = [], []
    dw = torch.zeros(s.W.shape, dtype=F64, device=DEV)
    W, b = s.Wb[:, :K].to(F64), s.W[:, K].to(F64)
    per = max(1, (1 << 26) // (c["hw"] ** 2 * c["ci"]))
    for n in range(0, c["batch"], per):
        x = s.x[n:n + per].to(F64)
        col, dz = _im2col(x, c["stride"]), s.dz[n:n + per].to(F64)
        d2 = dz.reshape(-1, c["co"])
        ys.append((col @ W.T + b).relu().view_as(dz))
        dw[:, :K] += d2.T @ col
        dw[:, K] += d2.sum(0)
        dxs.append(_col2im(d2 @ W, tuple(x.shape), c["stride"]) * (x > 0))
    return {"y": torch.cat(ys), "dw": dw, "dx": torch.cat(dxs)}


def _exact_train(s):
    net, c = s.net, s.c
    Pb, P = net.Pb.to(F64), net.P.to(F64)
    layers, feat = _layers(c["size"])
    off, par = 0, []
    for ci, co, _ in layers:
        row = (9 * ci + 1 + 7) // 8 * 8
        par.append((off, co, row, 9 * ci))
        off += co * row
    G = torch.zeros_like(P)
    logits = []
    Wf = Pb[off:off + 6 * feat].view(6, feat)
    bf = P[off + 6 * feat:]
    for n in range(0, c["batch"], 32):
        h = s.x[n:n + 32].to(F64)
        keep = []
        for o, co, row, K in par:
            col = _im2col(h, 2)
            W = Pb[o:o + co * row].view(co, row)[:, :K]
            y = (col @ W.T + P[o:o + co * row].view(co, row)[:, K]).relu()
            keep.append((tuple(h.shape), col, y))
            ho = (h.shape[1] - 1) // 2 + 1
            h = y.view(h.shape[0], ho, ho, co)
        f = h.reshape(h.shape[0], -1)
        out = f @ Wf.T + bf
        logits.append(out)
        d = (2.0 / (6 * c["batch"])) * (out - s.labels[n:n + 32].to(F64))
        G[off:off + 6 * feat] += (d.T @ f).reshape(-1)
        G[off + 6 * feat:] += d.sum(0)
        dy = (d @ Wf).reshape(keep[-1][2].shape)
        for li in range(len(par) - 1, -1, -1):
            o, co, row, K = par[li]
            shape, col, y = keep[li]
            dz = dy * (y > 0)
            blk = G[o:o + co * row].view(co, row)
            blk[:, :K] += dz.T @ col
            blk[:, K] += dz.sum(0)
            if li:
                W = Pb[o:o + co * row].view(co, row)[:, :K]
                dy = _col2im(dz @ W, shape, 2).reshape(keep[li - 1][2].shape)
    new = P - 1e-3 * G / (G.abs() + 1e-8)  # Adam's first step
    return {"logits": torch.cat(logits), "grad": G, "params": new}


def exact(case, seed):
    c = case
    limit = {"drr": 3e10, "drr_grad": 8e9, "ssd": 8e9}.get(c["kind"])
    if limit is not None and _sample_slots(c) > limit:
        return None
    if c["kind"] in ("fdk", "bp", "bp_grad", "fp_fwd", "fp_bp"):
        cost = c["nx"] * c["ny"] * c["nz"] * c["views"] * {"fdk": 1, "bp": 1, "bp_grad": 2}.get(c["kind"], 15)
        if cost > 3e10:
            return None
    s = prepare(case, seed)
    if c["kind"] == "conv":
        return _exact_conv(s)
    if c["kind"] == "train":
        return _exact_train(s)
    if c["kind"] in ("drr", "drr_grad", "ssd"):
        return _exact_rays(s)
    if c["kind"] == "fdk":
        q = _exact_filter(s.g, s.img, math.pi / c["views"])
        return {"filtered": q, "vol": _exact_bp(s.g, s, q, True)}
    if c["kind"] == "bp":
        return _exact_bp(s.g, s, s.img, c["weight"] == dp.W_FDK)
    if c["kind"] == "bp_grad":
        return _exact_bp_grad(s.g, s, c["weight"] == dp.W_FDK)
    return _exact_fp(s)
