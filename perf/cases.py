"""The workloads this library is timed on: each case is a call, or a short
sequence of calls, that a program using the library makes through its public
entry points, from the smallest requests to the benchmark's room.

A case is a dict of plain values whose ``kind`` says which calls it makes:

  bake       a bake request over a contiguous run of a room's camera points
  step       the benchmark's whole step: shading points, plan order, bake,
             fused loss and grid gradient
  rebake     one turn of the emitter loop: emission medians, emission upload,
             bake
  voxel      stage 1 with the voxel radiance cache: pooling, set-up, bake
  refine     the stage-3 refinement under a material grid
  grid_step  the fused loss-and-gradient step over plan-ordered points
  masked     grid fetch, emission-masked loss with the diffuse prior, and
             their backward passes, through autograd
  hash_fwd   inference with the hash-grid material network
  hash_train a training step of that network: forward, loss, backward

Rooms, cameras, roughness levels and sample counts are those of ``synth``;
every input is drawn from the seed.
"""
import dataclasses
import functools
import math

import numpy as np
import torch

import synth
from paper_2304_05669_amd import fipt

SIGMA = tuple(float(s) for s in np.asarray(synth.SIGMA_GRID, np.float32))
K = len(SIGMA)
PLANES = 3 + 6 * K
CAM_W, CAM_H = 320, 240                 # the rooms' camera size
# flops per lobe sample of a bake: the traversal's slab and triangle tests and
# the sampling, as the instrumented kernel counts them on the room
FLOPS_PER_SAMPLE = 1100.0
HG_FLOPS_PER_POINT = 2.0 * (64 * 64 + 64 * 64 + 5 * 64)
HG_TABLE = 32 * (1 << 19) * 2
HG_READS_PER_POINT = 161                # table entries of nonzero weight per point, measured on the room


def listed():
    return [
        # the smallest bake of the tests and of smoke(): one 64 x 64 camera
        # in the 20-triangle box
        dict(name="bake_tiny", kind="bake", room="tiny", points=4096, spp_d=64, spp_s=64, cache="triangle"),
        # the smallest request of the serving trace, odd in every size
        dict(name="bake_request", kind="bake", room="r2", points=10007, spp_d=37, spp_s=17, cache="vertex"),
        # the benchmark's step on the benchmark's room
        dict(name="room_step", kind="step", room="room", cams=24, spp=128, res=128),
        # the emitter loop's re-bake (256 samples per lobe) on a room of half a
        # million triangles
        dict(name="rebake", kind="rebake", room="r5", points=250000, spp=256),
        # stage 1 as the paper describes it: pixels pooled onto 256^3 voxels
        dict(name="voxel_stage", kind="voxel", room="r2", points=614400, spp=16, res=256),
        # stage 3 on part of a room
        dict(name="refine", kind="refine", room="room", points=76800, spp=64, res=128),
        # a training batch of the paper's size (8192 pixels) on a small grid,
        # with the tone map of Eq. 15
        dict(name="grid_step_batch", kind="grid_step", points=8192, res=32, tone=1),
        # every pixel of the benchmark's room at once, with that tone map
        dict(name="grid_step_room", kind="grid_step", points=1843200, res=128, tone=1),
        # the emission-masked loss with the diffuse prior on an odd point count
        dict(name="masked", kind="masked", points=600001, res=64, tone=1),
        # the material network evaluated at every pixel of the room
        dict(name="hash_forward", kind="hash_fwd", points=1843200),
        # its training step: a batch of the paper's size, and the whole room
        dict(name="hash_train_batch", kind="hash_train", points=8192),
        dict(name="hash_train_room", kind="hash_train", points=1843200),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["bake", "bake", "step", "rebake", "voxel", "refine", "grid_step", "grid_step", "masked",
                       "hash_fwd", "hash_train", "hash_train"])
    if kind == "bake":
        # requests of the serving trace, and smaller ones
        n, spp = _log(rng, 1000, 300000), _log(rng, 16, 256)
        spp = max(16, min(spp, int(2e8 / (n * (K + 1)))))
        return dict(kind=kind, room=rng.choice(["tiny", "r0", "r1", "r2", "room", "r4"]), points=n, spp_d=spp,
                    spp_s=max(1, int(spp * rng.uniform(0.4, 1.0))), cache=rng.choice(["vertex", "triangle"]))
    if kind == "step":
        return dict(kind=kind, room=rng.choice(["r0", "r1", "r2", "room", "r4"]), cams=rng.randint(1, 8),
                    spp=_log(rng, 16, 128), res=rng.choice([32, 64, 128]))
    if kind == "rebake":
        return dict(kind=kind, room=rng.choice(["room", "r4", "r5"]), points=_log(rng, 20000, 250000),
                    spp=_log(rng, 32, 256))
    if kind == "voxel":
        return dict(kind=kind, room=rng.choice(["r0", "r1", "r2", "room"]), points=_log(rng, 10000, 614400),
                    spp=_log(rng, 8, 32), res=rng.choice([64, 100, 128, 200, 256]))
    if kind == "refine":
        return dict(kind=kind, room=rng.choice(["r0", "r2", "room"]), points=_log(rng, 2000, 76800),
                    spp=_log(rng, 8, 64), res=rng.choice([32, 64, 128]))
    if kind == "grid_step":
        return dict(kind=kind, points=_log(rng, 1000, 1843200), res=rng.choice([32, 64, 100, 128]),
                    tone=rng.randint(0, 1))
    if kind == "masked":
        return dict(kind=kind, points=_log(rng, 1000, 1000000), res=rng.choice([32, 64, 100, 128]),
                    tone=rng.randint(0, 1))
    return dict(kind=kind, points=_log(rng, 1000, 1843200))


# ---- inputs ------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


@functools.lru_cache(maxsize=8)
def _mesh(room, seed, n_cams):
    """The tiny box, the benchmark's room or room i of the serving set ("ri"),
    its geometry, emission and cameras drawn from the seed."""
    if room == "tiny":
        return synth.tiny_box(seed=seed)
    if room == "room":
        return synth.room(seed=seed, n_cams=n_cams)
    return synth.serving_rooms(seed=seed, n_cams=n_cams, which=[int(room[1:])])[0]


def _scene(room, seed, n_cams, cache="vertex"):
    """The resident scene with its radiance set, and the mesh it came from."""
    sc = _mesh(room, 1000 + seed % 100000, n_cams)
    scene = fipt.Scene(sc.verts, sc.tris, device=0)
    em = torch.from_numpy(sc.emission).cuda()
    n = sc.n_verts if cache == "vertex" else sc.n_tris
    rad = 2.0 * torch.rand((3, n), generator=_gen(seed + 1), device="cuda")
    scene.set_radiance(rad, fipt.CACHE_VERTEX if cache == "vertex" else fipt.CACHE_TRIANGLE, em)
    return scene, sc, em


def _cams_for(points):
    return max(1, -(-points // (CAM_W * CAM_H)))


def _points(scene, sc, points):
    """`points` shading points as one run of the cameras' pixels."""
    cams = sc.cameras
    have = sum(c.width * c.height for c in cams)
    if have < points:      # the tiny box has one small camera: a larger one
        side = int(math.ceil(math.sqrt(points)))
        cams = [dataclasses.replace(cams[0], width=side, height=side)]
        have = side * side
    planes, tri = fipt.fipt_gen_points(scene, cams)
    first = (have - points) // 2
    return planes[:, first:first + points].contiguous(), tri[first:first + points].contiguous()


def _surface(points, seed):
    """Positions of `points` pixels of a room, and the room's box."""
    scene, sc, _ = _scene("r0", seed, _cams_for(points))
    planes, _ = _points(scene, sc, points)
    pos = planes[0:3].contiguous()
    torch.cuda.synchronize()
    scene.destroy()
    return pos, sc.bmin.tolist(), sc.bmax.tolist()


def _shading(n, g):
    """Shading planes with the ranges of baked ones."""
    s = torch.rand((PLANES, n), generator=g, device="cuda")
    s[0:3] *= 2.0
    s[3:3 + 3 * K] *= 1.5
    s[3 + 3 * K:] *= 0.3
    return s


def _grid(res, g):
    """A material grid: albedo and metallic U[0, 1], roughness U[0.02, 1]."""
    m = torch.rand((5, res, res, res), generator=g, device="cuda")
    m[3] = 0.02 + 0.98 * m[3]
    return m


def _hash_params(g):
    """A network in training, every level contributing: tables U(-1, 1),
    weights N(0, 1/16).  (At its start, tables of 1e-4, every roughness lies
    within rounding of 1/2, a level of the shading table where the gradient
    of the lerp jumps.)"""
    p = torch.empty(fipt.HG_PARAMS, device="cuda")
    p[:HG_TABLE] = 2.0 * torch.rand(HG_TABLE, generator=g, device="cuda") - 1.0
    p[HG_TABLE:] = torch.randn(fipt.HG_PARAMS - HG_TABLE, generator=g, device="cuda") / 4.0
    return p


def _mask(n, g):
    """Emission mask: small values, and 0.5 to 1 on one pixel in twenty."""
    a = 0.02 * torch.rand(n, generator=g, device="cuda") ** 2
    on = torch.rand(n, generator=g, device="cuda") < 0.05
    return torch.where(on, 0.5 + 0.5 * torch.rand(n, generator=g, device="cuda"), a)


def prepare(case, seed):
    kind = case["kind"]
    st = {"kind": kind, "case": case, "seed": int(seed)}
    g = _gen(seed)
    if kind == "bake":
        scene, sc, _ = _scene(case["room"], seed, _cams_for(case["points"]), case["cache"])
        st["scene"] = scene
        st["planes"], st["tri"] = _points(scene, sc, case["points"])
        st["out"] = torch.empty((PLANES, case["points"]), device="cuda")
    elif kind == "step":
        scene, sc, _ = _scene(case["room"], seed, case["cams"])
        planes, tri = fipt.fipt_gen_points(scene, sc.cameras)
        n = tri.shape[0]
        bmin, bmax = sc.bmin.tolist(), sc.bmax.tolist()
        plan = fipt.GridPlan(planes[0:3].cpu().numpy(), case["res"], bmin, bmax)
        st.update(scene=scene, cams=sc.cameras, planes=planes, tri=tri, plan=plan,
                  planes_q=torch.empty_like(planes), tri_q=torch.empty_like(tri),
                  shading=torch.empty((PLANES, n), device="cuda"), grid=_grid(case["res"], g),
                  obs=2.0 * torch.rand((3, n), generator=g, device="cuda"),
                  loss=torch.empty((fipt.LOSS_SLOTS,), dtype=torch.float64, device="cuda"))
        st["grad"] = torch.empty_like(st["grid"])
    elif kind == "rebake":
        scene, sc, em = _scene(case["room"], seed, _cams_for(case["points"]))
        planes, tri = _points(scene, sc, case["points"])
        th = tri.cpu().numpy()
        lit = torch.from_numpy(np.any(sc.emission > 0, axis=0).astype(np.uint8)).cuda()
        obs = torch.from_numpy(synth.emitter_observations(sc.emission, th, seed=2106 + seed)).cuda()
        st.update(scene=scene, planes=planes, tri=tri, lit=lit, obs=obs,
                  eplan=fipt.EmissionPlan(th, sc.n_tris), le=torch.empty_like(em),
                  out=torch.empty((PLANES, case["points"]), device="cuda"))
    elif kind == "voxel":
        scene, sc, em = _scene(case["room"], seed, _cams_for(case["points"]))
        planes, tri = _points(scene, sc, case["points"])
        st.update(scene=scene, planes=planes, tri=tri, em=em, bmin=sc.bmin.tolist(), bmax=sc.bmax.tolist(),
                  vplan=fipt.VoxelPlan(planes[0:3].cpu().numpy(), case["res"], sc.bmin.tolist(), sc.bmax.tolist()),
                  obs=2.0 * torch.rand((3, case["points"]), generator=g, device="cuda"),
                  cache=torch.empty((3, case["res"] ** 3), device="cuda"),
                  out=torch.empty((PLANES, case["points"]), device="cuda"))
    elif kind == "refine":
        scene, sc, _ = _scene(case["room"], seed, _cams_for(case["points"]))
        st["planes"], st["tri"] = _points(scene, sc, case["points"])
        st.update(scene=scene, bmin=sc.bmin.tolist(), bmax=sc.bmax.tolist(), grid=_grid(case["res"], g),
                  out=torch.empty((PLANES, case["points"]), device="cuda"))
    elif kind in ("grid_step", "masked"):
        n = case["points"]
        pos, bmin, bmax = _surface(n, seed)
        st.update(plan=fipt.GridPlan(pos.cpu().numpy(), case["res"], bmin, bmax), pos=pos, bmin=bmin, bmax=bmax,
                  grid=_grid(case["res"], g), shading=_shading(n, g),
                  obs=2.0 * torch.rand((3, n), generator=g, device="cuda"))
        if kind == "grid_step":
            st["loss"] = torch.empty((fipt.LOSS_SLOTS,), dtype=torch.float64, device="cuda")
            st["grad"] = torch.empty_like(st["grid"])
        else:
            st["grid"].requires_grad_(True)
            st["alpha"] = _mask(n, g).requires_grad_(True)
    else:
        n = case["points"]
        st["pos"], st["bmin"], st["bmax"] = _surface(n, seed)
        st["params"] = _hash_params(g)
        if kind == "hash_train":
            st["plan"] = fipt.HashGridPlan(st["pos"], st["bmin"], st["bmax"])
            st["params"].requires_grad_(True)
            st["shading"] = _shading(n, g)
            st["obs"] = 2.0 * torch.rand((3, n), generator=g, device="cuda")
        else:
            st["out"] = torch.empty((5, n), device="cuda")
    return st


# ---- the calls ---------------------------------------------------------------
def run(st):
    kind, case = st["kind"], st["case"]
    if kind == "bake":
        return fipt.fipt_bake(st["scene"], st["planes"], st["tri"], case["spp_d"], case["spp_s"], SIGMA, st["seed"],
                              out=st["out"])
    if kind == "step":
        n = st["tri"].shape[0]
        fipt.fipt_gen_points(st["scene"], st["cams"], planes=st["planes"], tri=st["tri"])
        st["plan"].permute(st["planes"], out=st["planes_q"])
        st["plan"].permute(st["tri"].view(1, n), out=st["tri_q"].view(1, n))
        fipt.fipt_bake(st["scene"], st["planes_q"], st["tri_q"], case["spp"], case["spp"], SIGMA, st["seed"],
                       out=st["shading"])
        buf, grad = st["plan"].render_loss(st["grid"], st["shading"], st["obs"], SIGMA, loss_buf=st["loss"],
                                           grad_grid=st["grad"])
        return {"planes": st["planes"], "tri": st["tri"], "shading": st["shading"], "loss": buf[0], "grad": grad}
    if kind == "rebake":
        le = st["eplan"].median(st["obs"], st["lit"], out=st["le"])
        st["scene"].set_emission(le)
        sh = fipt.fipt_bake(st["scene"], st["planes"], st["tri"], case["spp"], case["spp"], SIGMA, st["seed"],
                            out=st["out"])
        return {"le": le, "shading": sh}
    if kind == "voxel":
        cache = st["vplan"].pool(st["obs"], out=st["cache"])
        st["scene"].set_voxel_radiance(cache, case["res"], st["bmin"], st["bmax"], st["em"])
        sh = fipt.fipt_bake(st["scene"], st["planes"], st["tri"], case["spp"], case["spp"], SIGMA, st["seed"],
                            out=st["out"])
        return {"cache": cache, "shading": sh}
    if kind == "refine":
        return fipt.fipt_refine(st["scene"], st["planes"], st["tri"], case["spp"], case["spp"], SIGMA, st["seed"],
                                st["grid"], st["bmin"], st["bmax"], out=st["out"])
    if kind == "grid_step":
        buf, grad = st["plan"].render_loss(st["grid"], st["shading"], st["obs"], SIGMA, case["tone"],
                                           loss_buf=st["loss"], grad_grid=st["grad"])
        return {"loss": buf[0], "grad": grad}
    if kind == "masked":
        st["grid"].grad = st["alpha"].grad = None
        mat = fipt.GridGather.apply(st["grid"], st["plan"], st["bmin"], st["bmax"], st["pos"])
        loss = fipt.MaskedFactoredLoss.apply(mat, st["alpha"], st["shading"], st["obs"], SIGMA, case["tone"], 5e-4)
        loss.backward()
        return {"loss": loss.detach(), "grad": st["grid"].grad, "grad_alpha": st["alpha"].grad}
    if kind == "hash_fwd":
        return fipt.fipt_hashgrid_forward(st["params"], st["pos"], st["bmin"], st["bmax"], out=st["out"])
    st["params"].grad = None
    mat = fipt.HashGridMaterial.apply(st["params"], st["plan"])
    loss = fipt.FactoredLoss.apply(mat, st["shading"], st["obs"], SIGMA)
    loss.backward()
    return {"material": mat.detach(), "loss": loss.detach(), "grad": st["params"].grad}


def work(case):
    kind = case["kind"]
    if kind in ("bake", "rebake", "voxel", "refine", "step"):
        n = case["cams"] * CAM_W * CAM_H if kind == "step" else case["points"]
        samples = n * (case["spp_d"] + K * case["spp_s"] if kind == "bake" else case["spp"] * (K + 1))
        by = n * (40 + 4 * PLANES)
        if kind == "step":
            by += n * 12 + 2 * 20 * case["res"] ** 3
        elif kind == "rebake":
            by += 12 * n
        elif kind == "voxel":
            by += 16 * n + 12 * case["res"] ** 3
        elif kind == "refine":
            by += 20 * case["res"] ** 3
        return {"bytes": float(by), "flops": FLOPS_PER_SAMPLE * samples}
    n = case["points"]
    if kind in ("grid_step", "masked"):
        # position, Ld, the two bracketing levels, observation (and the mask
        # and its gradient); the grid and its gradient
        per = 84 + (8 if kind == "masked" else 0)
        return {"bytes": float(per * n + 2 * 20 * case["res"] ** 3), "flops": 400.0 * n}
    table = min(4.0 * HG_TABLE, 8.0 * HG_READS_PER_POINT * n)
    if kind == "hash_fwd":
        return {"bytes": table + 32.0 * n, "flops": n * (HG_FLOPS_PER_POINT + 4.0 * HG_READS_PER_POINT)}
    # the step: tables and positions in, the loss's 72 bytes per point in,
    # material out, the whole parameter gradient out
    return {"bytes": table + 104.0 * n + 4.0 * fipt.HG_PARAMS,
            "flops": n * 3.0 * (HG_FLOPS_PER_POINT + 4.0 * HG_READS_PER_POINT)}


# ---- the same values in 64 bits ----------------------------------------------
def _gather64(grid, pos, bmin, bmax):
    """Trilinear values of grid [C, R, R, R] at pos [3, n], float64."""
    R = grid.shape[1]
    flat = grid.reshape(grid.shape[0], -1)
    lo = torch.tensor(bmin, dtype=torch.float32, device="cuda").double()[:, None]
    hi = torch.tensor(bmax, dtype=torch.float32, device="cuda").double()[:, None]
    u = torch.clamp((pos.double() - lo) * ((R - 1) / (hi - lo)), 0.0, R - 1.0)
    c = torch.clamp(torch.floor(u), max=R - 2.0)
    f = u - c
    c = c.long()
    out = 0.0
    for k in range(8):
        d = (k & 1, (k >> 1) & 1, k >> 2)
        w = 1.0
        for a in range(3):
            w = w * (f[a] if d[a] else 1.0 - f[a])
        idx = (c[0] + d[0]) + R * ((c[1] + d[1]) + R * (c[2] + d[2]))
        out = out + w * flat[:, idx]
    return out


def _tone64(x, tone):
    if not tone:
        return x
    u = torch.log1p(torch.clamp(x, min=0.0))
    safe = torch.clamp(u, min=0.0031308)
    return torch.where(u <= 0.0031308, 12.92 * u, 1.055 * safe ** (1.0 / 2.4) - 0.055)


def _loss64(mat, sh, obs, tone, alpha=None, lam=0.0):
    sig = torch.tensor(SIGMA, dtype=torch.float64, device="cuda")
    a, s, m = mat[0:3], mat[3], mat[4]
    j = torch.clamp(torch.searchsorted(sig, s.detach().contiguous(), right=True) - 1, 0, K - 2)
    t = torch.clamp((s - sig[j]) / (sig[j + 1] - sig[j]), 0.0, 1.0)
    n = s.shape[0]
    at = torch.arange(n, device="cuda")
    l0, l1 = sh[3:3 + 3 * K].reshape(K, 3, n), sh[3 + 3 * K:].reshape(K, 3, n)

    def lerp(tab):
        return (1.0 - t) * tab[j, :, at].t().double() + t * tab[j + 1, :, at].t().double()

    r = a * (1.0 - m) * sh[0:3].double() + (0.04 * (1.0 - m) + a * m) * lerp(l0) + lerp(l1)
    y = obs.double()
    h = r if alpha is None else (1.0 - alpha) * r + alpha * y
    loss = ((_tone64(h, tone) - _tone64(y, tone)) ** 2).sum()
    if lam:
        loss = loss + lam * ((1.0 - s).abs().sum() + m.abs().sum())
    return loss


def _hash_levels(pos, bmin, bmax):
    """Per level: table slots [8, n] and trilinear weights [8, n] (float64)."""
    lo = torch.tensor(bmin, dtype=torch.float32, device="cuda")[:, None]
    hi = torch.tensor(bmax, dtype=torch.float32, device="cuda")[:, None]
    p = torch.clamp((pos - lo) * (1.0 / (hi - lo)), 0.0, 1.0)
    for lv in range(32):
        nl = float(16 * 2 ** lv)
        u = p * nl
        c = torch.minimum(torch.floor(u), torch.full_like(u, nl - 1.0))
        f = (u - c).double()
        c = c.double().long()
        idx, wgt = [], []
        for k in range(8):
            d = (k & 1, (k >> 1) & 1, k >> 2)
            x, y, z = (c[q] + d[q] for q in range(3))
            if lv < 3:
                r = (16 << lv) + 1
                idx.append(x + y * r + z * r * r)
            else:
                idx.append((x ^ (y * 2654435761) ^ (z * 805459861)) & ((1 << 19) - 1))
            wgt.append((f[0] if d[0] else 1 - f[0]) * (f[1] if d[1] else 1 - f[1]) * (f[2] if d[2] else 1 - f[2]))
        yield lv, torch.stack(idx), torch.stack(wgt)


def _hash64(st):
    """Encoding and weights in float64: enc [64, n], W1, W2, W3."""
    p = st["params"].detach()
    n = st["pos"].shape[1]
    tab = p[:HG_TABLE].reshape(32, 1 << 19, 2)
    enc = torch.empty((64, n), dtype=torch.float64, device="cuda")
    for lv, idx, w in _hash_levels(st["pos"], st["bmin"], st["bmax"]):
        for ft in range(2):
            enc[2 * lv + ft] = sum(w[k] * tab[lv, :, ft][idx[k]].double() for k in range(8))
    w1 = p[HG_TABLE:HG_TABLE + 4096].reshape(64, 64).double()
    w2 = p[HG_TABLE + 4096:HG_TABLE + 8192].reshape(64, 64).double()
    w3 = p[HG_TABLE + 8192:].reshape(5, 64).double()
    return enc, w1, w2, w3


def exact(case, seed):
    kind = case["kind"]
    if kind in ("bake", "step", "rebake", "refine"):
        return None     # Monte Carlo over brute-force ray casts: hours
    st = prepare(case, seed)
    if kind == "voxel":
        R = case["res"]
        lo = torch.tensor(st["bmin"], device="cuda").double()[:, None]
        hi = torch.tensor(st["bmax"], device="cuda").double()[:, None]
        v = torch.clamp(torch.floor((st["planes"][0:3].double() - lo) * R / (hi - lo)), 0, R - 1).long()
        v = (v[2] * R + v[1]) * R + v[0]
        cnt = torch.bincount(v, minlength=R ** 3).clamp(min=1).double()
        cache = torch.zeros((3, R ** 3), dtype=torch.float64, device="cuda")
        cache.index_add_(1, v, st["obs"].double())
        return {"cache": cache / cnt, "shading": None}
    if kind in ("grid_step", "masked"):
        grid = st["grid"].detach().double().requires_grad_(True)
        pos, alpha, lam = st["pos"], None, 0.0
        if kind == "grid_step":
            # shading and observations are in the plan's order
            order = torch.from_numpy(st["plan"].order().astype(np.int64)).cuda()
            pos = pos[:, order]
        else:
            alpha, lam = st["alpha"].detach().double().requires_grad_(True), 5e-4
        # the fetched material is stored in single precision
        mat = _gather64(grid, pos, st["bmin"], st["bmax"])
        mat = mat + (mat.detach().float().double() - mat.detach())
        loss = _loss64(mat, st["shading"], st["obs"], case["tone"], alpha, lam)
        loss.backward()
        out = {"loss": loss.detach(), "grad": grid.grad}
        return out if alpha is None else {**out, "grad_alpha": alpha.grad}
    enc, w1, w2, w3 = _hash64(st)
    if kind == "hash_fwd":
        return torch.sigmoid(w3 @ torch.relu(w2 @ torch.relu(w1 @ enc)))
    for t in (enc, w1, w2, w3):
        t.requires_grad_(True)
    mat = torch.sigmoid(w3 @ torch.relu(w2 @ torch.relu(w1 @ enc)))
    loss = _loss64(mat, st["shading"], st["obs"], 0)
    loss.backward()
    grad = torch.zeros(fipt.HG_PARAMS, dtype=torch.float64, device="cuda")
    tab = grad[:HG_TABLE].view(32, 1 << 19, 2)
    for lv, idx, w in _hash_levels(st["pos"], st["bmin"], st["bmax"]):
        ge = enc.grad[2 * lv:2 * lv + 2].t()
        for k in range(8):
            tab[lv].index_add_(0, idx[k], w[k][:, None] * ge)
    grad[HG_TABLE:] = torch.cat([w1.grad.reshape(-1), w2.grad.reshape(-1), w3.grad.reshape(-1)])
    return {"material": mat.detach(), "loss": loss.detach(), "grad": grad}
