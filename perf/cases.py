"""Workloads of the intersector, each through its public entry points: what is timed, on which inputs, and what comes back.

A case is a dict of plain values; its "kind" names the work:

  trace     closest hits of one or two ray sets (pinhole primary rays, cosine-weighted secondary rays)
  playback  an animation: every frame's geometry moved, then all frames' rays in one batched launch
  path      a path tracer's frame: primary hits, then bounce / compaction / hits per level
  compact   compaction of a bounce level's rays
  order     the ordering network's records and logits on the hits of a ray set
  train     optimizer steps of the ordering network

Scenes are those of the repository's synthetic workloads, generated on the GPU from the seed: displaced tori (32 x 16 cage, 512 patches,
10 % Gregory) and fields of randomly placed, scaled and turned tori (25 x 20 cages, 25 % Gregory)."""
import math

import numpy as np
import torch

from paper_1811_03510_amd import ccs

DEV = "cuda"
F64 = torch.float64
INNER, PV = [5, 6, 9, 10], [16, 17, 18, 19]


# --------------------------------------------------------------------- the cases
def listed():
    return [
        # picking, a probe's few rays: one small call, its latency counts
        {"name": "pick_1k", "kind": "trace", "objects": 1, "depth": 12, "local": True, "w": 32, "h": 32, "secondary": 0, "learned": False},
        # a preview image: the 512-patch torus, both ray classes in one launch
        {"name": "preview_32k", "kind": "trace", "objects": 1, "depth": 12, "local": True, "w": 128, "h": 128, "secondary": 16384, "learned": False},
        # close-up at a fine leaf size (64-bit path words), an odd number of rays
        {"name": "deep_l18", "kind": "trace", "objects": 1, "depth": 18, "local": True, "w": 201, "h": 133, "secondary": 0, "learned": False},
        # world frames (the default of a scene), a field of objects, a ragged image with one secondary ray per pixel
        {"name": "world_460k", "kind": "trace", "objects": 200, "depth": 10, "local": False, "w": 641, "h": 361, "secondary": 231401, "learned": False},
        # the learned child order on the same kind of scene
        {"name": "learned_260k", "kind": "trace", "objects": 200, "depth": 10, "local": True, "w": 480, "h": 270, "secondary": 129600, "learned": True},
        # the full frame of the benchmark: 1M patches, 1920 x 1080 primary rays and as many secondary ones
        {"name": "frame_1m", "kind": "trace", "objects": 2000, "depth": 10, "local": True, "w": 1920, "h": 1080, "secondary": 2073600, "learned": False},
        # animation playback of a small model: 16 refits, 16 uneven ray batches
        {"name": "playback_512", "kind": "playback", "objects": 1, "depth": 12, "local": True, "frames": 16, "rays": 24001},
        # animation playback of a large model: the refit's own share is large
        {"name": "playback_200k", "kind": "playback", "objects": 400, "depth": 10, "local": True, "frames": 2, "rays": 360000},
        # a path tracer's frame: 1280 x 720, two bounces, each level compacted
        {"name": "path_720p", "kind": "path", "objects": 400, "depth": 10, "local": True, "w": 1280, "h": 720, "bounces": 2},
        # compaction of a 4K bounce level, most paths ended
        {"name": "compact_4k", "kind": "compact", "n": 8294399, "active": 0.3},
        # records of the ordering network on 65,537 rays' hits and its logits on them (evaluation of a network)
        {"name": "order_65k", "kind": "order", "objects": 1, "depth": 12, "local": True, "rays": 65537},
        # training of the ordering network at the benchmark's batch size
        {"name": "train_100", "kind": "train", "rows": 400000, "steps": 100, "batch": 8192, "bf16": True},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["trace", "trace", "trace", "trace", "playback", "path", "compact", "order", "train"])
    objects = 1 if rng.random() < 0.4 else _log(rng, 8, 400)
    depth = 12 if objects == 1 else 10
    local = rng.random() < 0.7
    if kind == "trace":
        depth = rng.choice([8, 10, 12, 14, 18]) if objects == 1 else rng.choice([9, 10, 11])
        n = _log(rng, 256, 600000)
        w = max(8, int(math.sqrt(n * rng.uniform(1.0, 1.8))))
        return {"kind": kind, "objects": objects, "depth": depth, "local": local, "w": w, "h": max(1, n // w),
                "secondary": rng.choice([0, n, _log(rng, 64, 300000)]), "learned": depth <= 16 and rng.random() < 0.2}
    if kind == "playback":
        return {"kind": kind, "objects": objects, "depth": depth, "local": local, "frames": rng.randint(2, 16) if objects < 50 else rng.randint(1, 3),
                "rays": _log(rng, 2000, 300000 if objects < 50 else 400000) // (8 if objects < 50 else 1)}
    if kind == "path":
        n = _log(rng, 4000, 900000)
        w = int(math.sqrt(n * 1.78))
        return {"kind": kind, "objects": objects, "depth": depth, "local": local, "w": w, "h": max(1, n // w), "bounces": rng.randint(1, 3)}
    if kind == "compact":
        return {"kind": kind, "n": _log(rng, 1000, 8000000), "active": round(rng.uniform(0.05, 1.0), 3)}
    if kind == "order":
        return {"kind": kind, "objects": objects, "depth": depth, "local": local, "rays": _log(rng, 1000, 100000)}
    return {"kind": kind, "rows": _log(rng, 20000, 800000), "steps": rng.randint(8, 100), "batch": rng.choice([1000, 2048, 4096, 8192]),
            "bf16": rng.random() < 0.7}


# --------------------------------------------------------------- scenes and rays
def _gen(seed, k=0):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 64 + k)


def _rand(g, *shape):
    return torch.rand(shape, generator=g, device=DEV, dtype=F64)


def _randn(g, *shape):
    return torch.randn(shape, generator=g, device=DEV, dtype=F64)


def _ring(nt, np_):
    t = 2 * math.pi * torch.arange(nt, device=DEV, dtype=F64) / nt
    p = 2 * math.pi * torch.arange(np_, device=DEV, dtype=F64) / np_
    T, P = torch.meshgrid(t, p, indexing="ij")
    nrm = torch.stack((P.cos() * T.cos(), P.cos() * T.sin(), P.sin()), -1)
    return torch.stack((T.cos(), T.sin(), torch.zeros_like(T)), -1), nrm


def _bezier(cage):
    """Periodic bicubic B-spline cages (n, nu, nv, 3) to Bezier grids (n * nu * nv, 16, 3), slot 4 j + i."""
    def along(x, dim):
        m, p, q = x.roll(1, dim), x.roll(-1, dim), x.roll(-2, dim)
        return torch.stack(((m + 4 * x + p) / 6, (2 * x + p) / 3, (2 * p + x) / 3, (x + 4 * p + q) / 6), -2)
    U = along(cage, 1)                                     # (n, nu, nv, 4, 3)
    P = along(U, 2)                                        # (n, nu, nv, 4, 4, 3): [i][j]
    return P.transpose(-3, -2).reshape(-1, 16, 3)


def _patches(objects, seed):
    """Control points (n, 20, 3) fp64, types (n,) uint8, and the objects' bounding spheres (centre, radius)."""
    g = _gen(seed)
    nt, nph, frac = (32, 16, 0.10) if objects == 1 else (25, 20, 0.25)
    ring, nrm = _ring(nt, nph)
    if objects == 1:
        R, r = torch.full((1, 1, 1, 1), 1.0, device=DEV, dtype=F64), torch.full((1, 1, 1, 1), 0.35, device=DEV, dtype=F64)
    else:
        torus = _rand(g, objects, 1, 1, 1) < 0.5
        R, r = torch.where(torus, 1.0, 0.55).to(F64), torch.where(torus, 0.35, 0.5).to(F64)
    cage = R * ring + r * nrm + nrm * (0.02 * _randn(g, objects, nt, nph, 1))
    centre, scale = torch.zeros(objects, 3, device=DEV, dtype=F64), torch.ones(objects, device=DEV, dtype=F64)
    if objects > 1:
        scale = torch.exp(math.log(0.5) + math.log(4.0) * _rand(g, objects))
        q = _randn(g, objects, 4)
        w, x, y, z = (q / q.norm(dim=1, keepdim=True)).unbind(1)
        rot = torch.stack((1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y), 2 * (x * y + w * z), 1 - 2 * (x * x + z * z),
                           2 * (y * z - w * x), 2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)), 1).reshape(-1, 1, 1, 3, 3)
        centre = (2 * _rand(g, objects, 3) - 1) * _extent(objects)
        cage = (rot * cage.unsqueeze(-2)).sum(-1) * scale.view(-1, 1, 1, 1) + centre.view(-1, 1, 1, 3)
    grid = _bezier(cage)
    n = grid.shape[0]
    cp = torch.cat((grid, grid[:, INNER]), 1)
    types = torch.zeros(n, dtype=torch.uint8, device=DEV)
    sel = torch.randperm(n, generator=g, device=DEV)[: int(round(frac * n))]
    types[sel] = 1
    cell = sum((grid[sel, a] - grid[sel, b]).norm(dim=1) for a, b in ((3, 0), (15, 12), (12, 0), (15, 3))) / 4
    e = _randn(g, len(sel), 4, 3) * (0.05 * cell).view(-1, 1, 1)
    base = grid[sel][:, INNER]
    cp[sel.view(-1, 1), torch.tensor(INNER, device=DEV)] = base + e
    cp[sel.view(-1, 1), torch.tensor(PV, device=DEV)] = base - e
    return cp.to(torch.float32).contiguous(), types, centre, 1.7 * scale


def _extent(objects):
    return 40.0 * (objects / 2000.0) ** (1.0 / 3.0)  # the density of the 2000-object field


def _eye(objects):
    k = _extent(objects) / 40.0
    return ((0.0, -3.2, 2.0), 40.0) if objects == 1 else ((0.0, -110.0 * k, 30.0 * k), 50.0)


def _pinhole(eye, vfov, w, h, turn=0.0):
    """Rays from `eye` turned about z by `turn`, towards the origin."""
    c, s = math.cos(turn), math.sin(turn)
    eye = np.array([c * eye[0] - s * eye[1], s * eye[0] + c * eye[1], eye[2]])
    f = -eye / np.linalg.norm(eye)
    r = np.cross(f, (0.0, 0.0, 1.0))
    r /= np.linalg.norm(r)
    f, r, u = (torch.tensor(v, device=DEV, dtype=F64) for v in (f, r, np.cross(r, f)))
    th = math.tan(math.radians(vfov) / 2)
    x = (2 * (torch.arange(w, device=DEV, dtype=F64) + 0.5) / w - 1) * th * w / h
    y = (1 - 2 * (torch.arange(h, device=DEV, dtype=F64) + 0.5) / h) * th
    d = (f + x.view(1, -1, 1) * r + y.view(-1, 1, 1) * u).reshape(-1, 3)
    out = torch.zeros(len(d), 8, device=DEV, dtype=F64)
    out[:, :3] = torch.tensor(eye, device=DEV, dtype=F64)
    out[:, 4:7] = d / d.norm(dim=1, keepdim=True)
    out[:, 7] = math.inf
    return out.to(torch.float32)


def _bern(t):
    s = 1 - t
    return torch.stack((s * s * s, 3 * t * s * s, 3 * t * t * s, t * t * t), -1)


def _surface(g, greg, u, v):
    lam = torch.stack([torch.where(a + b > 0, a / (a + b).clamp_min(1e-300), 0.5) for b in (v, 1 - v) for a in (u, 1 - u)], 1)
    inner = torch.where(greg.view(-1, 1, 1), lam.unsqueeze(2) * (g[:, INNER] - g[:, PV]) + g[:, PV], g[:, INNER])
    g = g[:, :16].clone()
    g[:, INNER] = inner
    return ((_bern(v).unsqueeze(2) * _bern(u).unsqueeze(1)).reshape(-1, 16, 1) * g).sum(1)


def _secondary(cp, types, depth, eye, n, seed):
    """One cosine-weighted ray from each of n seeded surface points, the origin a leaf's size off the surface."""
    g, out = _gen(seed, 1), torch.zeros(n, 8, device=DEV, dtype=torch.float32)
    eye = torch.tensor(eye, device=DEV, dtype=F64)
    for b in range(0, n, 1 << 19):
        m = min(n - b, 1 << 19)
        idx = torch.randint(len(cp), (m,), generator=g, device=DEV)
        u, v, w1, w2 = 0.01 + 0.98 * _rand(g, m), 0.01 + 0.98 * _rand(g, m), _rand(g, m), _rand(g, m)
        p, greg, h = cp[idx].to(F64), types[idx] == 1, 1e-6
        x = _surface(p, greg, u, v)
        nrm = torch.linalg.cross(_surface(p, greg, u + h, v) - _surface(p, greg, u - h, v), _surface(p, greg, u, v + h) - _surface(p, greg, u, v - h))
        nrm = nrm / nrm.norm(dim=1, keepdim=True)
        nrm = nrm * torch.where(((eye - x) * nrm).sum(1, keepdim=True) < 0, -1.0, 1.0)
        sg = torch.where(nrm[:, 2] >= 0, 1.0, -1.0).to(F64)
        a = -1 / (sg + nrm[:, 2])
        c = nrm[:, 0] * nrm[:, 1] * a
        t1 = torch.stack((1 + sg * nrm[:, 0] ** 2 * a, sg * c, -sg * nrm[:, 0]), 1)
        t2 = torch.stack((c, sg + nrm[:, 1] ** 2 * a, -nrm[:, 1]), 1)
        r, phi = w1.sqrt(), 2 * math.pi * w2
        d = (r * phi.cos()).view(-1, 1) * t1 + (r * phi.sin()).view(-1, 1) * t2 + (1 - w1).sqrt().view(-1, 1) * nrm
        off = (p.amax(1) - p.amin(1)).sum(1, keepdim=True) * 2.0 ** -depth
        out[b:b + m, :3] = (x + off * nrm).to(torch.float32)
        out[b:b + m, 4:7] = (d / d.norm(dim=1, keepdim=True)).to(torch.float32)
    out[:, 7] = math.inf
    return out


def _moved(cp, f, frames, seed):
    """Frame f of an animation: a displacement that is a function of the rest position, so seams stay closed."""
    g = _gen(seed, 2)
    k = _randn(g, 3, 3)
    k = 2 * math.pi * k / k.norm(dim=1, keepdim=True)
    phase = 2 * math.pi * _rand(g, 3)
    amp = 0.05 * (cp[:, 3] - cp[:, 0]).norm(dim=1).mean().item()
    x = cp.to(F64)
    arg = (x.unsqueeze(2) * k).sum(-1) + phase + 2 * math.pi * f / frames
    return (x + amp * arg.sin()).to(torch.float32).contiguous()


def _network(seed):
    """A child-ordering network near the closest-first rule (the entry-distance input ranks the u-halves), with seeded noise."""
    g = _gen(seed, 3)
    W1, W2, W3 = 0.2 * _randn(g, 32, 16), 0.15 * _randn(g, 32, 32), 0.15 * _randn(g, 4, 32)
    W1[0], W1[1], W1[0, 12], W1[1, 12] = 0, 0, 8.0, -8.0
    W2[0], W2[1], W2[0, 0], W2[1, 1] = 0, 0, 1.0, 1.0
    W3[2:, 0], W3[:2, 1] = 1.0, 1.0
    z = torch.zeros(32, device=DEV, dtype=F64)
    return torch.cat([t.reshape(-1) for t in (W1, z, W2, z, W3, z[:4])]).to(torch.float32)


def _ray_sets(case, cp, types, seed):
    eye, fov = _eye(case["objects"])
    if case["kind"] == "order":
        return [_secondary(cp, types, case["depth"], eye, case["rays"], seed)]
    sets = [_pinhole(eye, fov, case["w"], case["h"], turn=0.37 * (seed % 17))]
    if case.get("secondary"):
        sets.append(_secondary(cp, types, case["depth"], eye, case["secondary"], seed))
    return sets


def _frames_of(case, cp, types, seed):
    """Per frame the moved control points and its rays: half primary from an orbiting camera, half secondary; uneven counts around the case's."""
    eye, fov = _eye(case["objects"])
    frames = []
    for f in range(case["frames"]):
        pts = _moved(cp, f, case["frames"], seed)
        n = max(64, int(case["rays"] * (0.25 + 1.5 * ((7 * f + 3) % 16) / 15)) if case["frames"] > 2 else case["rays"])
        side = max(8, int(math.sqrt(n / 2)))
        rays = torch.cat((_pinhole(eye, fov, side, side, 2 * math.pi * f / case["frames"]),
                          _secondary(pts, types, case["depth"], eye, max(1, n - side * side), seed + f)))
        frames.append((pts, rays))
    return frames


# ------------------------------------------------------------------- the passes
def _parts(hits):
    """Views of a hit array: distance, patch id, (u, v)."""
    return {"t": hits[:, 0], "id": hits.view(torch.int32)[:, 1], "uv": hits[:, 2:]}


def _hits(n):
    return torch.zeros(n, 4, device=DEV, dtype=torch.float32)


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": dict(case)}
    if kind == "compact":
        g, n = _gen(seed), case["n"]
        rays = torch.randn((n, 8), generator=g, device=DEV, dtype=torch.float32)
        on = torch.rand((n,), generator=g, device=DEV) < case["active"]
        rays[:, 3] = 0.0
        rays[:, 7] = torch.where(on, math.inf, -1.0)
        rays[~on, :3] = 0.0
        rays[~on, 4:7] = torch.tensor([0.0, 0.0, 1.0], device=DEV)
        return {**s, "rays": rays, "out": torch.zeros_like(rays), "index": torch.zeros(n, device=DEV, dtype=torch.int32),
                "work": torch.zeros(ccs.compact_work_words(n), device=DEV, dtype=torch.int32)}
    if kind == "train":
        g, n = _gen(seed), case["rows"]
        x = (2 * torch.rand((n, 16), generator=g, device=DEV) - 1).contiguous()
        y = (2 * (x[:, 12] + 0.3 * x[:, 0] > 0) + (x[:, 13] - 0.5 * x[:, 4] > 0)).to(torch.uint8)
        y[torch.rand((n,), generator=g, device=DEV) < 0.3] = ccs.NO_LABEL  # levels without a decision
        return {**s, "x": x, "y": y, "theta": _start_weights(seed)}
    cp, types, _, _ = _patches(case["objects"], seed)
    scene = ccs.Scene(cp, types, case["depth"], local_frames=case["local"])
    s["scene"] = scene
    if kind == "playback":
        scene.set_frames(case["frames"])
        s["frames"] = _frames_of(case, cp, types, seed)
        s["hits"] = [_hits(len(r)) for _, r in s["frames"]]
        return s
    s["rays"] = _ray_sets(case, cp, types, seed)
    s["hits"] = [_hits(len(r)) for r in s["rays"]]
    if kind == "trace" and case["learned"]:
        scene.set_policy(_network(seed))
    if kind == "path":
        g = _gen(seed, 4)
        n, m = len(s["rays"][0]), case["bounces"]
        s["uniforms"] = [torch.rand((n, 2), generator=g, device=DEV) for _ in range(m)]
        s["bounced"] = [torch.zeros(n, 8, device=DEV) for _ in range(m)]
        s["level"] = [torch.zeros(n, 8, device=DEV) for _ in range(m)]
        s["index"] = [torch.zeros(n, device=DEV, dtype=torch.int32) for _ in range(m)]
        s["work"] = torch.zeros(ccs.compact_work_words(n), device=DEV, dtype=torch.int32)
        s["hits"] += [_hits(n) for _ in range(m)]
    if kind == "order":
        scene.intersect(s["rays"][0], s["hits"][0])
        s["theta"] = _network(seed)
    return s


def run(s):
    case, kind = s["case"], s["case"]["kind"]
    if kind == "trace":
        if len(s["rays"]) == 1:
            s["scene"].intersect(s["rays"][0], s["hits"][0])
        else:
            s["scene"].intersect_batched([(0, r, h) for r, h in zip(s["rays"], s["hits"])])
        return [_parts(h) for h in s["hits"]]
    if kind == "playback":
        for f, (pts, _) in enumerate(s["frames"]):
            s["scene"].refit_frame(f, pts)
        s["scene"].intersect_batched([(f, r, h) for f, ((_, r), h) in enumerate(zip(s["frames"], s["hits"]))])
        return [_parts(h) for h in s["hits"]]
    if kind == "path":
        rays, n = s["rays"][0], len(s["rays"][0])
        hits, counts = s["scene"].intersect(rays, s["hits"][0]), []
        for k in range(case["bounces"]):
            bounced = s["scene"].bounce(rays, hits, s["uniforms"][k][:n], out=s["bounced"][k][:n])
            ccs.compact_rays(bounced, s["level"][k], s["index"][k], s["work"])
            n = int(s["work"][0].item())  # the next level's size, as a path tracer reads it
            rays = s["level"][k][:n]
            hits = s["scene"].intersect(rays, s["hits"][k + 1][:n])
            counts.append(n)
        return {"hits": [_parts(h) for h in s["hits"]], "rays": s["level"], "index": s["index"], "counts": counts}
    if kind == "compact":
        ccs.compact_rays(s["rays"], s["out"], s["index"], s["work"])
        return {"rays": s["out"], "index": s["index"], "count": s["work"][:1]}
    if kind == "order":
        features, labels = s["scene"].record(s["rays"][0], s["hits"][0])
        return {"features": features, "labels": labels, "logits": ccs.policy_infer(s["theta"], features)}
    theta = s["theta"].clone()
    loss = ccs.policy_train(theta, s["x"], s["y"], steps=case["steps"], batch=case["batch"], seed=5, bf16=case["bf16"])
    return {"theta": theta, "loss": loss}


def work(case):
    """Bytes read and written once; operations as this method's least arithmetic per ray (about 1.3 k per level of the leaf depth, measured by the work
    counters over the torus and the object fields; twice that in world frames)."""
    kind = case["kind"]
    if kind == "compact":
        return {"bytes": case["n"] * (32 + 36 * case["active"]), "flops": 10 * case["n"]}
    if kind == "train":
        rows = case["steps"] * min(case["batch"], case["rows"])
        return {"bytes": rows * 65 + case["steps"] * 4, "flops": rows * 6 * 1664}
    patches = 512 if case["objects"] == 1 else 500 * case["objects"]
    per_ray, touched = 1300 * case["depth"] * (1 if case["local"] else 2), 320
    if kind == "order":
        rows = case["rays"] * case["depth"]
        return {"bytes": case["rays"] * 48 + rows * (65 + 80) + min(patches, case["rays"]) * touched, "flops": rows * (1000 + 2 * 1664)}
    if kind == "playback":
        n = case["rays"] * case["frames"]
        return {"bytes": n * 48 + case["frames"] * patches * (240 + touched + 48), "flops": n * per_ray + case["frames"] * patches * 700}
    n = case["w"] * case["h"] + case.get("secondary", 0)
    if kind == "path":
        n += int(0.3 * n) * case["bounces"]
    return {"bytes": n * 48 + min(patches, n) * touched, "flops": n * per_ray}


def _start_weights(seed):
    """Seeded initial weights: uniform in +-sqrt(6 / fan-in), biases zero."""
    g = _gen(seed, 5)
    parts = []
    for rows, cols in ((32, 16), (32, 32), (4, 32)):
        parts += [((2 * _rand(g, rows, cols) - 1) * math.sqrt(6.0 / cols)).reshape(-1), torch.zeros(rows, device=DEV, dtype=F64)]
    return torch.cat(parts).to(torch.float32)


# ------------------------------------------------------- the same in 64 bits, plain
def _frames64(cp):
    """Patch frames: r0 along p30 - p00, r1 the part of p03 - p00 across it, r2 = r0 x r1."""
    eu, ev = cp[:, 3] - cp[:, 0], cp[:, 12] - cp[:, 0]
    r0 = eu / eu.norm(dim=1, keepdim=True)
    w = ev - (ev * r0).sum(1, keepdim=True) * r0
    r1 = w / w.norm(dim=1, keepdim=True)
    return torch.stack((r0, r1, torch.linalg.cross(r0, r1)), 1)


def _wbar(t0, t1, peak):
    t = torch.full_like(t0, peak).clamp(min=t0, max=t1)
    return 3 * t * (1 - t) ** 2 if peak < 0.5 else 3 * t * t * (1 - t)


def _crop(t0, t1):
    """(n, 4, 4): Bezier points to those of the restriction to [t0, t1]."""
    s0, s1, t = 1 - t0, 1 - t1, t1
    z = torch.zeros_like(t0)
    rows = []
    for k in range(4):  # blossom at (t0 x (3 - k), t1 x k)
        c = [torch.ones_like(t0), z, z, z]
        for a, b in [(s0, t0)] * (3 - k) + [(s1, t)] * k:
            c = [c[0] * a, c[1] * a + c[0] * b, c[2] * a + c[1] * b, c[3] * a + c[2] * b]
        rows.append(torch.stack(c, -1))
    return torch.stack(rows, 1)


def _bounds64(p, greg, u0, u1, v0, v1):
    """The lower bounding grid (n, 4 [j], 4 [i], 3) on the domain and the displacement (n, 3) of the upper one."""
    g = p[:, :16].clone()
    d = torch.zeros(len(p), 3, device=p.device, dtype=F64)
    for k in range(4):
        i, j = 1 + (k & 1), 1 + (k >> 1)
        du = (u0, u1) if i == 1 else (1 - u1, 1 - u0)
        dv = (v0, v1) if j == 1 else (1 - v1, 1 - v0)
        lo = (du[0] / (du[0] + dv[1])).unsqueeze(1)
        hi = (du[1] / (du[1] + dv[0])).unsqueeze(1)
        w = (_wbar(u0, u1, i / 3) * _wbar(v0, v1, j / 3)).unsqueeze(1)
        pu, pv = p[:, INNER[k]], p[:, PV[k]]
        A, B = pv + lo * (pu - pv), pv + hi * (pu - pv)
        g[:, INNER[k]] = torch.where(greg.unsqueeze(1), torch.minimum(A, B), pu)
        d = d + torch.where(greg.unsqueeze(1), w * (A - B).abs(), 0.0)
    g = g.view(-1, 4, 4, 3)
    g = (_crop(u0, u1).view(-1, 1, 4, 4, 1) * g.unsqueeze(2)).sum(3)            # along i
    return (_crop(v0, v1).view(-1, 4, 4, 1, 1) * g.unsqueeze(1)).sum(2), d      # along j


_HALVES = torch.tensor([[8, 0, 0, 0], [4, 4, 0, 0], [2, 4, 2, 0], [1, 3, 3, 1], [0, 2, 4, 2], [0, 0, 4, 4], [0, 0, 0, 8]], dtype=F64) / 8


def _slab(lo, hi, o, inv, tmin, tmax):
    a, b = (lo - o) * inv, (hi - o) * inv
    near = torch.maximum(torch.minimum(a, b).amax(-1), tmin)
    return near, near <= torch.minimum(torch.maximum(a, b).amin(-1), tmax)


def _pairs64(cp, rays, centre, radius):
    """(ray, patch) pairs whose boxes the ray meets; objects first by their bounding spheres."""
    per = len(cp) // len(centre)
    lo, hi = cp.amin(1), cp.amax(1)  # a Bezier patch's slots 16..19 repeat its inner points
    o, d = rays[:, :3], rays[:, 4:7]
    got = []
    for b in range(0, len(rays), 1 << 14):
        ob, db = o[b:b + (1 << 14)], d[b:b + (1 << 14)]
        q = centre.unsqueeze(0) - ob.unsqueeze(1)
        t = (q * db.unsqueeze(1)).sum(-1) / (db * db).sum(-1, keepdim=True)
        near = (q - t.clamp_min(0).unsqueeze(-1) * db.unsqueeze(1)).norm(dim=-1) <= radius + 0.1
        r, k = near.nonzero(as_tuple=True)
        for c in range(0, len(r), 1 << 14):
            rr = r[c:c + (1 << 14)]
            pp = k[c:c + (1 << 14)].unsqueeze(1) * per + torch.arange(per, device=DEV)
            inv = 1 / db[rr].unsqueeze(1)
            _, hit = _slab(lo[pp], hi[pp], ob[rr].unsqueeze(1), inv, rays[b + rr, 3].unsqueeze(1), rays[b + rr, 7].unsqueeze(1))
            x, y = hit.nonzero(as_tuple=True)
            got.append((b + rr[x], pp[x, y]))
    return torch.cat([x for x, _ in got]), torch.cat([y for _, y in got])


def _trace64(cp32, types, rays32, depth, local, centre, radius):
    """Closest leaf boxes of every ray, level by level over all subdomains that are met: {"t", "id": None, "uv"}."""
    cp, rays = cp32.to(F64), rays32.to(F64)
    ray, patch = _pairs64(cp, rays, centre, radius)
    best = torch.full((len(rays),), math.inf, device=DEV, dtype=F64)
    uv = torch.zeros(len(rays), 2, device=DEV, dtype=F64)
    halves = _HALVES.to(DEV)
    ident = torch.eye(3, device=DEV, dtype=F64)
    for b in range(0, len(ray), 1 << 17):
        r, p = ray[b:b + (1 << 17)], patch[b:b + (1 << 17)]
        iu, iv = torch.zeros_like(r), torch.zeros_like(r)
        base, greg = cp[p], types[p] == 1
        anchor = 0.5 * (base.amin(1) + base.amax(1))
        rot = _frames64(base) if local else ident.expand(len(r), 3, 3)
        base = ((base - anchor.unsqueeze(1)).unsqueeze(2) * rot.unsqueeze(1)).sum(-1)
        o = ((rays[r, :3] - anchor).unsqueeze(1) * rot).sum(-1)
        d = (rays[r, 4:7].unsqueeze(1) * rot).sum(-1)
        inv = torch.where(d == 0, 1e30, 1 / d)
        used = torch.where(greg.view(-1, 1, 1) | (torch.arange(20, device=DEV).view(1, 20, 1) < 16), base, base[:, :1])
        pad = (used.amax(1) - used.amin(1)).amax(1, keepdim=True) * 2.0 ** -19 if local else torch.zeros(len(r), 1, device=DEV, dtype=F64)
        at = torch.arange(len(r), device=DEV)
        for k in range(2 * depth):
            nu, nv = (k + 1) // 2, k // 2
            out = []
            for c in range(0, len(at), 1 << 18):
                a, x, y = at[c:c + (1 << 18)], iu[c:c + (1 << 18)], iv[c:c + (1 << 18)]
                u0, v0 = x.to(F64) * 2.0 ** -nu, y.to(F64) * 2.0 ** -nv
                g, disp = _bounds64(base[a], greg[a], u0, u0 + 2.0 ** -nu, v0, v0 + 2.0 ** -nv)
                g = g.transpose(1, 2) if k % 2 == 0 else g
                s = (halves.view(1, 7, 4, 1, 1) * g.unsqueeze(1)).sum(2)   # (n, 7, 4, 3), the split along dim 1
                for up in (0, 1):
                    part = s[:, 3 * up:3 * up + 4].reshape(-1, 16, 3)
                    t, hit = _slab(part.amin(1) - pad[a], part.amax(1) + disp + pad[a], o[a], inv[a], rays[r[a], 3], rays[r[a], 7])
                    hit = hit & (t <= best[r[a]])
                    h = hit.nonzero().squeeze(1)
                    out.append((a[h], 2 * x[h] + up if k % 2 == 0 else x[h], 2 * y[h] + up if k % 2 else y[h], t[h]))
            at, iu, iv, t = (torch.cat(z) for z in zip(*out))
        if len(at):
            rr = r[at]
            before = best.clone()
            best.scatter_reduce_(0, rr, t, "amin")
            win = (t == best[rr]) & (t < before[rr])
            uv[rr[win]] = (torch.stack((iu[win], iv[win]), 1).to(F64) + 0.5) * 2.0 ** -depth
    return {"t": best, "id": None, "uv": uv}


def _bf16(x):
    return x.to(torch.float32).to(torch.bfloat16).to(F64)


def _split_weights(th):
    W1, b1, W2, b2, W3, b3 = th.split([512, 32, 1024, 32, 128, 4])
    return W1.view(32, 16), b1, W2.view(32, 32), b2, W3.view(4, 32), b3


def _logits64(th, x):
    W1, b1, W2, b2, W3, b3 = _split_weights(th.to(F64))
    h = _bf16((_bf16(x) @ _bf16(W1).T + b1).relu())
    h = _bf16((h @ _bf16(W2).T + b2).relu())
    return h @ _bf16(W3).T + b3


def _mix(x):
    x = (x + 0x9E3779B97F4A7C15) & (2 ** 64 - 1)
    z = ((x ^ (x >> 30)) * 0xBF58476D1CE4E5B9) & (2 ** 64 - 1)
    z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & (2 ** 64 - 1)
    return x, z ^ (z >> 31)


def _train64(case, th, X, y):
    """Adam in 64 bits over the entry point's minibatches (a seeded affine permutation of the rows per epoch)."""
    n, batch = case["rows"], min(case["batch"], case["rows"])
    per_epoch = max(1, n // batch)
    th = th.to(F64)
    m, v, losses, epoch = torch.zeros_like(th), torch.zeros_like(th), [], -1
    q = _bf16 if case["bf16"] else (lambda z: z)
    for step in range(case["steps"]):
        if step // per_epoch != epoch:
            epoch = step // per_epoch
            x, a = _mix(5 ^ ((epoch * 0xD1B54A32D192ED03) & (2 ** 64 - 1)))
            a = a % n or 1
            while math.gcd(a, n) != 1:
                a = a + 1 if a + 1 < n else 1
            c = _mix(x)[1] % n
        rows = (a * (((step % per_epoch) * batch + torch.arange(batch, device=DEV)) % n) + c) % n
        rows = rows[y[rows] != ccs.NO_LABEL]
        W1, b1, W2, b2, W3, b3 = _split_weights(th)
        W1, W2, W3 = q(W1), q(W2), q(W3)
        x0 = q(X[rows].to(F64))
        a1 = x0 @ W1.T + b1
        h1 = q(a1.relu())
        a2 = h1 @ W2.T + b2
        h2 = q(a2.relu())
        z = h2 @ W3.T + b3
        hot = torch.nn.functional.one_hot(y[rows].long(), 4).to(F64)
        losses.append((z.logsumexp(1) - (z * hot).sum(1)).mean())
        d3 = z.softmax(1) - hot
        d2 = (d3 @ W3) * (a2 > 0)
        d1 = (d2 @ W2) * (a1 > 0)
        g = torch.cat([t.reshape(-1) for t in (d1.T @ x0, d1.sum(0), d2.T @ h1, d2.sum(0), d3.T @ h2, d3.sum(0))]) / max(1, len(rows))
        m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
        th = th - 3e-3 * (m / (1 - 0.9 ** (step + 1))) / ((v / (1 - 0.999 ** (step + 1))).sqrt() + 1e-8)
    return {"theta": th, "loss": torch.stack(losses)}


def exact(case, seed):
    kind = case["kind"]
    if kind in ("compact", "order"):  # a copy of its inputs; inputs defined by the kernel's own fp32 slab test at a box's boundary
        return None
    if kind == "train":
        s = prepare(case, seed)
        return _train64(case, s["theta"], s["x"], s["y"])
    if case["objects"] > 450 or case["depth"] > 16:  # too long level by level
        return None
    cp, types, centre, radius = _patches(case["objects"], seed)
    if kind == "playback":
        out = [_trace64(p, types, r, case["depth"], case["local"], centre, radius) for p, r in _frames_of(case, cp, types, seed)]
        return out
    sets = _ray_sets(case, cp, types, seed)
    out = [_trace64(cp, types, r, case["depth"], case["local"], centre, radius) for r in sets]
    if kind == "path":  # a later level starts from the hits of the one before
        return {"hits": out + [None] * case["bounces"], "rays": None, "index": None, "counts": None}
    return out
