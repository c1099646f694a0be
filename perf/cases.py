"""The work that programs have this library do, as timed cases.

Every case goes through the public Python entry points: NavSim (step, reset_to,
rollouts), Policy and ResetProposer.  Maps, poses, actions and weights are
drawn here from the case's seed; ``exact`` recomputes, in 64-bit arithmetic and
without the library, the outputs that are computed numbers.

Kinds (``case["kind"]``):

  step      one environment step of every env (``scan``: exact traversal or the
            paper's fixed-step march)
  reset_to  every env reset to given poses, its observation returned
  rollout   T steps with the paper's actor in the loop, as one HIP graph
  learned   one step whose resets come from the attached reset proposer
  propose   a batch of start/goal pairs at requested difficulty
  label     training pairs by the geodesic search
  train     optimisation steps of the proposer's network
  grad      loss and gradient of that network on explicit inputs
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2606_15846_amd import navsim, policy, reset_proposal

TWO_PI = 2 * math.pi
# Launch shapes a program sets once: none (the library's own), or what the
# autotuner finds for small maps (a byte map and workgroups of 1024) and for
# large ones (run walk on the bitmap and its transpose).
SHAPES = {
    "own": None,
    "bytes1024": dict(tile_envs=16, refill_at=40, groups=16, walk=4, threads=1024, balance=1),
    "runs512": dict(tile_envs=32, refill_at=32, groups=16, walk=5, threads=512, balance=1),
}
STEP = dict(kind="step", envs=4096, maps=16, side_lo=128, side_hi=128, res=0.05, rooms=False,
            beams=360, mixed=False, sectors=30, fov=TWO_PI, rmax=6.0, dt=0.1, rect=False,
            size=0.18, reverse=False, scan="traversal", shape="own")
PAIRS = dict(kind="label", maps=64, side_lo=256, side_hi=256, res=0.05, n=4096)


def listed():
    return [
        # a handful of envs, one small map: debugging, evaluation, latency
        dict(STEP, name="step 16 envs", envs=16, maps=1, side_lo=64, side_hi=64, res=0.1,
             beams=36, sectors=36, rmax=3.5),
        # the paper's TurtleBot2 training batch: 1024 envs, one floor plan of
        # 13.5 m, 1080 beams over 270 degrees, 20 m range, no tuning
        dict(STEP, name="step turtlebot2 1024", envs=1024, maps=1, side_lo=270, side_hi=270,
             rooms=True, beams=1080, fov=math.radians(270.0), rmax=20.0, size=0.2),
        # a training batch over 16 small maps, tuned shape
        dict(STEP, name="step 4096", shape="bytes1024"),
        # the large mixed batch: 128 uneven maps, four beam counts, both
        # footprints, tuned shape
        dict(STEP, name="step mixed 32768", envs=32768, maps=128, side_lo=96, side_hi=512,
             rooms=True, beams=1080, mixed=True, rmax=8.0, dt=0.05, reverse=True,
             shape="runs512"),
        # the paper's own range query (0.03 m march) instead of the exact one
        dict(STEP, name="step march 4096", scan="march"),
        # an experience batch: 32 steps with the actor in front of each
        dict(STEP, name="rollout actor 4096x32", kind="rollout", steps=32, noise=0.1,
             shape="bytes1024"),
        # a curriculum's start: every env to a given start and goal
        dict(STEP, name="reset_to 16384", kind="reset_to", envs=16384, maps=64, side_lo=256,
             side_hi=256, rooms=True),
        # a step with difficulty resets from the trained proposer
        dict(STEP, name="step learned 32768", kind="learned", envs=32768, maps=32, side_lo=256,
             side_hi=256, rooms=True, shape="runs512", proposals=32, tries=64),
        # start/goal pairs for a batch of new episodes
        dict(PAIRS, name="propose 8192", kind="propose", n=8192, proposals=32, tries=64),
        # training pairs for the proposer
        dict(PAIRS, name="label 16384", n=16384),
        # the proposer's training loop, 16 optimisation steps
        dict(PAIRS, name="train 1024x128x16", kind="train", n=1024, samples=128, steps=16),
        # one gradient on a batch that the program made itself
        dict(PAIRS, name="grad 1024", kind="grad", n=1024),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step", "march", "rollout", "reset_to", "learned",
                       "propose", "label", "train", "grad"])
    if kind in ("propose", "label", "train", "grad"):
        c = dict(PAIRS, kind=kind, maps=rng.randint(4, 64))
        c["side_lo"] = rng.randint(80, 256)
        c["side_hi"] = rng.randint(c["side_lo"], 256)
        if kind == "propose":
            c.update(n=_log(rng, 32, 8192), proposals=rng.choice([0, 8, 32]),
                     tries=rng.choice([16, 64]))
        elif kind == "label":
            c.update(n=_log(rng, 64, 16384))
        elif kind == "train":
            c.update(n=_log(rng, 48, 1024), samples=rng.randint(8, 128), steps=rng.randint(2, 16))
        else:
            c.update(n=_log(rng, 1, 4096))
        return c
    c = dict(STEP, kind="step" if kind == "march" else kind, rooms=rng.random() < 0.5,
             rect=rng.random() < 0.4, reverse=rng.random() < 0.5,
             rmax=round(rng.uniform(3.0, 20.0), 2), dt=rng.choice([0.05, 0.1]))
    c["size"] = round(rng.uniform(0.15, 0.25), 3)
    c["sectors"] = rng.choice([1, 10, 30, 36])
    c["beams"] = c["sectors"] * rng.randint(2, max(2, 1080 // c["sectors"] // 2))
    c["fov"] = rng.choice([TWO_PI, TWO_PI, math.radians(270.0), math.radians(97.5)])
    c["envs"] = _log(rng, 16, 16384)
    c["maps"] = min(c["envs"], _log(rng, 1, 64))
    c["side_lo"] = rng.randint(64, 256)
    c["side_hi"] = rng.randint(c["side_lo"], 256 if kind == "learned" else 384)
    c["mixed"] = c["sectors"] > 1 and rng.random() < 0.25
    c["shape"] = rng.choice(["own", "own", "runs512"])
    if kind == "march":
        c.update(scan="march", envs=min(c["envs"], 4096))
        c["beams"] = min(c["beams"], 12 * c["sectors"])
    elif kind == "rollout":
        c.update(steps=rng.randint(4, 16), noise=rng.choice([0.0, 0.1]),
                 envs=min(c["envs"], 4096))
    elif kind == "learned":
        c.update(proposals=rng.choice([8, 32]), tries=64, maps=min(c["maps"], 32))
    return c


# --- inputs -----------------------------------------------------------------
def _map(rng, w, h, res, rooms):
    """One floor plan: a border, then rooms of 2.5-4 m with one door per wall
    or rectangles and discs over about 15 % of the cells."""
    occ = np.zeros((h, w), np.uint8)
    occ[[0, -1], :] = 1
    occ[:, [0, -1]] = 1
    if rooms:
        door = int(round(1.0 / res))

        def cuts(n):
            out, at = [], 0
            while True:
                at += int(rng.uniform(2.5, 4.0) / res)
                if at >= n - int(2.0 / res):
                    return out
                out.append(at)
        xs, ys = cuts(w), cuts(h)
        for x in xs:
            occ[:, x:x + 2] = 1
        for y in ys:
            occ[y:y + 2, :] = 1
        for x in xs:  # one door in every wall between two rooms
            for y0, y1 in zip([0] + ys, ys + [h - 1]):
                d = int(rng.integers(y0 + 2, max(y0 + 3, y1 - door)))
                occ[d:min(d + door, y1), x:x + 2] = 0
        for y in ys:
            for x0, x1 in zip([0] + xs, xs + [w - 1]):
                d = int(rng.integers(x0 + 2, max(x0 + 3, x1 - door)))
                occ[y:y + 2, d:min(d + door, x1)] = 0
        occ[[0, -1], :] = 1
        occ[:, [0, -1]] = 1
        n = int(rng.integers(0, 30)) * w * h // (256 * 256)
    else:
        n = int(w * h * 0.15 / 100)
    jj, ii = np.mgrid[0:h, 0:w]
    for k in range(n):
        cx, cy = rng.uniform(0, w), rng.uniform(0, h)
        if rooms or k % 2:
            r = rng.uniform(0.1, 0.4) / res
            x0, x1 = max(0, int(cx - r)), min(w, int(cx + r) + 2)
            y0, y1 = max(0, int(cy - r)), min(h, int(cy + r) + 2)
            inside = (ii[y0:y1, x0:x1] - cx) ** 2 + (jj[y0:y1, x0:x1] - cy) ** 2 <= r * r
            occ[y0:y1, x0:x1] |= inside.astype(np.uint8)
        else:
            a, b = rng.integers(2, 17, 2)
            occ[int(cy):int(cy) + b, int(cx):int(cx) + a] = 1
    return occ


def _maps(case, rng):
    out = []
    for k in range(case["maps"]):
        w, h = (int(v) for v in rng.integers(case["side_lo"], case["side_hi"] + 1, 2))
        rooms = case.get("rooms", True) and (k % 2 == 1 or not case.get("mixed", False))
        out.append(_map(rng, w, h, case["res"], rooms))
    return out


def _clear_cells(occ, cells):
    """Cells with no occupied cell within `cells` rows and columns."""
    p = np.pad(occ, cells, constant_values=1).astype(np.int32)
    s = np.pad(p.cumsum(0).cumsum(1), ((1, 0), (1, 0)))
    k = 2 * cells + 1
    near = s[k:, k:] - s[:-k, k:] - s[k:, :-k] + s[:-k, :-k]
    free = np.flatnonzero(near == 0)
    if not free.size:
        raise ValueError("map without free space")
    return free


class Scene:
    """Configuration, maps and host arrays of a batch of envs."""

    def __init__(self, case, seed):
        rng = np.random.default_rng([seed, 11])
        self.case = case
        N = case["envs"]
        size = case["size"]
        lo = -0.5 if case["reverse"] else 0.0
        self.cfg = dict(
            num_envs=N, num_beams=case["beams"], num_sectors=case["sectors"], fov_rad=case["fov"],
            max_range_m=case["rmax"], dt_s=case["dt"], horizon=200, goal_radius_m=0.2,
            c_progress=2.0, r_success=10.0, r_collision=-10.0, footprint=int(case["rect"]),
            radius_m=size, length_m=3.9 * size, width_m=1.7 * size, v_min=lo, v_max=0.5,
            w_min=-1.0, w_max=1.0, goal_min_dist_m=1.0, reset_max_tries=64, seed=seed)
        self.maps = _maps(case, rng)
        self.res = [case["res"]] * len(self.maps)
        self.env_map = ((np.arange(N, dtype=np.int64) * len(self.maps)) // N).astype(np.int32)
        self.profiles = None
        if case["mixed"]:
            m, per = case["sectors"], max(1, case["beams"] // case["sectors"] // 6)
            self.profiles = [dict(num_beams=min(case["beams"], m * per * int(rng.choice([1, 2, 4, 6]))),
                                  footprint=int(rng.integers(0, 2)), radius_m=size,
                                  length_m=3.9 * size, width_m=1.7 * size) for _ in self.maps]
        self.rng = rng

    def beams_of(self, k):
        return self.profiles[k]["num_beams"] if self.profiles else self.cfg["num_beams"]

    def robot_of(self, k):
        q = self.profiles[k] if self.profiles else self.cfg
        return q["footprint"], q["radius_m"], q["length_m"], q["width_m"]

    def poses(self):
        """A collision-free start and goal for every env: x, y, heading, goal x, y."""
        out = np.zeros((self.cfg["num_envs"], 5), np.float32)
        for k, occ in enumerate(self.maps):
            e = np.flatnonzero(self.env_map == k)
            if not e.size:
                continue
            fp, r, ln, wd = self.robot_of(k)
            rc = r if fp == 0 else 0.5 * math.hypot(ln, wd)
            free = _clear_cells(occ, int(math.ceil(rc / self.res[k] + 0.5)))
            w = occ.shape[1]
            a, b = self.rng.choice(free, (2, e.size))
            j = self.rng.uniform(-0.4, 0.4, (4, e.size))
            out[e, 0] = (a % w + 0.5 + j[0]) * self.res[k]
            out[e, 1] = (a // w + 0.5 + j[1]) * self.res[k]
            out[e, 2] = self.rng.uniform(-math.pi, math.pi, e.size)
            out[e, 3] = (b % w + 0.5 + j[2]) * self.res[k]
            out[e, 4] = (b // w + 0.5 + j[3]) * self.res[k]
        return out

    def start(self):
        """Mid-episode env states (the mix of ages that a running batch has)
        and eight batches of normalised actions."""
        p, N = self.poses(), self.cfg["num_envs"]
        z = np.zeros(N, np.float32)
        d = np.hypot(p[:, 3].astype(np.float64) - p[:, 0], p[:, 4].astype(np.float64) - p[:, 1])
        st = dict(x=p[:, 0], y=p[:, 1], th=p[:, 2], v=z, w=z, gx=p[:, 3], gy=p[:, 4],
                  dprev=d.astype(np.float32), t=self.rng.integers(0, 200, N).astype(np.int32),
                  ep=np.zeros(N, np.uint32))
        acts = self.rng.uniform(-1.0, 1.0, (8, N, 2)).astype(np.float32)
        return st, acts

    def build(self):
        sim = navsim.NavSim(self.cfg, self.maps, self.res, self.env_map, device=0,
                            profiles=self.profiles)
        shape = SHAPES[self.case["shape"]]
        if shape:
            sim.set_tuning(**shape)
        if self.case["scan"] == "march":
            sim.set_scan(navsim.NAVSIM_SCAN_MARCH, 0.03)
        return sim


def _pair_scene(case, seed):
    """The proposer's maps behind a minimal simulator."""
    c = dict(STEP, envs=max(64, case["maps"]), rooms=True)
    c.update({k: case[k] for k in ("maps", "side_lo", "side_hi", "res")})
    return Scene(c, seed)


def _bins(seed, n):
    return np.random.default_rng([seed, 12]).integers(0, 8, n).astype(np.int32)


def _pairs(rp, maps, per_map):
    """Labelled training pairs, as flat device arrays."""
    ids = np.repeat(np.arange(maps, dtype=np.int32), per_map)
    lab = rp.label(ids, 0)
    nb = rp.nb
    m = torch.from_numpy(ids).to(rp.device).repeat_interleave(nb)
    b = torch.arange(nb, dtype=torch.int32, device=rp.device).repeat(ids.size)
    s = lab["start"].repeat_interleave(nb)
    g = lab["goal"].reshape(-1)
    ok = g >= 0
    return dict(map=m[ok].contiguous(), bin=b[ok].contiguous(), start=s[ok].contiguous(),
                goal=g[ok].contiguous())


def _trained(sim, case):
    """A proposer after a short training (draws land in the asked bin often
    enough that the network serves most requests)."""
    rp = reset_proposal.ResetProposer(sim)
    rp.train(_pairs(rp, case["maps"], max(8, 8192 // case["maps"])), 400, batch=1024, samples=64)
    return rp


def _grad_inputs(case, seed):
    """Weights (bfloat16 values, as the products see them) and a batch."""
    rng = np.random.default_rng([seed, 13])
    dims = [1024 + 8 + 16, 256, 256, 256, 5]
    flat, at = [], 0
    for i, o in zip(dims, dims[1:]):
        w = rng.uniform(-1, 1, (o, i)) / math.sqrt(i)
        b = rng.uniform(-1, 1, o) / math.sqrt(i)
        for t in (w, b):
            t = torch.from_numpy(t.astype(np.float32)).to(torch.bfloat16).float().reshape(-1)
            flat.append(torch.nn.functional.pad(t, (0, -t.numel() % 8)))
    n = case["n"]
    x = np.zeros((n, dims[0]), np.float32)
    x[:, :1024] = rng.random((n, 1024)) < 0.35
    x[np.arange(n), 1024 + rng.integers(0, 8, n)] = 1.0
    x[:, 1032:] = rng.uniform(-1, 1, (n, 16))
    t = rng.uniform(0, 1, (n, 5)).astype(np.float32)
    t[:, 2] = 0.0
    return dims, torch.cat(flat), torch.from_numpy(x).to(torch.bfloat16), torch.from_numpy(t)


def prepare(case, seed):
    kind, dev = case["kind"], torch.device("cuda", 0)
    s = dict(kind=kind, case=case, i=0)
    if kind in ("propose", "label", "train", "grad"):
        sc = _pair_scene(case, seed)
        s["sim"] = sim = sc.build()
        n = case["n"]
        if kind == "propose":
            s["rp"] = _trained(sim, case) if case["proposals"] else reset_proposal.ResetProposer(sim)
            i32 = dict(dtype=torch.int32, device=dev)
            rng = np.random.default_rng([seed, 14])
            s["req"] = (torch.from_numpy(rng.integers(0, case["maps"], n).astype(np.int32)).to(dev),
                        torch.from_numpy(_bins(seed, n)).to(dev), torch.arange(n, **i32),
                        torch.from_numpy(rng.integers(0, 50, n).astype(np.int32)).to(dev))
            s["out"] = dict(pose=torch.empty(n, 5, device=dev), hops=torch.empty(n, **i32),
                            source=torch.empty(n, **i32), checks=torch.empty(n, **i32))
            return s
        s["rp"] = rp = reset_proposal.ResetProposer(sim)
        if kind == "label":
            s["ids"] = np.random.default_rng([seed, 14]).integers(0, case["maps"], n).astype(np.int32)
        elif kind == "train":
            s["pairs"] = _pairs(rp, case["maps"], 32)
            s["loss"] = torch.empty(case["steps"], device=dev)
        else:
            _, p, x, t = _grad_inputs(case, seed)
            rp.set_params(p.numpy())
            s["x"], s["t"] = x.view(torch.int16).to(dev), t.to(dev)
        return s
    sc = Scene(case, seed)
    s["sim"] = sim = sc.build()
    if kind == "reset_to":
        s["pose"] = torch.from_numpy(sc.poses()).to(dev)
        return s
    st, acts = sc.start()
    sim.set_state(st)
    if kind == "rollout":
        s["pol"] = pol = policy.Policy(sim)
        pol.init_params(seed)
        s["buf"] = sim.rollout_buffers(case["steps"])
        s["obs0"] = torch.rand(case["envs"], case["sectors"] + 4, device=dev,
                               generator=torch.Generator(dev).manual_seed(seed))
        return s
    if kind == "learned":
        s["rp"] = rp = _trained(sim, case)
        rp.attach(_bins(seed, case["envs"]), case["proposals"], case["tries"],
                  max(1, case["envs"] // 16))
    s["acts"] = [a.contiguous() for a in torch.from_numpy(acts).to(dev)]
    return s


def run(s):
    kind = s["kind"]
    if kind in ("step", "learned"):
        act = s["acts"][s["i"] % len(s["acts"])]
        s["i"] += 1
        obs, reward, term, trunc, info = s["sim"].step(act)
        return dict(obs=obs, reward=reward, terminated=term, truncated=trunc,
                    final_obs=info["final_obs"])
    if kind == "reset_to":
        return s["sim"].reset_to(s["pose"])
    if kind == "rollout":
        T = s["case"]["steps"]
        if s["i"]:
            s["obs0"].copy_(s["buf"]["obs"][-1])
        b = s["pol"].rollout(T, s["i"], s["obs0"], noise_std=s["case"]["noise"], buffers=s["buf"])
        s["i"] += T
        return b
    if kind == "propose":
        return s["rp"].propose_into(*s["req"], s["case"]["proposals"], s["case"]["tries"], s["out"])
    if kind == "label":
        out = s["rp"].label(s["ids"], s["i"])
        s["i"] += s["case"]["n"]
        return out
    if kind == "train":
        s["rp"].train(s["pairs"], s["case"]["steps"], batch=s["case"]["n"],
                      samples=s["case"]["samples"], loss=s["loss"])
        return dict(loss=s["loss"], params=s["rp"].get_params())
    rows, g = s["rp"].loss_grad(s["x"], s["t"])
    return dict(loss=rows, grad=g)


# --- what a pass cannot do without --------------------------------------------
def _net_flops(rows, first):
    return 2.0 * rows * (first * 256 + 2 * 256 * 256 + 256 * 5)


def work(case):
    kind, area = case["kind"], ((case["side_lo"] + case["side_hi"]) / 2.0) ** 2
    bits = case["maps"] * area / 8
    if kind == "grad":
        n, params = case["n"], 1048 * 256 + 2 * 65536 + 1280
        return dict(bytes=n * (1048 * 2 + 24) + params * 8, flops=3 * _net_flops(n, 1048))
    if kind == "train":
        rows, params = case["n"] * case["samples"], 1048 * 256 + 2 * 65536 + 1280
        return dict(bytes=case["steps"] * params * 24.0,
                    flops=case["steps"] * (_net_flops(rows, 16) + 3 * _net_flops(case["n"], 1048)))
    if kind == "label":
        # every reached cell once, with its random key (about 40 integer operations)
        return dict(bytes=bits + case["n"] * 72.0, flops=case["n"] * area * 0.6 * 40)
    if kind == "propose":
        # the draws, and one search of the map's cells for the pair that is taken
        return dict(bytes=bits + case["n"] * 44.0,
                    flops=_net_flops(case["n"] * case["proposals"], 16) + case["n"] * area * 0.6)
    # a ray visits about a third of the cells within its range and the map; two
    # operations a visit
    N, m = case["envs"], case["sectors"]
    beams = case["beams"] * (0.55 if case["mixed"] else 1.0)
    cells = 0.35 * min(case["rmax"] / case["res"], 0.7 * math.sqrt(area))
    ray = 2.0 * N * beams * cells
    if kind == "reset_to":
        return dict(bytes=bits + N * (20 + 40 + 4 * (m + 4)), flops=ray)
    b, f = bits + N * (80 + 8 + 6 + 4 * (m + 4)), ray
    if kind == "rollout":
        T = case["steps"]
        return dict(bytes=bits + T * N * (80 + 8 + 6 + 4 * (m + 4)),
                    flops=T * (ray + 2.0 * N * ((m + 4) * 100 + 20000 + 200)))
    if kind == "learned":
        f += 0.015 * N * (_net_flops(case["proposals"], 16) + area * 0.6)
    return dict(bytes=b, flops=f)


# --- 64-bit recomputation -------------------------------------------------------
def _f(v):
    """The double of the float32 that the library was given."""
    return float(np.float32(v))


def _ranges(sc, case, pose, env):
    """Range of every beam from the float64 poses [n][3] of the envs `env`,
    as a list of [K_e] rows: the distance at which the ray enters the first
    occupied or outside cell, or the first such sample of the march."""
    dev = pose.device
    rmax, out = _f(case["rmax"]), [None] * len(env)
    em = sc.env_map[env]
    for k in np.unique(em):
        rows = np.flatnonzero(em == k)
        occ = torch.from_numpy(np.pad(sc.maps[k], 1, constant_values=1)).to(dev)
        K, s = sc.beams_of(k), _f(sc.res[k])
        fov = _f(case["fov"])
        kk = torch.arange(K, dtype=torch.float64, device=dev)
        if fov >= TWO_PI - 1e-6:
            al = -math.pi + kk * (TWO_PI / K)
        else:
            al = -0.5 * fov + kk * (fov / (K - 1)) if K > 1 else kk * 0.0
        p = pose[torch.from_numpy(rows).to(dev)]
        ang = p[:, 2:3] + al[None, :]
        n = rows.size * K
        dx, dy = torch.cos(ang).reshape(n), torch.sin(ang).reshape(n)
        ox, oy = (p[:, i:i + 1].expand(-1, K).reshape(n) for i in (0, 1))
        ix, iy = torch.floor(ox / s).long(), torch.floor(oy / s).long()
        hmax, wmax = occ.shape[0] - 1, occ.shape[1] - 1

        def hit(i, j):
            return occ[(j + 1).clamp(0, hmax), (i + 1).clamp(0, wmax)] != 0
        rng = torch.full((n,), rmax, dtype=torch.float64, device=dev)
        live = torch.arange(n, device=dev)
        if case["scan"] == "march":
            h, q = _f(0.03), 0
            while live.numel() and q * h <= rmax:
                t = q * h
                b = hit(torch.floor((ox[live] + t * dx[live]) / s).long(),
                        torch.floor((oy[live] + t * dy[live]) / s).long())
                rng[live[b]] = t
                live, q = live[~b], q + 1
        else:
            b = hit(ix, iy)
            rng[b] = 0.0
            live = live[~b]
            sx, sy = torch.where(dx > 0, 1, -1), torch.where(dy > 0, 1, -1)
            while live.numel():
                i, j = ix[live], iy[live]
                tx = ((i + (sx[live] > 0)) * s - ox[live]) / dx[live]
                ty = ((j + (sy[live] > 0)) * s - oy[live]) / dy[live]
                tx, ty = tx.nan_to_num(math.inf, math.inf, math.inf), ty.nan_to_num(math.inf, math.inf, math.inf)
                xs = tx <= ty
                t = torch.where(xs, tx, ty)
                i, j = torch.where(xs, i + sx[live], i), torch.where(xs, j, j + sy[live])
                ix[live], iy[live] = i, j
                far = t > rmax
                b = hit(i, j) & ~far
                rng[live[b]] = t[b]
                live = live[~(b | far)]
        for q, r in enumerate(rng.reshape(rows.size, K)):
            out[rows[q]] = r
    return out


def _observe(sc, case, pose, goal, vw, env):
    """Observation rows of the envs `env` at float64 poses."""
    m = case["sectors"]
    n = len(env)
    if not n:
        return torch.zeros(0, m + 4, dtype=torch.float64, device=pose.device)
    lid = torch.stack([r.reshape(m, -1).amin(1) for r in _ranges(sc, case, pose, env)])
    dx, dy = goal[:, 0] - pose[:, 0], goal[:, 1] - pose[:, 1]
    phi = torch.atan2(dy, dx) - pose[:, 2]
    phi = torch.atan2(torch.sin(phi), torch.cos(phi))
    return torch.cat([lid, torch.hypot(dx, dy)[:, None], phi[:, None], vw], 1)


def _collides(sc, pose):
    """Whether each env's footprint overlaps an occupied or outside cell."""
    out = torch.zeros(pose.shape[0], dtype=torch.bool, device=pose.device)
    for k, occ in enumerate(sc.maps):
        e = torch.from_numpy(np.flatnonzero(sc.env_map == k)).to(pose.device)
        if not e.numel():
            continue
        fp, r, ln, wd = sc.robot_of(k)
        r, hl, hw, s = _f(r), 0.5 * _f(ln), 0.5 * _f(wd), _f(sc.res[k])
        rc = r if fp == 0 else math.hypot(hl, hw)
        big = torch.from_numpy(occ).to(pose.device)
        h, w = occ.shape
        p = pose[e]
        win = int(2 * rc / s) + 3
        g = torch.arange(win, device=pose.device)
        i = (torch.floor((p[:, 0] - rc) / s).long()[:, None, None] + g[None, None, :]).expand(-1, win, win)
        j = (torch.floor((p[:, 1] - rc) / s).long()[:, None, None] + g[None, :, None]).expand(-1, win, win)
        full = (i < 0) | (j < 0) | (i >= w) | (j >= h) | (big[j.clamp(0, h - 1), i.clamp(0, w - 1)] != 0)
        x, y = p[:, 0, None, None], p[:, 1, None, None]
        if fp == 0:
            ex = x - torch.minimum(torch.maximum(x, i * s), (i + 1) * s)
            ey = y - torch.minimum(torch.maximum(y, j * s), (j + 1) * s)
            over = ex * ex + ey * ey < r * r
        else:
            c, sn = torch.cos(p[:, 2])[:, None, None], torch.sin(p[:, 2])[:, None, None]
            ux, uy = (i + 0.5) * s - x, (j + 0.5) * s - y
            hc = 0.5 * s
            cell = hc * (c.abs() + sn.abs())
            over = ((ux.abs() < hc + hl * c.abs() + hw * sn.abs())
                    & (uy.abs() < hc + hl * sn.abs() + hw * c.abs())
                    & ((c * ux + sn * uy).abs() < hl + cell)
                    & ((c * uy - sn * ux).abs() < hw + cell))
        out[e] = (full & over).flatten(1).any(1)
    return out


def exact(case, seed):
    kind = case["kind"]
    dev = torch.device("cuda", 0) if torch.cuda.is_available() else torch.device("cpu")
    if kind == "grad":
        dims, flat, x, t = _grad_inputs(case, seed)
        flat, x, t = (v.to(dev).double() for v in (flat, x, t))
        ps, at = [], 0
        for i, o in zip(dims, dims[1:]):
            w = flat[at:at + o * i].reshape(o, i).clone().requires_grad_()
            at += o * i + -(o * i) % 8
            b = flat[at:at + o].clone().requires_grad_()
            at += o + -o % 8
            ps += [w, b]
        y = x
        for l in range(4):
            y = y @ ps[2 * l].T + ps[2 * l + 1]
            y = torch.nn.functional.leaky_relu(y, _f(0.01)) if l < 3 else y
        wt = torch.tensor([1.0, 1.0, 0.0, 1.0, 1.0], dtype=torch.float64, device=dev)
        rows = ((y - t) ** 2 * wt).sum(1)
        g = torch.autograd.grad(rows.mean(), ps)
        return dict(loss=rows.detach(),
                    grad=torch.cat([torch.nn.functional.pad(v.reshape(-1), (0, -v.numel() % 8)) for v in g]))
    if kind == "reset_to":
        sc = Scene(case, seed)
        p = torch.from_numpy(sc.poses()).to(dev).double()
        z = torch.zeros(p.shape[0], 2, dtype=torch.float64, device=dev)
        return _observe(sc, case, p[:, :3], p[:, 3:], z, np.arange(p.shape[0]))
    if kind not in ("step", "learned"):
        return None
    sc = Scene(case, seed)
    st, acts = sc.start()
    st = {k: torch.from_numpy(np.asarray(v, np.float64)).to(dev) for k, v in st.items()}
    c = {k: _f(v) if isinstance(v, float) else v for k, v in sc.cfg.items()}
    a = torch.from_numpy(acts[0]).to(dev).double()
    v = (c["v_min"] + (a[:, 0] + 1) / 2 * (c["v_max"] - c["v_min"])).float().double()
    w = (c["w_min"] + (a[:, 1] + 1) / 2 * (c["w_max"] - c["w_min"])).float().double()
    th = st["th"] + w * c["dt_s"]
    th = torch.where(th >= math.pi, th - TWO_PI, torch.where(th < -math.pi, th + TWO_PI, th))
    # the state is held in float32
    pose = torch.stack([st["x"] + v * torch.cos(st["th"]) * c["dt_s"],
                        st["y"] + v * torch.sin(st["th"]) * c["dt_s"], th], 1).float().double()
    goal = torch.stack([st["gx"], st["gy"]], 1)
    d = torch.hypot(goal[:, 0] - pose[:, 0], goal[:, 1] - pose[:, 1])
    coll, won = _collides(sc, pose), d < c["goal_radius_m"]
    reward = torch.where(won, c["r_success"],
                         torch.where(coll, c["r_collision"], c["c_progress"] * (st["dprev"] - d)))
    ended = (coll | won | (st["t"] + 1 >= 200)).nonzero()[:, 0]
    final = torch.zeros(pose.shape[0], case["sectors"] + 4, dtype=torch.float64, device=dev)
    final[ended] = _observe(sc, case, pose[ended], goal[ended], torch.stack([v, w], 1)[ended],
                            ended.cpu().numpy())
    # a reset draws its poses from the library's counter-based generator, and
    # obs shows them: no value here
    return dict(obs=None, reward=reward, terminated=None, truncated=None, final_obs=final)
