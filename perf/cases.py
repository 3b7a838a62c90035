"""Timed cases of the AdamW-GS step library, over the range of its public entry points.

Each case is one pass of a training program's loop, or of one of its rarer
events, through the Python binding: the per-iteration step (visibility and
step in one launch, or in two), the dense step, the step of many scenes,
multi-view visibility, relocation, densification and spatial reordering.
``exact`` gives the same results in FP64 with plain torch, written from the
definitions in ``include/gsopt.h``.
"""
from __future__ import annotations

import math
import random

import torch

import paper_2601_16736_amd as gs

DEV = torch.device("cuda")

# (name, dim, lr, DAR kind): the 59 values of a degree-3 SH primitive with the
# public 3DGS learning rates, as one SH group or split into DC and rest.
GROUPS5 = [("means", 3, 1.6e-4, gs.GS_DAR_NONE), ("scales", 3, 5e-3, gs.GS_DAR_LOGSCALE_EXP),
           ("quats", 4, 1e-3, gs.GS_DAR_NONE), ("opacity", 1, 5e-2, gs.GS_DAR_OPACITY_SIGMOID),
           ("sh", 48, 2.5e-3, gs.GS_DAR_NONE)]
GROUPS6 = GROUPS5[:4] + [("sh_dc", 3, 2.5e-3, gs.GS_DAR_NONE), ("sh_rest", 45, 1.25e-4, gs.GS_DAR_NONE)]
# first column of each group in a packed [n][64] row
PACKED_COLUMNS = {"sh": 0, "quats": 48, "means": 52, "scales": 55, "opacity": 58}
PACKED_ROW = 64

REG_NORM = 1e5                # 1000 x 1000 pixels
RSR_ALPHA1, RSR_ALPHA2, RSR_RATIO = 0.2, 0.04, 0.05
AIU_RATIO, AIU_SCALE = 0.05, 1.0
NOISE_LR, NOISE_K, NOISE_T = 5e5, 100.0, 0.005
FIRST_ITERATION = 1201        # in the middle of training
N_CAMERAS = 200


# ------------------------------------------------------------------ cases
def _case(name, kind, n, **options):
    c = {"kind": kind, "n": n, "layout": "groups5", "bf16": False, "order": "morton", "z_far": 17.5, "views": 1,
         "rsr": False, "aiu": False, "noise": False, "schedule": "auto", "scenes": 0, "scene_seed": 0}
    if name:
        c = {"name": name, **c}
    c.update(options)
    return c


def listed():
    return [
        # one training iteration of a 3M-primitive scene kept in Morton order,
        # 29 % visible: the benchmark's headline, and its BF16-moment form
        _case("view_f32_3m", "view", 3_000_000),
        _case("view_bf16_3m", "view", 3_000_000, bf16=True),
        # the start of training: a sparse point cloud, where launches and the
        # host path count; unsorted, as loaded
        _case("view_f32_54k", "view", 54_275, order="none", layout="groups6"),
        # visibility, then the masked step, on a scene that was never sorted
        # (visible rows scattered), SH split as 3DGS stores it
        _case("masked_f32_1m_unsorted", "two_launch", 1_234_567, order="none", layout="groups6", schedule="masked"),
        # synchronous Adam over every primitive (the densification phase of
        # the "half" schedule)
        _case("dense_f32_600k", "dense", 600_001, schedule="dense"),
        # an iteration with Re-State and the implicit update of invisible rows
        _case("view_f32_2m_rsr_aiu", "view", 2_000_000, rsr=True, aiu=True),
        # an MCMC iteration: 1 % of the primitives relocated, then the step
        # with position noise
        _case("mcmc_f32_1m", "mcmc", 1_000_000, noise=True),
        # 16 scenes of 0.2M to 4M primitives stepped by one plan, contiguous
        # groups, BF16 moments
        _case("batched_bf16_16_scenes", "batched", 16_000_000, bf16=True, order="none", scenes=16),
        # fewer scenes whose state is packed in one row per primitive
        _case("batched_f32_5_scenes_packed", "batched", 3_000_000, order="none", scenes=5, layout="packed",
              scene_seed=3),
        # a batch of eight training views culled in one pass
        _case("visibility_8_views_3m", "multi", 3_000_000, views=8),
        # a densification event: 10 % pruned, 5 % cloned
        _case("densify_f32_1500k", "densify", 1_500_000),
        # the spatial reorder that follows densification
        _case("reorder_f32_1m", "reorder", 1_000_003, order="none"),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(["view", "two_launch", "dense", "mcmc", "batched", "multi", "densify", "reorder"],
                       weights=[8, 4, 1, 2, 2, 1, 1, 1])[0]
    z_far = rng.choice([12.5, 15.0, 17.5, 17.5, 20.0, 25.0, 1000.0])
    order = rng.choice(["morton", "morton", "none"])
    bf16 = rng.random() < 0.4
    layout = rng.choice(["groups5", "groups6", "groups5", "groups6", "packed"])
    if kind == "view":
        return _case(None, kind, _log_uniform(rng, 10_000, 6_000_000), layout=layout, bf16=bf16, order=order,
                     z_far=z_far, views=rng.choice([1, 1, 1, 4]), rsr=rng.random() < 0.2, aiu=rng.random() < 0.1)
    if kind == "two_launch":
        return _case(None, kind, _log_uniform(rng, 10_000, 4_000_000), layout=layout, bf16=bf16, order=order,
                     z_far=z_far, schedule=rng.choice(["masked", "compacted"]), rsr=rng.random() < 0.2)
    if kind == "dense":
        return _case(None, kind, _log_uniform(rng, 10_000, 3_000_000), layout=layout, bf16=bf16, schedule="dense")
    if kind == "mcmc":
        return _case(None, kind, _log_uniform(rng, 100_000, 6_000_000), layout=rng.choice(["groups5", "groups6"]),
                     bf16=bf16, order=order, z_far=z_far, noise=True)
    if kind == "batched":
        scenes = rng.randint(2, 12)
        return _case(None, kind, _log_uniform(rng, 100_000, 1_000_000) * scenes, layout=layout, bf16=bf16,
                     order="none", scenes=scenes, scene_seed=rng.randrange(1000), rsr=rng.random() < 0.2)
    if kind == "multi":
        return _case(None, kind, _log_uniform(rng, 30_000, 6_000_000), order=order, z_far=z_far,
                     views=rng.randint(2, 16))
    if kind == "densify":
        return _case(None, kind, _log_uniform(rng, 50_000, 3_000_000), layout=rng.choice(["groups5", "groups6"]),
                     bf16=bf16)
    return _case(None, kind, _log_uniform(rng, 50_000, 3_000_000), layout=rng.choice(["groups5", "groups6"]),
                 bf16=bf16, order="none")


# ----------------------------------------------------------------- inputs
def _specs(case):
    return GROUPS6 if case["layout"] == "groups6" else GROUPS5


def _generator(seed, salt):
    g = torch.Generator(device=DEV)
    g.manual_seed(1_000_003 * (seed + 1) + salt)
    return g


def _scene_sizes(case):
    """Primitives and visible fraction of each scene of a batched case: sizes
    spread over a factor of 20, summing to about n."""
    r = random.Random(case["scene_seed"])
    w = [math.exp(r.uniform(math.log(0.2), math.log(4.0))) for _ in range(case["scenes"])]
    total = sum(w)
    return [(max(1, int(case["n"] * x / total)), r.uniform(0.02, 0.60)) for x in w]


def _spread3(x):
    x = (x | (x << 16)) & 0x030000FF
    x = (x | (x << 8)) & 0x0300F00F
    x = (x | (x << 4)) & 0x030C30C3
    return (x | (x << 2)) & 0x09249249


def _morton_order(means):
    """Primitive indices in the order of their means' 30-bit Morton codes
    (10 bits per axis over the bounding box, FP32 arithmetic), ties in index order."""
    lo = means.amin(0)
    ext = means.amax(0) - lo
    scale = (1024.0 / ext.double()).float()
    q = ((means - lo) * scale).clamp(0.0, 1023.0).to(torch.int64)
    code = _spread3(q[:, 0]) | (_spread3(q[:, 1]) << 1) | (_spread3(q[:, 2]) << 2)
    return torch.sort(code, stable=True).indices


def _means(case, n, seed):
    g = _generator(seed, 1)
    if case["kind"] == "mcmc":        # a clustered scene: 64 Gaussians
        centres = 20.0 * torch.rand((64, 3), generator=g, device=DEV) - 10.0
        which = torch.randint(0, 64, (n,), generator=g, device=DEV)
        m = centres[which] + 1.5 * torch.randn((n, 3), generator=g, device=DEV)
    else:
        m = 20.0 * torch.rand((n, 3), generator=g, device=DEV) - 10.0
    return m[_morton_order(m)].contiguous() if case["order"] == "morton" else m


def _arrays(case, n, seed):
    """theta, gradients, moments and step counts of a scene in mid-training:
    lists of [n][dim] tensors, one per group."""
    g = _generator(seed, 2)
    mdt = torch.bfloat16 if case["bf16"] else torch.float32
    a = {"theta": [], "grad": [], "m": [], "v": []}
    for name, dim, _, _ in _specs(case):
        x = torch.randn((n, dim), generator=g, device=DEV)
        if name == "means":
            x = _means(case, n, seed)
        elif name == "scales":        # log-scales of a trained scene, around 0.01
            x = math.log(0.01) + 0.5 * x
        elif name == "opacity":       # logits, many nearly transparent
            x = 2.0 * x - 1.0
        elif name == "sh_rest":
            x = 0.1 * x
        a["theta"].append(x)
        a["grad"].append(1e-3 * torch.randn((n, dim), generator=g, device=DEV))
        a["m"].append((1e-4 * torch.randn((n, dim), generator=g, device=DEV)).to(mdt))
        a["v"].append((1e-6 * torch.rand((n, dim), generator=g, device=DEV) + 1e-9).to(mdt))
    a["t"] = torch.randint(0, 400, (n,), generator=g, device=DEV, dtype=torch.int32)
    return a


def _cameras(case, seed):
    """Cameras on a Fibonacci sphere of radius 15 that look at the origin
    (60 degrees, 1000 x 1000), in the seed's shuffled order."""
    f = 500.0 / math.tan(math.radians(30.0))
    cams = []
    for k in range(N_CAMERAS):
        z = 1.0 - 2.0 * (k + 0.5) / N_CAMERAS
        rho, phi = math.sqrt(1.0 - z * z), math.pi * (3.0 - math.sqrt(5.0)) * (k + 0.5)
        eye = [15.0 * rho * math.cos(phi), 15.0 * rho * math.sin(phi), 15.0 * z]
        fwd = [-e / 15.0 for e in eye]
        up = (0.0, 1.0, 0.0) if abs(fwd[2]) > 0.99 else (0.0, 0.0, 1.0)
        right = [fwd[1] * up[2] - fwd[2] * up[1], fwd[2] * up[0] - fwd[0] * up[2], fwd[0] * up[1] - fwd[1] * up[0]]
        length = math.sqrt(sum(c * c for c in right))
        right = [c / length for c in right]
        down = [fwd[1] * right[2] - fwd[2] * right[1], fwd[2] * right[0] - fwd[0] * right[2],
                fwd[0] * right[1] - fwd[1] * right[0]]
        view = []
        for row in (right, down, fwd):
            view += row + [-sum(r * e for r, e in zip(row, eye))]
        cams.append(gs.Camera(view, f, f, 500.0, 500.0, 1000, 1000, 0.2, case["z_far"]))
    random.Random(seed).shuffle(cams)
    return cams


def _config(case, seed):
    sched = {"auto": gs.GS_SCHED_AUTO, "masked": gs.GS_SCHED_MASKED, "compacted": gs.GS_SCHED_COMPACTED,
             "dense": gs.GS_SCHED_DENSE}[case["schedule"]]
    names = [s[0] for s in _specs(case)]
    return gs.StepConfig(seed=seed, iteration=FIRST_ITERATION - 1, reg_norm=REG_NORM,
                         moment_dtype=gs.GS_MOMENT_BF16 if case["bf16"] else gs.GS_MOMENT_F32, schedule=sched,
                         rsr_enable=case["rsr"], rsr_alpha1=RSR_ALPHA1, rsr_alpha2=RSR_ALPHA2, rsr_ratio=RSR_RATIO,
                         aiu_enable=case["aiu"], aiu_ratio=AIU_RATIO, aiu_scale=AIU_SCALE,
                         noise_enable=case["noise"],
                         noise_groups=tuple(names.index(k) for k in ("means", "scales", "quats", "opacity")),
                         noise_lr=NOISE_LR, noise_k=NOISE_K, noise_t=NOISE_T)


def _dar(case, kind):
    """lambda of a regularised group: the MCMC setting, or AdamW-GS's own."""
    if kind == gs.GS_DAR_NONE:
        return 0.0
    if case["kind"] == "mcmc":
        return 0.01
    return 1e-3 if kind == gs.GS_DAR_OPACITY_SIGMOID else 1e-5


def _scene(case, n, seed):
    """The scene's groups as the binding takes them, and the tensors behind
    them (per group, or one packed tensor per role)."""
    return _as_groups(case, _arrays(case, n, seed), n)


def _as_groups(case, a, n):
    specs = _specs(case)
    if case["layout"] == "packed":
        whole = {}
        for role in ("theta", "grad", "m", "v"):
            p = torch.zeros((n, PACKED_ROW), dtype=a[role][0].dtype, device=DEV)
            for (name, dim, _, _), x in zip(specs, a[role]):
                p[:, PACKED_COLUMNS[name]:PACKED_COLUMNS[name] + dim] = x
            whole[role] = [p]
            a[role] = [p[:, PACKED_COLUMNS[s[0]]:PACKED_COLUMNS[s[0]] + s[1]] for s in specs]
    else:
        whole = {role: a[role] for role in ("theta", "grad", "m", "v")}
    groups = [gs.Group(a["theta"][k], a["grad"][k], a["m"][k], a["v"][k], lr, dar_kind=dar,
                       dar_lambda=_dar(case, dar), dar_clip=10.0) for k, (_, _, lr, dar) in enumerate(specs)]
    out = {"theta": whole["theta"], "m": whole["m"], "v": whole["v"], "t": a["t"]}
    return groups, a["t"], out


def _scene_rows(case):
    """Row range of each scene in the arrays that a batched case keeps for
    all of its scenes, starts at multiples of 64 rows (256-byte lines in
    every group)."""
    at, out = 0, []
    for size, _ in _scene_sizes(case):
        out.append((at, at + size))
        at += (size + 63) // 64 * 64
    return out, at


def _all_scenes(case, seed):
    """A batched case's arrays: every scene's rows in one tensor per group
    and role."""
    ranges, total = _scene_rows(case)
    whole = None
    for k, (lo, hi) in enumerate(ranges):
        a = _arrays(case, hi - lo, 1000 * seed + k)
        if whole is None:
            whole = {r: [torch.zeros((total, x.shape[1]), dtype=x.dtype, device=DEV) for x in a[r]]
                     for r in ("theta", "grad", "m", "v")}
            whole["t"] = torch.zeros(total, dtype=torch.int32, device=DEV)
        for r in ("theta", "grad", "m", "v"):
            for w, x in zip(whole[r], a[r]):
                w[lo:hi] = x
        whole["t"][lo:hi] = a["t"]
    return whole


def _bernoulli(n, p, seed):
    return (torch.rand(n, generator=_generator(seed, 3), device=DEV) < p).to(torch.uint8)


def _kept(n, seed):
    """Keep mask of a pruning: all but a tenth of the primitives, picked at random."""
    keep = torch.ones(n, dtype=torch.uint8, device=DEV)
    keep[torch.randperm(n, generator=_generator(seed, 3), device=DEV)[:n // 10]] = 0
    return keep


def _relocated(n):
    return max(1, n // 100)


def prepare(case, seed):
    kind, n = case["kind"], case["n"]
    s = {"kind": kind, "n": n, "bf16": case["bf16"], "at": 0}
    mdt = gs.GS_MOMENT_BF16 if case["bf16"] else gs.GS_MOMENT_F32
    s["moment_dtype"] = mdt
    if kind == "batched":
        ranges, total = _scene_rows(case)
        groups, t, s["out"] = _as_groups(case, _all_scenes(case, seed), total)
        scenes = []
        for k, ((lo, hi), (size, p)) in enumerate(zip(ranges, _scene_sizes(case))):
            part = [gs.Group(g.param[lo:hi], g.grad[lo:hi], g.exp_avg[lo:hi], g.exp_avg_sq[lo:hi], g.lr,
                             dar_kind=g.dar_kind, dar_lambda=g.dar_lambda, dar_clip=g.dar_clip) for g in groups]
            scenes.append(gs.Scene(part, size, t[lo:hi], visible=_bernoulli(size, p, 1000 * seed + k),
                                   schedule=gs.GS_SCHED_MASKED))
        s["plan"] = gs.gs_batch_create(scenes, mdt)
        s["cfg"] = _config(case, seed)
        return s
    if kind == "multi":
        s["means"] = _means(case, n, seed)
        s["cams"] = _cameras(case, seed)
        s["views"] = case["views"]
        s["mask"] = torch.empty(n, dtype=torch.uint8, device=DEV)
        s["bits"] = torch.empty(n, dtype=torch.int32, device=DEV)
        return s
    s["groups"], s["t"], s["out"] = _scene(case, n, seed)
    s["cfg"] = _config(case, seed)
    if kind == "densify":
        kept, k = n - n // 10, n // 20
        rows = kept + k
        s["keep"], s["kept"] = _kept(n, seed), kept
        s["src_idx"] = torch.randint(0, kept, (k,), generator=_generator(seed, 4), device=DEV,
                                     dtype=torch.int32)
        dst, out = [], {"theta": [], "m": [], "v": []}
        for g in s["groups"]:
            x, m, v = (torch.zeros((rows, g.dim), dtype=q.dtype, device=DEV)
                       for q in (g.param, g.exp_avg, g.exp_avg_sq))
            dst.append(gs.Group(x, None, m, v, g.lr))
            out["theta"].append(x)
            out["m"].append(m)
            out["v"].append(v)
        s["dst"] = dst
        s["t_dst"] = out["t"] = torch.zeros(rows, dtype=torch.int32, device=DEV)
        s["kept_count"] = out["kept_count"] = torch.zeros(1, dtype=torch.int32, device=DEV)
        s["out"] = out
        s["ws"] = torch.empty(gs.gs_prune_workspace_size(n), dtype=torch.uint8, device=DEV)
        return s
    if kind == "reorder":
        s["perm"] = torch.empty(n, dtype=torch.int32, device=DEV)
        s["ws"] = torch.empty(gs.gs_spatial_order_workspace_size(n), dtype=torch.uint8, device=DEV)
        return s
    if kind in ("view", "two_launch", "mcmc"):
        s["cams"] = _cameras(case, seed)
        s["views"] = case["views"]
        s["means"] = s["groups"][0].param
    if kind == "two_launch":
        s["mask"] = torch.empty(n, dtype=torch.uint8, device=DEV)
        s["vis_idx"] = s["vis_count"] = None
        if case["schedule"] == "compacted":
            s["vis_idx"] = torch.empty(n, dtype=torch.int32, device=DEV)
            s["vis_count"] = torch.zeros(1, dtype=torch.int32, device=DEV)
    if kind == "mcmc":
        s["selected"] = torch.empty(_relocated(n), dtype=torch.int32, device=DEV)
        s["ws"] = torch.empty(gs.gs_relocate_workspace_size(n), dtype=torch.uint8, device=DEV)
    return s


# ------------------------------------------------------------------- pass
def _next_views(s):
    """The views of this iteration: the next ones of the shuffled rig."""
    k = s["at"]
    s["at"] = k + s["views"]
    return [s["cams"][(k + j) % N_CAMERAS] for j in range(s["views"])]


def run(s):
    kind = s["kind"]
    if kind == "multi":
        gs.gs_visibility_multi(s["means"], _next_views(s), mask=s["mask"], view_bits=s["bits"])
        return {"mask": s["mask"], "bits": s["bits"]}
    if kind == "densify":
        gs.gs_prune(s["keep"], s["groups"], s["dst"], s["moment_dtype"], s["t"], s["t_dst"], s["kept_count"], s["ws"])
        gs.gs_append(s["dst"], s["moment_dtype"], s["kept"], s["src_idx"], s["t_dst"])
        return s["out"]
    if kind == "reorder":
        gs.gs_spatial_order(s["groups"][0].param, s["perm"], s["ws"])
        o = s["out"]
        moved = gs.apply_spatial_order(o["theta"] + o["m"] + o["v"] + [o["t"]], s["perm"])
        k = len(o["theta"])
        return {"theta": moved[:k], "m": moved[k:2 * k], "v": moved[2 * k:3 * k], "t": moved[3 * k],
                "perm": s["perm"]}
    cfg = s["cfg"]
    cfg.iteration += 1
    if kind == "batched":
        s["plan"].step(cfg)
    elif kind == "dense":
        gs.adamw_gs_step(s["groups"], s["n"], s["t"], cfg)
    elif kind == "view":
        gs.adamw_gs_step_view(s["groups"], s["n"], s["t"], cfg, s["means"], _next_views(s))
    elif kind == "two_launch":
        gs.gs_visibility(s["means"], _next_views(s)[0], mask=s["mask"], vis_idx=s["vis_idx"],
                         vis_count=s["vis_count"])
        gs.adamw_gs_step(s["groups"], s["n"], s["t"], cfg, visible=s["mask"], vis_idx=s["vis_idx"],
                         vis_count=s["vis_count"])
        return {**s["out"], "mask": s["mask"]}
    else:                                                    # mcmc
        opacity = s["groups"][cfg.noise_groups[3]].param
        gs.gs_relocate_reset(opacity, _relocated(s["n"]), s["groups"], s["moment_dtype"], s["t"], True, s["ws"],
                             selected=s["selected"])
        gs.adamw_gs_step_view(s["groups"], s["n"], s["t"], cfg, s["means"], _next_views(s))
        return {**s["out"], "selected": s["selected"]}
    return s["out"]


# ------------------------------------------------------------------- work
def _visible_fraction(case):
    """Share of a scene's primitives that the case's views see, from a sample."""
    r = torch.Generator().manual_seed(5)
    x = 20.0 * torch.rand((20_000, 3), generator=r, dtype=torch.float64) - 10.0
    if case["kind"] == "mcmc":
        x = x[:64][torch.randint(0, 64, (20_000,), generator=r)] + 1.5 * torch.randn((20_000, 3), generator=r,
                                                                                       dtype=torch.float64)
    cams = _cameras(case, 0)
    total = 0.0
    for trial in range(4):
        seen = torch.zeros(len(x), dtype=torch.bool)
        for c in cams[trial * case["views"]:(trial + 1) * case["views"]]:
            view = torch.tensor(c.view, dtype=torch.float64).reshape(3, 4)
            p = x @ view[:, :3].T + view[:, 3]
            u, v = c.fx * p[:, 0] / p[:, 2] + c.cx, c.fy * p[:, 1] / p[:, 2] + c.cy
            seen |= (p[:, 2] > c.z_near) & (p[:, 2] < c.z_far) & (u >= 0) & (u <= 1000) & (v >= 0) & (v <= 1000)
        total += float(seen.double().mean()) / 4
    return total


def work(case):
    """Each input read once and each output written once: per stepped row
    theta, gradient and moments read, theta and moments written, t both."""
    n, kind, ms = case["n"], case["kind"], 2 if case["bf16"] else 4
    row = 59 * (4 + 4 + 4 + 4 * ms) + 8
    if kind == "batched":
        visible = sum(size * p for size, p in _scene_sizes(case))
        total = sum(size for size, _ in _scene_sizes(case))
        extra = RSR_RATIO * (total - visible) * 59 * 4 * ms if case["rsr"] else 0.0
        return {"bytes": visible * row + total + extra, "flops": visible * 59 * 20}
    if kind == "multi":
        return {"bytes": n * (12 + 1 + 4), "flops": n * case["views"] * 40}
    if kind == "densify":
        state = 59 * (4 + 2 * ms) + 4
        return {"bytes": 0.9 * n * 2 * state + n + 0.05 * n * (59 * 4 + state + 4), "flops": 0}
    if kind == "reorder":
        return {"bytes": n * (12 + 2 * (59 * (4 + 2 * ms) + 4) + 4), "flops": 0}
    if kind == "dense":
        return {"bytes": n * row, "flops": n * 59 * 20}
    visible = n * _visible_fraction(case)
    moved = visible * row + n * 12
    if case["rsr"]:
        moved += RSR_RATIO * (n - visible) * 59 * 4 * ms
    if case["aiu"]:
        moved += AIU_RATIO * (n - visible) * (59 * (8 + 2 * ms) + 4)
    if kind == "two_launch":
        moved += n
    if kind == "mcmc":
        moved += n * 4 + _relocated(n) * (59 * 2 * ms + 8)
    return {"bytes": moved, "flops": visible * 59 * 20}


# ----------------------------------------------------------- FP64 results
_M64 = (1 << 64) - 1
_GAMMA = 0x9E3779B97F4A7C15
_TAG_RSR, _TAG_NOISE, _TAG_AIU = 1, 48, 64


def _signed(x):
    x &= _M64
    return x - (1 << 64) if x >> 63 else x


def _shift_right(z, k):
    return (z >> k) & ((1 << (64 - k)) - 1)


def _mix(z):
    """SplitMix64's output function on int64 tensors (wrapping products)."""
    z = (z ^ _shift_right(z, 30)) * _signed(0xBF58476D1CE4E5B9)
    z = (z ^ _shift_right(z, 27)) * _signed(0x94D049BB133111EB)
    return z ^ _shift_right(z, 31)


def _draws(state, k):
    """Outputs k (an int64 tensor) of the stream with this state."""
    return _mix(_signed(state) + k * _signed(_GAMMA))


def _stream(seed, tag, iteration):
    def out(s, k):
        return int(_draws(s, torch.tensor([k], dtype=torch.int64))[0]) & _M64
    return out(out(seed, tag + 1), iteration + 1)


def _sampled(seed, tag, n, ratio):
    i = torch.arange(n, device=DEV, dtype=torch.int64)
    return _shift_right(_draws(_stream(seed, tag, FIRST_ITERATION), i + 1), 32) < int(math.floor(ratio * 2 ** 32))


def _f32(x):
    return x.to(torch.float32).to(torch.float64)


def _one_view(means, cam):
    """The FP32 cull: every operation in FP64 on FP32 values, then rounded,
    which rounds as the FP32 operation does."""
    s = lambda q: float(torch.tensor(q, dtype=torch.float32))     # noqa: E731
    x, y, z = (means[:, a].double() for a in range(3))
    p = []
    for k in range(3):
        r = [s(q) for q in cam.view[4 * k:4 * k + 4]]
        p.append(_f32(_f32(_f32(_f32(r[0] * x) + _f32(r[1] * y)) + _f32(r[2] * z)) + r[3]))
    u = _f32(_f32(_f32(s(cam.fx) * p[0]) / p[2]) + s(cam.cx))
    v = _f32(_f32(_f32(s(cam.fy) * p[1]) / p[2]) + s(cam.cy))
    return ((p[2] > s(cam.z_near)) & (p[2] < s(cam.z_far)) & (u >= 0) & (u <= float(cam.width)) & (v >= 0)
            & (v <= float(cam.height)))


def _noise_move(a, names, seed, n):
    """eta_{R_o} R_mu of every primitive, from the state before the step."""
    i = torch.arange(n, device=DEV, dtype=torch.int64)
    st = _stream(seed, _TAG_NOISE, FIRST_ITERATION)
    d1, d2 = _draws(st, 2 * i + 1), _draws(st, 2 * i + 2)
    top = lambda d: (_shift_right(d, 40) + 1).double() / 2 ** 24           # noqa: E731
    low = lambda d: (_shift_right(d, 8) & 0xFFFFFF).double() / 2 ** 24     # noqa: E731
    r1, r2 = torch.sqrt(-2.0 * torch.log(top(d1))), torch.sqrt(-2.0 * torch.log(top(d2)))
    p1, p2 = 2.0 * math.pi * low(d1), 2.0 * math.pi * low(d2)
    gamma = torch.stack([r1 * torch.cos(p1), r1 * torch.sin(p1), r2 * torch.cos(p2)], 1)
    q = a["theta"][names.index("quats")].double()
    w, x, y, z = (q / q.norm(dim=1, keepdim=True)).unbind(1)
    rot = torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                       2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                       2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)], 1).reshape(n, 3, 3)
    e = (rot * gamma[:, :, None]).sum(1) * torch.exp(2.0 * a["theta"][names.index("scales")].double())
    sigma_gamma = (rot * e[:, None, :]).sum(2)
    o = torch.sigmoid(a["theta"][names.index("opacity")].double())
    return NOISE_LR * GROUPS5[0][2] * torch.sigmoid(-NOISE_K * (o - NOISE_T)) * sigma_gamma


def _step_exact(case, a, vis, seed, n):
    """The step of the arrays a over the visible rows vis, in place, in FP64."""
    specs = _specs(case)
    names = [s[0] for s in specs]
    rsr = _sampled(seed, _TAG_RSR, n, RSR_RATIO) if case["rsr"] else None
    aiu = (_sampled(seed, _TAG_AIU, n, AIU_RATIO) & ~vis & (a["t"] > 0)) if case["aiu"] else None
    move = _noise_move(a, names, seed, n) if case["noise"] else None
    a["t"] = a["t"] + vis.to(torch.int32)
    t = a["t"].double()[:, None]
    b1, b2 = -torch.expm1(t * math.log(0.9)), -torch.expm1(t * math.log(0.999))
    vis = vis[:, None]
    for k, (name, _, lr, dar) in enumerate(specs):
        th, g, m, v = (a[r][k].double() for r in ("theta", "grad", "m", "v"))
        if rsr is not None:
            m = torch.where(rsr[:, None], RSR_ALPHA1 * m, m)
            v = torch.where(rsr[:, None], RSR_ALPHA2 * v, v)
        m2 = torch.where(vis, 0.9 * m + (1.0 - 0.9) * g, m)
        v2 = torch.where(vis, 0.999 * v + (1.0 - 0.999) * g * g, v)
        d = torch.sqrt(v2 / b2) + 1e-15
        u = (m2 / b1) / d
        if dar != gs.GS_DAR_NONE:
            slope = torch.sigmoid(th) * torch.sigmoid(-th) if dar == gs.GS_DAR_OPACITY_SIGMOID else torch.exp(th)
            u = u + torch.clamp(_dar(case, dar) / REG_NORM * slope / d, max=10.0)
        new = th - lr * u
        if name == "means" and move is not None:
            new = new - move
        new = torch.where(vis, new, th)
        if aiu is not None:
            new = torch.where(aiu[:, None], th - lr * AIU_SCALE * (m2 / b1) / d, new)
        a["theta"][k], a["m"][k], a["v"][k] = new, m2, v2


def _as_out(case, a):
    """The arrays in the layout that run() returns."""
    if case["layout"] != "packed":
        return {"theta": a["theta"], "m": a["m"], "v": a["v"], "t": a["t"]}
    out = {"t": a["t"]}
    for role in ("theta", "m", "v"):
        p = torch.zeros((len(a["t"]), PACKED_ROW), dtype=torch.float64, device=DEV)
        for (name, dim, _, _), x in zip(_specs(case), a[role]):
            p[:, PACKED_COLUMNS[name]:PACKED_COLUMNS[name] + dim] = x
        out[role] = [p]
    return out


def exact(case, seed):
    kind, n = case["kind"], case["n"]
    if kind == "multi":
        means, cams = _means(case, n, seed), _cameras(case, seed)
        bits = torch.zeros(n, dtype=torch.int64, device=DEV)
        for k in range(case["views"]):
            bits |= _one_view(means, cams[k]).to(torch.int64) << k
        return {"mask": (bits != 0).to(torch.uint8), "bits": bits.to(torch.int32)}
    if kind == "batched":
        ranges, total = _scene_rows(case)
        whole = None
        for k, ((lo, hi), (size, p)) in enumerate(zip(ranges, _scene_sizes(case))):
            a = _arrays(case, size, 1000 * seed + k)
            # scene k of a plan draws with the call's seed + k
            _step_exact(case, a, _bernoulli(size, p, 1000 * seed + k) != 0, seed + k, size)
            if whole is None:
                whole = {r: [torch.zeros((total, x.shape[1]), dtype=torch.float64, device=DEV) for x in a[r]]
                         for r in ("theta", "m", "v")}
                whole["t"] = torch.zeros(total, dtype=torch.int32, device=DEV)
            for r in ("theta", "m", "v"):
                for w, x in zip(whole[r], a[r]):
                    w[lo:hi] = x
            whole["t"][lo:hi] = a["t"]
        return _as_out(case, whole)
    a = _arrays(case, n, seed)
    if kind == "densify":
        keep = _kept(n, seed) != 0
        src = torch.randint(0, n - n // 10, (n // 20,), generator=_generator(seed, 4), device=DEV,
                            dtype=torch.int32).long()
        out = {"kept_count": keep.sum().to(torch.int32).reshape(1)}
        kept = {r: [x[keep] for x in a[r]] for r in ("theta", "m", "v")}
        out["theta"] = [torch.cat([x, x[src]]).double() for x in kept["theta"]]
        for r in ("m", "v"):
            out[r] = [torch.cat([x, torch.zeros_like(x[src])]).double() for x in kept[r]]
        t = a["t"][keep]
        out["t"] = torch.cat([t, torch.zeros_like(t[src])])
        return out
    if kind == "reorder":
        perm = _morton_order(a["theta"][0])
        out = {r: [x[perm].double() for x in a[r]] for r in ("theta", "m", "v")}
        return {**out, "t": a["t"][perm], "perm": perm.to(torch.int32)}
    names = [s[0] for s in _specs(case)]
    extra = {}
    if kind == "mcmc":
        low = torch.sort(a["theta"][names.index("opacity")][:, 0], stable=True).indices[:_relocated(n)]
        extra["selected"] = torch.sort(low).values.to(torch.int32)
        for r in ("m", "v"):
            for x in a[r]:
                x[low] = 0
        a["t"][low] = 0
    if kind == "dense":
        vis = torch.ones(n, dtype=torch.bool, device=DEV)
    else:
        cams = _cameras(case, seed)
        vis = torch.zeros(n, dtype=torch.bool, device=DEV)
        for k in range(case["views"]):
            vis |= _one_view(a["theta"][0], cams[k])
    if kind == "two_launch":
        extra["mask"] = vis.to(torch.uint8)
    _step_exact(case, a, vis, seed, n)
    return {**_as_out(case, a), **extra}
