"""Timed cases of the rendering path, through the package's public classes.

Each case is a dict of plain values whose "kind" names the entry point:

query      Field.query at n points (point look-ups, picking, baking a volume)
occupancy  Field.build_occupancy, the grid a field needs before it is rendered with empty-space skipping
closest    Mesh.closest_hit (picking, collision queries), with a refit first where the mesh is animated
render     Renderer.render of one camera: rays, bounces, hit ids, radiance, throughput
fields     Renderer.render_fields: several placed fields among meshes
cameras    a batch of cameras with bounce limits of their own, one captured graph, Russian roulette
train      one batch of proposal training: targets from the field, then loss and gradients
"""
import functools
import math

import numpy as np
import torch

from paper_2309_04581_amd import meshrf as M
from paper_2309_04581_amd import scenegen as sg

OFF, ON = False, True


def listed():
    return [
        # a handful of points of a small field: an interactive look-up, where the launch is what counts
        {"name": "query_probe", "kind": "query", "layout": "tiny", "half": OFF, "n": 1000, "posed": OFF},
        # a volume sampled at scattered points (baking, density export): 16 levels, FP32
        {"name": "query_batch", "kind": "query", "layout": "mid", "half": OFF, "n": 3000001, "posed": OFF},
        # the empty-space grid of a sparse 16-level field, rebuilt whenever the field changes
        {"name": "occupancy_128", "kind": "occupancy", "layout": "mid", "half": OFF, "res": 128},
        # ray casts against the meshes alone: picking and collision queries on 100 spheres
        {"name": "closest_hit", "kind": "closest", "balls": 100, "refit": OFF, "n": 500003},
        # the smallest frame: 64x64, 8-level field, mirror cube, 4 bounces (preview thumbnails, tests)
        {"name": "frame_tiny", "kind": "render", "scene": "tiny", "w": 64, "h": 64, "samples": 64, "bounces": 4,
         "half": OFF, "sampler": "uniform", "occ": OFF, "light_sampling": OFF, "shadows": OFF, "refit": OFF},
        # the ordinary frame: 800x800, 16 levels, glass, mirror and diffuse meshes, 8 bounces
        {"name": "frame_mid", "kind": "render", "scene": "mid", "w": 800, "h": 800, "samples": 256, "bounces": 8,
         "half": OFF, "sampler": "uniform", "occ": ON, "light_sampling": OFF, "shadows": OFF, "refit": OFF},
        # the same frame the fast way: proposal sampler, FP16 table, BF16 MLPs
        {"name": "frame_proposal", "kind": "render", "scene": "mid", "w": 800, "h": 800, "samples": 256, "bounces": 8,
         "half": ON, "sampler": "proposal", "occ": ON, "light_sampling": OFF, "shadows": OFF, "refit": OFF},
        # an emitting panel with light sampling at every diffuse hit
        {"name": "frame_emitter", "kind": "render", "scene": "emitter", "w": 800, "h": 800, "samples": 256,
         "bounces": 8, "half": OFF, "sampler": "uniform", "occ": ON, "light_sampling": ON, "shadows": OFF,
         "refit": OFF},
        # an animated cloth at a ragged size: a refit and a frame of the 8-level field
        {"name": "frame_cloth", "kind": "render", "scene": "cloth", "w": 801, "h": 603, "samples": 256, "bounces": 8,
         "half": OFF, "sampler": "uniform", "occ": OFF, "light_sampling": OFF, "shadows": OFF, "refit": ON},
        # three placed fields with disjoint boxes among meshes
        {"name": "three_fields", "kind": "fields", "fields": 3, "spacing": 2.9, "w": 800, "h": 450, "samples": 516,
         "half": OFF, "occ": ON},
        # sixteen cameras, 16.2 million rays, up to 16 bounces, replayed from a graph with the tuned launch shape
        {"name": "sixteen_cameras", "kind": "cameras", "cams": 16, "scale": 1.0},
        # one training batch of the proposal sampler: 2^14 segments, 32 bins
        {"name": "train_batch", "kind": "train", "layout": "mid", "n": 16384, "bins": 32, "samples": 256},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["query", "query", "occupancy", "closest", "render", "render", "render", "render", "fields",
                       "cameras", "train"])
    if kind == "query":
        return {"kind": kind, "layout": rng.choice(["tiny", "mid", "mid"]), "half": rng.random() < 0.4,
                "n": _log_int(rng, 500, 3000000), "posed": rng.random() < 0.3}
    if kind == "occupancy":
        return {"kind": kind, "layout": rng.choice(["tiny", "mid"]), "half": rng.random() < 0.4,
                "res": rng.randint(24, 128)}
    if kind == "closest":
        return {"kind": kind, "balls": _log_int(rng, 1, 100), "refit": rng.random() < 0.5,
                "n": _log_int(rng, 500, 500000)}
    if kind == "fields":
        h = _log_int(rng, 40, 450)
        return {"kind": kind, "fields": rng.randint(2, 3), "spacing": rng.choice([1.2, 2.9]),
                "w": int(h * rng.uniform(1.0, 1.7)), "h": h, "samples": rng.randint(128, 516),
                "half": rng.random() < 0.3, "occ": rng.random() < 0.5}
    if kind == "cameras":
        return {"kind": kind, "cams": rng.randint(2, 15), "scale": round(rng.uniform(0.15, 0.8), 3)}
    if kind == "train":
        return {"kind": kind, "layout": rng.choice(["tiny", "mid"]), "n": _log_int(rng, 512, 16384),
                "bins": rng.choice([20, 32, 48]), "samples": rng.randint(64, 256)}
    scene = rng.choice(["tiny", "mid", "mid", "cloth", "emitter"])
    h = _log_int(rng, 32, 700)
    sampler = rng.choice(["uniform", "uniform", "proposal"])
    return {"kind": kind, "scene": scene, "w": int(h * rng.uniform(0.7, 1.3)), "h": h,
            "samples": rng.randint(48, 256), "bounces": rng.randint(2, 8), "half": rng.random() < 0.4,
            "sampler": sampler, "occ": scene != "tiny" and rng.random() < 0.6,
            "light_sampling": scene == "emitter" and rng.random() < 0.6, "shadows": scene == "mid" and rng.random() < 0.2,
            "refit": scene == "cloth"}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _rng(seed, what):
    return np.random.default_rng([int(seed) & 0x7FFFFFFF, what])


def _field_params(layout, seed, amp=1.0, offset=1.0):
    s = 100 + int(seed) % (1 << 30)
    return (sg.mid_field if layout == "mid" else sg.tiny_field)(seed=s, table_amp=amp, density_offset=offset)


def _types(half):
    return dict(table_dtype=M.MR_F16, mlp_dtype=M.MR_BF16) if half else {}


def _pose(seed):
    r = _rng(seed, 3)
    return sg.pose_matrix(sg.rotation(r.normal(size=3), r.uniform(0.2, 2.0)), r.uniform(-0.3, 0.3, size=3))


def _query_inputs(case, seed):
    f = _field_params(case["layout"], seed)
    if case["posed"]:
        f.pose = _pose(seed)
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    x = torch.rand(case["n"], 3, device="cuda", generator=g) * 2.0 - 1.0
    d = torch.randn(case["n"], 3, device="cuda", generator=g)
    d = d / d.norm(dim=1, keepdim=True)
    return f, x, d


@functools.lru_cache(maxsize=None)
def _static_mesh(name, balls=0):
    if name == "mid":
        return sg.mid_mesh()
    if name == "emitter":
        return sg.emitter_scene(8, 8).mesh
    if name == "balls":
        return sg.balls_mesh(balls)
    return {"tiny": sg.mirror_cube_mesh, "cloth": sg.cloth_mesh}[name]()


def _closest_inputs(case, seed):
    m = _static_mesh("balls", case["balls"])
    v = m.vertices
    if case["refit"]:   # the spheres breathe and drift with the seed
        r = _rng(seed, 1)
        v = (v * r.uniform(0.9, 1.1) + r.uniform(-0.05, 0.05, size=3)).astype(np.float32)
    g = torch.Generator(device="cuda").manual_seed(int(seed) + 1)
    o = torch.randn(case["n"], 3, device="cuda", generator=g)
    o = o / o.norm(dim=1, keepdim=True) * 2.5
    d = (torch.rand(case["n"], 3, device="cuda", generator=g) * 1.8 - 0.9) - o
    return m, v, o, d / d.norm(dim=1, keepdim=True)


def _scene(case, seed):
    r = _rng(seed, 2)
    name, w, h = case["scene"], case["w"], case["h"]
    layout = "mid" if name in ("mid", "emitter") else "tiny"
    # the literal configurations have nearly homogeneous tables (amplitude
    # 1e-4); 0.1 keeps their densities and gives the features a say
    f = _field_params(layout, seed, amp=0.1)
    jitter = r.uniform(-0.05, 0.05, size=3)
    cam = sg.Camera(pos=(float(jitter[0]), float(jitter[1]), float(-2.5 + jitter[2])), look_at=(0.0, 0.0, 0.0),
                    fov_deg=60.0, width=w, height=h, max_bounces=case["bounces"])
    lights = sg.seeded_light(int(seed)) if layout == "mid" else sg.no_lights()
    return sg.Scene(name=name, field=f, mesh=_static_mesh(name), lights=lights, cameras=[cam], t_near=0.05, t_far=4.0,
                    n_samples=case["samples"], max_bounces=case["bounces"], occupancy_res=128,
                    seed=int(seed) & 0xFFFFFFFF)


class _Graph:
    """A captured render, with everything its launches read and write."""

    def __init__(self, handle, keep):
        self.handle, self.keep = handle, keep

    def __del__(self):
        M.mr_graph_destroy(self.handle)


def prepare(case, seed):
    kind = case["kind"]
    st = {"case": case}
    if kind == "query":
        f, st["x"], st["d"] = _query_inputs(case, seed)
        st["field"] = M.Field(f, **_types(case["half"]))
    elif kind == "occupancy":
        st["field"] = M.Field(_field_params(case["layout"], seed, offset=-5.0), **_types(case["half"]))
    elif kind == "closest":
        m, v, st["o"], st["d"] = _closest_inputs(case, seed)
        st["mesh"], st["v"] = M.Mesh(m), torch.from_numpy(v).cuda()
    elif kind == "render":
        sc = _scene(case, seed)
        st["scene"], st["field"], st["mesh"] = sc, M.Field(sc.field, **_types(case["half"])), M.Mesh(sc.mesh)
        if case["occ"]:
            st["field"].build_occupancy(sc.occupancy_res, sc.occupancy_thresh)
        st["prop"] = None
        if case["sampler"] == "proposal":
            st["prop"] = M.Field(sg.make_proposal(seed=int(seed) % (1 << 30), table_amp=0.5),
                                 table_dtype=M.MR_F16 if case["half"] else M.MR_F32)
        st["opts"] = M.make_opts(sc, sampler=M.MR_SAMPLER_PROPOSAL if st["prop"] else M.MR_SAMPLER_UNIFORM,
                                 proposal=st["prop"], use_occupancy=case["occ"],
                                 shadow_mask=0.2 if case["shadows"] else None, sample_emitters=case["light_sampling"])
        st["o"], st["d"], _ = M.camera_rays(sg.cameras_array(sc.cameras))
        st["r"] = M.Renderer(sc.n_rays, sc.max_bounces)
        if case["refit"]:
            st["v"] = torch.from_numpy(sg.cloth_vertices(int(seed) % 997)).cuda()
    elif kind == "fields":
        sc = sg.fields_scene(case["fields"], case["w"], case["h"], spacing=case["spacing"], table_amp=0.1,
                             n_samples=case["samples"])
        for k, f in enumerate(sc.fields):   # other tables for another seed, same layout and placement
            g = sg.mid_field(seed=100 + int(seed) % (1 << 30) + k, table_amp=0.1)
            f.table, f.mlp = g.table, g.mlp
        st["fields"] = [M.Field(f, **_types(case["half"])) for f in sc.fields]
        if case["occ"]:
            for f in st["fields"]:
                f.build_occupancy(sc.occupancy_res, sc.occupancy_thresh)
        st["scene"], st["mesh"] = sc, M.Mesh(sc.mesh)
        st["opts"] = M.make_opts(sc, use_occupancy=case["occ"])
        st["o"], st["d"], _ = M.camera_rays(sg.cameras_array(sc.cameras))
        st["r"] = M.Renderer(sc.n_rays, sc.max_bounces)
    elif kind == "cameras":
        cams = sg.multicam_cameras(44)[16 - case["cams"]:]
        r = _rng(seed, 4)
        for c in cams:
            c.width, c.height = max(8, int(c.width * case["scale"])), max(8, int(c.height * case["scale"]))
            c.pos = tuple(float(p + q) for p, q in zip(c.pos, r.uniform(-0.02, 0.02, size=3)))
        sc = sg.multicam_scene(44)
        sc.cameras, sc.field, sc.seed = cams, _field_params("tiny", seed, amp=0.1), int(seed) & 0xFFFFFFFF
        o, d, ci = M.camera_rays(sg.cameras_array(cams))
        limits = torch.empty(sc.n_rays, dtype=torch.int32, device="cuda")
        M.mr_camera_bounce_limits(ci, sc.n_rays, [c.max_bounces for c in cams], limits)
        F, G = M.Field(sc.field), M.Mesh(sc.mesh)
        R = M.Renderer(sc.n_rays, sc.max_bounces, with_hits=False)
        opts = M.apply_launch(M.make_opts(sc), (0, 4, 384, 0, 8, 2))
        h = M.mr_render_graph_create(F.handle, G.handle, sc.n_rays, o, d, sc.max_bounces, limits, sc.lights, opts,
                                     R.out, R.workspace, R.ws_bytes)
        st["r"], st["graph"] = R, _Graph(h, (F, G, R, o, d, limits))
    elif kind == "train":
        st["field"] = M.Field(_field_params(case["layout"], seed))
        p = sg.make_proposal(seed=int(seed) % (1 << 30), table_amp=0.5)
        st["prop"] = M.Field(p)
        o, d = sg.random_rays(case["n"], seed=int(seed) % (1 << 30))
        st["o"], st["d"] = torch.from_numpy(o).cuda(), torch.from_numpy(d).cuda()
        st["trainer"] = M.ProposalTrainer(st["prop"], n_bins=case["bins"])
        st["loss"] = torch.empty(1, device="cuda")
        st["g_table"] = torch.empty(p.table.size, device="cuda")
        st["g_mlp"] = torch.empty(p.mlp.size, device="cuda")
    return st


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "query":
        r = st["field"].query(st["x"], st["d"])
        return r["sigma"], r["rgb"]
    if kind == "occupancy":
        return st["field"].build_occupancy(case["res"], 0.01, export=True)
    if kind == "closest":
        if case["refit"]:
            st["mesh"].refit(st["v"])
        return st["mesh"].closest_hit(st["o"], st["d"])
    if kind == "train":
        lohi, tgt = st["trainer"].targets(st["field"], st["o"], st["d"], 0.05, 4.0, case["samples"])
        M.mr_proposal_grad(st["prop"].handle, case["n"], st["o"], st["d"], lohi, tgt, case["bins"], st["loss"],
                           st["g_table"], st["g_mlp"])
        return lohi, tgt, st["loss"], st["g_table"], st["g_mlp"]
    R = st["r"]
    if kind == "cameras":
        M.mr_graph_launch(st["graph"].handle)
        return R.radiance, R.throughput, R.bounces, R.counters
    sc = st["scene"]
    if kind == "fields":
        R.render_fields(st["fields"], st["mesh"], st["o"], st["d"], sc.lights, st["opts"])
    else:
        if case["refit"]:
            st["mesh"].refit(st["v"])
        R.render(st["field"], st["mesh"], st["o"], st["d"], sc.lights, st["opts"])
    return R.radiance, R.throughput, R.bounces, R.hit_ids, R.counters


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

_TABLE = {"tiny": 8 * 2 * 2 ** 14, "mid": 16 * 2 * 2 ** 19}   # values
_DENSITY = 2 * (32 * 64 + 64 * 16)
_FLOPS = {"tiny": _DENSITY + 2 * (20 * 64 + 64 * 3), "mid": _DENSITY + 2 * (32 * 64 + 64 * 64 + 64 * 3)}


def work(case):
    """Each input read once, each output written once, and the MLP products of the field samples.  The sample
    counts of the renders are fractions of rays x intervals, from the renderer's own counters on these scenes."""
    kind, n = case["kind"], case.get("n", 0)
    tab = _TABLE.get(case.get("layout"), 0) * (2 if case.get("half") else 4)
    if kind == "query":
        return {"bytes": tab + n * (24 + 16), "flops": n * _FLOPS[case["layout"]]}
    if kind == "occupancy":
        cells = case["res"] ** 3
        return {"bytes": tab + cells * 1.125, "flops": 8 * cells * 2 * (32 * 64 + 64)}
    if kind == "closest":
        return {"bytes": n * 32 + (case["balls"] * 80 + 2) * 112, "flops": 0}
    if kind == "train":
        samples = 0.45 * n * case["samples"]
        return {"bytes": tab + 2 * 5 * 2 ** 17 * 8 + n * (24 + 16 + 8 * case["bins"]),
                "flops": samples * _DENSITY + 3 * 2 * n * case["bins"] * 176}
    if kind == "cameras":
        rays = sum(max(8, int(c.width * case["scale"])) * max(8, int(c.height * case["scale"]))
                   for c in sg.multicam_cameras(44)[16 - case["cams"]:])
        return {"bytes": _TABLE["tiny"] * 4 + rays * (24 + 4 + 28), "flops": rays * 30 * _FLOPS["tiny"]}
    rays = case["w"] * case["h"]
    if kind == "fields":
        return {"bytes": case["fields"] * _TABLE["mid"] * (2 if case["half"] else 4) + rays * (24 + 28 + 36),
                "flops": rays * 0.09 * case["samples"] * _FLOPS["mid"]}
    layout = "mid" if case["scene"] in ("mid", "emitter") else "tiny"
    per_ray = 42 if case["sampler"] == "proposal" else 0.31 * case["samples"]
    return {"bytes": _TABLE[layout] * (2 if case["half"] else 4) + rays * (24 + 28 + 4 * (case["bounces"] + 1)),
            "flops": rays * per_ray * _FLOPS[layout]}


# ---------------------------------------------------------------------------
# the same values in 64 bits, from the definitions
# ---------------------------------------------------------------------------

def _bf16(a):
    return a.to(torch.bfloat16).to(torch.float64)


def _encode64(x, table, res, log2_table, lo=-1.0, hi=1.0):
    """Hash-grid features (n, 2 L) of field-frame points x (n, 3) in 64 bits; table (L, T, 2)."""
    xh = ((x - lo) / (hi - lo)).clamp(0.0, 1.0)
    T = 1 << log2_table
    out = []
    for l, N in enumerate(res):
        N = int(N)
        p = xh * N
        v = p.floor().clamp(max=N - 1)
        w = p - v
        v = v.long()
        f = 0.0
        for c in range(8):
            k = [(c >> a) & 1 for a in range(3)]
            q = [v[:, a] + k[a] for a in range(3)]
            if (N + 1) ** 3 <= T:
                i = q[0] + q[1] * (N + 1) + q[2] * (N + 1) ** 2
            else:
                i = (q[0] ^ (q[1] * 2654435761 & 0xFFFFFFFF) ^ (q[2] * 805459861 & 0xFFFFFFFF)) & (T - 1)
            t = 1.0
            for a in range(3):
                t = t * (w[:, a] if k[a] else 1.0 - w[:, a])
            f = f + t[:, None] * table[l][i]
        out.append(f)
    return torch.cat(out, dim=1)


def _sh64(d, n):
    x, y, z = d[:, 0], d[:, 1], d[:, 2]
    pi = math.pi
    c = [0.5 * math.sqrt(1 / pi) * torch.ones_like(x), -math.sqrt(3 / (4 * pi)) * y, math.sqrt(3 / (4 * pi)) * z,
         -math.sqrt(3 / (4 * pi)) * x]
    if n == 16:
        a, b = math.sqrt(15 / pi), math.sqrt(5 / pi)
        c += [a / 2 * x * y, -a / 2 * y * z, b / 4 * (3 * z * z - 1), -a / 2 * x * z, a / 4 * (x * x - y * y),
              -math.sqrt(35 / (2 * pi)) / 4 * y * (3 * x * x - y * y), math.sqrt(105 / pi) / 2 * x * y * z,
              -math.sqrt(21 / (2 * pi)) / 4 * y * (5 * z * z - 1), math.sqrt(7 / pi) / 4 * z * (5 * z * z - 3),
              -math.sqrt(21 / (2 * pi)) / 4 * x * (5 * z * z - 1), math.sqrt(105 / pi) / 4 * z * (x * x - y * y),
              -math.sqrt(35 / (2 * pi)) / 4 * x * (x * x - 3 * y * y)]
    return torch.stack(c, dim=1)


class _Field64:
    """A field in 64 bits on the parameters as the handle holds them (an FP16 table and, in the BF16 engine, rounded
    hidden layers; the SH columns and the output layer stay FP32)."""

    def __init__(self, f, half):
        self.f = f
        t = torch.from_numpy(f.table).cuda()
        self.table = (t.half() if half else t).double()
        self.layers, off = [], 0
        shapes = f.layer_shapes()
        for i, (o, n) in enumerate(shapes):
            W = torch.from_numpy(f.mlp[off:off + o * n].reshape(o, n).copy()).cuda()
            W64 = W.double()
            if half and i < len(shapes) - 1:
                W64 = _bf16(W)
                if i == 2:
                    W64[:, f.d_out:] = W.double()[:, f.d_out:]
            self.layers.append(W64)
            off += o * n

    def raw(self, x):
        f = self.f
        e = _encode64(x, self.table, f.resolutions, f.log2_table)
        h = torch.relu(e @ self.layers[0][:, :e.shape[1]].T)
        return h @ self.layers[1].T

    def sigma(self, x):
        return torch.nn.functional.softplus(self.raw(x)[:, 0] + self.f.density_offset, threshold=1e9)

    def __call__(self, x, d):
        raw = self.raw(x)
        c = torch.cat([raw, _sh64(d, self.f.sh)], dim=1)
        c = torch.relu(c @ self.layers[2][:, :c.shape[1]].T)
        for W in self.layers[3:-1]:
            c = torch.relu(c @ W.T)
        sigma = torch.nn.functional.softplus(raw[:, 0] + self.f.density_offset, threshold=1e9)
        return sigma, torch.exp(c @ self.layers[-1].T)


def _box64(o, d, t0, t1):
    """[lo, hi] of rays in the box [-1, 1]^3 and [t0, t1]; hi <= lo on a miss."""
    a, b = (-1.0 - o) / d, (1.0 - o) / d
    lo = torch.minimum(a, b).amax(dim=1).clamp(min=t0)
    hi = torch.maximum(a, b).amin(dim=1).clamp(max=t1)
    return lo, hi


def _targets64(F, o, d, t0, t1, n_samples, bins):
    lo, hi = _box64(o, d, t0, t1)
    hit = hi > lo
    lo, hi = torch.where(hit, lo, torch.zeros_like(lo)), torch.where(hit, hi, torch.zeros_like(hi))
    delta = (t1 - t0) / n_samples
    k = torch.arange(n_samples, device=o.device, dtype=torch.float64)
    a = torch.maximum(t0 + k[None] * delta, lo[:, None])
    b = torch.minimum(t0 + (k[None] + 1.0) * delta, hi[:, None])
    ok = (b > a) & hit[:, None]
    D = torch.where(ok, b - a, torch.zeros_like(a))
    x = o[:, None, :] + (0.5 * (a + b))[:, :, None] * d[:, None, :]
    tau = torch.zeros_like(D)
    tau[ok] = F.sigma(x[ok])
    tau = tau * D
    T = torch.exp(-(tau.cumsum(dim=1) - tau))
    w = T * -torch.expm1(-tau)
    bw = ((hi - lo) / bins)[:, None]
    hist = []
    for j in range(bins):
        c0, c1 = lo[:, None] + j * bw, lo[:, None] + (j + 1) * bw
        ov = (torch.minimum(b, c1) - torch.maximum(a, c0)).clamp(min=0.0)
        hist.append(torch.where(ok, w * ov / D.clamp(min=1e-300), torch.zeros_like(w)).sum(dim=1))
    return torch.stack([lo, hi], dim=1), torch.stack(hist, dim=1)


def _exact_train(case, seed):
    F = _Field64(_field_params(case["layout"], seed), False)
    p = sg.make_proposal(seed=int(seed) % (1 << 30), table_amp=0.5)
    o, d = (torch.from_numpy(a).cuda().double() for a in sg.random_rays(case["n"], seed=int(seed) % (1 << 30)))
    parts = [_targets64(F, o[i:i + 2048], d[i:i + 2048], 0.05, 4.0, case["samples"], case["bins"])
             for i in range(0, case["n"], 2048)]
    lohi, tgt = (torch.cat(v) for v in zip(*parts))
    bins = case["bins"]
    table = torch.from_numpy(p.table).cuda().double().requires_grad_()
    mlp = torch.from_numpy(p.mlp).cuda().double().requires_grad_()
    W1, W2 = mlp[:p.hidden * 10].reshape(p.hidden, 10), mlp[p.hidden * 10:]
    lo, D = lohi[:, :1], (lohi[:, 1:] - lohi[:, :1]) / bins
    tm = lo + (torch.arange(bins, device="cuda") + 0.5)[None] * D
    x = (o[:, None, :] + tm[:, :, None] * d[:, None, :]).reshape(-1, 3)
    z = torch.relu(_encode64(x, table, p.resolutions, p.log2_table) @ W1.T) @ W2 + p.density_offset
    tau = torch.nn.functional.softplus(z, threshold=1e9).reshape(-1, bins) * D
    w = torch.exp(-(tau.cumsum(dim=1) - tau)) * -torch.expm1(-tau)
    miss = torch.relu(tgt - w)
    loss = (miss * miss / (tgt + 1e-7) * (lohi[:, 1:] > lohi[:, :1])).sum() / case["n"]
    g_table, g_mlp = torch.autograd.grad(loss, (table, mlp))
    return lohi, tgt, loss.detach().reshape(1), g_table.reshape(-1), g_mlp


def _exact_closest(case, seed):
    """Every ray against every triangle (Moller-Trumbore), the nearest t; the triangle ids are whole numbers."""
    m, v, o, d = _closest_inputs(case, seed)
    o, d = o.double(), d.double()
    V = torch.from_numpy(v).cuda().double()[torch.from_numpy(m.indices).cuda().long()]
    best = torch.full((case["n"],), math.inf, device="cuda", dtype=torch.float64)
    a, e1, e2 = V[:, 0], V[:, 1] - V[:, 0], V[:, 2] - V[:, 0]
    # with n = e1 x e2 and s = o - a: det = -d.n, t = s.n / det, u = (s x d).-e2 / det, v = (s x d).e1 / det,
    # each a product of per-ray and per-triangle vectors
    nrm = torch.linalg.cross(e1, e2)
    od = torch.linalg.cross(o, d)
    step = max(1, (1 << 25) // len(a))
    for i in range(0, case["n"], step):
        O, Dd, OD = o[i:i + step], d[i:i + step], od[i:i + step]
        det = -(Dd @ nrm.T)
        t = (O @ nrm.T - (a * nrm).sum(1)) / det
        # (s x d) = o x d - a x d;  (a x d).e = d.(e x a)
        u = -(OD @ e2.T - Dd @ torch.linalg.cross(e2, a).T) / det
        w = (OD @ e1.T - Dd @ torch.linalg.cross(e1, a).T) / det
        ok = (u >= 0) & (w >= 0) & (u + w <= 1) & (t > 0)
        best[i:i + step] = torch.where(ok, t, torch.full_like(t, math.inf)).amin(dim=1)
    return best, None


def exact(case, seed):
    kind = case["kind"]
    if kind == "query":
        f, x, d = _query_inputs(case, seed)
        F = _Field64(f, case["half"])
        x, d = x.double(), d.double()
        if f.pose is not None:
            P = torch.from_numpy(np.asarray(f.pose, np.float32)).cuda().double()
            x, d = (x - P[:, 3]) @ P[:, :3], d @ P[:, :3]
        parts = [F(x[i:i + (1 << 18)], d[i:i + (1 << 18)]) for i in range(0, case["n"], 1 << 18)]
        return tuple(torch.cat(v) for v in zip(*parts))
    if kind == "closest":
        return _exact_closest(case, seed)
    if kind == "train":
        return _exact_train(case, seed)
    # whole renders branch at every bounce and march millions of samples; an occupancy grid is whole numbers
    return None
