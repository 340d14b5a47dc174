"""The work that a user of this framework has it do, as measured cases.

Every case goes through the package's public calls on inputs drawn from a
seed: ray queries, whole frames, batches of frames, a served request stream,
hierarchy builds, frames of moving geometry and the post-process passes.
Scenes come from `scenegen` (the inputs that the tests and the benchmark
use); `exact` holds a brute-force float64 model of what the calls compute.

  listed()            the cases
  draw(rng)           one more case of the same ranges
  prepare(case, seed) what a program has in hand before the call
  run(state)          one pass through the public calls, and its outputs
  work(case)          bytes and operations that a pass cannot do without
  exact(case, seed)   the outputs in float64, where they have such a value
"""
import math

import numpy as np
import torch

import paper_2001_09792_amd as rg
import scenegen as sg
from paper_2001_09792_amd import serve

# pairs of ray and triangle that the brute-force model may test (a few seconds)
PAIRS_CUDA, PAIRS_CPU = 1.2e10, 2e8


def listed():
    return [
        # a picking or visibility query: few rays, latency and launches count
        dict(name="rays_1k", kind="rays", scene="two_level", tris=184320, meshes=3, instances=64, n=1000,
             query="closest", options=False, width=4, leaf=4, builder="lbvh"),
        # the benchmark's step: camera rays and 8 occlusion rays per hit over 10M unique triangles
        dict(name="ao_step_1080p", kind="ao", scene="incoherent", tris=10035200, meshes=16, instances=1024, w=1920,
             h=1080, query="closest", options=False, width=4, leaf=1, builder="treelet"),
        # occlusion queries with visibility masks, culling and opacity masks, an odd image size
        dict(name="ao_any_options", kind="ao", scene="incoherent", tris=627200, meshes=4, instances=256, w=1001,
             h=563, query="any", options=True, width=4, leaf=1, builder="treelet"),
        # an interactive preview: the smallest configuration's frame
        dict(name="frame_256_d1", kind="frame", scene="small", tris=1282, meshes=1, instances=1, w=256, h=256,
             depth=1, mode=0, width=4, leaf=4, builder="lbvh"),
        # a full frame with reflections, refractions and shadows
        dict(name="frame_1080p_d4", kind="frame", scene="two_level", tris=184320, meshes=3, instances=64, w=1920,
             h=1080, depth=4, mode=0, width=8, leaf=1, builder="treelet"),
        # an ambient-occlusion frame at a preview size, hierarchy of the package's defaults
        dict(name="ao_frame_360p", kind="frame", scene="uneven", tris=60000, meshes=4, instances=24, w=640, h=360,
             depth=0, mode=1, width=4, leaf=4, builder="lbvh"),
        # frames of unrelated scenes and sizes rendered together
        dict(name="batch_24", kind="batch", frames=24, tris_min=1000, tris_max=200000, instances=128, pix_min=4096,
             pix_max=1048576, depth=2, width=4, leaf=1, builder="lbvh"),
        # a request stream over resident scenes, all requests waiting at the start
        dict(name="serve_24", kind="serve", requests=24, small=4, large=2, tris=627200, budget_gib=16, width=4,
             leaf=1, builder="treelet"),
        # loading one large mesh
        dict(name="build_linear_627k", kind="build", scene="uneven", tris=627200, meshes=1, instances=1, n=4096,
             later=True, width=4, leaf=1, builder="lbvh"),
        # loading a scene of a few meshes with the hierarchy that traces fastest
        dict(name="build_treelet_scene", kind="build", scene="two_level", tris=184320, meshes=3, instances=64,
             n=4096, later=False, width=8, leaf=1, builder="treelet"),
        # a frame of an animation: vertices and instances moved, then the camera's rays
        dict(name="dynamic_720p", kind="dynamic", scene="incoherent", tris=2508800, meshes=16, instances=512, w=1280,
             h=720, width=4, leaf=1, builder="treelet"),
        # the post-process passes on a full frame
        dict(name="post_1080p", kind="post", w=1920, h=1080, radius=8, materials=64),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["rays", "ao", "frame", "batch", "serve", "build", "dynamic", "post"])
    width, leaf = rng.choice([(2, 1), (4, 1), (4, 4), (4, 1), (8, 1), (8, 2)])
    shape = dict(width=width, leaf=leaf, builder=rng.choice(["lbvh", "treelet", "ploc"]))
    instances = _log_int(rng, 1, 1024)
    scene = dict(scene="uneven", tris=_log_int(rng, 1000, 1000000), meshes=min(instances, rng.randint(1, 8)),
                 instances=instances)
    image = dict(w=_log_int(rng, 64, 1920), h=_log_int(rng, 48, 1080))
    if kind == "rays":
        return dict(kind=kind, **scene, n=_log_int(rng, 1, 2000000), query=rng.choice(["closest", "any", "found"]),
                    options=rng.random() < 0.3, **shape)
    if kind == "ao":
        return dict(kind=kind, **scene, **image, query=rng.choice(["closest", "any"]),
                    options=rng.random() < 0.3, **shape)
    if kind == "frame":
        mode = 1 if rng.random() < 0.25 else 0
        return dict(kind=kind, **scene, **image, depth=0 if mode else rng.randint(0, 4), mode=mode, **shape)
    if kind == "batch":
        return dict(kind=kind, frames=rng.randint(2, 32), tris_min=1000, tris_max=_log_int(rng, 5000, 200000),
                    instances=_log_int(rng, 2, 128), pix_min=4096, pix_max=_log_int(rng, 16384, 1048576),
                    depth=rng.randint(0, 2), **shape)
    if kind == "serve":
        return dict(kind=kind, requests=rng.randint(1, 32), small=rng.randint(1, 4), large=rng.randint(0, 2),
                    tris=_log_int(rng, 10000, 1000000), budget_gib=rng.choice([8, 16]), **shape)
    if kind == "build":
        return dict(kind=kind, **scene, n=4096, later=shape["builder"] == "lbvh" and rng.random() < 0.5, **shape)
    if kind == "dynamic":
        return dict(kind=kind, **scene, **image, **shape)
    return dict(kind=kind, **image, radius=rng.choice([0, 1, 3, 8, 8, 12, 16]), materials=_log_int(rng, 2, 256))


# ------------------------------------------------------------------ inputs
def _mesh(kind, tris, seed):
    """An icosphere, torus or displaced grid near `tris` triangles."""
    m = int(max(3, round(math.sqrt(tris / 2.0))))
    if kind == 0 and tris < 100000:
        return sg.icosphere(int(max(0, round(math.log(max(tris, 20) / 20.0, 4)))))
    return sg.grid(m, m, 0.15, 4.0, seed) if kind == 2 else sg.torus(m, m, 1.0, 0.3, 0.05, 5.0, seed)


def _materials(rng, n):
    rows = []
    for k in rng.integers(0, 3, n):
        if k == sg.DIFFUSE:
            rows.append((sg.DIFFUSE, tuple(rng.uniform(0.2, 0.9, 3)), 1.5))
        else:
            rows.append((int(k), (0.9, 0.9, 0.9) if k == sg.MIRROR else (1.0, 1.0, 1.0), 1.5))
    return sg.materials(rows)


def _scene(case, seed):
    """The case's scene: one of the benchmark's configurations, or instances
    of meshes of the case's triangle count spread at their density."""
    w, h, depth = case.get("w", 256), case.get("h", 256), case.get("depth", 1)
    if case["scene"] == "small":
        s = sg.config_small()
        rng = np.random.default_rng(seed)
        s.camera = sg.Camera((float(rng.uniform(-1, 1)), 1.0, 4.0), (0.0, 0.0, 0.0), (0.0, 1.0, 0.0), 60.0)
        s.light = sg.Light((float(rng.uniform(3, 5)), 6.0, 3.0))
        s.width, s.height, s.max_depth = w, h, depth
        return s
    if case["scene"] == "two_level":
        return sg.config_two_level(seed=seed, width=w, height=h, max_depth=depth)
    n_inst, n_mesh = case["instances"], case["meshes"]
    rng = np.random.default_rng(np.random.SeedSequence([seed, 1]))
    if case["scene"] == "incoherent":
        m = int(round(math.sqrt(case["tris"] / n_mesh / 2.0)))
        meshes = [sg.torus(m, m, 1.0, 0.35, 0.25 * 0.35, 6.0, 3000 + 16 * seed + k) for k in range(n_mesh)]
    else:
        meshes = [_mesh(k % 3 if n_mesh > 1 else 1, case["tris"] / n_mesh, 100 * seed + k) for k in range(n_mesh)]
    c = 2.0 * n_inst ** (1.0 / 3.0)
    return sg.Scene("case", meshes, sg.random_instances(rng, n_inst, extent=c),
                    (np.arange(n_inst) % n_mesh).astype(np.uint32), np.arange(n_inst, dtype=np.uint32) % 256,
                    _materials(rng, min(n_inst, 256)),
                    sg.Camera((0.0, 0.0, 2.2 * c + 2.0), (0.0, 0.0, 0.0), (0.0, 1.0, 0.0), 60.0),
                    sg.Light((c + 5.0, 2.0 * c + 10.0, c + 8.0)), w, h, depth, case.get("mode", 0), seed)


def _device_meshes(scene):
    out = []
    for m in scene.blas:
        pm = None if m.prim_mat is None else torch.from_numpy(
            np.ascontiguousarray(m.prim_mat, np.uint16).view(np.int16)).cuda()
        out.append((torch.from_numpy(np.ascontiguousarray(m.verts, np.float32)).cuda(),
                    torch.from_numpy(np.ascontiguousarray(m.idx, np.uint32).view(np.int32)).cuda(), pm))
    return out


def _upload(case, scene, flags=None, alpha=None):
    if alpha is None:
        return rg.upload_scene(scene, width=case["width"], leaf_max=case["leaf"], builder=case["builder"])
    blas = []
    for (v, i, pm), a in zip(_device_meshes(scene), alpha):
        b = rg.build_blas(v, i, pm, case["width"], case["leaf"], builder=case["builder"])
        if a is not None:
            rg.set_alpha(b, torch.from_numpy(a[0].view(np.int64)).cuda(), a[1])
        blas.append(b)
    return rg.build_tlas(blas, scene.xform, scene.blas_id, scene.inst_mat, case["width"], builder=case["builder"],
                         inst_flags=flags)


def _random_rays(case, seed):
    """Rays as a query meets them: origins inside the instances' spread, any direction."""
    ext = 20.0 if case["scene"] == "two_level" else 2.0 * case["instances"] ** (1.0 / 3.0)
    return sg.random_rays(case["n"], 7000 + seed, extent=ext)


def _post_inputs(case, seed):
    """A frame as the tracer leaves it: a sky gradient behind discs and
    half-planes of one material each, shaded, unfiltered edges; beside it the
    material per pixel and the roughness per material."""
    rng = np.random.default_rng(np.random.SeedSequence([seed, 2]))
    w, h, n = case["w"], case["h"], case["materials"]
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    y = (torch.arange(h, device=dev, dtype=torch.float64)[:, None] + 0.5).expand(h, w)
    x = (torch.arange(w, device=dev, dtype=torch.float64)[None, :] + 0.5).expand(h, w)
    v = y / h
    img = torch.stack([1.0 - 0.5 * v, 1.0 - 0.3 * v, torch.ones_like(v)], -1)
    mat = torch.full((h, w), -1, dtype=torch.int32, device=dev)
    for k in range(40):
        cx, cy = rng.uniform(0, w), rng.uniform(0, h)
        if k % 4:
            inside = (x - cx) ** 2 + (y - cy) ** 2 <= (rng.uniform(0.02, 0.25) * max(w, h)) ** 2
        else:
            a = rng.uniform(0, 2 * math.pi)
            inside = math.cos(a) * (x - cx) + math.sin(a) * (y - cy) > rng.uniform(0.2, 0.5) * max(w, h)
        col = torch.tensor(rng.uniform(0.0, 1.0, 3) * (2.0 if rng.random() < 0.2 else 1.0), device=dev)
        ramp = 0.6 + 0.4 * torch.cos(rng.uniform(2, 9) * x / w + rng.uniform(2, 9) * v + rng.uniform(0, 6))
        if rng.random() < 0.3:
            c = int(rng.integers(4, 24))
            ramp = torch.where(((x // c + y // c) % 2) == 0, ramp, 0.55 * ramp)
        img = torch.where(inside[..., None], ramp[..., None] * col, img)
        mat = torch.where(inside, torch.tensor(int(rng.integers(0, n)), dtype=torch.int32, device=dev), mat)
    return img.float().contiguous(), mat.contiguous(), torch.from_numpy(sg.roughness_table(n, seed)).to(dev)


def _batch_scenes(case, seed):
    """Scenes of the seed; the images' sizes are the case's own."""
    scenes = sg.config_batched(seed=seed, n_scenes=case["frames"], tri_range=(case["tris_min"], case["tris_max"]),
                               max_inst=case["instances"], pix_range=(case["pix_min"], case["pix_max"]),
                               max_depth=case["depth"])
    rng = np.random.default_rng(case["frames"])
    for c in scenes:
        c.width = int(round(math.sqrt(math.exp(rng.uniform(math.log(case["pix_min"]), math.log(case["pix_max"]))))))
        c.height = int(round(c.width * rng.uniform(0.6, 1.0)))
    return scenes


def prepare(case, seed):
    s = dict(case=case)
    kind = case["kind"]
    if kind == "post":
        s["image"], s["mat"], s["rough"] = _post_inputs(case, seed)
        s["post"] = rg.Post(case["w"], case["h"])
        s["blurred"], s["final"] = torch.empty_like(s["image"]), torch.empty_like(s["image"])
        return s
    if kind == "batch":
        frames = [(rg.upload_scene(c, width=case["width"], leaf_max=case["leaf"], builder=case["builder"]),
                   c.materials, c.camera, c.light, c.width, c.height, c.max_depth)
                  for c in _batch_scenes(case, seed)]
        s["batch"] = rg.Batch(frames)
        return s
    if kind == "serve":
        entries = []
        for k in range(case["small"]):
            c = sg.config_two_level(seed=5000 + 64 * seed + k)
            entries.append((_upload(case, c), c))
        for k in range(case["large"]):
            c = _scene(dict(scene="incoherent", tris=case["tris"], meshes=4, instances=256), 64 * seed + k)
            entries.append((_upload(case, c), c))
        table = [(tl, rg.materials_array(c.materials), c.camera, c.light) for tl, c in entries]
        s["cache"] = serve.ResidentCache(lambda k: (table[k], table[k][0].buf.numel()))
        s["engine"] = rg.Engine(**rg.Engine.for_budget(case["budget_gib"] << 30, max_jobs=64, width=case["width"]))
        s["requests"] = lambda: serve.poisson_requests(case["requests"], math.inf, len(table), 5)
        return s
    scene = _scene(case, seed)
    s["scene"] = scene
    if kind == "build":
        s["meshes"] = _device_meshes(scene)
        s["rays"] = rg.rays_to_device(_random_rays(case, seed))
        return s
    if kind == "dynamic":
        s["moved"] = [torch.from_numpy(sg.animate_mesh(m, 0.15, amp=0.02, seed=seed + k)).cuda()
                      for k, m in enumerate(scene.blas)]
        s["xform"] = sg.animate_instances(scene.xform, 0.15, seed=seed)
        s["tlas"] = _upload(case, scene)
        s["idx"] = [i for _, i, _ in _device_meshes(scene)]
        s["top"] = rg.TlasBuilder(s["tlas"].blas, scene.blas_id, scene.inst_mat, case["width"])
    elif kind in ("rays", "ao") and case["options"]:
        flags, alpha = sg.option_inputs(scene, seed=seed)
        s["tlas"] = _upload(case, scene, flags, alpha)
        s["opts"] = dict(cull=rg.RAY_CULL_BACK, mask=0x02)
    else:
        s["tlas"] = _upload(case, scene)
    s.setdefault("opts", {})
    if kind == "frame":
        s["renderer"] = rg.Renderer(case["w"], case["h"], case["depth"], case["mode"])
        s["mats"] = rg.materials_array(scene.materials)
        s["pm"] = torch.empty((case["h"], case["w"]), dtype=torch.int32, device="cuda") if case["mode"] == 0 else None
        return s
    if kind == "rays":
        s["rays"] = rg.rays_to_device(_random_rays(case, seed))
        s["hits"] = rg.alloc_hits(case["n"])
        s["occ"] = torch.empty(case["n"], dtype=torch.uint8, device="cuda")
        return s
    n = case["w"] * case["h"]
    s["cam"] = torch.empty((8, n), dtype=torch.float32, device="cuda")
    s["hits"] = rg.alloc_hits(n)
    if kind == "ao":
        s["ao"] = torch.zeros((8, 8 * n), dtype=torch.float32, device="cuda")
        s["src"] = torch.zeros(8 * n, dtype=torch.int32, device="cuda")
        s["count"] = torch.zeros(1, dtype=torch.int32, device="cuda")
        need = rg.c_u64()
        rg._check("rg_ao_rays_scratch", rg._lib.rg_ao_rays_scratch(n, rg.ctypes.byref(need)))
        s["scratch"] = torch.empty(max(256, need.value), dtype=torch.uint8, device="cuda")
        # the number of rays is known from an earlier frame of the same view
        rg.camera_rays(scene.camera, case["w"], case["h"], out=s["cam"])
        rg.trace_closest(s["tlas"], s["cam"], out=s["hits"])
        s["n_ao"] = 8 * int((s["hits"]["inst"] != -1).sum().item())
        s["ao_hits"] = {k: v.zero_() for k, v in rg.alloc_hits(8 * n).items()}
        s["occ"] = torch.zeros(8 * n, dtype=torch.uint8, device="cuda")
    return s


# -------------------------------------------------------------------- runs
def _run_rays(s):
    q = s["case"]["query"]
    if q == "closest":
        return rg.trace_closest(s["tlas"], s["rays"], out=s["hits"], **s["opts"])
    found = {k: s["hits"][k] for k in ("inst", "prim")} if q == "found" else None
    occ = rg.trace_any(s["tlas"], s["rays"], occluded=s["occ"], found=found, **s["opts"])
    # which triangle an any-hit query stops at is open: its being one is the result
    return dict(occluded=occ) if found is None else dict(occluded=occ, found=found["inst"] != -1)


def _run_ao(s):
    c, scene = s["case"], s["scene"]
    rg.camera_rays(scene.camera, c["w"], c["h"], out=s["cam"])
    rg.trace_closest(s["tlas"], s["cam"], out=s["hits"])
    rg.ao_rays(s["tlas"], s["cam"], s["hits"], scene.seed, 5.0, out=s["ao"], src=s["src"], count=s["count"],
               scratch=s["scratch"])
    m = s["n_ao"]
    rays = s["ao"][:, :m]
    if m and c["query"] == "closest":
        rg.trace_closest(s["tlas"], rays, out={k: v[:m] for k, v in s["ao_hits"].items()}, **s["opts"])
    elif m:
        rg.trace_any(s["tlas"], rays, occluded=s["occ"][:m], **s["opts"])
    # the buffers are sized for a hit at every pixel: zero past the rays there are
    return dict(camera=s["cam"], primary=s["hits"], ao=s["ao"], src=s["src"], count=s["count"],
                result=s["ao_hits"] if c["query"] == "closest" else s["occ"])


def _run_frame(s):
    scene = s["scene"]
    img = s["renderer"].render(s["tlas"], s["mats"], scene.camera, scene.light, scene.seed, primary_mat=s["pm"])
    return dict(image=img, primary=s["pm"])


def _run_serve(s):
    ex = serve.EngineExecutor(s["engine"], s["cache"], keep_images=True)
    serve.serve(s["requests"](), ex, serve.RealClock())
    return [ex.images[k] for k in sorted(ex.images)]


def _run_build(s):
    c, scene = s["case"], s["scene"]
    opts = dict(width=c["width"], leaf_max=c["leaf"])
    if c["later"]:
        pending = [rg.build_blas_async(v, i, pm, **opts) for v, i, pm in s["meshes"]]
        blas = [p.finish() for p in pending]
    else:
        blas = [rg.build_blas(v, i, pm, builder=c["builder"], **opts) for v, i, pm in s["meshes"]]
    tl = rg.build_tlas(blas, scene.xform, scene.blas_id, scene.inst_mat, c["width"], builder=c["builder"])
    out = dict(hits=rg.trace_closest(tl, s["rays"]), box=np.array([list(b.desc.lo) + list(b.desc.hi) for b in blas]),
               tris=[], slots=[])
    for b in blas:  # the documented parts of the structure that do not hang on the order of its nodes
        t, k, n = int(b.desc.tris_off), int(b.desc.slots_off), b.n_tris
        out["tris"].append(b.buf[t:t + 40 * n].view(torch.int32))
        out["slots"].append(b.buf[k:k + 4 * n].view(torch.int32))
    return out


def _run_dynamic(s):
    c, scene = s["case"], s["scene"]
    rg.refit_blas_many(s["tlas"].blas, s["moved"], s["idx"])
    tl = s["top"].build(s["xform"])
    rg.camera_rays(scene.camera, c["w"], c["h"], out=s["cam"])
    return rg.trace_closest(tl, s["cam"], out=s["hits"])


def _run_post(s):
    blurred = s["post"].roughness_blur(s["image"], s["mat"], s["rough"], s["case"]["radius"], out=s["blurred"])
    return dict(blurred=blurred, final=s["post"].fxaa(blurred, out=s["final"]))


def run(state):
    return dict(rays=_run_rays, ao=_run_ao, frame=_run_frame, batch=lambda s: s["batch"].render(), serve=_run_serve,
                build=_run_build, dynamic=_run_dynamic, post=_run_post)[state["case"]["kind"]](state)


# -------------------------------------------------------------------- work
def _trace_work(rays, tris, instances, width):
    """A ray and its hit, the geometry at most once (40 bytes a triangle, at
    least one triangle a ray), one box test per child on the way down both
    levels and one triangle test."""
    levels = math.log(max(instances, 2), width) + math.log(max(tris, 2), width)
    return dict(bytes=rays * 52 + 40 * min(tris, rays * 4), flops=rays * (levels * width * 18 + 60))


def work(case):
    k = case["kind"]
    if k == "post":
        n = case["w"] * case["h"]
        return dict(bytes=n * (12 + 4 + 12 + 12 + 12), flops=n * (2 * 8 * (2 * case["radius"] + 1) + 60))
    if k == "rays":
        return _trace_work(case["n"], case["tris"], case["instances"], case["width"])
    if k == "serve":
        pix = case["requests"] * sum(w * h for w, h in serve.RESOLUTIONS) / len(serve.RESOLUTIONS)
        t = _trace_work(2 * pix, 184320 * case["small"] + case["tris"] * case["large"], 64, case["width"])
        return dict(bytes=12 * pix + 40 * (184320 * case["small"] + case["tris"] * case["large"]), flops=t["flops"])
    if k == "batch":
        mid = lambda lo, hi: (hi - lo) / math.log(hi / lo)  # noqa: E731  (mean of a log-uniform draw)
        pix = case["frames"] * mid(case["pix_min"], case["pix_max"])
        tris = case["frames"] * mid(case["tris_min"], case["tris_max"])
        t = _trace_work(2 * pix, tris / case["frames"], case["instances"], case["width"])
        return dict(bytes=12 * pix + 40 * min(tris, 4 * pix), flops=t["flops"])
    tris, inst, width = case["tris"], case["instances"], case["width"]
    if k == "build":
        # vertices and indices in; triangles, slots and nodes out; a comparison sort's key comparisons
        return dict(bytes=tris * (12 + 6 + 40 + 4 + 32 * width / (width - 1)) + inst * 160 + case["n"] * 52,
                    flops=tris * (2 * math.log2(max(tris, 2)) + 60))
    pix = case["w"] * case["h"]
    t = _trace_work(pix, tris, inst, width)
    if k == "dynamic":
        return dict(bytes=t["bytes"] + tris * (12 + 6 + 40 + 32 * width / (width - 1)) + inst * 160,
                    flops=t["flops"] + tris * 60)
    if k == "frame":
        rays = 9 * pix if case["mode"] else 2 * pix
        return dict(bytes=12 * pix + 40 * min(tris, 4 * pix),
                    flops=_trace_work(rays, tris, inst, width)["flops"])
    # camera rays that hit spawn 8 more: six in ten, as the benchmark's view has it
    ao = _trace_work(0.6 * 8 * pix, tris, inst, width)
    return dict(bytes=t["bytes"] + ao["bytes"] + 0.6 * 8 * pix * 36, flops=t["flops"] + ao["flops"])


# ------------------------------------------------------------------- exact
def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _world_triangles(scene):
    """Per instance: float64 world-space corners [T, 3, 3]."""
    dev = _device()
    meshes = [torch.from_numpy(m.verts.astype(np.float64)[m.idx]).to(dev) for m in scene.blas]
    X = torch.from_numpy(np.asarray(scene.xform, np.float64).reshape(-1, 3, 4)).to(dev)
    for k in range(X.shape[0]):
        yield k, meshes[int(scene.blas_id[k])] @ X[k, :, :3].T + X[k, :, 3]


def _pairs(rays, scene):
    return rays * float(sum(scene.blas[b].idx.shape[0] for b in scene.blas_id))


def _nearest(scene, o, d, tmin, tmax):
    """Brute-force closest hit in float64: t, u, v, instance, triangle."""
    n, dev = o.shape[0], o.device
    best = torch.full((n,), math.inf, dtype=torch.float64, device=dev)
    bu, bv = torch.zeros_like(best), torch.zeros_like(best)
    bi = torch.full((n,), -1, dtype=torch.int64, device=dev)
    bp = bi.clone()
    step = 1 << 14
    for k, tri in _world_triangles(scene):
        for a in range(0, tri.shape[0], step):
            p0 = tri[a:a + step, 0]
            e1, e2 = tri[a:a + step, 1] - p0, tri[a:a + step, 2] - p0
            rows = max(1, (1 << 24) // p0.shape[0])
            for r in range(0, n, rows):
                dd, s = d[r:r + rows, None], o[r:r + rows, None] - p0
                pv = torch.linalg.cross(dd, e2[None])
                det = (e1 * pv).sum(-1)
                q = torch.linalg.cross(s, e1[None].expand_as(s))
                u, v = (s * pv).sum(-1) / det, (dd * q).sum(-1) / det
                t = (e2 * q).sum(-1) / det
                ok = (u >= 0) & (v >= 0) & (u + v <= 1) & (t >= tmin) & (t <= tmax[r:r + rows, None])
                t = torch.where(ok, t, math.inf)
                m, j = t.min(1)
                better = m < best[r:r + rows]
                at = torch.arange(m.shape[0], device=dev)
                for to, new in ((best, m), (bu, u[at, j]), (bv, v[at, j]), (bi, torch.full_like(j, k)),
                                (bp, j + a)):
                    to[r:r + rows] = torch.where(better, new, to[r:r + rows])
    return best, bu, bv, bi, bp


def _camera64(cam, w, h):
    dev = _device()
    eye, target, up = (torch.tensor(np.asarray(v, np.float32).astype(np.float64), device=dev)
                       for v in (cam.eye, cam.target, cam.up))
    norm = lambda v: v / torch.linalg.norm(v, dim=-1, keepdim=True)  # noqa: E731
    f = norm(target - eye)
    r = norm(torch.linalg.cross(f, up))
    u = torch.linalg.cross(r, f)
    th = math.tan(0.5 * math.radians(cam.vfov_deg))
    y, x = torch.meshgrid(torch.arange(h, device=dev, dtype=torch.float64),
                          torch.arange(w, device=dev, dtype=torch.float64), indexing="ij")
    sx, sy = (2 * (x + 0.5) / w - 1) * th * (w / h), (1 - 2 * (y + 0.5) / h) * th
    d = norm(f + sx.reshape(-1, 1) * r + sy.reshape(-1, 1) * u)
    return eye.expand_as(d).contiguous(), d


def _whitted(scene, o, d, depth):
    """The recursive shading model of a frame, per pixel, in float64."""
    dev, n = o.device, o.shape[0]
    out = torch.zeros((n, 3), dtype=torch.float64, device=dev)
    kinds = torch.tensor(np.asarray([int(m["type"]) for m in scene.materials]), device=dev)
    rgb = torch.tensor(np.asarray([m["rgb"] for m in scene.materials], np.float64), device=dev)
    ior = torch.tensor(np.asarray([m["ior"] for m in scene.materials], np.float64), device=dev)
    imat = torch.tensor(scene.inst_mat.astype(np.int64), device=dev)
    bid = torch.tensor(scene.blas_id.astype(np.int64), device=dev)
    X = torch.from_numpy(np.asarray(scene.xform, np.float64).reshape(-1, 3, 4)).to(dev)
    light = torch.tensor(np.asarray(scene.light.pos, np.float32).astype(np.float64), device=dev)
    power = torch.tensor(np.asarray(scene.light.intensity, np.float64), device=dev)
    norm = lambda v: v / torch.linalg.norm(v, dim=-1, keepdim=True)  # noqa: E731
    pix, beta = torch.arange(n, device=dev), torch.ones((n, 3), dtype=torch.float64, device=dev)
    for level in range(depth + 1):
        m = o.shape[0]
        if m == 0:
            break
        inf = torch.full((m,), math.inf, dtype=torch.float64, device=dev)
        t, _, _, inst, prim = _nearest(scene, o, d, 0.0, inf)
        sky = inst < 0
        a = 0.5 * (norm(d[sky])[:, 1:2] + 1)
        blue = torch.tensor([[0.5, 0.7, 1.0]], dtype=torch.float64, device=dev)
        out.index_add_(0, pix[sky], beta[sky] * ((1 - a) + a * blue))
        hit = ~sky
        o, d, t, inst, prim, pix, beta = o[hit], norm(d[hit]), t[hit] * torch.linalg.norm(d[hit], dim=-1), inst[hit], \
            prim[hit], pix[hit], beta[hit]
        if o.shape[0] == 0:
            break
        p = o + t[:, None] * d
        ng, mat = torch.zeros_like(p), torch.zeros_like(inst)
        for b, mesh in enumerate(scene.blas):
            at = bid[inst] == b
            tri = torch.from_numpy(mesh.verts.astype(np.float64)[mesh.idx]).to(dev)[prim[at]]
            no = torch.linalg.cross(tri[:, 1] - tri[:, 0], tri[:, 2] - tri[:, 0])
            inv = torch.linalg.inv(X[inst[at], :, :3])
            ng[at] = norm((inv.transpose(1, 2) @ no[..., None])[..., 0])
            own = imat[inst[at]]
            if mesh.prim_mat is not None:
                per = torch.from_numpy(mesh.prim_mat.astype(np.int64)).to(dev)[prim[at]]
                own = torch.where(own == sg.PER_PRIM, per, own)
            mat[at] = own
        s = torch.where((ng * d).sum(-1) < 0, 1.0, -1.0).double()
        nf = s[:, None] * ng
        eps = 1e-4 * p.abs().max(-1).values.clamp(min=1.0)[:, None]
        kind, col = kinds[mat], rgb[mat]
        dif = kind == sg.DIFFUSE
        out.index_add_(0, pix[dif], beta[dif] * col[dif] * scene.light.ambient)
        c = (nf * norm(light - p)).sum(-1)
        lit = dif & (c > 0)
        so = p[lit] + eps[lit] * nf[lit]
        if so.shape[0]:
            sd = light - so
            far = torch.full((so.shape[0],), 1 - 1e-4, dtype=torch.float64, device=dev)
            free = torch.isinf(_nearest(scene, so, sd, 0.0, far)[0])
            out.index_add_(0, pix[lit][free], (beta[lit] * col[lit] * power * c[lit][:, None])[free])
        if level == depth:
            break
        dnf = (d * nf).sum(-1, keepdim=True)
        refl = d - 2 * dnf * nf
        entering = (d * ng).sum(-1, keepdim=True) < 0
        eta = torch.where(entering, 1 / ior[mat][:, None], ior[mat][:, None])
        kappa = 1 - eta ** 2 * (1 - dnf ** 2)
        sk = kappa.clamp(min=0).sqrt()
        r0 = ((ior[mat] - 1) / (ior[mat] + 1))[:, None] ** 2
        fres = r0 + (1 - r0) * (1 - torch.where(entering, -dnf, sk)) ** 5
        glass, mirror = kind == sg.GLASS, kind == sg.MIRROR
        fres = torch.where(kappa < 0, torch.ones_like(fres), fres)
        through = glass & (kappa[:, 0] >= 0)
        o, d, pix, beta = (
            torch.cat([(p + eps * nf)[mirror | glass], (p - eps * nf)[through]]),
            torch.cat([refl[mirror | glass], (eta * d + (-eta * dnf - sk) * nf)[through]]),
            torch.cat([pix[mirror | glass], pix[through]]),
            torch.cat([(beta * torch.where(mirror[:, None], col, fres))[mirror | glass],
                       (beta * (1 - fres))[through]]))
    return out


def _blur64(img, mat, rough, radius):
    """The roughness blur in float64: two 1-D passes over taps of the centre's material."""
    h, w = mat.shape
    known = (mat >= 0) & (mat < rough.shape[0])
    r = torch.where(known, rough.double()[mat.clamp(0, rough.shape[0] - 1).long()].clamp(0, 1), 0.0)
    live = (r >= 1.0 / 256.0) & (radius > 0)
    sig = torch.where(live, r * radius / 3.0, 1.0)
    v = img.double()
    for axis in (1, 0):
        num, den = v.clone(), torch.ones((h, w, 1), dtype=torch.float64, device=v.device)
        for k in range(1, radius + 1):
            if k >= v.shape[axis]:
                break
            wt = torch.exp(-k * k / (2 * sig * sig))[..., None]
            size = v.shape[axis] - k
            for to, frm in ((0, k), (k, 0)):
                a, b = (lambda x, f=frm: x.narrow(axis, f, size)), (lambda x, g=to: x.narrow(axis, g, size))
                ok = (a(mat) == b(mat))[..., None] * b(wt)
                b(num).add_(ok * a(v))
                b(den).add_(ok)
        v = torch.where(live[..., None], num / den, v)
    return v


def exact(case, seed):
    kind = case["kind"]
    if kind == "post":
        return dict(blurred=_blur64(*_post_inputs(case, seed), case["radius"]), final=None)
    most = PAIRS_CUDA if torch.cuda.is_available() else PAIRS_CPU
    if kind in ("batch", "serve"):
        return None
    scene = _scene(case, seed)
    if kind == "ao":
        o, d = _camera64(scene.camera, case["w"], case["h"])
        n = o.shape[0]
        ends = torch.stack([torch.zeros(n), torch.full((n,), math.inf)]).double().to(o.device)
        return dict(camera=torch.cat([o.T, d.T, ends]))
    if kind == "frame":
        if case["mode"] or _pairs(case["w"] * case["h"] * 2 * (2 ** case["depth"]), scene) > most:
            return None
        o, d = _camera64(scene.camera, case["w"], case["h"])
        img = _whitted(scene, o, d, case["depth"])
        return dict(image=img.reshape(case["h"], case["w"], 3), primary=None)
    if kind == "dynamic":
        scene.blas = [sg.Mesh(sg.animate_mesh(m, 0.15, amp=0.02, seed=seed + k), m.idx)
                      for k, m in enumerate(scene.blas)]
        scene.xform = sg.animate_instances(scene.xform, 0.15, seed=seed)
        if _pairs(case["w"] * case["h"], scene) > most:
            return None
        o, d = _camera64(scene.camera, case["w"], case["h"])
        far = torch.full((o.shape[0],), math.inf, dtype=torch.float64, device=o.device)
    else:
        if case.get("options") or case.get("query", "closest") != "closest":
            return None
        out = {}
        if kind == "build":
            out["box"] = np.array([np.concatenate([m.verts[m.idx].reshape(-1, 3).min(0),
                                                   m.verts[m.idx].reshape(-1, 3).max(0)]) for m in scene.blas],
                                  np.float64)
        if _pairs(case["n"], scene) > most:
            return out or None
        r = torch.from_numpy(_random_rays(case, seed).astype(np.float64)).to(_device())
        o, d, far = r[:, :3].contiguous(), r[:, 3:6].contiguous(), r[:, 7].contiguous()
    t, u, v, _, _ = _nearest(scene, o, d, 0.0, far)
    hits = dict(t=t, u=u, v=v, inst=None, prim=None)
    return dict(hits=hits, **out) if kind == "build" else hits
