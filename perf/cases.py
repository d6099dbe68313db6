"""Performance cases of the framework, through its public entry points.

Every case is one pass of something a user's program repeats: an iteration
of fine-stage or coarse-stage training, a rendered view, a differentiable
render inside the user's own optimisation, a step of the image-fitting toy.
Sizes are those of the repository's configurations (the tiny 32^3, the full
160^3, the precision and the stress 256^3 shapes, the coarse 100^3 stage, the
progressive-scaling stages) or lie between them.

Inputs are drawn on the GPU from the seed alone.  The state is that of a run
that has been going for a while (Adam moments of a plausible size, an
activity mask derived from them), not the first iteration: nearly every
iteration a user pays for is one of those.  What an optimisation returns is
its updated state: the raw gradient of a ReLU network jumps by a sample's
whole share where rounding moves a unit across its kink, so that two equally
exact evaluations agree on the state but not on every gradient entry.

``exact`` evaluates the same pass in float64 with plain torch.  The sampler's
discrete decisions and the sample points are defined as float32 arithmetic
by the interface, so they are taken in float32 there too; everything that
follows from the points is float64.
"""

from __future__ import annotations

import math

import torch

from paper_2111_11215_amd import api, autograd, train
from paper_2111_11215_amd._lib import DVGO_BF16, DVGO_F32

DEV = "cuda"
LO, HI = (-1.0, -1.0, -1.0), (1.0, 1.0, 1.0)
BG = (1.0, 1.0, 1.0)
COARSE_N = 100
ITER = 2000            # iterations the state has behind it
LR_GRID, LR_MLP, LR_PROP, DECAY = 0.1, 1e-3, 3e-3, 20000
BETAS, EPS = (0.9, 0.999), 1e-8
W_PT, W_BG = 1e-2, 1e-3          # the fine objective's auxiliary weights
CW_PT, CW_BG = 0.1, 0.01         # the coarse objective's
TAU, FINE_TAU = 1e-4, 1e-4


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def _train(n, rays, prec, scene="spheres", pe_x=0, aux=False, prop=False, morton=False, cap=0):
    return {"kind": "train", "n": n, "rays": rays, "prec": prec, "scene": scene, "pe_x": pe_x, "aux": aux,
            "prop": prop, "morton": morton, "cap": cap}


def _image(n, H, W, prec, scene="spheres", pe_x=0, fine=False):
    return {"kind": "image", "n": n, "H": H, "W": W, "prec": prec, "scene": scene, "pe_x": pe_x, "fine": fine}


def _coarse(n, rays):
    return {"kind": "coarse", "n": n, "rays": rays}


def _autograd(n, rays, prec, scene="spheres", pe_x=0):
    return {"kind": "autograd", "n": n, "rays": rays, "prec": prec, "scene": scene, "pe_x": pe_x}


def _toy(H, W, gh, gw, mode):
    return {"kind": "toy", "H": H, "W": W, "gh": gh, "gw": gw, "mode": mode}


def listed():
    return [
        # the smallest training iteration (the smoke test's): latency and launches count
        dict(_train(32, 512, "f32", scene="uniform", cap=128), name="train_tiny_f32"),
        # the tiny configuration's whole batch, Morton-ordered, bfloat16
        dict(_train(32, 4096, "bf16", scene="uniform", morton=True, cap=128), name="train_tiny_bf16_morton"),
        # the full configuration in plain float32: the precision the paper trains in
        dict(_train(160, 8192, "f32"), name="train_full_f32"),
        # the same in the benchmark's headline form: bfloat16 with the learned proposal
        dict(_train(160, 8192, "bf16", prop=True), name="train_full_bf16_proposal"),
        # the paper's network (encoded position) and whole objective, float32
        dict(_train(160, 8192, "f32", pe_x=5, aux=True), name="train_paper_f32"),
        # the same in bfloat16 at a progressive-scaling stage, a ragged batch
        dict(_train(100, 5003, "bf16", pe_x=5, aux=True), name="train_paper_bf16_ragged"),
        # the stress shapes: every vertex steps, every in-box sample evaluated
        dict(_train(256, 32768, "bf16", scene="uniform", cap=800), name="train_stress_bf16"),
        # an iteration of the coarse stage
        dict(_coarse(COARSE_N, 8192), name="coarse_full"),
        # a held-out view at test time, the paper's image size
        dict(_image(160, 800, 800, "bf16"), name="image_800_bf16"),
        # a small float32 preview with both free-space rules, ragged
        dict(_image(160, 151, 203, "f32", fine=True), name="image_small_f32_fine"),
        # the differentiable render under a user's own loss, with the
        # framework's dense Adam steps
        dict(_autograd(128, 4096, "f32"), name="autograd_f32"),
        # the image-fitting toy: a handful of small launches
        dict(_toy(256, 256, 128, 128, 2), name="toy_256_post"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges, no dearer than the stress case."""
    kind = rng.choice(["train"] * 5 + ["image"] * 2 + ["coarse", "autograd", "toy"])
    if kind == "toy":
        H, W = rng.randint(64, 512), rng.randint(64, 512)
        stride = rng.uniform(2.0, 16.0)
        return _toy(H, W, max(2, int(H / stride)), max(2, int(W / stride)), rng.randint(0, 2))
    if kind == "coarse":
        return _coarse(rng.randint(40, 128), _log_int(rng, 256, 12288))
    prec = rng.choice(["f32", "bf16"])
    pe_x = rng.choice([0, 0, 5])
    scene = rng.choice(["spheres", "spheres", "uniform"])
    n = _log_int(rng, 24, 192)
    if kind == "image":
        fine = bool(rng.randint(0, 1)) and scene == "spheres"
        top = 640 if scene == "spheres" else 160
        return _image(n, rng.randint(32, top), rng.randint(32, top), prec, scene, pe_x, fine)
    most = 16384 if scene == "spheres" else (8192 if prec == "bf16" else 4096)
    if kind == "autograd":
        return _autograd(n, _log_int(rng, 64, most // 2), prec, scene, pe_x)
    return _train(n, _log_int(rng, 64, most), prec, scene, pe_x, aux=bool(rng.randint(0, 1)),
                  prop=prec == "bf16" and bool(rng.randint(0, 1)), morton=rng.random() < 0.2)


# ---------------------------------------------------------------------------
# inputs, from the seed alone
# ---------------------------------------------------------------------------
def _gen(seed, part):
    return torch.Generator(device=DEV).manual_seed(1000003 * int(seed) + part)


def _rand(g, *shape, lo=0.0, hi=1.0):
    return torch.rand(*shape, generator=g, device=DEV) * (hi - lo) + lo


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device=DEV)


def _spheres(seed):
    """64 soft spheres: centres, radii, peak densities, colours, edge 0.01."""
    g = _gen(seed, 1)
    return (_rand(g, 64, 3, lo=-0.7, hi=0.7), _rand(g, 64, lo=0.1, hi=0.25), 50.0 * (1.0 - _rand(g, 64)),
            _rand(g, 64, 3), 0.01)


def _scene(sp, x):
    """Density and density-weighted colour of the sphere scene at points x."""
    c, r, rho, rgb, edge = sp
    sig = torch.zeros(x.shape[:-1], device=x.device)
    col = torch.zeros_like(x)
    for k in range(c.shape[0]):
        s = rho[k] * torch.sigmoid((r[k] - torch.linalg.vector_norm(x - c[k], dim=-1)) / edge)
        sig += s
        col += s[..., None] * rgb[k]
    return sig, col / sig.clamp_min(1e-12)[..., None]


def _vertices(n):
    ax = torch.linspace(-1.0, 1.0, n, device=DEV)
    return torch.stack(torch.meshgrid(ax, ax, ax, indexing="ij"), dim=-1)


def _cameras(seed, n, radius=4.0):
    """Centres uniform on the upper hemisphere and their camera-to-world
    rotations (columns right, up, back), looking at the origin; float64."""
    g = _gen(seed, 2)
    z = torch.rand(n, generator=g, device=DEV, dtype=torch.float64) * 0.98
    phi = torch.rand(n, generator=g, device=DEV, dtype=torch.float64) * (2.0 * math.pi)
    rxy = torch.sqrt(1.0 - z * z)
    c = radius * torch.stack([rxy * torch.cos(phi), rxy * torch.sin(phi), z], dim=-1)
    fwd = -c / torch.linalg.vector_norm(c, dim=-1, keepdim=True)
    up = torch.tensor([0.0, 0.0, 1.0], dtype=torch.float64, device=DEV).expand_as(fwd)
    right = torch.linalg.cross(fwd, up)
    right = right / torch.linalg.vector_norm(right, dim=-1, keepdim=True)
    return c, torch.stack([right, torch.linalg.cross(right, fwd), -fwd], dim=-1)


def _pixel_rays(c, R, H, W, focal, pi, pj):
    dc = torch.stack([(pj + 0.5 - 0.5 * W) / focal, -(pi + 0.5 - 0.5 * H) / focal, -torch.ones_like(pi)], dim=-1)
    d = (R @ dc[..., None])[..., 0]
    d = d / torch.linalg.vector_norm(d, dim=-1, keepdim=True)
    return c.expand_as(d).float().contiguous(), d.float().contiguous()


def _batch(seed, B, tiny):
    """B rays through random pixels of the training cameras, with jitter."""
    H, focal, ncam = (64, 80.0, 8) if tiny else (800, 1000.0, 100)
    c, R = _cameras(seed, ncam)
    flat = torch.randint(0, ncam * H * H, (B,), generator=_gen(seed, 3), device=DEV)
    cam, rem = flat // (H * H), flat % (H * H)
    o, d = _pixel_rays(c[cam], R[cam], H, H, focal, (rem // H).double(), (rem % H).double())
    return o, d, _rand(_gen(seed, 4), B)


def _targets(seed, o, d, sp):
    """The colours to fit: the sphere scene composited at 128 points per ray,
    or uniform colours for the random grids."""
    if sp is None:
        return _rand(_gen(seed, 5), o.shape[0], 3)
    out = []
    for a in range(0, o.shape[0], 4096):
        oo, dd = o[a:a + 4096], d[a:a + 4096]
        t = 2.2 + (torch.arange(128, device=DEV) + 0.5) * (3.6 / 128)
        sig, col = _scene(sp, oo[:, None] + t[None, :, None] * dd[:, None])
        tau = torch.cumsum(sig * (3.6 / 128), dim=1)
        T = torch.exp(-torch.cat([torch.zeros_like(tau[:, :1]), tau], dim=1))
        w = T[:, :-1] - T[:, 1:]
        out.append((w[..., None] * col).sum(1) + T[:, -1:])
    return torch.cat(out).contiguous()


def _xavier(g, dims):
    parts = []
    for fi, fo in zip(dims[:-1], dims[1:]):
        a = math.sqrt(6.0 / (fi + fo))
        parts += [_rand(g, fo, fi, lo=-a, hi=a).reshape(-1), 0.1 * _randn(g, fo)]
    return torch.cat(parts).contiguous()


def _step_of(case):
    """Half a voxel, and the cap that covers the box diagonal."""
    step = 0.5 * 2.0 / (case["n"] - 1)
    return step, case.get("cap") or int(math.ceil(2.0 * math.sqrt(3.0) / step)) + 1


def _shift(case):
    """Softplus shift of the low-density initialisation (alpha 1e-2; the
    coarse stage's 1e-6)."""
    alpha = 1e-6 if case["kind"] == "coarse" else 1e-2
    return math.log(math.expm1(-math.log1p(-alpha) / (2.0 / (case["n"] - 1))))


def _moments(g, shape, size, where=None):
    """Adam moments of a run in progress, around gradients of ``size``."""
    m, v = 0.3 * size * _randn(g, *shape), (size * _rand(g, *shape, lo=0.5, hi=1.5)) ** 2
    if where is not None:
        k = where.reshape(where.shape + (1,) * (len(shape) - where.dim()))
        m, v = m * k, v * k
    return m.contiguous(), v.contiguous()


def _raw_of(sig, shift):
    s = sig.clamp_min(1e-12).double()
    return (s + torch.log(-torch.expm1(-s)) - shift).float()


def _inputs(case, seed):
    """Grids, network and (spheres) the coarse grid of a fine-stage case,
    with the Adam moments of the training cases."""
    n, g = case["n"], _gen(seed, 6)
    I = {"shift": _shift(case), "coarse_raw": None}
    I["step"], I["max_samples"] = _step_of(case)
    active = None
    if case["scene"] == "uniform":
        I["sp"] = None
        I["density"] = _rand(g, n, n, n, lo=-1.0, hi=1.0)
        I["feat"] = _rand(g, n, n, n, 12, lo=-1.0, hi=1.0)
    else:
        sp = I["sp"] = _spheres(seed)
        I["coarse_raw"] = _raw_of(_scene(sp, _vertices(COARSE_N))[0], 0.0)
        # vertices that samples reach: those in or beside a kept cell
        keep = _keep_cells(I["coarse_raw"], _raw_threshold(TAU, I["step"], 0.0))
        wide = torch.nn.functional.max_pool3d(keep[None, None].float(), 3, 1, 1)[0, 0] > 0
        i = ((_vertices(n) + 1.0) * ((COARSE_N - 1) / 2.0)).floor().long().clamp(0, COARSE_N - 2)
        active = wide[i[..., 0], i[..., 1], i[..., 2]]
        raw = _raw_of(_scene(sp, _vertices(n))[0], I["shift"]).clamp(-4.0, 60.0) + 0.3 * _randn(g, n, n, n)
        I["density"] = torch.where(active, raw, torch.zeros_like(raw)).contiguous()
        I["feat"] = (0.7 * _randn(g, n, n, n, 12) * active[..., None]).contiguous()
    I["mlp"] = _xavier(g, (72 if case["pe_x"] else 39, 128, 128, 3))
    if case["kind"] != "image":
        # sized by the gradients of the first iterations (dL/dc is about
        # 2e-5 there), which the second moment remembers longest
        I["m_density"], I["v_density"] = _moments(g, (n, n, n), 2e-5, active)
        I["m_feat"], I["v_feat"] = _moments(g, (n, n, n, 12), 2e-5, active)
        I["m_mlp"], I["v_mlp"] = _moments(g, (I["mlp"].numel(),), 1e-3)
        if case.get("prop"):
            flat = _xavier(g, (54, 64, 64, 32))
            flat[-32 * 64 - 32:-32] *= 3.0
            flat[-32:] += 0.5
            I["prop"] = flat
            I["m_prop"], I["v_prop"] = _moments(g, (flat.numel(),), 1e-3)
    return I


def _model(case, I):
    bf16 = case["prec"] == "bf16"
    aux = bool(case.get("aux"))
    cfg = train.FineConfig(step=I["step"], max_samples=I["max_samples"], bg=BG, lr_grid=LR_GRID, lr_mlp=LR_MLP,
                           decay_steps=DECAY, betas=BETAS, eps=EPS, precision=DVGO_BF16 if bf16 else DVGO_F32,
                           bf16_feat=bf16, morton=bool(case.get("morton")), w_pt_rgb=W_PT if aux else 0.0,
                           w_bg_entropy=W_BG if aux else 0.0)
    coarse = None
    if I["coarse_raw"] is not None:
        thr = api.coarse_raw_threshold(TAU, I["step"])
        coarse = (api.coarse_mask_build(I["coarse_raw"], LO, HI, thr), LO, HI, (COARSE_N,) * 3)
    return train.FineModel(I["density"], I["feat"], I["mlp"], LO, HI, I["shift"], cfg, coarse=coarse)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "toy":
        V, target, m, v = _toy_inputs(case, seed)
        st = train.AdamState.of(V)
        st.m.copy_(m)
        st.v.copy_(v)
        return {"case": case, "st": st, "target": target, "t": ITER}
    if kind == "coarse":
        C = _coarse_inputs(case, seed)
        model = train.CoarseModel(case["n"], LO, HI, C["cams"], 800, 800, 1000.0, lr=LR_GRID, w_pt=CW_PT,
                                  w_bg=CW_BG, decay_steps=DECAY, bg=BG)
        for st, k in ((model.st_density, "density"), (model.st_rgb, "rgb")):
            st.p.copy_(C[k])
            st.m.copy_(C["m_" + k])
            st.v.copy_(C["v_" + k])
        model.t = ITER
        return {"case": case, "model": model, "o": C["o"], "d": C["d"], "j": C["j"], "target": C["target"]}
    I = _inputs(case, seed)
    S = {"case": case, "model": _model(case, I)}
    if kind == "image":
        c, R = _cameras(seed, 1)
        S["c2w"] = R[0].float().tolist()
        S["origin"] = c[0].float().tolist()
        S["fine"] = (I["density"], api.coarse_raw_threshold(FINE_TAU, I["step"], I["shift"])) if case["fine"] else None
        return S
    S["o"], S["d"], S["j"] = _batch(seed, case["rays"], case["scene"] == "uniform" and case["n"] <= 64)
    S["target"] = _targets(seed, S["o"], S["d"], I["sp"])
    model = S["model"]
    for st, k in ((model.st_density, "density"), (model.st_feat, "feat"), (model.st_mlp, "mlp")):
        st.m.copy_(I["m_" + k])
        st.v.copy_(I["v_" + k])
    model.t = model.t_grid = ITER
    if kind == "autograd":
        for k in ("density", "feat", "mlp"):
            I[k].requires_grad_(True)
        return S
    d, f = model.st_density, model.st_feat
    api.grid_active_init(d.m, d.v, f.m, f.v, model.active)
    if case["prop"]:
        prop = train.ProposalModel(I["prop"], LO, HI, lr=LR_PROP)
        prop.st.m.copy_(I["m_prop"])
        prop.st.v.copy_(I["v_prop"])
        prop.t = ITER
        S["prop"] = prop
    return S


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def _state_out(prefix, st):
    return {prefix: st.p, prefix + "_m": st.m, prefix + "_v": st.v}


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "toy":
        st = state["st"]
        state["t"] += 1
        loss, _ = api.toy2d_loss_grad(st.p, state["target"], case["mode"], 1.0, grad=st.g)
        api.adam_step(st.p, st.g, st.m, st.v, 0.1, state["t"])
        return dict(_state_out("V", st), loss=loss)
    if kind == "coarse":
        m = state["model"]
        res = m.train_step(state["o"], state["d"], state["target"], state["j"])
        return dict(_state_out("density", m.st_density), **_state_out("rgb", m.st_rgb), loss=res["loss"],
                    n_kept=res["samples"].n_kept)
    model = state["model"]
    c = model.cfg
    if kind == "image":
        return api.render_image(model.grid, model.mlp, state["c2w"], state["origin"], case["H"], case["W"],
                                1.25 * case["W"], c.step, c.max_samples, coarse=model.coarse, bg=c.bg,
                                precision=c.precision, use_shadow=c.bf16_feat, fine=state["fine"])
    if kind == "autograd":
        states = (model.st_density, model.st_feat, model.st_mlp)
        params = [st.p for st in states]
        s = model.sample(state["o"], state["d"], state["j"])
        rgb, depth, acc = autograd.render(*params, s, LO, HI, model.grid.act_shift, c.bg, c.precision,
                                          model.grid.feat_shadow)
        loss = (rgb - state["target"]).square().sum(1).mean() + 1e-3 * depth.mean() + 1e-2 * acc.mean()
        grads = torch.autograd.grad(loss, params)
        model.t += 1
        for st, grad, lr in zip(states, grads, (c.lr_grid, c.lr_grid, c.lr_mlp)):
            api.adam_step(st.p, grad, st.m, st.v, model.lr(lr), model.t, c.betas, c.eps, shadow=st.shadow)
        return dict(_state_out("density", model.st_density), **_state_out("feat", model.st_feat),
                    **_state_out("mlp", model.st_mlp), rgb=rgb, depth=depth, acc=acc, loss=loss, n_kept=s.n_kept)
    if case["prop"]:
        res = train.proposal_train_step(model, state["prop"], state["o"], state["d"], state["target"], state["j"])
    else:
        res = model.train_step(state["o"], state["d"], state["target"], state["j"])
    s = res["samples"]
    out = dict(_state_out("density", model.st_density), **_state_out("feat", model.st_feat),
               **_state_out("mlp", model.st_mlp), loss=res["loss"], rgb=res["rgb"], n_kept=s.n_kept,
               ray_offset=s.ray_offset)
    if model.st_feat.shadow is not None:
        out["feat_bf16"] = model.st_feat.shadow.view(torch.bfloat16)
    if case["prop"]:
        out.update(_state_out("prop", state["prop"].st), mask=res["mask"])
    return out


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def work(case):
    kind = case["kind"]
    if kind == "toy":
        # image read, grid p, m, v read and written; per pixel the bilinear
        # interpolation, activation and its transpose
        pix, nv = case["H"] * case["W"], case["gh"] * case["gw"]
        return {"bytes": 4.0 * pix + 24.0 * nv, "flops": 60.0 * pix + 15.0 * nv}
    n = case["n"]
    nv = float(n) ** 3
    if kind == "coarse":
        samples = case["rays"] * 0.86 * n
        return {"bytes": 4 * 24.0 * nv + 4.0 * nv + 40.0 * case["rays"], "flops": 300.0 * samples + 60.0 * nv}
    # evaluated samples: about 0.33 n per ray inside the coarse mask, 0.86 n
    # without one (means over the configurations' rays)
    dense = case["scene"] == "uniform"
    rays = case["H"] * case["W"] if kind == "image" else case["rays"]
    samples = rays * (0.86 if dense else 0.33 if kind != "image" or not case["fine"] else 0.2) * n
    n_in = 72 if case["pe_x"] else 39
    fwd = 2.0 * ((n_in - 27) * 128 + 128 * 128 + 3 * 128)
    fbytes = 24.0 if case["prec"] == "bf16" else 48.0
    share = 1.0 if dense else 0.4      # vertices that samples can reach
    touched = min(nv * share, 4.0 * samples)
    flops = samples * fwd
    if kind == "image":
        return {"bytes": touched * (4.0 + fbytes) + 20.0 * rays, "flops": flops}
    flops += samples * (fwd + 2.0 * ((n_in + 1) * 128 + 128 * 128 + 3 * 128))
    if kind == "autograd":
        share = 1.0      # the dense Adam steps every vertex
    step = nv * share * (13 * 24.0 + (24.0 if case["prec"] == "bf16" else 0.0))
    return {"bytes": step + 40.0 * rays, "flops": flops}


# ---------------------------------------------------------------------------
# the same pass in float64
# ---------------------------------------------------------------------------
F64 = torch.float64


def _raw_threshold(tau, step, shift):
    y = -math.log1p(-tau) / step
    thr = y + math.log(-math.expm1(-y)) - shift
    t = torch.tensor(thr, dtype=torch.float32)
    if t.double().item() > thr:
        t = torch.nextafter(t, torch.tensor(-math.inf))
    return t.item()


def _keep_cells(raw, thr):
    return torch.nn.functional.max_pool3d(raw[None, None], 2, 1)[0, 0] >= thr


def _cell_f32(x, n):
    """Cell index of float32 points in the float32 recipe."""
    scale = torch.tensor(float(n - 1), dtype=torch.float32) / torch.tensor(2.0)
    return ((x - (-1.0)) * scale.item()).floor().clamp(0.0, float(n - 2)).long()


def _sample(o, d, j, step, max_samples, keep=None, fine=None):
    """Kept samples of rays o + t d: (mask [R, K], points [R, K, 3], t [R, K]),
    by the sampler's float32 recipe."""
    inv = 1.0 / d
    t0, t1 = (-1.0 - o) * inv, (1.0 - o) * inv
    tn = torch.minimum(t0, t1).amax(1).clamp_min(0.0)
    tx = torch.maximum(t0, t1).amin(1)
    k = torch.arange(max_samples, device=DEV, dtype=torch.float32)
    kp = k[None] + j[:, None] if j is not None else k[None].expand(o.shape[0], -1)
    t = tn[:, None] + kp * step
    mask = (t < tx[:, None]) & (tn < tx)[:, None]
    x = o[:, None] + t[..., None] * d[:, None]
    if keep is not None:
        i = _cell_f32(x, COARSE_N)
        mask &= keep[i[..., 0], i[..., 1], i[..., 2]]
    if fine is not None:
        mask &= _trilerp(fine[0][..., None].double(), x)[..., 0] >= fine[1]
    return mask, x, t


def _trilerp(grid, x):
    """Trilinear interpolation of grid [n,n,n,C] at points x (any shape)."""
    n, C = grid.shape[0], grid.shape[3]
    flat = grid.reshape(-1, C)
    u = (x.double() + 1.0) * ((n - 1) / 2.0)
    i = u.floor().clamp(0.0, n - 2.0)
    f = (u - i).clamp(0.0, 1.0)
    i = i.long()
    base = (i[..., 0] * n + i[..., 1]) * n + i[..., 2]
    out = 0.0
    for c in range(8):
        b = ((c >> 2) & 1, (c >> 1) & 1, c & 1)
        w = 1.0
        for a in range(3):
            w = w * (f[..., a] if b[a] else 1.0 - f[..., a])
        at = base + (b[0] * n + b[1]) * n + b[2]
        out = out + w[..., None] * flat.index_select(0, at.reshape(-1)).reshape(at.shape + (C,))
    return out


def _pe(x, k):
    out = [x]
    for q in range(k):
        out += [torch.sin(x * 2.0 ** q), torch.cos(x * 2.0 ** q)]
    return torch.cat(out, dim=-1)


def _net(flat, z):
    n_in = z.shape[1]
    o, h = 0, z
    for fo, fi in ((128, n_in), (128, 128), (3, 128)):
        w, b = flat[o:o + fo * fi].reshape(fo, fi), flat[o + fo * fi:o + fo * fi + fo]
        o += fo * fi + fo
        h = torch.addmm(b, h, w.t())
        h = torch.relu(h) if fo == 128 else torch.sigmoid(h)
    return h


def _composite(raw, col, mask, t, step, shift):
    """rgb (without background), depth, acc, T_end, weights of padded rays."""
    sd = torch.nn.functional.softplus(raw + shift, threshold=500.0) * step * mask
    tau = torch.cumsum(sd, dim=1)
    excl = torch.cat([torch.zeros_like(tau[:, :1]), tau[:, :-1]], dim=1)
    w = torch.exp(-excl) * -torch.expm1(-sd)
    rgb = (w[..., None] * col).sum(1)
    return rgb, (w * t).sum(1), w.sum(1), torch.exp(-tau[:, -1]), w


def _padded(mask, values):
    out = torch.zeros(mask.shape + values.shape[1:], dtype=F64, device=DEV)
    return out.masked_scatter(mask.reshape(mask.shape + (1,) * (values.dim() - 1)).expand_as(out), values)


def _entropy(T):
    p = T.clamp(1e-6, 1.0 - 1e-6)
    return -p * torch.log(p) - (1.0 - p) * torch.log1p(-p)


def _render(P, case, I, o, d, j, keep, fine=None):
    """rgb, depth, acc, T_end, and the per-sample terms of rays, float64."""
    mask, x, t = _sample(o, d, j, I["step"], I["max_samples"], keep, fine)
    x, t = x[mask], t.double()
    raw = _trilerp(P["density"][..., None], x)[..., 0]
    z = [_trilerp(P["feat"], x)]
    if case["pe_x"]:
        z.append(_pe(x.double(), 5))
    ray = mask.nonzero()[:, 0]
    z.append(_pe(d.double(), 4)[ray])
    col = _padded(mask, _net(P["mlp"], torch.cat(z, dim=1)))
    rgb, depth, acc, T, w = _composite(_padded(mask, raw), col, mask, t, I["step"], I["shift"])
    return rgb + T[:, None] * torch.tensor(BG, dtype=F64, device=DEV), depth, acc, T, w, col, mask


def _ray_chunk(case, max_samples):
    return max(64, min(8192, int(1.2e6 / (0.9 * max_samples)) * (1 if case["scene"] == "uniform" else 3)))


def _adam(p, m, v, g, lr, t, beta=BETAS):
    m = beta[0] * m.double() + (1.0 - beta[0]) * g
    v = beta[1] * v.double() + (1.0 - beta[1]) * g * g
    p = p.double() - lr * (m / (1.0 - beta[0] ** t)) / (torch.sqrt(v / (1.0 - beta[1] ** t)) + EPS)
    return p, m, v


def exact(case, seed):
    kind = case["kind"]
    if kind == "toy":
        return _toy_exact(case, seed)
    if kind == "coarse":
        return _coarse_exact(case, seed)
    if case.get("prop"):
        return None      # the masks are decisions of the bfloat16 proposal network
    I = _inputs(case, seed)
    bf16 = case["prec"] == "bf16"
    keep = None
    if I["coarse_raw"] is not None:
        keep = _keep_cells(I["coarse_raw"], _raw_threshold(TAU, I["step"], 0.0))
    names = ("density", "feat", "mlp")
    P = {k: I[k].double() for k in names}
    if bf16:      # the gathers read the bfloat16 copy of the features
        P["feat"] = I["feat"].bfloat16().double()
    chunk = _ray_chunk(case, I["max_samples"])
    if kind == "image":
        fine = (I["density"], _raw_threshold(FINE_TAU, I["step"], I["shift"])) if case["fine"] else None
        c, R = _cameras(seed, 1)
        H, W = case["H"], case["W"]
        pix = torch.arange(H * W, device=DEV)
        o, d = _pixel_rays(c, R.float().double(), H, W, 1.25 * W, (pix // W).double(), (pix % W).double())
        got = []
        with torch.no_grad():
            for a in range(0, H * W, chunk):
                got.append(_render(P, case, I, o[a:a + chunk], d[a:a + chunk], None, keep, fine)[:3])
        return {k: torch.cat([x[i] for x in got]) for i, k in enumerate(("rgb", "depth", "acc"))}
    B = case["rays"]
    o, d, j = _batch(seed, B, case["scene"] == "uniform" and case["n"] <= 64)
    target = _targets(seed, o, d, I["sp"]).double()
    for k in names:
        P[k].requires_grad_(True)
    got, loss = [], 0.0
    for a in range(0, B, chunk):
        e = slice(a, min(a + chunk, B))
        rgb, depth, acc, T, w, col, mask = _render(P, case, I, o[e], d[e], j[e], keep)
        L = (rgb - target[e]).square().sum() / B
        if kind == "autograd":
            L = L + 1e-3 * depth.sum() / B + 1e-2 * acc.sum() / B
        elif case["aux"]:
            L = L + W_PT * (w.detach() * (col - target[e, None]).square().sum(-1) * mask).sum() / B
            L = L + W_BG * _entropy(T).sum() / B
        L.backward()
        got.append((rgb.detach(), depth.detach(), acc.detach()))
        loss += L.detach()
    rgb, depth, acc = (torch.cat(x) for x in zip(*got))
    grads = {k: P[k].grad for k in names}
    out = {"rgb": rgb, "loss": loss, "n_kept": None}
    if kind == "autograd":
        out.update(depth=depth, acc=acc)
    else:
        out.update(loss=loss.reshape(1), ray_offset=None)
    t = ITER + 1
    decay = 0.1 ** (t / DECAY)
    for k in names:
        lr = (LR_MLP if k == "mlp" else LR_GRID) * decay
        out[k], out[k + "_m"], out[k + "_v"] = _adam(I[k], I["m_" + k], I["v_" + k], grads[k], lr, t)
    if bf16 and kind == "train":
        out["feat_bf16"] = out["feat"]
    return out


# ---------------------------------------------------------------------------
# coarse stage and toy: inputs and float64 passes
# ---------------------------------------------------------------------------
def _coarse_inputs(case, seed):
    n, g, sp = case["n"], _gen(seed, 7), _spheres(seed)
    c, R = _cameras(seed, 100)
    C = {"cams": torch.cat([R.reshape(-1, 9), c], dim=1).float().contiguous()}
    C["o"], C["d"], C["j"] = _batch(seed, case["rays"], False)
    C["target"] = _targets(seed, C["o"], C["d"], sp)
    sig, col = _scene(sp, _vertices(n))
    C["density"] = _raw_of(sig, _shift(case)).clamp(-2.0, 40.0) + 0.3 * _randn(g, n, n, n)
    C["rgb"] = torch.logit(col.clamp(0.05, 0.95)) + 0.3 * _randn(g, n, n, n, 3)
    C["m_density"], C["v_density"] = _moments(g, (n, n, n), 1e-5)
    C["m_rgb"], C["v_rgb"] = _moments(g, (n, n, n, 3), 1e-5)
    return C


def _view_scale(n, cams):
    """n_j / n_max: the share of cameras that see each vertex."""
    x = _vertices(n).reshape(-1, 3).double()
    cnt = torch.zeros(x.shape[0], dtype=F64, device=DEV)
    for cam in cams.double():
        p = (x - cam[9:]) @ cam[:9].reshape(3, 3)
        z = -p[:, 2]
        u, v = 1000.0 * p[:, 0] / z + 400.0, -1000.0 * p[:, 1] / z + 400.0
        cnt += ((z > 0) & (u >= 0) & (u < 800) & (v >= 0) & (v < 800)).double()
    return (cnt / cnt.max()).reshape(n, n, n)


def _coarse_exact(case, seed):
    n, B, C = case["n"], case["rays"], _coarse_inputs(case, seed)
    shift = _shift(case)
    step = 0.5 * 2.0 / (n - 1)
    max_samples = int(math.ceil(math.sqrt(3.0) * 2.0 / step)) + 1
    dens = C["density"].double().requires_grad_(True)
    rgbg = C["rgb"].double().requires_grad_(True)
    target, loss = C["target"].double(), 0.0
    for a in range(0, B, 2048):
        e = slice(a, min(a + 2048, B))
        mask, x, t = _sample(C["o"][e], C["d"][e], C["j"][e], step, max_samples)
        x = x[mask]
        raw = _padded(mask, _trilerp(dens[..., None], x)[..., 0])
        col = _padded(mask, torch.sigmoid(_trilerp(rgbg, x)))
        rgb, _, _, T, w = _composite(raw, col, mask, t.double(), step, shift)
        rgb = rgb + T[:, None] * torch.tensor(BG, dtype=F64, device=DEV)
        L = (rgb - target[e]).square().sum() / B + CW_BG * _entropy(T).sum() / B
        L = L + CW_PT * (w.detach() * (col - target[e, None]).square().sum(-1) * mask).sum() / B
        L.backward()
        loss += L.detach()
    t = ITER + 1
    lr = LR_GRID * 0.1 ** (t / DECAY)
    out = {"loss": loss.reshape(1), "n_kept": None}
    scale = _view_scale(n, C["cams"])
    for k, g, s in (("density", dens.grad, scale), ("rgb", rgbg.grad, 1.0)):
        out[k], out[k + "_m"], out[k + "_v"] = _adam(C[k], C["m_" + k], C["v_" + k], g, lr * s, t)
    return out


def _toy_inputs(case, seed):
    """A grid half-way through its fit, the binary image of 12 discs and the
    moments of the fit."""
    H, W, g = case["H"], case["W"], _gen(seed, 8)
    y = (torch.arange(H, device=DEV) + 0.5)[:, None] / H
    x = (torch.arange(W, device=DEV) + 0.5)[None, :] / W
    p = _rand(g, 12, 3)
    img = torch.zeros(H, W, device=DEV)
    for k in range(12):
        r = 0.03 + 0.12 * p[k, 2]
        img = torch.maximum(img, ((y - p[k, 0]) ** 2 + (x - p[k, 1]) ** 2 < r * r).float())
    V = (3.0 * _randn(g, case["gh"], case["gw"])).contiguous()
    m, v = _moments(g, (case["gh"], case["gw"]), 1e-4)
    return V, img.contiguous(), m, v


def _toy_exact(case, seed):
    V0, target, m, v = _toy_inputs(case, seed)
    V = V0.double().requires_grad_(True)
    H, W, gh, gw, mode = case["H"], case["W"], case["gh"], case["gw"], case["mode"]
    u = ((torch.arange(H, device=DEV, dtype=F64) + 0.5) * ((gh - 1) / H))[:, None]
    w = ((torch.arange(W, device=DEV, dtype=F64) + 0.5) * ((gw - 1) / W))[None, :]
    i, k = u.floor().clamp(0, gh - 2), w.floor().clamp(0, gw - 2)
    fu, fv = (u - i).clamp(0, 1), (w - k).clamp(0, 1)
    base = i.long() * gw + k.long()
    softplus = lambda z: torch.nn.functional.softplus(z, threshold=500.0)  # noqa: E731
    alpha = lambda s: -torch.expm1(-s)  # noqa: E731

    def interp(z):
        z = z.reshape(-1)
        return ((1 - fu) * (1 - fv) * z[base] + (1 - fu) * fv * z[base + 1] + fu * (1 - fv) * z[base + gw]
                + fu * fv * z[base + gw + 1])

    a = interp(alpha(softplus(V))) if mode == 0 else alpha(interp(softplus(V))) if mode == 1 \
        else alpha(softplus(interp(V)))
    loss = (a - target.double()).square().mean()
    loss.backward()
    p, mm, vv = _adam(V0, m, v, V.grad, 0.1, ITER + 1)
    return {"V": p, "V_m": mm, "V_v": vv, "loss": loss.detach().reshape(1)}
