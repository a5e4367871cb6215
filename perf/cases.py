"""Performance cases of the selective-refinement framework.

Each case is work that a program built on this package does through its public
entry points (``paper_2511_18672_amd.binding`` and ``Refiner``), at the sizes of
the repository's own workloads or at generic ones:

  loop       ``Refiner.run``: the whole partial-denoising loop of a small request
  step       one refinement step of packed requests: select and compact, gather
             with injection, denoiser and DDIM update, scatter out of place
  cached     a partial step with the latent cache: the selected queries attend
             to every token of the request through cached keys and values
  attention  the varlen attention entry point on ragged segments
  latents    selection, gather and scatter alone, on long sequences
  frontend   the mask front-end over regression output frames

``exact`` restates every floating path in plain float64 torch from the method's
definitions (linear betas over 1000 steps, deterministic DDIM, adaLN
transformer); it shares no code with the package.
"""
import math

import numpy as np
import torch

from paper_2511_18672_amd import binding as B
from paper_2511_18672_amd.refiner import Refiner

DEV = "cuda"

TINY = dict(D=64, heads=4, head_dim=16, mlp=256)
SMALL = dict(D=512, heads=8, head_dim=64, mlp=2048)
WIDE = dict(D=1024, heads=16, head_dim=64, mlp=4096)
XL = dict(D=1152, heads=16, head_dim=72, mlp=4608)


def listed():
    step = dict(kind="step", dtype="bf16", attention="joint", full=0, t_lo=0.5, t_hi=0.5, steps=25, at=0)
    return [
        # the smallest request there is: 2 frames of 8x8 latents, 5 or so of 32 tokens, one step of an fp32
        # denoiser; its time is launches and host calls
        dict(kind="loop", name="tiny_loop_f32", **TINY, L=1, dtype="f32", reqs="2x8x8", rho="0.16", t=0.5, steps=1),
        # a small preview request: 8 frames of 32x32 latents, half of 2048 tokens, ten steps of a 4-block denoiser
        dict(kind="loop", name="small_loop", **SMALL, L=4, dtype="bf16", reqs="8x32x32", rho="0.5", t=0.6, steps=10),
        # the same request through an fp32 model (the precision option for checking or delicate content)
        dict(step, name="small_step_f32", **dict(SMALL, dtype="f32"), L=4, reqs="8x32x32", rho="0.5"),
        # the main workload: 14 views of 576x1024 (72x128 latents), 30 % of 32256 tokens, all 12 blocks
        dict(step, name="headline_step", **WIDE, L=12, reqs="14x72x128", rho="0.3"),
        # the same views when the regression was nearly good enough: 5 % selected, two blocks
        dict(step, name="light_step", **WIDE, L=2, reqs="14x72x128", rho="0.05"),
        # 21 views, 8 frames refined whole and 15 % of the others, per-frame start times, the wide 72-dim-head model,
        # at the step from which every frame is active
        dict(step, name="frame_region_step", **XL, L=2, reqs="21x64x64", rho="0.15", full=8, t_lo=0.3, t_hi=0.7, at=14),
        # a server's batch of four requests of different sizes and selected fractions in one call, up to whole frames
        dict(step, name="batched_step", **WIDE, L=1, reqs="6x32x32+14x72x128+21x64x64+8x64x64",
             rho="0.1+0.3+0.6+1.0"),
        # the same views with the latent cache between two full steps: 9677 queries against 32256 keys
        dict(step, name="cached_step", **WIDE, L=1, reqs="14x72x128", rho="0.3", at=2) | {"kind": "cached"},
        # a denoiser whose blocks alternate attention within a frame and across frames
        dict(step, name="factorised_step", **dict(WIDE, attention="factorised"), L=2, reqs="14x72x128", rho="0.3"),
        # attention alone over many requests of very different lengths, as a batch of small selections gives
        dict(kind="attention", name="attention_ragged", heads=16, head_dim=64, dtype="bf16",
             q="1+17+96+129+333+640+1021+1500+2049+3100", kv="64+17+96+129+1333+640+1021+4500+2049+3100"),
        # selection, gather with noise and scatter of one long sequence: 128 frames of 512x512 latents, 2^23 tokens
        dict(kind="latents", name="latents_large", reqs="128x512x512", rho="0.3", layout="tokens", dtype="f32",
             noise=True),
        # the mask of 14 rendered views of 576x1024 from their sharpness and opacity
        dict(kind="frontend", name="frontend_views", reqs="14x72x128"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_reqs(rng, tokens, count, frames=24):
    """`count` requests of together about `tokens` tokens; even latent sides of any residue."""
    out = []
    for _ in range(count):
        t = max(4, tokens // count)
        f = max(1, min(frames, _log_int(rng, 1, 24), t // 4))
        hp = max(1, int(round(math.sqrt(t / f) * rng.uniform(0.7, 1.3))))
        wp = max(1, t // (f * hp))
        out.append("%dx%dx%d" % (f, 2 * min(hp, 512), 2 * min(wp, 512)))
    return "+".join(out)


def draw(rng):
    kind = rng.choice(["loop", "step", "step", "step", "step", "cached", "attention", "latents", "frontend"])
    if kind == "loop":
        f32 = rng.random() < 0.5
        model = rng.choice([TINY, dict(D=128, heads=4, head_dim=32, mlp=512)] if f32 else
                           [dict(D=128, heads=2, head_dim=64, mlp=512), SMALL])
        return dict(kind="loop", **model, L=rng.randint(1, 4), dtype="f32" if f32 else "bf16",
                    reqs=_draw_reqs(rng, _log_int(rng, 16, 2500), 1), rho="%.3f" % rng.uniform(0.1, 1.0),
                    t=round(rng.uniform(0.2, 0.6), 2), steps=rng.randint(1, 10))
    if kind in ("step", "cached"):
        f32 = kind == "step" and rng.random() < 0.25
        model = SMALL if f32 else rng.choice([SMALL, WIDE, WIDE, XL])
        count = rng.choice([1, 1, 1, 2, 3, 5])
        tokens = _log_int(rng, 200, 3000 if f32 else 30000)
        lo = round(rng.uniform(0.3, 0.6), 2)
        case = dict(kind=kind, **model, L=rng.randint(1, 2), dtype="f32" if f32 else "bf16",
                    attention=rng.choice(["joint", "joint", "factorised"]), reqs=_draw_reqs(rng, tokens, count, 12),
                    rho="+".join("%.3f" % math.exp(rng.uniform(math.log(0.03), 0.0)) for _ in range(count)),
                    full=0, t_lo=lo, t_hi=lo, steps=25, at=rng.choice([0, 1, 12]))
        return case
    if kind == "attention":
        nseg = rng.randint(1, 12)
        q = [_log_int(rng, 1, 4000) for _ in range(nseg)]
        kv = [n if rng.random() < 0.6 else _log_int(rng, 1, 8000) for n in q]
        return dict(kind="attention", heads=rng.choice([2, 8, 16]), head_dim=rng.choice([64, 64, 72]), dtype="bf16",
                    q="+".join(map(str, q)), kv="+".join(map(str, kv)))
    if kind == "latents":
        return dict(kind="latents", reqs=_draw_reqs(rng, _log_int(rng, 20000, 6 << 20), rng.choice([1, 1, 3]), 128),
                    rho="", layout=rng.choice(["tokens", "nchw"]), dtype=rng.choice(["f32", "f32", "bf16"]),
                    noise=rng.random() < 0.6) | {"rho": "%.3f" % rng.uniform(0.05, 0.9)}
    return dict(kind="frontend", reqs=_draw_reqs(rng, _log_int(rng, 200, 30000), rng.choice([1, 1, 2]), 16))


# ---------------------------------------------------------------------------
# shapes
# ---------------------------------------------------------------------------
class _Req:
    def __init__(self, text):
        self.frames, self.h, self.w = (int(v) for v in text.split("x"))
        self.tpf = (self.h // 2) * (self.w // 2)
        self.tokens = self.frames * self.tpf


class _Cfg:
    def __init__(self, c):
        self.D, self.heads, self.head_dim, self.mlp, self.L = c["D"], c["heads"], c["head_dim"], c["mlp"], c["L"]
        self.dtype, self.attention = c["dtype"], c.get("attention", "joint")


def _reqs(case):
    return [_Req(t) for t in case["reqs"].split("+")]


def _rhos(case, reqs):
    v = [float(t) for t in case["rho"].split("+")]
    return v if len(v) == len(reqs) else v[:1] * len(reqs)


def _count(n, rho):
    return min(n, int(math.floor(rho * n + 0.5)))


def _selected(case, reqs):
    if case.get("full"):
        return [case["full"] * r.tpf + (r.frames - case["full"]) * _count(r.tpf, rho)
                for r, rho in zip(reqs, _rhos(case, reqs))]
    return [_count(r.tokens, rho) for r, rho in zip(reqs, _rhos(case, reqs))]


def _tdt(name):
    return torch.bfloat16 if name == "bf16" else torch.float32


# ---------------------------------------------------------------------------
# inputs (drawn on the GPU from the seed)
# ---------------------------------------------------------------------------
def _gen(seed, stream):
    return torch.Generator(device=DEV).manual_seed((int(seed) * 1000003 + stream) % (1 << 62))


def _randn(gen, *shape):
    return torch.randn(*shape, generator=gen, device=DEV, dtype=torch.float32)


def _uncertainty(reqs, seed):
    """Per-token maps of 20 Gaussian blobs a frame plus a little noise, float32 [N]."""
    gen = _gen(seed, 3)
    out = []
    for r in reqs:
        hp, wp = r.h // 2, r.w // 2
        sigma = 8.0
        cy = torch.rand(r.frames, 20, 1, generator=gen, device=DEV) * r.h
        cx = torch.rand(r.frames, 20, 1, generator=gen, device=DEV) * r.w
        gy = torch.exp(-((2.0 * torch.arange(hp, device=DEV) + 0.5 - cy) ** 2) / (2 * sigma * sigma))
        gx = torch.exp(-((2.0 * torch.arange(wp, device=DEV) + 0.5 - cx) ** 2) / (2 * sigma * sigma))
        u = torch.zeros(r.frames, hp, wp, device=DEV)
        for i in range(20):
            u += gy[:, i, :, None] * gx[:, i, None, :]
        u += 0.1 * torch.rand(r.frames, hp, wp, generator=gen, device=DEV)
        out.append(u.reshape(-1))
    return torch.cat(out)


def _threshold(v, rho):
    k = _count(v.numel(), rho)
    if k >= v.numel():
        return -math.inf
    return float(torch.sort(v)[0][v.numel() - k - 1])


def _thresholds(case, reqs, u):
    """Per-frame thresholds: the request's rho, or `full` whole frames (largest mean) and rho in each other one."""
    thr, t0 = [], 0
    for r, rho in zip(reqs, _rhos(case, reqs)):
        v = u[t0:t0 + r.tokens]
        t0 += r.tokens
        if case.get("full"):
            fr = v.view(r.frames, r.tpf)
            top = set(torch.argsort(fr.double().mean(1), descending=True)[:case["full"]].tolist())
            thr += [-math.inf if f in top else _threshold(fr[f], rho) for f in range(r.frames)]
        else:
            thr += [_threshold(v, rho)] * r.frames
    return torch.tensor(thr, dtype=torch.float32, device=DEV)


def _weights(c, seed):
    """Named parameters, every value an N(0, 0.02^2) draw in the model's type."""
    gen, dt = _gen(seed, 0), _tdt(c["dtype"])
    D, mlp, L = c["D"], c["mlp"], c["L"]
    shapes = [("PE_W", 0, (D, 16)), ("PE_B", 0, (D,)), ("T1_W", 0, (D, 256)), ("T1_B", 0, (D,)),
              ("T2_W", 0, (D, D)), ("T2_B", 0, (D,)), ("COND_W", 0, ((6 * L + 2) * D, D)),
              ("COND_B", 0, ((6 * L + 2) * D,)), ("OUT_W", 0, (16, D)), ("OUT_B", 0, (16,))]
    for l in range(L):
        shapes += [("QKV_W", l, (3 * D, D)), ("QKV_B", l, (3 * D,)), ("O_W", l, (D, D)), ("O_B", l, (D,)),
                   ("FC1_W", l, (mlp, D)), ("FC1_B", l, (mlp,)), ("FC2_W", l, (D, mlp)), ("FC2_B", l, (D,))]
    return {(p, l): (_randn(gen, *s) * 0.02).to(dt) for p, l, s in shapes}


def _blob(cfg, weights):
    desc = B.model_desc(cfg)
    esz = 2 if cfg.dtype == "bf16" else 4
    blob = torch.zeros(B.sphinx_model_blob_bytes(desc) // esz, dtype=_tdt(cfg.dtype), device=DEV)
    for (p, l), w in weights.items():
        off, cnt = B.sphinx_model_param(desc, p, l)
        assert cnt == w.numel()
        blob[off // esz:off // esz + cnt] = w.reshape(-1)
    return blob


def _latents(case, reqs, seed):
    n = 16 * sum(r.tokens for r in reqs)
    dt = _tdt(case["dtype"])
    return _randn(_gen(seed, 1), n).to(dt), _randn(_gen(seed, 2), n).to(dt)


def _starts(case, reqs, seed):
    G = sum(r.frames for r in reqs)
    rng = np.random.default_rng(seed)
    t = rng.uniform(case["t_lo"], case["t_hi"], G) if case["t_hi"] > case["t_lo"] else np.full(G, case["t_lo"])
    if case["t_hi"] > case["t_lo"]:
        t[rng.integers(G)] = case["t_hi"]  # the latest start, so that step `at` finds the same frames active
        t = np.where(t < 0.31, 0.31, t)
    return np.rint(1000.0 * t).astype(np.int32) - 1


# ---------------------------------------------------------------------------
# prepare and run
# ---------------------------------------------------------------------------
def prepare(case, seed):
    return {"loop": _prepare_loop, "step": _prepare_step, "cached": _prepare_step, "attention": _prepare_attention,
            "latents": _prepare_latents, "frontend": _prepare_frontend}[case["kind"]](case, seed)


def run(state):
    return _RUN[state["kind"]](state)


def _prepare_loop(case, seed):
    reqs, cfg = _reqs(case), _Cfg(case)
    u = _uncertainty(reqs, seed)
    thr = _thresholds(case, reqs, u)
    z0, eps = _latents(case, reqs, seed)
    blob = _blob(cfg, _weights(case, seed))
    starts = np.full(sum(r.frames for r in reqs), int(round(1000 * case["t"])) - 1, np.int32)
    ref = Refiner(reqs, cfg, blob, starts, np.full(len(reqs), case["steps"], np.int32), u.cpu().numpy(),
                  thr.cpu().numpy(), z0.float().cpu().numpy(), eps.float().cpu().numpy())
    return {"kind": "loop", "refiner": ref}


def _run_loop(s):
    r = s["refiner"]
    state = r.run()
    return {"state": state, "mask": r.mask, "idx": r.idx[:r.n_sel]}


def _prepare_step(case, seed):
    reqs, cfg = _reqs(case), _Cfg(case)
    N, R = sum(r.tokens for r in reqs), len(reqs)
    creqs = B.make_requests(reqs)
    s = dict(kind=case["kind"], reqs=creqs, N=N, dt=B.dtype_code(case["dtype"]))
    s["u"] = _uncertainty(reqs, seed)
    s["thr"] = _thresholds(case, reqs, s["u"])
    z, s["eps"] = _latents(case, reqs, seed)  # token-major state and noise
    s["z"] = z.float()
    s["out"] = s["z"].clone()
    s["blob"] = _blob(cfg, _weights(case, seed))
    s["desc"] = B.model_desc(cfg, s["blob"].data_ptr())
    starts, nsteps = _starts(case, reqs, seed), np.full(R, case["steps"], np.int32)
    s["plan"] = {k: torch.from_numpy(v).to(DEV)
                 for k, v in B.plan_step(creqs, starts, nsteps, case["at"]).items()}
    s["mask"] = torch.empty(N, dtype=torch.uint8, device=DEV)
    s["idx"] = torch.empty(N, dtype=torch.int32, device=DEV)
    s["cu"] = torch.empty(R + 1, dtype=torch.int32, device=DEV)
    s["x"] = torch.empty(16 * N, dtype=torch.float32, device=DEV)
    s["ws_sel"] = torch.empty(B.sphinx_select_workspace_bytes(N), dtype=torch.uint8, device=DEV)
    s["ws"] = torch.empty(B.sphinx_refine_workspace_bytes(s["desc"], creqs, N), dtype=torch.uint8, device=DEV)
    if case["kind"] == "cached":
        s["ctx"] = {k: torch.from_numpy(v).to(DEV)
                    for k, v in B.sphinx_plan_cache(creqs, starts, nsteps, case["at"], case["steps"]).items()
                    if k in ("a_ctx", "b_ctx")}
        s["kv"] = _cache(case, N, seed)
    return s


def _cache(case, N, seed):
    """Keys and values of an earlier full step: the scale of a projection of normalised rows."""
    std = 0.02 * math.sqrt(case["D"])
    return (_randn(_gen(seed, 5), case["L"], N, 2 * case["D"]) * std).to(_tdt(case["dtype"]))


def _run_step(s):
    p = s["plan"]
    cu = B.select_mask(s["reqs"], s["u"], s["thr"], p["active"], s["mask"], s["idx"], s["cu"], s["ws_sel"])
    n = int(cu[-1])
    B.gather(s["reqs"], B.TOKENS, s["z"], B.F32, s["eps"], s["dt"], s["idx"], n, p["a"], p["b"], s["x"])
    B.refine_step(s["desc"], s["reqs"], s["idx"], n, cu, p["tau"], p["c1"], p["c2"], s["x"], s["ws"])
    B.scatter_blend(s["reqs"], s["x"], s["idx"], n, s["z"], B.F32, B.TOKENS, s["out"], B.F32, B.TOKENS)
    return {"x": s["x"][:16 * n], "out": s["out"], "mask": s["mask"], "idx": s["idx"][:n]}


def _run_cached(s):
    p, c = s["plan"], s["ctx"]
    cu = B.select_mask(s["reqs"], s["u"], s["thr"], p["active"], s["mask"], s["idx"], s["cu"], s["ws_sel"])
    n = int(cu[-1])
    B.sphinx_gather_ctx(s["reqs"], B.TOKENS, s["z"], B.F32, s["eps"], s["dt"], s["idx"], n, s["mask"], p["a"], p["b"],
                        c["a_ctx"], c["b_ctx"], s["x"])
    B.sphinx_refine_step_cached(s["desc"], s["reqs"], s["idx"], n, cu, p["tau"], p["c1"], p["c2"], s["x"], s["kv"],
                                s["ws"])
    B.sphinx_scatter_masked(s["reqs"], s["x"], s["idx"], n, s["mask"], s["out"], B.F32, B.TOKENS)
    return {"x": s["x"][:16 * n], "out": s["out"], "kv": s["kv"], "mask": s["mask"], "idx": s["idx"][:n]}


def _segments(case):
    return [int(v) for v in case["q"].split("+")], [int(v) for v in case["kv"].split("+")]


def _prepare_attention(case, seed):
    lq, lk = _segments(case)
    H, d = case["heads"], case["head_dim"]
    gen, D = _gen(seed, 6), H * d
    # q as the projection leaves it: scaled by log2(e)/sqrt(d), and rounded to the model's type
    q = (_randn(gen, sum(lq), D) * (math.log2(math.e) / math.sqrt(d))).to(_tdt(case["dtype"]))
    kv = _randn(gen, sum(lk), 2 * D).to(_tdt(case["dtype"]))
    return dict(kind="attention", dt=B.dtype_code(case["dtype"]), H=H, d=d, q=q, kv=kv, o=torch.empty_like(q),
                cu_q=np.concatenate([[0], np.cumsum(lq)]).astype(np.int32),
                cu_k=np.concatenate([[0], np.cumsum(lk)]).astype(np.int32))


def _run_attention(s):
    D = s["H"] * s["d"]
    B.sphinx_varlen_attention(s["dt"], s["H"], s["d"], s["q"], D, s["kv"], s["kv"][:, D:], 2 * D, s["o"], s["cu_q"],
                              s["cu_k"])
    return s["o"]


def _prepare_latents(case, seed):
    reqs = _reqs(case)
    N, G = sum(r.tokens for r in reqs), sum(r.frames for r in reqs)
    rng = np.random.default_rng(seed)
    s = dict(kind="latents", reqs=B.make_requests(reqs), dt=B.dtype_code(case["dtype"]),
             layout=B.TOKENS if case["layout"] == "tokens" else B.NCHW)
    s["u"] = _uncertainty(reqs, seed)
    s["thr"] = _thresholds(case, reqs, s["u"])
    s["z"] = _randn(_gen(seed, 1), 16 * N).to(_tdt(case["dtype"]))
    s["out"] = s["z"].clone()
    s["eps"] = _randn(_gen(seed, 2), 16 * N).to(torch.bfloat16) if case["noise"] else None
    s["active"] = torch.ones(G, dtype=torch.uint8, device=DEV)
    a = rng.uniform(0.5, 0.9, G).astype(np.float32) if case["noise"] else np.ones(G, np.float32)
    b = np.sqrt(1 - a * a).astype(np.float32) if case["noise"] else np.zeros(G, np.float32)
    s["a"], s["b"] = torch.from_numpy(a).to(DEV), torch.from_numpy(b).to(DEV)
    s["mask"] = torch.empty(N, dtype=torch.uint8, device=DEV)
    s["idx"] = torch.empty(N, dtype=torch.int32, device=DEV)
    s["cu"] = torch.empty(len(reqs) + 1, dtype=torch.int32, device=DEV)
    s["x"] = torch.empty(16 * sum(_selected(case, reqs)), dtype=torch.float32, device=DEV)
    s["ws"] = torch.empty(B.sphinx_select_workspace_bytes(N), dtype=torch.uint8, device=DEV)
    return s


def _run_latents(s):
    cu = B.select_mask(s["reqs"], s["u"], s["thr"], s["active"], s["mask"], s["idx"], s["cu"], s["ws"])
    n = int(cu[-1])
    B.gather(s["reqs"], s["layout"], s["z"], s["dt"], s["eps"], B.BF16, s["idx"], n, s["a"], s["b"], s["x"])
    B.scatter_blend(s["reqs"], s["x"], s["idx"], n, s["out"], s["dt"], s["layout"], s["out"], s["dt"], s["layout"])
    return {"x": s["x"][:16 * n], "out": s["out"], "mask": s["mask"], "idx": s["idx"][:n], "cu": s["cu"]}


def _prepare_frontend(case, seed):
    """Textured frames with blurred discs (motion blur) and an opacity map with holes (disocclusions)."""
    reqs, gen = _reqs(case), _gen(seed, 7)
    rgb, opacity = [], []
    for r in reqs:
        H, W = 8 * r.h, 8 * r.w
        yy = torch.arange(H, device=DEV, dtype=torch.float32)[:, None]
        xx = torch.arange(W, device=DEV, dtype=torch.float32)[None, :]
        for _ in range(r.frames):
            v = torch.rand(64, generator=gen, device=DEV)
            img = torch.stack([128 + 80 * torch.sin(6.28 * (6 * v[3 * c] * yy / H + 6 * v[3 * c + 1] * xx / W +
                                                            v[3 * c + 2])) for c in range(3)])
            img = (img + 96 * (torch.rand(3, H, W, generator=gen, device=DEV) - 0.5)).clamp(0, 255)
            soft = torch.nn.functional.avg_pool2d(img[None], 7, 1, 3, count_include_pad=False)[0]
            inside = torch.zeros(H, W, dtype=torch.bool, device=DEV)
            op = torch.ones(H, W, device=DEV)
            for k in range(5):
                rad = (0.05 + 0.1 * v[20 + k]) * min(H, W)
                inside |= (yy - v[25 + k] * H) ** 2 + (xx - v[30 + k] * W) ** 2 < rad * rad
                sig = (0.02 + 0.04 * v[35 + k]) * min(H, W)
                op -= 0.95 * torch.exp(-((yy - v[40 + k] * H) ** 2 + (xx - v[45 + k] * W) ** 2) / (2 * sig * sig))
            rgb.append(torch.where(inside, soft, img).round().to(torch.uint8).permute(1, 2, 0).reshape(-1))
            opacity.append((op + 0.02 * _randn(gen, H, W)).clamp(0, 1).reshape(-1))
    N, G = sum(r.tokens for r in reqs), sum(r.frames for r in reqs)
    creqs = B.make_requests(reqs)
    return dict(kind="frontend", reqs=creqs, rgb=torch.cat(rgb), opacity=torch.cat(opacity),
                mask=torch.empty(N, dtype=torch.uint8, device=DEV),
                u=torch.empty(N, dtype=torch.float32, device=DEV),
                otsu=torch.empty(G, dtype=torch.int32, device=DEV),
                ws=torch.empty(B.sphinx_mask_frontend_workspace_bytes(creqs), dtype=torch.uint8, device=DEV))


def _run_frontend(s):
    B.sphinx_mask_frontend(s["reqs"], s["rgb"], s["opacity"], 0.5, s["mask"], s["u"], s["otsu"], s["ws"])
    return {"mask": s["mask"], "u": s["u"], "otsu": s["otsu"]}


_RUN = {"loop": _run_loop, "step": _run_step, "cached": _run_cached, "attention": _run_attention,
        "latents": _run_latents, "frontend": _run_frontend}


# ---------------------------------------------------------------------------
# work and tolerance
# ---------------------------------------------------------------------------
def _model_flops(c, n, pairs):
    D = c["D"]
    return c["L"] * (2.0 * n * (4 * D * D + 2 * D * c["mlp"]) + 4.0 * D * pairs) + 64.0 * n * D


def _weight_count(c):
    D, L = c["D"], c["L"]
    return (D * 17 + 257 * D + D * D + D + (6 * L + 2) * D * (D + 1) + 16 * D + 16 +
            L * (4 * D * D + 4 * D + 2 * D * c["mlp"] + c["mlp"] + D))


def _pairs(c, reqs, sel):
    """Query-key pairs of one block (joint, or the mean of a spatial and a temporal block), selections taken as even."""
    tot = 0.0
    for r, k in zip(reqs, sel):
        keys = r.tokens if c["kind"] == "cached" else k
        if c.get("attention", "joint") == "joint":
            tot += float(k) * keys
        else:
            blocks = [k * keys / r.frames if l % 2 == 0 else k * keys / r.tpf for l in range(c["L"])]
            tot += sum(blocks) / c["L"]
    return tot


def work(case):
    kind = case["kind"]
    if kind == "attention":
        lq, lk = _segments(case)
        D = case["heads"] * case["head_dim"]
        return {"bytes": 2.0 * D * (2 * sum(lq) + 2 * sum(lk)),
                "flops": 4.0 * D * sum(float(a) * b for a, b in zip(lq, lk))}
    reqs = _reqs(case)
    N = sum(r.tokens for r in reqs)
    if kind == "frontend":  # RGB and opacity read, mask and map written; integer stencil work is no matrix work
        return {"bytes": 256.0 * N * 7 + 5.0 * N, "flops": 60.0 * 256 * N}
    sel = _selected(case, reqs)
    n, e = sum(sel), 2 if case["dtype"] == "bf16" else 4
    if kind == "latents":
        # map read, mask and indices written; state rows (and noise) read, gathered rows written, read and scattered
        return {"bytes": 5.0 * N + 4.0 * n + n * (16 * e + (32 if case["noise"] else 0) + 64 + 16 * e),
                "flops": 32.0 * n}
    weights = float(_weight_count(case)) * e
    if kind == "loop":
        steps = case["steps"]
        return {"bytes": steps * (weights + 192.0 * n) + 16.0 * N * (2 * e + 4) + 9.0 * N,
                "flops": steps * _model_flops(case, n, _pairs(case, reqs, sel))}
    bytes_ = weights + 5.0 * N + 4.0 * n + 64.0 * n + 16.0 * e * n + 64.0 * n
    if kind == "step":
        bytes_ += 128.0 * N
    else:
        bytes_ += 64.0 * n + 2.0 * case["D"] * e * N * case["L"]
    return {"bytes": bytes_, "flops": _model_flops(case, n, _pairs(case, reqs, sel))}


def tolerance(case):
    """About four times the distance to float64 that the path shows at these sizes (fp32 steps 6e-8; bf16 steps 1.7e-4
    and loops 2.4e-4 on the latents, which the update moves little; cached bf16 keys and values 1.3e-3; bf16
    attention alone 2.3e-3)."""
    kind = case["kind"]
    if kind == "frontend":
        return "exact"  # integer arithmetic throughout
    if kind == "latents":
        # one multiply-add per value; bf16 states round it once more
        return {"rel": 2e-7, "max": 1e-6} if case["dtype"] == "f32" else {"rel": 1e-3, "max": 1e-2}
    if case["dtype"] == "f32":
        return {"rel": 5e-7, "max": 1e-5}
    if kind == "attention":
        return {"rel": 8e-3, "max": 0.1}
    if kind == "cached":
        return {"rel": 5e-3, "max": 0.05}
    return {"rel": 1e-3 if kind == "loop" else 7e-4, "max": 0.03}


# ---------------------------------------------------------------------------
# float64 references
# ---------------------------------------------------------------------------
def _alpha_bar():
    return np.cumprod(1.0 - np.linspace(1e-4, 2e-2, 1000))


def _plan64(reqs, starts, nsteps, step):
    """Per frame: active, newly, tau, injection (a, b) and DDIM (c1, c2) on the request's shared grid."""
    ab = _alpha_bar()
    at = lambda t: 1.0 if t < 0 else float(ab[t])
    out, g = [], 0
    for r in reqs:
        s = starts[g:g + r.frames]
        smax = int(s.max())
        grid = lambda i: ((nsteps - i) * (smax + 1)) // nsteps - 1
        t, tn = grid(step), grid(step + 1)
        c1 = math.sqrt(at(tn) / at(t))
        c2 = math.sqrt(1 - at(tn)) - math.sqrt(at(tn) * (1 - at(t)) / at(t))
        for f in range(r.frames):
            active = t <= s[f]
            newly = active and (step == 0 or grid(step - 1) > s[f])
            out.append((active, newly, t, math.sqrt(at(t)) if newly else 1.0, math.sqrt(1 - at(t)) if newly else 0.0,
                        c1 if active else 1.0, c2 if active else 0.0))
        g += r.frames
    return out


def _sin_cos(pos, half, base_count):
    w = torch.exp(-math.log(1e4) * torch.arange(base_count, device=DEV, dtype=torch.float64) / base_count)
    a = pos.double()[:, None] * w
    return torch.cat([torch.sin(a), torch.cos(a)], 1)


def _softmax_pv(q, k, v, mask=None):
    s = q @ k.transpose(-1, -2)
    if mask is not None:
        s = s.masked_fill(~mask, -math.inf)
    return torch.softmax(s, -1) @ v


def _attend64(c, reqs, block, idx, cu, q, k, v, kd, vd):
    """Attention of one block; kd, vd: every token's keys and values with the latent cache, else None."""
    n, H, d = q.shape[0], c["heads"], c["head_dim"]
    o = torch.empty_like(q)
    split = lambda t: t.reshape(-1, H, d).transpose(0, 1)  # [H][rows][d]
    t0 = 0
    for r, (lo, hi) in zip(reqs, zip(cu[:-1], cu[1:])):
        if hi > lo:
            loc = idx[lo:hi] - t0
            if c["attention"] == "joint":
                groups = [(slice(lo, hi), slice(t0, t0 + r.tokens))]
            elif block % 2 == 0:
                f = loc // r.tpf
                groups = []
                for ff in torch.unique(f).tolist():
                    rows = torch.nonzero(f == ff).flatten()
                    groups.append((slice(lo + int(rows[0]), lo + int(rows[-1]) + 1),
                                   slice(t0 + ff * r.tpf, t0 + (ff + 1) * r.tpf)))
            else:
                groups = None
            if groups is not None:
                for rows, toks in groups:
                    qq, kk, vv = split(q[rows]), *((split(k[rows]), split(v[rows])) if kd is None else
                                                  (split(kd[toks]), split(vd[toks])))
                    for h in range(H):
                        o[rows, h * d:(h + 1) * d] = _softmax_pv(qq[h], kk[h], vv[h])
            else:  # across the frames of a position: dense [position][head][frame][d] with absent members masked
                def dense(t):
                    z = torch.zeros(r.tokens, H * d, device=DEV, dtype=torch.float64)
                    z[loc] = t[lo:hi]
                    return z
                shape = lambda t: t.reshape(r.frames, r.tpf, H, d).permute(1, 2, 0, 3)
                there = torch.zeros(r.tokens, dtype=torch.bool, device=DEV)
                there[loc] = True
                if kd is None:
                    kk, vv, keep = dense(k), dense(v), there.clone()
                else:
                    kk, vv, keep = kd[t0:t0 + r.tokens], vd[t0:t0 + r.tokens], torch.ones_like(there)
                keep = keep.reshape(r.frames, r.tpf).t()
                keep = torch.where(keep.any(1, keepdim=True), keep, torch.ones_like(keep))
                res = _softmax_pv(shape(dense(q)), shape(kk), shape(vv), keep[:, None, None, :])
                o[lo:hi] = res.permute(2, 0, 1, 3).reshape(r.tokens, H * d)[loc]
        t0 += r.tokens
    return o


def _layer_norm(h):
    m = h.mean(1, keepdim=True)
    return (h - m) / torch.sqrt(((h - m) ** 2).mean(1, keepdim=True) + 1e-6)


def _denoise64(c, reqs, w, x, idx, cu, tau, kv=None):
    """eps_hat of the gathered rows x [n][16] at their timesteps tau [n]; kv [L][N][2D] is updated in place."""
    W = lambda p, l=0: w[(p, l)].double()
    lin = lambda a, p, b, l=0: a @ W(p, l).t() + W(b, l)
    silu = lambda a: a / (1 + torch.exp(-a))
    D, L = c["D"], c["L"]
    times, inv = torch.unique(tau, return_inverse=True)
    wk = torch.exp(-math.log(1e4) * torch.arange(128, device=DEV, dtype=torch.float64) / 128)
    arg = times.double()[:, None] * wk
    cond = lin(silu(lin(torch.cat([torch.cos(arg), torch.sin(arg)], 1), "T1_W", "T1_B")), "T2_W", "T2_B")
    mod = lin(silu(cond), "COND_W", "COND_B")[inv].view(x.shape[0], 6 * L + 2, D)
    f, y, xx, t0 = [], [], [], 0
    for r, lo, hi in zip(reqs, cu[:-1], cu[1:]):
        loc = idx[lo:hi] - t0
        f.append(loc // r.tpf)
        y.append(loc % r.tpf // (r.w // 2))
        xx.append(loc % r.tpf % (r.w // 2))
        t0 += r.tokens
    f, y, xx = torch.cat(f), torch.cat(y), torch.cat(xx)
    h = lin(x, "PE_W", "PE_B") + torch.cat([_sin_cos(y, D // 2, D // 4), _sin_cos(xx, D // 2, D // 4)], 1)
    h = h + _sin_cos(f, D, D // 2)
    for l in range(L):
        sh1, sc1, g1, sh2, sc2, g2 = (mod[:, 6 * l + i] for i in range(6))
        q, k, v = lin(_layer_norm(h) * (1 + sc1) + sh1, "QKV_W", "QKV_B", l).split(D, 1)
        kd = vd = None
        if kv is not None:
            kv[l, idx] = torch.cat([k, v], 1)
            kd, vd = kv[l, :, :D], kv[l, :, D:]
        o = _attend64(c, reqs, l, idx, cu, q / math.sqrt(c["head_dim"]), k, v, kd, vd)
        h = h + (1 + g1) * lin(o, "O_W", "O_B", l)
        a = lin(_layer_norm(h) * (1 + sc2) + sh2, "FC1_W", "FC1_B", l)
        a = 0.5 * a * (1 + torch.tanh(math.sqrt(2 / math.pi) * (a + 0.044715 * a ** 3)))
        h = h + (1 + g2) * lin(a, "FC2_W", "FC2_B", l)
    return lin(_layer_norm(h) * (1 + mod[:, 6 * L + 1]) + mod[:, 6 * L], "OUT_W", "OUT_B")


def _frames_of(reqs):
    return torch.cat([torch.arange(r.frames, device=DEV).repeat_interleave(r.tpf) + g for r, g in
                      zip(reqs, np.cumsum([0] + [r.frames for r in reqs[:-1]]).tolist())])


def _to_tokens(reqs, z):
    """NCHW latents of all requests -> [N][16] token rows."""
    out, o = [], 0
    for r in reqs:
        v = z[o:o + 16 * r.tokens].view(r.frames, 4, r.h // 2, 2, r.w // 2, 2)
        out.append(v.permute(0, 2, 4, 1, 3, 5).reshape(r.tokens, 16))
        o += 16 * r.tokens
    return torch.cat(out)


def _to_nchw(reqs, t):
    out, o = [], 0
    for r in reqs:
        v = t[o:o + r.tokens].view(r.frames, r.h // 2, r.w // 2, 4, 2, 2)
        out.append(v.permute(0, 3, 1, 4, 2, 5).reshape(-1))
        o += r.tokens
    return torch.cat(out)


def _step64(case, reqs, w, u, thr, z, eps, starts, step, kv=None):
    """One step in float64 on token rows z [N][16]; returns (state, selected rows, mask, idx)."""
    plan = _plan64(reqs, starts, case["steps"], step)
    col = lambda i: torch.tensor([float(p[i]) for p in plan], device=DEV, dtype=torch.float64)
    fr = _frames_of(reqs)
    mask = (u > thr[fr]) & (col(0)[fr] > 0)
    idx = torch.nonzero(mask).flatten()
    bounds = np.cumsum([0] + [r.tokens for r in reqs])
    cu = [int(mask[:b].sum()) for b in bounds]
    g = fr[idx]
    x = col(3)[g][:, None] * z[idx] + col(4)[g][:, None] * eps[idx]
    e = _denoise64(case, reqs, w, x, idx, cu, col(2)[g], kv)
    x = col(5)[g][:, None] * x + col(6)[g][:, None] * e
    out = z.clone()
    out[idx] = x
    return out, x, mask.to(torch.uint8), idx.to(torch.int32)


def exact(case, seed):
    kind = case["kind"]
    if kind == "frontend":
        return None  # whole numbers, which have to stay the same
    if kind == "attention":
        s = _prepare_attention(case, seed)
        H, d, D = s["H"], s["d"], s["H"] * s["d"]
        o = torch.empty(s["q"].shape, dtype=torch.float64, device=DEV)
        for i in range(len(s["cu_q"]) - 1):
            a, b, e, f = s["cu_q"][i], s["cu_q"][i + 1], s["cu_k"][i], s["cu_k"][i + 1]
            for h in range(H):
                c = slice(h * d, (h + 1) * d)
                q = s["q"][a:b, c].double() * math.log(2.0)  # the base-2 softmax
                o[a:b, c] = _softmax_pv(q, s["kv"][e:f, c].double(), s["kv"][e:f, D:][:, c].double())
        return o
    reqs = _reqs(case)
    if kind == "latents":
        s = _prepare_latents(case, seed)
        fr = _frames_of(reqs)
        mask = s["u"] > s["thr"][fr]
        idx = torch.nonzero(mask).flatten()
        tok = (lambda t: t.view(-1, 16)) if case["layout"] == "tokens" else (lambda t: _to_tokens(reqs, t))
        x = s["a"].double()[fr[idx]][:, None] * tok(s["z"])[idx].double()
        if case["noise"]:
            x = x + s["b"].double()[fr[idx]][:, None] * tok(s["eps"])[idx].double()
        out = tok(s["z"]).double()
        out = out.clone() if case["layout"] == "tokens" else out
        out[idx] = x
        out = out.reshape(-1) if case["layout"] == "tokens" else _to_nchw(reqs, out)
        return {"x": x.reshape(-1), "out": out, "mask": None, "idx": None, "cu": None}
    w = _weights(case, seed)
    u = _uncertainty(reqs, seed)
    thr = _thresholds(case, reqs, u)
    z, eps = (t.double() for t in _latents(case, reqs, seed))
    if kind == "loop":
        z, eps = _to_tokens(reqs, z), _to_tokens(reqs, eps)
        starts = np.full(sum(r.frames for r in reqs), int(round(1000 * case["t"])) - 1, np.int32)
        c = dict(case, attention="joint")
        for i in range(case["steps"]):
            z, _, mask, idx = _step64(c, reqs, w, u, thr, z, eps, starts, i)
        return {"state": _to_nchw(reqs, z), "mask": None, "idx": None}
    kv = _cache(case, sum(r.tokens for r in reqs), seed).double() if kind == "cached" else None
    out, x, mask, idx = _step64(case, reqs, w, u, thr, z.view(-1, 16), eps.view(-1, 16),
                                _starts(case, reqs, seed), case["at"], kv)
    res = {"x": x.reshape(-1), "out": out.reshape(-1), "mask": None, "idx": None}
    return res | ({"kv": kv} if kind == "cached" else {})
