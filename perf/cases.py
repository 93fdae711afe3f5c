"""Performance cases of libgspn: what a program that uses the line scan has it do.

A case is a plain dict.  Kinds:

* "fwd"         inference: one forward scan (scan_fwd; with layout="blocked"
                the producer wrote the per-direction tensors in scan order);
* "fwd_norm"    inference with the weights given as logits (scan_fwd_norm);
* "train"       one training step of the operator: the training pair
                scan_fwd_train + scan_bwd_reserve, y and every gradient;
* "train_norm"  the training pair of the entry points that take logits;
* "latent"      the latent-space propagation sublayer (latent_fwd).

Buffers that a program keeps between steps (outputs, workspace, reserve) are
made by prepare(); every pass fills them anew.
"""
from __future__ import annotations

import math

import torch

import paper_2606_00746_amd as gspn

DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def _scan(name, kind, B, C, G, H, W, dtype="bf16", dirs=15, layout="pixel", sigma=1.0):
    return {"name": name, "kind": kind, "B": B, "C": C, "G": G, "H": H, "W": W, "dtype": dtype,
            "dirs": dirs, "layout": layout, "sigma": sigma}


def _latent(name, B, C, Cc, H, W, dirs=15):
    return {"name": name, "kind": "latent", "B": B, "C": C, "Cc": Cc, "H": H, "W": W,
            "dtype": "bf16", "dirs": dirs}


def listed():
    return [
        # the smallest call: one direction of a 16x16 fp32 map, launch latency
        _scan("fwd-f32-16x16", "fwd", 1, 8, 1, 16, 16, "f32", dirs=1),
        # one image of a detector's rectangular feature map, weights as logits
        _scan("infer-48x80-logits", "fwd_norm", 1, 256, 8, 48, 80),
        # 14x14 token grid of a small ViT, training
        _scan("train-14x14", "train", 32, 384, 12, 14, 14),
        # second stage of a hierarchical encoder (56 -> 28), training
        _scan("train-28x28", "train", 64, 192, 16, 28, 28),
        # odd token grid (518 pixels in 14-pixel patches), training
        _scan("train-37x37", "train", 16, 384, 12, 37, 37),
        # first stage of a hierarchical encoder, training
        _scan("train-56x56", "train", 64, 96, 8, 56, 56),
        # high-resolution encoder stage, training: the headline benchmark
        _scan("train-64x64", "train", 8, 768, 24, 64, 64),
        # the same stage with per-channel weights predicted as logits
        _scan("train-64x64-perchannel", "train_norm", 8, 768, 768, 64, 64),
        # fp32 storage (full-precision fine-tuning) on a rectangular map
        _scan("train-f32-40x56", "train", 4, 192, 6, 40, 56, "f32"),
        # dense-prediction map, training, planes longer than a wave
        _scan("train-128x128", "train", 2, 192, 6, 128, 128),
        # extreme-resolution inference with peaky weights
        _scan("fwd-256x256", "fwd", 1, 1024, 32, 256, 256, sigma=2.0),
        # latent sublayer of a ViT at 1036 pixels (74x74 tokens), inference
        _latent("latent-74x74", 32, 1152, 64, 74, 74),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["train", "train", "train", "train", "train_norm", "fwd", "fwd", "fwd_norm",
                       "latent"])
    dirs = rng.choice([15, 15, 15, 15, 3, 12, 1, 7])
    if kind == "latent":
        H = _log_int(rng, 20, 80)
        W = H if rng.random() < 0.6 else _log_int(rng, 20, 80)
        Cc = rng.choice([16, 32, 64, 96])
        C = 8 * _log_int(rng, 24, 144)
        B = max(1, min(32, int(32 * 1152 * 74 * 74 * rng.uniform(0.1, 0.9) / (C * H * W * Cc / 64))))
        return {"kind": "latent", "B": B, "C": C, "Cc": Cc, "H": H, "W": W, "dtype": "bf16",
                "dirs": dirs}
    train = kind.startswith("train")
    top = 160 if train else 256
    H = _log_int(rng, 7, top)
    W = H if rng.random() < 0.5 else max(7, min(top, int(H * rng.uniform(0.5, 2.0))))
    dtype = "f32" if rng.random() < 0.25 else "bf16"
    cpg = rng.choice([1, 8, 32, _log_int(rng, 2, 48), _log_int(rng, 2, 48)])
    # elements of x: from one small image to the largest listed maps (longer
    # planes of a training step up to the listed 128x128 one)
    most = 6.2e6 if train and max(H, W) > 64 else 2.0e7
    n = math.exp(rng.uniform(math.log(3e4), math.log(most * (0.5 if dtype == "f32" else 1.0))))
    groups = max(1, int(n / (H * W * cpg)))
    B = min(64, groups, rng.choice([1, 2, 4, 8, 16, 32, 64]))
    G = max(1, groups // B)
    layout = "blocked" if kind == "fwd" and rng.random() < 0.4 else "pixel"
    return {"kind": kind, "B": B, "C": G * cpg, "G": G, "H": H, "W": W, "dtype": dtype,
            "dirs": dirs, "layout": layout, "sigma": rng.choice([1.0, 1.0, 2.0])}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _bits(dirs):
    return [b for b in (1, 2, 4, 8) if dirs & b]


def _blocked(t, dirs, H, W):
    """Pixel-major [D, ..., H, W] -> blocked line-major [D, ..., H*W]."""
    out = torch.empty(t.shape[:-2] + (H * W,), dtype=t.dtype, device=t.device)
    for s, bit in enumerate(_bits(dirs)):
        p = t[s] if bit < 4 else t[s].transpose(-1, -2)
        L = p.shape[-2]
        out[s] = torch.cat([p[..., q:q + 8, :].transpose(-1, -2).flatten(-2)
                            for q in range(0, L, 8)], dim=-1)
    return out


def _draw_scan(c, seed):
    """Pixel-major inputs in the storage type, from the seed alone."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    dt = DTYPES[c["dtype"]]
    B, C, G, H, W = (c[k] for k in "BCGHW")
    bits = _bits(c["dirs"])
    D = len(bits)

    def normal(*shape):
        return torch.randn(shape, generator=gen, device="cuda")

    t = {"x": normal(B, C, H, W).to(dt),
         "lam": normal(D, B, C, H, W).sigmoid_().to(dt),
         "u": normal(D, B, C, H, W).sigmoid_().to(dt)}
    logits = normal(D, B, G, 3, H, W).mul_(c["sigma"])
    if c["kind"].endswith("norm"):
        t["w"] = logits.to(dt)
    else:
        # softmax over the taps on the grid; the others are 0
        for s, bit in enumerate(bits):
            if bit < 4:
                logits[s, ..., 0, :, 0] = -math.inf
                logits[s, ..., 2, :, W - 1] = -math.inf
            else:
                logits[s, ..., 0, 0, :] = -math.inf
                logits[s, ..., 2, H - 1, :] = -math.inf
        t["w"] = logits.softmax(3).to(dt)
    if c["kind"].startswith("train"):
        t["dy"] = normal(B, C, H, W).to(dt)
    return t


def _draw_latent(c, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    B, C, Cc, H, W = (c[k] for k in ("B", "C", "Cc", "H", "W"))
    D = len(_bits(c["dirs"]))

    def normal(*shape, fan=1):
        return torch.randn(shape, generator=gen, device="cuda").mul_(fan ** -0.5).bfloat16()

    return {"x": normal(B, C, H, W), "p_down": normal(Cc, C, fan=C),
            "l_u": normal(D, Cc, Cc, fan=Cc), "l_lam": normal(D, Cc, Cc, fan=Cc),
            "l_w": normal(D, Cc, 3, Cc, fan=Cc), "p_up": normal(C, Cc, fan=Cc)}


def _workspace(ops, t, dirs):
    n = max(gspn.workspace_size(op, t["x"], t["w"], dirs) for op in ops)
    return torch.empty(max(n, 1), dtype=torch.uint8, device="cuda")


def prepare(c, seed):
    dirs = c["dirs"]
    s = {"kind": c["kind"], "dirs": dirs}
    if c["kind"] == "latent":
        s.update(_draw_latent(c, seed))
        s["y"] = torch.empty_like(s["x"])
        return s
    t = _draw_scan(c, seed)
    if c["layout"] == "blocked":
        for k in ("w", "lam", "u"):
            t[k] = _blocked(t[k], dirs, c["H"], c["W"])
    s.update(t)
    s["y"] = torch.empty_like(t["x"])
    s["layout"] = c["layout"]
    if c["kind"] == "fwd":
        op = gspn.OP_FWD if c["layout"] == "pixel" else gspn.OP_FWD_BLOCKED
        s["ws"] = _workspace([op], t, dirs)
    elif c["kind"] == "fwd_norm":
        s["ws"] = _workspace([gspn.OP_FWD_NORM], t, dirs)
    else:
        norm = c["kind"] == "train_norm"
        s["ws"] = _workspace([gspn.OP_FWD_NORM_TRAIN, gspn.OP_BWD_NORM_RESERVE] if norm
                             else [gspn.OP_FWD_TRAIN, gspn.OP_BWD_RESERVE], t, dirs)
        nrs = gspn.reserve_size(t["x"], t["w"], dirs, norm=norm)
        s["reserve"] = torch.empty(nrs, dtype=torch.uint8, device="cuda") if nrs else None
        s["grads"] = tuple(torch.empty_like(t[k]) for k in ("x", "w", "lam", "u"))
    return s


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def run(s):
    kind, dirs = s["kind"], s["dirs"]
    if kind == "latent":
        return gspn.latent_fwd(s["x"], s["p_down"], s["l_u"], s["l_lam"], s["l_w"], s["p_up"],
                               dirs, y=s["y"])
    x, w, lam, u = s["x"], s["w"], s["lam"], s["u"]
    if kind == "fwd":
        return gspn.scan_fwd(x, w, lam, u, dirs, y=s["y"], layout=s["layout"], workspace=s["ws"])
    if kind == "fwd_norm":
        return gspn.scan_fwd_norm(x, w, lam, u, dirs, y=s["y"], workspace=s["ws"])
    norm = kind == "train_norm"
    fwd = gspn.scan_fwd_norm_train if norm else gspn.scan_fwd_train
    bwd = gspn.scan_bwd_norm_reserve if norm else gspn.scan_bwd_reserve
    y, reserve = fwd(x, w, lam, u, dirs, y=s["y"], reserve=s["reserve"], workspace=s["ws"])
    dx, dw, dlam, du = bwd(x, w, lam, u, s["dy"], reserve, dirs, out=s["grads"],
                           workspace=s["ws"])
    return {"y": y, "dx": dx, "dw": dw, "dlam": dlam, "du": du}


def work(c):
    """Each input read once, each output written once; multiply-adds as two."""
    N, C, D = c["B"] * c["H"] * c["W"], c["C"], len(_bits(c["dirs"]))
    if c["kind"] == "latent":
        Cc = c["Cc"]
        return {"bytes": 2 * (2 * N * C + 2 * C * Cc + 5 * D * Cc * Cc),
                "flops": 2 * N * (2 * C * Cc + 5 * D * Cc * Cc) + 10 * N * Cc * D}
    es, G = (4 if c["dtype"] == "f32" else 2), c["G"]
    nbytes = es * N * (C * (2 + 2 * D) + 3 * G * D)
    flops = 10 * N * C * D
    if c["kind"].startswith("train"):
        nbytes += es * N * (C * (3 + 4 * D) + 6 * G * D)
        flops += 30 * N * C * D
    return {"bytes": nbytes, "flops": flops}


def tolerance(c):
    if c["dtype"] == "f32":
        return {"rel": 2e-6}
    if c["kind"] == "latent":
        return {"rel": 2e-2}
    return {"rel": 8e-3}


# ---------------------------------------------------------------------------
# the same results in 64 bits, by plain torch
# ---------------------------------------------------------------------------

def _frame(t, bit):
    """Pixel-major [..., H, W] as [..., L, P] in scan order of a direction
    (a view up to a flip; its own inverse up to the transpose)."""
    if bit >= 4:
        t = t.transpose(-1, -2)
    return t.flip(-2) if bit in (2, 8) else t


def _unframe(t, bit):
    if bit in (2, 8):
        t = t.flip(-2)
    return t.transpose(-1, -2) if bit >= 4 else t


def _shift(h, k):
    """h[..., j + k - 1], 0 off the line."""
    if k == 1:
        return h
    out = torch.zeros_like(h)
    if k == 0:
        out[..., 1:] = h[..., :-1]
    else:
        out[..., :-1] = h[..., 1:]
    return out


def _mask_taps(w):
    """[B, G, 3, L, P] in a direction's frame: taps off the grid set to 0."""
    w = w.clone()
    w[:, :, 0, :, 0] = 0
    w[:, :, 2, :, -1] = 0
    return w


def _normalize(logits):
    """Row-stochastic weights of framed logits, and the sigmoids on the grid."""
    s = _mask_taps(logits.sigmoid())
    return s / s.sum(2, keepdim=True).clamp_min(1e-30), s


def _exact_scan(x, w, lam, u, dy, dirs, norm):
    B, C, H, W = x.shape
    G = w.shape[2]
    cpg = C // G
    y = torch.zeros_like(x)
    dx = dw = dlam = du = None
    if dy is not None:
        dx, dw, dlam, du = (torch.zeros_like(t) for t in (x, w, lam, u))
    for s, bit in enumerate(_bits(dirs)):
        def channels(t):                    # [B, G, cpg, L, P]
            f = _frame(t, bit)
            return f.reshape((B, G, cpg) + f.shape[-2:])
        raw = _frame(w[s], bit)
        wf, sig = _normalize(raw) if norm else (_mask_taps(raw), None)
        xf, lf, uf = channels(x), channels(lam[s]), channels(u[s])
        L = xf.shape[-2]
        hs = []
        for i in range(L):
            h = lf[..., i, :] * xf[..., i, :]
            if i:
                for k in range(3):
                    h += wf[:, :, None, k, i] * _shift(hs[-1], k)
            hs.append(h)
        hf = torch.stack(hs, -2)
        del hs
        back = (lambda t: _unframe(t.flatten(1, 2), bit))   # noqa: E731
        y += back(uf * hf)
        if dy is None:
            continue
        gf = channels(dy)
        a, dwf = None, torch.zeros_like(wf)
        dxf, dlf = torch.empty_like(hf), torch.empty_like(hf)
        for i in range(L - 1, -1, -1):
            an = uf[..., i, :] * gf[..., i, :]
            if a is not None:
                for k in range(3):
                    an += _shift(wf[:, :, None, k, i + 1] * a, 2 - k)
            a = an
            dlf[..., i, :] = a * xf[..., i, :]
            dxf[..., i, :] = a * lf[..., i, :]
            if i:
                for k in range(3):
                    dwf[:, :, k, i] = (a * _shift(hf[..., i - 1, :], k)).sum(2)
        if norm:
            S = sig.sum(2, keepdim=True).clamp_min(1e-30)
            dwf = sig * (1 - sig) * (dwf - (wf * dwf).sum(2, keepdim=True)) / S
        dx += back(dxf)
        dlam[s] = back(dlf)
        du[s] = back(gf * hf)
        dw[s] = _unframe(_mask_taps(dwf), bit)
    if dy is None:
        return y
    return {"y": y, "dx": dx, "dw": dw, "dlam": dlam, "du": du}


def exact(c, seed):
    if c["kind"] == "latent":
        t = _draw_latent(c, seed)
        y = torch.empty(t["x"].shape, dtype=torch.float64, device="cuda")
        p = {k: t[k].double() for k in ("p_down", "l_u", "l_lam", "l_w", "p_up")}
        Cc, H, W = c["Cc"], c["H"], c["W"]
        for b in range(c["B"]):
            xc = p["p_down"] @ t["x"][b].double().flatten(1)
            lam = torch.stack([m @ xc for m in p["l_lam"]]).view(-1, 1, Cc, H, W)
            u = torch.stack([m @ xc for m in p["l_u"]]).view(-1, 1, Cc, H, W)
            w = torch.stack([m.flatten(0, 1) @ xc for m in p["l_w"]]).view(-1, 1, Cc, 3, H, W)
            yc = _exact_scan(xc.view(1, Cc, H, W), w, lam, u, None, c["dirs"], True)
            y[b] = (p["p_up"] @ yc.view(Cc, H * W)).view(-1, H, W)
        return y
    t = {k: v.double() for k, v in _draw_scan(c, seed).items()}
    return _exact_scan(t["x"], t["w"], t["lam"], t["u"], t.get("dy"), c["dirs"],
                       c["kind"].endswith("norm"))
