"""The work this framework is timed on: whole frames, reads of long banks, the
layer stack, the step after the mask decoder and the bare attention, over the
sizes, types and options they run with.

A case is a dict of plain values.  `kind` says which call it makes:

  frames   a looped clip: one rs3_frame call (select, read, write) per frame.
           The clip's frames follow each other in a ring bank that is already
           full of them, so every pass meets the bank in the same state.
  read     select and read one frame against a full bank, nothing written.
  stack    select and run the L-layer memory-attention stack on the kept rows.
  close    the closure of the decoded masks and the palette.
  attend   the attention on tensors that are already projected (the dense,
           unpruned layer a user compares the sparse readout with).

Tokens are Gaussian, masks are rotated ellipses, and W_q is scaled so that a
query attends to a few keys, as trained memory attention does.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_2608_22526_amd as rs3
from paper_2608_22526_amd.session import Session

LOGIT_SCALE = 3.0   # standard deviation of the attention logits
R_S, C_BOX = 4, 14  # prior radius and box cap, the defaults of the method
LN_EPS = 1e-5


# ---- the cases ---------------------------------------------------------------
def _frames(name, m, n, C, H, d_kv, n_obj, f_max, loop, rho, lo, hi, kind="frames", s=1, dtype="bf16", absorb=False,
            rope=0.0, shared_x=True, union=True, full_prior=False, dense=False):
    return dict(name=name, kind=kind, m=m, n=n, s=s, C=C, H=H, d_kv=d_kv, dtype=dtype, n_obj=n_obj, shared_x=shared_x,
                union=union, f_max=f_max, loop=loop, rho=rho, lo=lo, hi=hi, absorb=absorb, rope=rope,
                full_prior=full_prior, dense=dense)


def listed():
    return [
        # the smallest call: the fp32 configuration on a 16x16 grid, two-frame
        # bank; a frame is launch and memory latency.  The fp32 cases keep
        # every token of a written frame (sparse reads of a dense memory)
        _frames("tiny_f32", 16, 16, 64, 1, 32, 1, 2, 1, 0.25, 0.30, 0.30, dtype="f32", dense=True),
        # fp32 at a grid of 32x32 and model width 256 in four heads, for users
        # who need 1e-4 agreement
        _frames("f32_4x64", 32, 32, 256, 4, 64, 1, 4, 3, 0.25, 0.15, 0.40, dtype="f32", dense=True),
        # the benchmark's workload: one object, 64x64 grid, one pinned and six
        # recent frames, the single head folded onto the raw bank rows
        _frames("sam2_single", 64, 64, 256, 1, 64, 1, 7, 6, 0.22, 0.10, 0.40, absorb=True),
        # the same with rotary positions, which need the projected bank and a
        # head of 256
        _frames("sam2_rope", 64, 64, 256, 1, 64, 1, 7, 6, 0.22, 0.10, 0.40, rope=10000.0),
        # eight objects on one shared grid, a bank and a keep-set each
        _frames("multi_obj8", 64, 64, 256, 1, 64, 8, 7, 6, 0.22, 0.05, 0.25, absorb=True, union=False),
        # a serving batch: 64 objects, each with its own grid
        _frames("objects64", 64, 64, 256, 1, 64, 64, 7, 2, 0.22, 0.05, 0.25, absorb=True, union=False, shared_x=False),
        # a ragged 480p grid at stride 16 with three objects in one keep-set,
        # four projected heads of 64
        _frames("video_480p", 30, 54, 256, 4, 64, 3, 6, 5, 0.30, 0.05, 0.25, s=16),
        # a long video: one read against 64 frames of memory
        _frames("long_video", 64, 64, 256, 1, 64, 1, 64, 63, 0.30, 0.10, 0.30, kind="read", absorb=True),
        # high resolution: 128x128 grid, eight heads of 32, 16-frame bank, the
        # whole grid as prior; the largest
        _frames("highres", 128, 128, 256, 8, 64, 1, 16, 5, 0.25, 0.05, 0.50, full_prior=True),
        # the four-layer stack on the kept rows of the benchmark's grid
        dict(name="stack4", kind="stack", m=64, n=64, f_max=7, rho=0.22, lo=0.10, hi=0.40, layers=4, H_s=1, F=2048),
        # eight decoded masks at 1024x1024, closed with the method's 9x9 square
        dict(name="close_1024", kind="close", n_obj=8, H=1024, W=1024, k=9, dtype="bf16"),
        # the dense layer of the 64x64 grid: every query against seven whole
        # frames, two heads of 128
        dict(name="attend_dense", kind="attend", n_q=4096, n_kv=28672, H=2, d_h=128, dtype="bf16"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_frames(rng, kind):
    dtype = "f32" if kind == "frames" and rng.random() < 0.2 else "bf16"
    top = 32 if dtype == "f32" else 128
    m = _log_int(rng, 12, top)
    n = max(12, min(top, int(round(m * rng.uniform(0.6, 1.8)))))
    if dtype == "f32":
        m, n = 8 * ((m + 7) // 8), 8 * ((n + 7) // 8)
    absorb = dtype == "bf16" and rng.random() < 0.5
    if absorb:
        C, H, d_kv = 256, 1, 64
    else:
        C, H = rng.choice([(64, 1), (64, 2), (256, 1), (256, 2), (256, 4), (256, 8)])
        d_kv = rng.choice([32, 64])
    n_obj = 1 if rng.random() < 0.4 else _log_int(rng, 2, 64 if absorb else 8)
    shared = rng.random() < 0.6
    union = n_obj == 1 or (shared and rng.random() < 0.4)
    if kind == "read":
        f_max, loop = _log_int(rng, 2, 64), 0
        loop = f_max - 1
    else:
        loop = rng.choice([1, 2, 3, 5, 6])
        f_max = 1 + loop * rng.choice([1, 2, 3])
    lo = rng.uniform(0.05, 0.30)
    rope = 10000.0 if not absorb and rng.random() < 0.3 else 0.0
    return dict(_frames("", m, n, C, H, d_kv, n_obj, f_max, loop, round(rng.uniform(0.1, 0.5), 3), round(lo, 3),
                        round(lo + rng.uniform(0.0, 0.2), 3), kind=kind, s=rng.choice([1, 1, 4, 16]), dtype=dtype,
                        absorb=absorb, rope=rope, shared_x=shared, union=union, full_prior=rng.random() < 0.2,
                        dense=dtype == "f32" or rng.random() < 0.1))


def _draw_one(rng):
    kind = rng.choice(["frames", "frames", "frames", "read", "read", "stack", "close", "attend"])
    if kind in ("frames", "read"):
        c = _draw_frames(rng, kind)
    elif kind == "stack":
        m = _log_int(rng, 16, 64)
        lo = round(rng.uniform(0.10, 0.30), 3)
        c = dict(kind="stack", m=m, n=max(16, min(64, int(round(m * rng.uniform(0.6, 1.8))))), f_max=rng.randint(2, 8),
                 rho=round(rng.uniform(0.1, 0.5), 3), lo=lo, hi=round(lo + 0.1, 3), layers=rng.randint(1, 4),
                 H_s=rng.choice([1, 2, 4, 8]), F=rng.choice([512, 1024, 2048]))
    elif kind == "close":
        H = _log_int(rng, 120, 1100)
        c = dict(kind="close", n_obj=_log_int(rng, 1, 8), H=H, W=min(2000, int(round(H * rng.uniform(0.7, 1.9)))),
                 k=rng.choice([3, 5, 9, 9, 9, 15]), dtype=rng.choice(["bf16", "bf16", "f32"]))
    else:
        H, d_h = rng.choice([(1, 64), (1, 256), (2, 128), (4, 64), (8, 32), (8, 64), (8, 128)])
        f32 = d_h <= 64 and rng.random() < 0.25
        c = dict(kind="attend", n_q=_log_int(rng, 64, 512 if f32 else 4096),
                 n_kv=_log_int(rng, 64, 1024 if f32 else 28672), H=H, d_h=d_h, dtype="f32" if f32 else "bf16")
    c.pop("name", None)
    return c


def draw(rng):
    """One more case of the same ranges, no larger than the largest listed."""
    every = {c["name"]: work(c) for c in listed()}
    most = max(w["bytes"] for w in every.values())
    while True:
        c = _draw_one(rng)
        w = work(c)
        # fp32 runs at a tenth of the bf16 rate, and the scan of pixel masks
        # at a fraction of the token rate: both stay near their listed cases
        flops = every["f32_4x64" if c.get("dtype") == "f32" else "highres"]["flops"]
        if w["bytes"] <= most and w["flops"] <= flops and _pixels(c) <= 8 << 20:
            return c


# ---- inputs ------------------------------------------------------------------
def _gen(seed, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1000003 + stream * 7919) % (1 << 62))
    return g


def _normal(seed, stream, shape, dtype):
    t = torch.randn(shape, generator=_gen(seed, stream), device="cuda", dtype=torch.float32)
    return t.to(torch.bfloat16) if dtype == "bf16" else t


def _ellipses(seed, stream, count, H, W, lo, hi):
    """`count` rotated ellipses, uint8 [count][H][W], of area fraction lo..hi."""
    r = np.random.default_rng([seed, stream])
    p = []
    for _ in range(count):
        area, kappa, th = r.uniform(lo, hi), math.exp(r.uniform(-math.log(2.0), math.log(2.0))), r.uniform(0.0, math.pi)
        a, b = math.sqrt(area * H * W * kappa / math.pi), math.sqrt(area * H * W / (math.pi * kappa))
        ex = math.hypot(a * math.cos(th), b * math.sin(th))
        ey = math.hypot(a * math.sin(th), b * math.cos(th))
        cx = r.uniform(ex, W - ex) if 2 * ex < W else W / 2
        cy = r.uniform(ey, H - ey) if 2 * ey < H else H / 2
        p.append((cy, cx, a, b, math.cos(th), math.sin(th)))
    q = torch.tensor(p, dtype=torch.float32, device="cuda").T.reshape(6, count, 1, 1)
    dy = torch.arange(H, device="cuda").reshape(1, H, 1) + 0.5 - q[0]
    dx = torch.arange(W, device="cuda").reshape(1, 1, W) + 0.5 - q[1]
    u, v = (dx * q[4] + dy * q[5]) / q[2], (dy * q[4] - dx * q[5]) / q[3]
    return (u * u + v * v <= 1.0).to(torch.uint8)


def _host(w, dtype):
    """float32 weights as the host array a layer takes (uint16 = bf16 bits)."""
    t = torch.from_numpy(w)
    return t.to(torch.bfloat16).view(torch.int16).numpy().view(np.uint16) if dtype == "bf16" else w


def _wide(a):
    """A host weight array in 64 bits on the GPU."""
    t = torch.from_numpy(a.view(np.int16)).view(torch.bfloat16) if a.dtype == np.uint16 else torch.from_numpy(a)
    return t.to("cuda", torch.float64)


def _matrix(r, rows, cols, scale=1.0):
    return r.standard_normal((rows, cols), dtype=np.float32) * np.float32(scale / math.sqrt(rows))


def _layer_weights(seed, C, d_kv, dtype):
    r = np.random.default_rng([seed, 6])
    shapes = (("Wq", C, LOGIT_SCALE), ("Wk", d_kv, 1.0), ("Wv", d_kv, 1.0), ("Wo", C, 1.0))
    return SimpleNamespace(**{k: _host(_matrix(r, rows, C, sc), dtype) for k, rows, sc in shapes})


def _memory(c, seed, frames, d_kv, dtype, n_obj, s):
    """Memory tokens and masks of `frames` frames and of the pinned one."""
    mn = c["m"] * c["n"]
    K = _normal(seed, 2, (frames + 1, n_obj, mn, d_kv), dtype)
    V = _normal(seed, 3, (frames + 1, n_obj, mn, d_kv), dtype)
    masks = _ellipses(seed, 4, (frames + 1) * n_obj, c["m"] * s, c["n"] * s, c["lo"], c["hi"])
    return K, V, masks.reshape(frames + 1, n_obj, c["m"] * s, c["n"] * s)


def _clip(c, seed):
    """Everything a frames or read case works on (frame `loop` is pinned)."""
    mn, L = c["m"] * c["n"], c["loop"]
    K, V, masks = _memory(c, seed, L, c["d_kv"], c["dtype"], c["n_obj"], c["s"])
    n_x = 1 if c["shared_x"] else c["n_obj"]
    frames = L if c["kind"] == "frames" else 1
    X = _normal(seed, 1, (frames, n_x, mn, c["C"]), c["dtype"])
    every = torch.ones_like(masks)
    read, masks = every if c["full_prior"] else masks, every if c["dense"] else masks
    return SimpleNamespace(X=X, K=K, V=V, masks=masks, read=read, W=_layer_weights(seed, c["C"], c["d_kv"], c["dtype"]))


def _budget(c):
    return int(math.floor(c["rho"] * c["m"] * c["n"]))


def _stack_weights(seed, layers, C, d_kv, F):
    out = []
    for i in range(layers):
        r = np.random.default_rng([seed, 8, i])
        shapes = {"Wqs": (C, C, LOGIT_SCALE), "Wks": (C, C, 1), "Wvs": (C, C, 1), "Wos": (C, C, 0.5),
                  "Wq": (C, C, LOGIT_SCALE), "Wk": (d_kv, C, 1), "Wv": (d_kv, C, 1), "Wo": (C, C, 0.5),
                  "W1": (C, F, 1), "W2": (F, C, 0.5)}
        w = {k: _host(_matrix(r, a, b, sc), "bf16") for k, (a, b, sc) in shapes.items()}
        for k in ("ln1", "ln2", "ln3"):
            w[k + "_g"] = 1.0 + 0.1 * r.standard_normal(C).astype(np.float32)
            w[k + "_b"] = 0.1 * r.standard_normal(C).astype(np.float32)
        out.append(w)
    return out


def _stack_inputs(c, seed):
    K, V, masks = _memory(c, seed, c["f_max"] - 1, 64, "bf16", 1, 1)
    X = _normal(seed, 1, (1, c["m"] * c["n"], 256), "bf16")
    return SimpleNamespace(X=X, K=K, V=V, masks=masks, W=_layer_weights(seed, 256, 64, "bf16"),
                           layers=_stack_weights(seed, c["layers"], 256, 64, c["F"]))


def _logits(c, seed):
    """Decoder logits: positive inside an ellipse, with single-pixel holes."""
    inside = _ellipses(seed, 4, c["n_obj"], c["H"], c["W"], 0.05, 0.30).bool()
    mag = (2.0 + _normal(seed, 1, inside.shape, "f32")).abs()
    holes = torch.rand(inside.shape, generator=_gen(seed, 5), device="cuda") < 0.04
    x = torch.where(inside & ~holes, mag, -mag)
    return x.to(torch.bfloat16) if c["dtype"] == "bf16" else x


def _qkv(c, seed):
    q, k, v = (_normal(seed, i, (rows, c["H"], c["d_h"]), "f32") for i, rows in ((1, c["n_q"]), (2, c["n_kv"]), (3, c["n_kv"])))
    q = q * LOGIT_SCALE
    return tuple(t.to(torch.bfloat16) if c["dtype"] == "bf16" else t for t in (q, k, v))


# ---- the framework's calls -----------------------------------------------------
def _session(c, W):
    mn = c["m"] * c["n"]
    return Session(m=c["m"], n=c["n"], s=c["s"], C=c["C"], H=c["H"], d_kv=c["d_kv"], dtype=c["dtype"],
                   n_obj=c["n_obj"], shared_x=c["shared_x"], union_objects=c["union"], cap=(c["f_max"] + 1) * mn,
                   f_max=c["f_max"], n_pin=1, weights=W, r_s=R_S, c=C_BOX, max_sel=_budget(c), absorb=c["absorb"],
                   rope_theta=c["rope"] or None)


def prepare(case, seed):
    c, kind = case, case["kind"]
    if kind in ("frames", "read"):
        d = _clip(c, seed)
        sess = _session(c, d.W)
        L = c["loop"]
        sess.commit(d.K[L], d.V[L], d.masks[L], 0, True)
        for t in range(c["f_max"] - 1):
            sess.commit(d.K[t % L], d.V[t % L], d.masks[t % L], t + 1, False)
        Y = torch.empty((len(d.X), c["n_obj"], c["m"] * c["n"], c["C"]), dtype=d.X.dtype, device="cuda")
        return SimpleNamespace(c=c, d=d, sess=sess, Y=Y, t=c["f_max"], k=[_budget(c)] * sess.n_groups)
    if kind == "stack":
        d = _stack_inputs(c, seed)
        sc = dict(c, s=1, C=256, H=1, d_kv=64, dtype="bf16", n_obj=1, shared_x=True, union=True, absorb=True, rope=0.0)
        sess = _session(sc, d.W)
        for t in range(c["f_max"]):
            j = (t - 1) % c["f_max"]
            sess.commit(d.K[j], d.V[j], d.masks[j], t, t == 0)
        st = rs3.Stack(d.layers, C=256, H_s=c["H_s"], d_kv=64, F=c["F"])
        ws = torch.zeros(st.workspace_size(_budget(c)), dtype=torch.uint8, device="cuda")
        return SimpleNamespace(c=c, d=d, sess=sess, st=st, ws=ws, Y=torch.empty_like(d.X), k=[_budget(c)])
    if kind == "close":
        n, H, W = c["n_obj"], c["H"], c["W"]
        return SimpleNamespace(c=c, x=_logits(c, seed), dt=rs3.RS3_BF16 if c["dtype"] == "bf16" else rs3.RS3_F32,
                               closed=torch.empty((n, H, W), dtype=torch.uint8, device="cuda"),
                               pal=torch.empty((H, W), dtype=torch.uint8, device="cuda"),
                               ws=torch.zeros(rs3.close_workspace_size(n, H, W), dtype=torch.uint8, device="cuda"))
    q, k, v = _qkv(c, seed)
    dt = rs3.RS3_BF16 if c["dtype"] == "bf16" else rs3.RS3_F32
    ws = rs3.attend_workspace_size(c["n_q"], c["n_kv"], c["H"], c["d_h"], dt)
    return SimpleNamespace(c=c, q=q, k=k, v=v, dt=dt, ws=torch.zeros(max(ws, 256), dtype=torch.uint8, device="cuda"),
                           O=torch.empty((c["n_q"], c["H"], c["d_h"]), dtype=torch.float32, device="cuda"))


def run(state):
    s, c = state, state.c
    if c["kind"] == "frames":
        d, L = s.d, c["loop"]
        for j in range(L):
            s.sess.frame(d.read[j - 1 if j else L - 1], d.X[j], s.k, s.Y[j], d.K[j], d.V[j], d.masks[j], s.t, False)
            s.t += 1
        return {"Y": list(s.Y), "sel_count": s.sess.sel_count, "kept_count": s.sess.kept_count}
    if c["kind"] == "read":
        s.sess.select(s.d.read[c["loop"] - 1], s.d.X[0], s.k)
        s.sess.readout(s.d.X[0], s.Y[0])
        return {"Y": s.Y[0], "sel_count": s.sess.sel_count}
    if c["kind"] == "stack":
        s.sess.select(s.d.masks[c["f_max"] - 2], s.d.X, s.k)
        s.st.readout(s.sess.grid, s.d.X, s.sess.banks[0], s.sess.sel_idx, s.sess.sel_count, s.k[0], s.Y, ws=s.ws)
        return {"Y": s.Y, "sel_count": s.sess.sel_count}
    if c["kind"] == "close":
        rs3.close_masks(c["n_obj"], c["H"], c["W"], s.x, s.dt, c["k"], s.closed, s.pal, s.ws)
        return {"closed": s.closed, "palette": s.pal}
    rs3.attend(s.q, s.k, s.v, c["n_q"], c["n_kv"], c["H"], c["d_h"], s.dt, s.O, s.ws)
    return {"O": s.O}


# ---- what a pass cannot do without ----------------------------------------------
def _pixels(c):
    """Mask pixels whose box a pass finds (masks finer than the grid)."""
    if c["kind"] not in ("frames", "read") or c["s"] == 1:
        return 0
    return (c["loop"] if c["kind"] == "frames" else 1) * c["n_obj"] * c["m"] * c["n"] * c["s"] ** 2


def _grown(cells, mn):
    """About how many cells an ellipse of `cells` cells has after the prior's
    dilation (a square of radius R_S)."""
    return min(mn, cells + 2.2 * R_S * math.sqrt(math.pi * cells) + 4 * R_S * R_S)


def work(case):
    c = case
    b = 4 if c.get("dtype") == "f32" else 2
    if c["kind"] == "close":
        px = c["n_obj"] * c["H"] * c["W"]
        return {"bytes": px * (b + 1) + c["H"] * c["W"], "flops": 0}
    if c["kind"] == "attend":
        D = c["H"] * c["d_h"]
        return {"bytes": (c["n_q"] + 2 * c["n_kv"]) * D * b + c["n_q"] * D * 4, "flops": 4 * c["n_q"] * c["n_kv"] * D}
    mn = c["m"] * c["n"]
    area = 0.5 * (c["lo"] + c["hi"]) * mn
    if c["kind"] == "stack":
        nq = min(_budget(c), _grown(area, mn))
        N, F = area * c["f_max"], c["F"]
        flops = c["layers"] * nq * (8 * 256 * 256 + 4 * 256 * nq + 4 * 64 * N + 4 * 256 * 64 + 4 * 256 * F)
        weights = c["layers"] * 2 * (4 * 256 * 256 + 2 * 256 * 64 + 2 * 256 * F)
        return {"bytes": 2 * mn * 256 * 2 + mn + N * 2 * 64 * 2 + weights, "flops": flops + 2 * mn * 256}
    n_obj, C, d_kv = c["n_obj"], c["C"], c["d_kv"]
    Da = d_kv if c["absorb"] else C
    prior = mn if c["full_prior"] else _grown(area * (n_obj if c["union"] else 1) ** 0.8, mn)
    kept = mn if c["dense"] else area
    nq, N = min(_budget(c), prior), kept * c["f_max"]
    n_x = 1 if c["shared_x"] else n_obj
    flops = n_obj * nq * (4 * N * Da + 4 * C * Da) + 2 * n_x * mn * C
    # tokens in and out, masks, resident keys and values, Wq and Wo
    data = (n_x + n_obj) * mn * C * b + n_obj * mn * c["s"] ** 2 + n_obj * N * 2 * Da * b + 2 * C * Da * b
    if c["kind"] == "frames":   # the write: mask, rows in, raw and attention rows out
        data += n_obj * (mn + kept * (4 * d_kv + 2 * Da) * b)
        flops += 0 if c["absorb"] else n_obj * kept * 4 * d_kv * C
    frames = c["loop"] if c["kind"] == "frames" else 1
    return {"bytes": frames * data, "flops": frames * flops}


def tolerance(case):
    """Largest differences of another implementation at the same precision:
    about four times what another order of the sums (other key splits), or
    the distance to exact() where there is no such switch, shows."""
    if case["kind"] == "close":
        return "exact"
    if case.get("dtype") == "f32":
        return {"rel": 2e-6, "max": 3e-5}
    if case["kind"] == "attend":
        return {"rel": 1.6e-2, "max": 0.25}
    if case["kind"] == "stack":
        return {"rel": 1e-2, "max": 0.15}
    return {"rel": 6e-3, "max": 0.1}


# ---- the same in 64 bits ----------------------------------------------------------
def _axial(c, d_h, cells):
    """Axial rotary factors, complex [len(cells)][d_h/2]."""
    p = torch.arange(d_h // 4, device="cuda", dtype=torch.float64)
    freq = c["rope"] ** (-4.0 * p / d_h)
    col, row = (cells % c["n"]).double(), (cells // c["n"]).double()
    ang = torch.cat([col[:, None] * freq, row[:, None] * freq], 1)
    return torch.polar(torch.ones_like(ang), ang)


def _turn(x, H, f):
    """x [rows][H*d_h] with each head's channel pairs turned by f[row]."""
    z = torch.view_as_complex(x.reshape(x.shape[0], H, -1, 2).contiguous()) * f[:, None, :]
    return torch.view_as_real(z).reshape(x.shape)


def _attention(q, k, v, H, bias=None):
    """softmax(q k^T / sqrt(d_h) + bias) v per head, in row blocks."""
    d = q.shape[1] // H
    out = torch.zeros_like(q)
    step = max(16, (1 << 28) // max(1, k.shape[0]) // 8)
    for h in range(H):
        cols = slice(h * d, (h + 1) * d)
        kt, vh = k[:, cols].T.contiguous(), v[:, cols].contiguous()
        for r in range(0, q.shape[0], step):
            s = q[r:r + step, cols] @ kt / math.sqrt(d)
            out[r:r + step, cols] = torch.softmax(s if bias is None else s + bias, 1) @ vh
    return out


def _select(c, read, X, k, union):
    """The kept cells of each group, ascending: inside the dilated masks the k
    of largest energy, ties to the lower cell."""
    s = c.get("s", 1)
    cells = (read[:, ::s, ::s] != 0).float()[:, None]
    prior = torch.nn.functional.max_pool2d(cells, 2 * R_S + 1, 1, R_S)[:, 0].reshape(cells.shape[0], -1) > 0
    if union:
        prior = prior.any(0, keepdim=True)
    out = []
    for g in range(prior.shape[0]):
        e = X[0 if X.shape[0] == 1 else g].double().square().sum(1)
        cand = prior[g].nonzero()[:, 0]
        if len(cand) > k:
            cand = cand[torch.sort(e[cand], descending=True, stable=True)[1][:k]].sort()[0]
        out.append(cand)
    return out


def _kept(K, V, mask, s):
    cells = (mask[::s, ::s].reshape(-1) != 0).nonzero()[:, 0]
    return K[cells].double(), V[cells].double(), cells


def _exact_clip(c, seed):
    d = _clip(c, seed)
    W = {k: _wide(v) for k, v in vars(d.W).items()}
    L, H, s = c["loop"], c["H"], c["s"]
    d_h, rep = c["C"] // H, (c["f_max"] - 1) // L
    Y = []
    sel = []
    for j in range(len(d.X)):
        i = (j - 1) % L if c["kind"] == "frames" else L - 1
        sel.append(_select(c, d.read[i], d.X[j], _budget(c), c["union"]))
        Y.append(d.X[j].double().expand(c["n_obj"], -1, -1).clone())
    for o in range(c["n_obj"]):
        parts = [_kept(d.K[i, o], d.V[i, o], d.masks[i, o], s) for i in range(L + 1)]
        k, v, pos = (torch.cat([p[i] for p in parts]) for i in range(3))
        # a clip frame is in the bank `rep` times, the pinned one once
        bias = torch.full((len(pos),), math.log(rep), dtype=torch.float64, device="cuda")
        bias[len(pos) - len(parts[L][2]):] = 0.0
        k, v = k @ W["Wk"], v @ W["Wv"]
        if c["rope"]:
            k = _turn(k, H, _axial(c, d_h, pos))
        for j in range(len(d.X)):
            r = sel[j][0 if c["union"] else o]
            x = Y[j][o, r]
            q = x @ W["Wq"]
            if c["rope"]:
                q = _turn(q, H, _axial(c, d_h, r))
            Y[j][o, r] = x + _attention(q, k, v, H, bias) @ W["Wo"]
    if c["kind"] == "read":
        return {"Y": Y[0], "sel_count": None}
    return {"Y": Y, "sel_count": None, "kept_count": None}


def _norm(z, g, b):
    z = z - z.mean(1, keepdim=True)
    z = z / torch.sqrt(z.square().mean(1, keepdim=True) + LN_EPS)
    return z * torch.from_numpy(g).to(z) + torch.from_numpy(b).to(z)


def _exact_stack(c, seed):
    d = _stack_inputs(c, seed)
    rows = _select(c, d.masks[c["f_max"] - 2], d.X, _budget(c), True)[0]
    parts = [_kept(d.K[i, 0], d.V[i, 0], d.masks[i, 0], 1) for i in range(c["f_max"])]
    k, v = (torch.cat([p[i] for p in parts]) for i in (0, 1))
    Y = d.X.double()
    z = Y[0, rows]
    for host in d.layers:
        w = {n: _wide(a) for n, a in host.items() if n.startswith("W")}
        a = _norm(z, host["ln1_g"], host["ln1_b"])
        z = z + _attention(a @ w["Wqs"], a @ w["Wks"], a @ w["Wvs"], c["H_s"]) @ w["Wos"]
        a = _norm(z, host["ln2_g"], host["ln2_b"])
        z = z + _attention(a @ w["Wq"], k @ w["Wk"], v @ w["Wv"], 1) @ w["Wo"]
        a = _norm(z, host["ln3_g"], host["ln3_b"])
        z = z + torch.relu(a @ w["W1"]) @ w["W2"]
    Y[0, rows] = z
    return {"Y": Y, "sel_count": None}


def exact(case, seed):
    """What run() returns, in 64 bits (None: bytes and counts)."""
    c = case
    if c["kind"] == "close":
        return None
    if c["kind"] == "stack":
        return _exact_stack(c, seed)
    if c["kind"] == "attend":
        q, k, v = (t.double().reshape(t.shape[0], -1) for t in _qkv(c, seed))
        return {"O": _attention(q, k, v, c["H"]).reshape(c["n_q"], c["H"], c["d_h"])}
    return _exact_clip(c, seed)
