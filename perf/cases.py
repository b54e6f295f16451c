"""The work that a MambaByte program has this library do, as cases that can be timed and checked.

A case is one layer's call, or the calls that a program makes together, through the package's public
entry points.  The sizes are those of the MambaByte layers (D = 2048, 3584 and 4608 channels, 16 states,
a convolution of 4 taps, 8,192-byte training contexts, 65,536-byte extrapolation, 16-byte drafts) and the
odd ones that byte prompts, drafts and other models bring: a prompt has any number of bytes.

kind      what it stands for
decode    one generated byte: conv1d_step, then scan_step, states updated in place
verify    a speculative verification: the drafted bytes scanned from the cached state, their top-3 check,
          and the state at the last accepted byte
prefill   a prompt or a long document: optionally the convolution, then the scan, with what decoding
          needs afterwards (h_last, the convolution's state)
conv      the convolution alone
train     forward and backward of the differentiable scan
"""
import math

import torch

import paper_2401_13660_amd as mb

N = 16          # states per channel
K = 4           # taps of the convolution
DEV = "cuda:0"
BETA = 3        # candidates a drafted byte may be among
MODEL_DIMS = (2048, 3584, 4608)


def listed():
    return [
        # one generated byte of one prompt: latency and launches
        dict(name="decode_b1", kind="decode", batch=1, dim=3584, dtype="bf16"),
        # one generated byte of a batch of prompts
        dict(name="decode_b32", kind="decode", batch=32, dim=3584, dtype="bf16"),
        # 16 drafted bytes for a batch of prompts
        dict(name="verify_b32_L16", kind="verify", batch=32, dim=3584, L=16, dtype="bf16", out="f32"),
        # drafts come in any number of bytes (three subwords)
        dict(name="verify_b8_L13", kind="verify", batch=8, dim=2048, L=13, dtype="bf16", out="bf16"),
        # a short prompt, of any number of bytes, into an empty cache
        dict(name="prompt_b1_L1013", kind="prefill", batch=1, dim=3584, L=1013, dtype="bf16", out="bf16",
             conv=True, h0=False, gate=True),
        # one full context into an empty cache
        dict(name="prefill_b1_L8192", kind="prefill", batch=1, dim=3584, L=8192, dtype="bf16", out="bf16",
             conv=True, h0=False, gate=True),
        # the 972M layer over a training batch's contexts, forward only (evaluation); fp32 out
        dict(name="scan_b4_L8192", kind="prefill", batch=4, dim=3584, L=8192, dtype="bf16", out="f32",
             conv=False, h0=False, gate=True),
        # the 1.6B layer over a 65,536-byte document
        dict(name="scan_b1_L65536", kind="prefill", batch=1, dim=4608, L=65536, dtype="bf16", out="f32",
             conv=False, h0=False, gate=True),
        # fp32 activations, a continued document of odd length, no gate
        dict(name="scan_f32_b2_L2047", kind="prefill", batch=2, dim=2048, L=2047, dtype="f32", out="f32",
             conv=False, h0=True, gate=False),
        # the 972M layer's convolution
        dict(name="conv_b4_L8192", kind="conv", batch=4, dim=3584, L=8192, dtype="bf16"),
        # one layer's share of a training step
        dict(name="train_b4_L8192", kind="train", batch=4, dim=3584, L=8192, dtype="bf16"),
        # fine-tuning in fp32 on short texts with a small model
        dict(name="train_f32_b2_L1024", kind="train", batch=2, dim=1536, L=1024, dtype="f32"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _dim(rng):
    """A model's width, or any other."""
    return rng.choice(MODEL_DIMS) if rng.random() < 0.5 else min(4608, max(256, _log(rng, 256, 4608)))


def draw(rng):
    kind = rng.choice(("decode", "verify", "prefill", "prefill", "conv", "train"))
    dtype = "f32" if rng.random() < 0.25 else "bf16"
    c = dict(kind=kind, dim=_dim(rng), dtype=dtype)
    if kind == "decode":
        c["batch"] = _log(rng, 1, 64)
        return c
    if kind == "verify":
        c["batch"], c["L"] = _log(rng, 1, 32), rng.randint(4, 40)
        c["out"] = "f32" if dtype == "f32" else rng.choice(("f32", "bf16"))
        return c
    c["batch"] = rng.choice((1, 1, 2, 3, 4))
    if kind == "train":
        c["L"] = 16 * min(_log(rng, 16, 512), 4 * 3584 * 512 // (c["batch"] * c["dim"]))
        return c
    # half of the lengths are whole contexts, half are whatever a document has
    L = _log(rng, 64, 65536)
    L = min(L, (4 * 3584 * 8192) // (c["batch"] * c["dim"]))
    c["L"] = max(64, L // 64 * 64) if rng.random() < 0.5 else L
    if kind == "prefill":
        c["out"] = "f32" if dtype == "f32" else rng.choice(("f32", "bf16"))
        c["conv"] = rng.random() < 0.5
        c["h0"] = rng.random() < 0.4
        c["gate"] = rng.random() < 0.8
    return c


# ---- inputs -------------------------------------------------------------------

_DT = {"bf16": torch.bfloat16, "f32": torch.float32}


class _Draws:
    """Seeded draws on the GPU, in the order asked for."""

    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(seed)

    def normal(self, *shape, dtype=torch.float32, scale=1.0):
        x = torch.randn(shape, generator=self.g, device=DEV)
        return (x * scale if scale != 1.0 else x).to(dtype)

    def uniform(self, lo, hi, *shape):
        return torch.rand(shape, generator=self.g, device=DEV) * (hi - lo) + lo


def _layer(r, dim):
    """A layer's weights: A around -(n + 1) as training leaves it, softplus(dt_bias) in [1e-3, 0.1]."""
    n = torch.arange(1, N + 1, device=DEV, dtype=torch.float32)
    dt = r.uniform(1e-3, 0.1, dim)
    b = 1.0 / math.sqrt(K)
    return dict(A=-(n * torch.exp(r.normal(dim, N, scale=0.25))).contiguous(), dt_bias=torch.log(torch.expm1(dt)),
                D=r.uniform(0.5, 1.5, dim), w=r.uniform(-b, b, dim, K), bias=r.uniform(-b, b, dim))


def prepare(case, seed):
    r = _Draws(seed)
    b, d, act = case["batch"], case["dim"], _DT[case["dtype"]]
    kind, L = case["kind"], case.get("L", 1)
    s = dict(case=case, **_layer(r, d))
    if kind == "decode":
        s.update(x=r.normal(b, d, dtype=act), delta=r.normal(b, d, dtype=act), z=r.normal(b, d, dtype=act),
                 B=r.normal(b, N, dtype=act), C=r.normal(b, N, dtype=act), h=r.normal(b, d, N, scale=0.1),
                 conv_state=r.normal(b, d, K - 1, dtype=act).float())
        return s
    if kind == "conv":
        s["x"] = r.normal(b, d, L, dtype=act)
        return s
    conv = kind == "prefill" and case["conv"]
    gate = kind != "prefill" or case["gate"]
    s["x" if conv else "u"] = r.normal(b, d, L, dtype=act)
    s.update(delta=r.normal(b, d, L, dtype=act), B=r.normal(b, N, L, dtype=act), C=r.normal(b, N, L, dtype=act),
             z=r.normal(b, d, L, dtype=act) if gate else None, h0=None)
    if kind == "verify" or (kind == "prefill" and case["h0"]):
        s["h0"] = r.normal(b, d, N, scale=0.1)
    if kind == "verify":
        s["logits"] = r.normal(b, L, 256, scale=2.0)
        best = s["logits"].argmax(-1)
        other = torch.randint(0, 256, (b, L), generator=r.g, device=DEV)
        keep = torch.rand((b, L), generator=r.g, device=DEV) < 0.93     # most drafted bytes pass
        s["draft"] = torch.where(keep, best, other).to(torch.int32).contiguous()
    if kind == "train":
        s["dy"] = r.normal(b, d, L, dtype=act)
        for k in ("u", "delta", "A", "B", "C", "D", "dt_bias", "z"):
            s[k].requires_grad_(True)
    return s


# ---- one pass -------------------------------------------------------------------

def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "decode":
        u = mb.conv1d_step(s["conv_state"], s["x"], s["w"], s["bias"])
        y = mb.scan_step(s["h"], u, s["delta"], s["A"], s["B"], s["C"], D=s["D"], dt_bias=s["dt_bias"],
                         z_t=s["z"], out_dtype=u.dtype)
        return {"y": y, "h": s["h"], "u": u, "conv_state": s["conv_state"]}
    if kind == "verify":
        args = (s["u"], s["delta"], s["A"], s["B"], s["C"])
        kw = dict(D=s["D"], dt_bias=s["dt_bias"], z=s["z"], h0=s["h0"], out_dtype=_DT[c["out"]],
                  return_last_state=True)
        y, h_last = mb.scan_fwd(*args, **kw)
        accepted, last_pos, ranks = mb.verify_rank(s["logits"], s["draft"], BETA, return_ranks=True)
        y2, h_last2, h_at = mb.scan_fwd(*args, positions=last_pos[None], **kw)
        return {"y": y, "h_last": h_last, "accepted": accepted, "ranks": ranks, "y2": y2, "h_last2": h_last2,
                "h_at": h_at}
    if kind == "conv":
        y, state = mb.conv1d(s["x"], s["w"], s["bias"], return_state=True)
        return {"y": y, "state": state}
    if kind == "prefill":
        out, u = {}, s.get("u")
        if c["conv"]:
            u, out["conv_state"] = mb.conv1d(s["x"], s["w"], s["bias"], return_state=True)
            out["u"] = u
        out["y"], out["h_last"] = mb.scan_fwd(u, s["delta"], s["A"], s["B"], s["C"], D=s["D"], dt_bias=s["dt_bias"],
                                              z=s["z"], h0=s["h0"], out_dtype=_DT[c["out"]], return_last_state=True)
        return out
    names = ("u", "delta", "A", "B", "C", "D", "dt_bias", "z")
    y, h_last = mb.selective_scan(*(s[k] for k in names))
    grads = torch.autograd.grad(y, [s[k] for k in names], s["dy"])
    return {"y": y.detach(), "h_last": h_last.detach(), **{"d" + k: g for k, g in zip(names, grads)}}


# ---- what a pass cannot do without -------------------------------------------------

def work(case):
    b, d, L = case["batch"], case["dim"], case.get("L", 1)
    e = 2 if case["dtype"] == "bf16" else 4
    kind, el, st = case["kind"], b * d * L, 4 * b * d * N
    weights = 4 * d * (N + 2)
    taps = 4 * d * (K + 1) + 4 * b * d * (K - 1)
    # per state: dlt A, exp, dlt u B, h (2), C h (2); per element: softplus, dlt u, skip, gate
    scan_flops = el * (7 * N + 15)
    conv_flops = el * (2 * K + 5)
    bc = 2 * b * N * L * e
    if kind == "decode":
        return {"bytes": el * 5 * e + bc + 2 * st + weights + taps + 4 * b * d * (K - 1),
                "flops": scan_flops + conv_flops}
    if kind == "conv":
        return {"bytes": 2 * el * e + taps, "flops": conv_flops}
    if kind == "train":
        # forward: u, delta, z in, y out; backward: dy in, du, ddelta, dz out; the chunks' states recomputed
        return {"bytes": el * 8 * e + 2 * bc + st + 2 * weights, "flops": el * (7 * N + 15 + 19 * N + 30)}
    o = 2 if case["out"] == "bf16" else 4
    if kind == "verify":
        return {"bytes": el * (3 * e + o) + bc + 3 * st + weights + 4 * b * L * 257 + el * o, "flops": 2 * scan_flops}
    io = el * ((3 if case["gate"] else 2) * e + o) + bc + weights + st * (2 if case["h0"] else 1)
    return {"bytes": io + (el * e + taps if case["conv"] else 0),
            "flops": scan_flops + (conv_flops if case["conv"] else 0)}


def tolerance(case):
    """fp32 results: 1e-7 to 4e-7 from `exact` (2-norm), sums over time and channels in another order.
    bf16 results: one rounding, 1.7e-3 from `exact`.  Where the scan reads the convolution's bf16 output, a
    rounding that falls the other way there moves single results by more than their own rounding, so only the
    2-norm is stated."""
    if case["dtype"] == "f32" or case.get("out") == "f32" and not case.get("conv"):
        t = {"rel": 2e-6, "max": 1e-4}
    else:
        t = {"rel": 7e-3}
        if case["kind"] != "decode" and not case.get("conv"):
            t["max"] = 1.6e-2
    if case["kind"] == "verify":
        t["differ"] = 0.0          # ranks and accepted lengths are whole numbers
    return t


# ---- 64 bits ----------------------------------------------------------------------

def _conv64(x, state, w, bias):
    """x (b, d, L), state (b, d, K-1): silu(causal depthwise convolution), in float64, and the next state."""
    L = x.shape[2]
    xin = torch.cat([state.double(), x.double()], 2)
    pre = bias.double()[None, :, None].expand(x.shape).clone()
    for i in range(K):
        pre += w.double()[None, :, i:i + 1] * xin[:, :, i:i + L]
    return pre * torch.sigmoid(pre), xin[:, :, L:]


def _scan64(u, delta, A, B, C, D, dt_bias, z, h0, keep=()):
    """The recurrence in time order in float64: y, h_last and the states after the timesteps in `keep`."""
    b, d, L = u.shape
    A = A.double()
    h = torch.zeros(b, d, N, dtype=torch.float64, device=DEV) if h0 is None else h0.double().clone()
    dlt = torch.nn.functional.softplus(delta.double() + dt_bias.double()[:, None], threshold=700)
    y = torch.empty(L, b, d, dtype=torch.float64, device=DEV)
    at = {-1: h.clone()} if keep else {}
    dl_t, dx_t = dlt.permute(2, 0, 1).contiguous(), (dlt * u.double()).permute(2, 0, 1).contiguous()
    B_t, C_t = B.double().permute(2, 0, 1).contiguous(), C.double().permute(2, 0, 1).contiguous()
    for t in range(L):
        h.mul_(torch.exp_(dl_t[t, :, :, None] * A)).addcmul_(dx_t[t, :, :, None], B_t[t, :, None, :])
        torch.sum(h * C_t[t, :, None, :], 2, out=y[t])
        if t in keep:
            at[t] = h.clone()
    out = y.permute(1, 2, 0) + D.double()[:, None] * u.double()
    if z is not None:
        out = out * torch.nn.functional.silu(z.double())
    return out, h, at


def _train64(s):
    """Forward and reverse recurrence in float64, all states kept."""
    u, delta, A, B, C, D, dt_bias, z, dy = (s[k].detach().double() for k in
                                            ("u", "delta", "A", "B", "C", "D", "dt_bias", "z", "dy"))
    b, d, L = u.shape
    tm = lambda x: x.permute(2, 0, 1).contiguous()  # noqa: E731  time first
    v = delta + dt_bias[:, None]
    dlt = torch.nn.functional.softplus(v, threshold=700)
    sig = torch.sigmoid(z)
    g = z * sig
    dl_t, u_t, ds_t, B_t, C_t = tm(dlt), tm(u), tm(dy * g), tm(B), tm(C)
    hs = torch.zeros(L + 1, b, d, N, dtype=torch.float64, device=DEV)
    sums = torch.empty(L, b, d, dtype=torch.float64, device=DEV)
    for t in range(L):
        torch.mul(hs[t], torch.exp_(dl_t[t, :, :, None] * A), out=hs[t + 1])
        hs[t + 1].addcmul_((dl_t[t] * u_t[t])[:, :, None], B_t[t, :, None, :])
        torch.sum(hs[t + 1] * C_t[t, :, None, :], 2, out=sums[t])
    pre = sums.permute(1, 2, 0) + D[:, None] * u
    du_t, ddl_t = torch.empty_like(sums), torch.empty_like(sums)
    dB_t, dC_t = torch.empty_like(B_t), torch.empty_like(C_t)
    dA = torch.zeros(d, N, dtype=torch.float64, device=DEV)
    carry = torch.zeros(b, d, N, dtype=torch.float64, device=DEV)
    for t in range(L - 1, -1, -1):
        abar = torch.exp_(dl_t[t, :, :, None] * A)
        lam = carry.addcmul_(ds_t[t, :, :, None], C_t[t, :, None, :])
        torch.sum(ds_t[t, :, :, None] * hs[t + 1], 1, out=dC_t[t])
        torch.sum(lam * (dl_t[t] * u_t[t])[:, :, None], 1, out=dB_t[t])
        lb = (lam * B_t[t, :, None, :]).sum(2)
        carry = lam * abar
        w = carry * hs[t]
        du_t[t] = dl_t[t] * lb
        ddl_t[t] = u_t[t] * lb + (w * A).sum(2)
        dA += (w * dl_t[t, :, :, None]).sum(0)
    bt = lambda x: x.permute(1, 2, 0)  # noqa: E731
    ddelta = bt(ddl_t) * torch.sigmoid(v)
    ds = dy * g
    return {"y": pre * g, "h_last": hs[L].clone(), "du": bt(du_t) + D[:, None] * ds, "ddelta": ddelta, "dA": dA,
            "dB": bt(dB_t), "dC": bt(dC_t), "dD": (ds * u).sum((0, 2)), "ddt_bias": ddelta.sum((0, 2)),
            "dz": dy * pre * sig * (1 + z * (1 - sig))}


def exact(case, seed):
    s = prepare(case, seed)
    kind, act = case["kind"], _DT[case["dtype"]]
    zeros = torch.zeros(case["batch"], case["dim"], K - 1, device=DEV)
    with torch.no_grad():
        if kind == "train":
            return _train64(s)
        if kind == "conv":
            y, state = _conv64(s["x"], zeros, s["w"], s["bias"])
            return {"y": y, "state": state}
        if kind == "decode":
            u, conv_state = _conv64(s["x"][:, :, None], s["conv_state"], s["w"], s["bias"])
            used = u.to(act)                    # conv1d_step hands the scan its input in the activations' type
            y, h, _ = _scan64(used, s["delta"][:, :, None], s["A"], s["B"][:, :, None], s["C"][:, :, None], s["D"],
                              s["dt_bias"], s["z"][:, :, None], s["h"])
            return {"y": y[:, :, 0], "h": h, "u": u[:, :, 0], "conv_state": conv_state}
        if kind == "verify":
            lg, dr = s["logits"], s["draft"].long()
            ranks = 1 + (lg > lg.gather(2, dr[:, :, None])).sum(2)
            accepted = (ranks <= BETA).int().cumprod(1).sum(1)
            y, h, at = _scan64(s["u"], s["delta"], s["A"], s["B"], s["C"], s["D"], s["dt_bias"], s["z"], s["h0"],
                               keep=range(case["L"]))
            h_at = torch.stack([at[int(a) - 1][i] for i, a in enumerate(accepted)])[None]
            return {"y": y, "h_last": h, "accepted": accepted.int(), "ranks": ranks.int(), "y2": y, "h_last2": h,
                    "h_at": h_at}
        out, u = {}, s.get("u")
        if case["conv"]:
            out["u"], out["conv_state"] = _conv64(s["x"], zeros, s["w"], s["bias"])
            u = out["u"].to(act)
        out["y"], out["h_last"], _ = _scan64(u, s["delta"], s["A"], s["B"], s["C"], s["D"], s["dt_bias"], s["z"],
                                             s["h0"])
        return out
