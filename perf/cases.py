"""The work whose speed counts: passes through the library's public entry points at the sizes users run.

Kinds of pass
    step    one POET-X linear in training: blocks built from the packed parameters, forward, whole backward pass
    fwd     forward alone, blocks at hand (evaluation, prefill, and a handful of tokens as in decoding)
    bwd     the one-call backward alone
    series  the blocks and the series backward of a whole decoder layer, once per step

A case is a dict: kind, n (d_out), m (d_in), b (block), k (series order), tokens, dtype ("f32" / "bf16"), variant
("fast" keeps B, "mem" recomputes it, "xq" is mem on an INT8 weight), layout ("feature" / "token").  `series` cases
have nb (number of blocks) in place of n, m and tokens.  Values and scales follow workloads/configs.py.
"""
from __future__ import annotations

import math

import torch

import paper_2603_05500_amd as px


def _lin(name, kind, n, m, b, k, tokens, dtype="bf16", variant="fast", layout="feature"):
    return {"name": name, "kind": kind, "n": n, "m": m, "b": b, "k": k, "tokens": tokens, "dtype": dtype,
            "variant": variant, "layout": layout}


def listed():
    return [
        # the smallest configuration, a single fp32 linear: launches and latency are all there is
        _lin("single256-f32-step", "step", 256, 256, 32, 4, 512, "f32"),
        # fp32 at a size where arithmetic counts, with a token count that is no multiple of anything
        _lin("mid-f32-step", "step", 1024, 768, 64, 4, 1001, "f32"),
        # llama60m, gate: small blocks, ragged last block (1376 = 21 * 64 + 32), batch of 4 x 256
        _lin("llama60m-gate-step", "step", 1376, 512, 64, 4, 1024),
        # llama1b, q, a handful of tokens in a framework's own layout: generation from the model in training
        _lin("llama1b-q-decode", "fwd", 2048, 2048, 256, 4, 16, layout="token"),
        # llama1b, down: evaluation on a batch whose token count is odd
        _lin("llama1b-down-eval", "fwd", 2048, 5632, 256, 4, 1999),
        # llama3b, gate: a training batch with a ragged token count, token-major activations
        _lin("llama3b-gate-ragged-step", "step", 8192, 3072, 256, 5, 4090, layout="token"),
        # one 4096 x 4096 projection at 2048 tokens: the single-layer latency setting of the paper
        _lin("llama8b-q-2k-step", "step", 4096, 4096, 256, 5, 2048),
        # llama8b, gate at the full batch of 4 x 4096: the largest forward product
        _lin("llama8b-gate-fwd", "fwd", 14336, 4096, 256, 5, 16384),
        # llama8b, down at the full batch: the largest backward
        _lin("llama8b-down-bwd", "bwd", 4096, 14336, 256, 5, 16384),
        # llama8b, o with the larger block side, full batch
        _lin("llama8b-b512-o-step", "step", 4096, 4096, 512, 5, 16384),
        # llama8b, k on an INT8 base weight: few output features, recomputation, dequantisation
        _lin("llama8b-k-xq-step", "step", 1024, 4096, 256, 5, 4096, variant="xq"),
        # series of a whole llama8b layer: 320 blocks of 256 built and differentiated in one call each
        {"name": "llama8b-layer-series", "kind": "series", "nb": 320, "b": 256, "k": 5, "dtype": "bf16"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    what = rng.choice(("f32", "small", "large", "large", "large", "series"))
    if what == "series":
        b = rng.choice((64, 256, 256, 512))
        nb = _log(rng, 2, 320 if b < 512 else 80)
        return {"kind": "series", "nb": nb, "b": b, "k": rng.randint(3, 5), "dtype": "bf16"}
    if what == "f32":        # fp32 linears
        b = rng.choice((32, 64))
        n, m = (max(16 * rng.randint(8, 64), b) for _ in range(2))
        return dict(kind=rng.choice(("step", "fwd", "bwd")), n=n, m=m, b=b, k=4, tokens=_log(rng, 16, 2048), dtype="f32",
                    variant="fast", layout=rng.choice(("feature", "token")))
    if what == "small":      # small models: small blocks, feature counts that b need not divide
        b = rng.choice((64, 64, 128))
        n, m = (32 * rng.randint(8, 48) for _ in range(2))
        return dict(kind=rng.choice(("step", "fwd", "bwd")), n=n, m=m, b=b, k=4, tokens=_log(rng, 16, 4096), dtype="bf16",
                    variant=rng.choice(("fast", "fast", "mem")), layout=rng.choice(("feature", "token")))
    b = rng.choice((256, 256, 512))
    n, m = (512 * max(2, min(28, _log(rng, 2, 28))) for _ in range(2))
    # tokens so that no drawn pass does more than the largest listed one of its sort
    if rng.random() < 0.5:   # whole sequences
        tokens = min(256 * _log(rng, 1, 64), 27 * 16384 * 4096 * 14336 // (100 * n * m) // 256 * 256)
    else:                    # whatever a batch happens to hold
        tokens = min(_log(rng, 8, 6000), 4090 * 8192 * 3072 // (n * m))
    return dict(kind=rng.choice(("step", "fwd", "bwd")), n=n, m=m, b=b, k=rng.choice((4, 5)), tokens=tokens, dtype="bf16",
                variant=rng.choice(("fast", "fast", "mem", "xq")), layout=rng.choice(("feature", "feature", "token")))


# ------------------------------------------------------------------------------------ inputs
def _sigma_theta(b):
    return 0.01 if b <= 128 else 0.005


def _dt(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def _nblk(d, b):
    return -(-d // b)


def _skew(theta, b, d):
    """Packed rows -> skew matrices [nb][b][b]; rows and columns past the tail side are zero."""
    nb = theta.shape[0]
    iu = torch.triu_indices(b, b, 1, device=theta.device)
    q = torch.zeros((nb, b, b), dtype=theta.dtype, device=theta.device)
    q[:, iu[0], iu[1]] = theta
    q = q - q.transpose(1, 2)
    r = d - b * (nb - 1)
    if r < b:
        mask = torch.ones((nb, b, b), dtype=theta.dtype, device=theta.device)
        mask[-1, r:, :] = 0
        mask[-1, :, r:] = 0
        q = q * mask
    return q


def _residual(q, k):
    """G - I = 2 (Q + .. + Q^k) + Q^(k+1)."""
    h = q
    for _ in range(k):
        h = 2 * q + torch.bmm(h, q)
    return h


def _draws(case, seed):
    """Everything a pass is given, from the seed alone."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    dt, b, k = _dt(case), case["b"], case["k"]

    def normal(shape, sigma=1.0, to=torch.float32):
        return (torch.randn(shape, generator=g, device="cuda", dtype=torch.float32) * sigma).to(to)

    L = b * (b - 1) // 2
    if case["kind"] == "series":
        return {"theta": normal((case["nb"], L), _sigma_theta(b)), "dG": normal((case["nb"], b, b))}
    n, m, N = case["n"], case["m"], case["tokens"]
    tm = case["layout"] == "token"
    d = {}
    # one packed buffer for both sides, R first: a single build serves both where b divides both dimensions
    d["theta"] = normal((_nblk(m, b) + _nblk(n, b), L), _sigma_theta(b))
    d["pi_R"] = torch.randperm(m, generator=g, device="cuda").to(torch.int32)
    d["pi_P"] = torch.randperm(n, generator=g, device="cuda").to(torch.int32)
    d["W"] = normal((n, m), 0.02, dt)
    if case["kind"] != "fwd":
        d["dZ"] = normal((N, n) if tm else (n, N), 1.0, dt)
    d["X"] = normal((N, m) if tm else (m, N), 1.0, dt)
    if case["kind"] == "bwd" and case["variant"] == "fast":
        d["B"] = normal((n, N), 0.02 * math.sqrt(m), dt)   # what the forward pass saved
    if case["variant"] == "xq":
        # symmetric absmax codes per output row, then the row scales at the next multiple of 256 bytes
        w = d["W"].float()
        top = w.abs().amax(1)
        scale = torch.where(top > 0, top / 127.0, torch.ones_like(top))
        code = torch.round(w / scale[:, None]).clamp_(-127, 127)
        wq = torch.zeros(px.poetx_weight_q8_bytes(n, m), dtype=torch.uint8, device="cuda")
        off = (n * m + 255) // 256 * 256
        wq[:n * m] = code.to(torch.int8).view(torch.uint8).reshape(-1)
        wq[off:off + 4 * n] = scale.view(torch.uint8)
        d["Wq"] = wq
        d["W"] = (scale[:, None] * code).to(dt)            # what the codes stand for
    if case["kind"] != "step":                             # blocks at hand, from these very parameters
        for side, dim, th in (("R", m, d["theta"][:_nblk(m, b)]), ("P", n, d["theta"][_nblk(m, b):])):
            e = _residual(_skew(th, b, dim), k)
            if dt == torch.float32:
                d["blk_" + side] = e + torch.eye(b, device="cuda")
            else:
                e = e.to(dt)
                d["blk_" + side] = torch.stack((e, e.transpose(1, 2)), 1).contiguous()
    return d


def prepare(case, seed):
    px.load_library()
    s = _draws(case, seed)
    b, k = case["b"], case["k"]
    code = px.F32 if case["dtype"] == "f32" else px.BF16
    s["case"], s["prec"] = dict(case), px.CNP_FP32 if code == px.F32 else px.CNP_BF16
    dt = _dt(case)
    bytes_ = lambda n: torch.empty(max(int(n), 256), dtype=torch.uint8, device="cuda")
    if case["kind"] == "series":
        nb = case["nb"]
        d = nb * b
        s["E"] = torch.empty((nb, 2, b, b), dtype=torch.bfloat16, device="cuda")
        s["dtheta"] = torch.empty_like(s["theta"])
        s["ws"] = bytes_(max(px.poetx_cnp_workspace_bytes(d, b), px.poetx_cnp_bwd_workspace_bytes(d, b, k)))
        return s
    n, m, N = case["n"], case["m"], case["tokens"]
    tm = case["layout"] == "token"
    flags = {"fast": 0, "mem": px.FLAG_RECOMPUTE_B, "xq": px.FLAG_RECOMPUTE_B | px.FLAG_W_INT8}[case["variant"]]
    s["desc"] = px.make_desc(m, n, b, k, N, code, flags=flags, layout=px.TOKEN_MAJOR if tm else px.FEATURE_MAJOR)
    s["weight"] = s["Wq"] if case["variant"] == "xq" else s["W"]
    s["ws"] = bytes_(px.poetx_linear_workspace_bytes(s["desc"]))
    nbR = _nblk(m, b)
    s["theta_R"], s["theta_P"] = s["theta"][:nbR], s["theta"][nbR:]
    if case["kind"] == "step":
        nbt = s["theta"].shape[0]
        s["blk"] = torch.empty((nbt, b, b) if code == px.F32 else (nbt, 2, b, b), dtype=dt, device="cuda")
        s["blk_R"], s["blk_P"] = s["blk"][:nbR], s["blk"][nbR:]
        s["cws"] = bytes_(px.poetx_cnp_workspace_bytes(b * nbt, b))
    if case["kind"] != "bwd":
        s["Z"] = torch.empty((N, n) if tm else (n, N), dtype=dt, device="cuda")
        s["B"] = torch.empty((n, N), dtype=dt, device="cuda") if case["variant"] == "fast" else None
    elif case["variant"] != "fast":
        s["B"] = None
    if case["kind"] != "fwd":
        s["dX"] = torch.empty_like(s["X"])
        s["dtheta"] = torch.empty_like(s["theta"])
        s["dtheta_R"], s["dtheta_P"] = s["dtheta"][:nbR], s["dtheta"][nbR:]
    return s


# ------------------------------------------------------------------------------------ the pass
def run(s):
    c = s["case"]
    b, k = c["b"], c["k"]
    if c["kind"] == "series":
        d = c["nb"] * b
        px.poetx_cnp_build(s["theta"], d, b, k, s["prec"], E_bf16=s["E"], ws=s["ws"])
        px.poetx_cnp_bwd(s["theta"], s["dG"], d, b, k, s["prec"], s["dtheta"], False, s["ws"])
        return {"E": s["E"], "dtheta": s["dtheta"]}
    n, m = c["n"], c["m"]
    out = {}
    if c["kind"] == "step":
        kind = "G_f32" if c["dtype"] == "f32" else "E_bf16"
        if m % b == 0 and n % b == 0:
            px.poetx_cnp_build(s["theta"], m + n, b, k, s["prec"], ws=s["cws"], **{kind: s["blk"]})
        else:
            px.poetx_cnp_build(s["theta_R"], m, b, k, s["prec"], ws=s["cws"], **{kind: s["blk_R"]})
            px.poetx_cnp_build(s["theta_P"], n, b, k, s["prec"], ws=s["cws"], **{kind: s["blk_P"]})
        out["blocks"] = s["blk"]
    if c["kind"] != "bwd":
        px.poetx_linear_fwd(s["desc"], s["X"], s["weight"], s["pi_R"], s["pi_P"], s["blk_R"], s["blk_P"], s["Z"], s["B"],
                            s["ws"])
        out["Z"] = s["Z"]
        if s["B"] is not None:
            out["B"] = s["B"]
    if c["kind"] != "fwd":
        px.poetx_linear_bwd(s["desc"], s["X"], s["dZ"], s["B"], s["weight"], s["pi_R"], s["pi_P"], s["blk_R"], s["blk_P"],
                            s["theta_R"], s["theta_P"], s["dX"], s["dtheta_R"], s["dtheta_P"], False, s["ws"])
        out["dX"], out["dtheta"] = s["dX"], s["dtheta"]
    return out


def work(case):
    b, k = case["b"], case["k"]
    es = 4 if case["dtype"] == "f32" else 2
    L4 = 4 * (b * (b - 1) // 2)                      # packed parameters of a block
    blk = 4 * b * b                                  # a stored block: fp32, or a bf16 pair
    prod = 2.0 * b ** 3
    if case["kind"] == "series":
        nb = case["nb"]
        return {"bytes": nb * (2 * L4 + blk + 4 * b * b), "flops": nb * 3 * k * prod}
    n, m, N = case["n"], case["m"], case["tokens"]
    nb = _nblk(m, b) + _nblk(n, b)
    w = n * m + 4 * n if case["variant"] == "xq" else es * n * m
    keep = case["variant"] == "fast"
    fwd_f = 2.0 * N * m * n + 2.0 * N * (m + n) * b
    bwd_f = 2.0 * N * m * n + 4.0 * N * (m + n) * b + (0 if keep else 2.0 * N * m * n + 2.0 * N * m * b)
    idx = 4 * (m + n)
    if case["kind"] == "fwd":
        return {"bytes": es * N * (m + n + (n if keep else 0)) + w + nb * blk + idx, "flops": fwd_f}
    if case["kind"] == "bwd":
        return {"bytes": es * N * (2 * m + n + (n if keep else 0)) + w + nb * (blk + 2 * L4) + idx,
                "flops": bwd_f + nb * 2 * k * prod}
    return {"bytes": es * N * (2 * m + 2 * n + (n if keep else 0)) + w + nb * (blk + 2 * L4) + idx,
            "flops": fwd_f + bwd_f + nb * 3 * k * prod}


def tolerance(case):
    # bf16: every intermediate is rounded once (2^-9 relative), up to four of them in a row; fp32: sums over up to a
    # few thousand terms in another order
    return {"rel": 1e-5} if case["dtype"] == "f32" else {"rel": 1.2e-2}


# ------------------------------------------------------------------------------------ 64-bit reference
def _apply(v, pi, g, trans=False):
    """Psi^T Diag(op G) Psi v for d x N columns; the tail block is padded with zero rows."""
    nb, b = g.shape[0], g.shape[1]
    d, N = v.shape
    x = torch.zeros((nb * b, N), dtype=v.dtype, device=v.device)
    x[:d] = v[pi]
    y = torch.bmm((g.transpose(1, 2) if trans else g).contiguous(), x.view(nb, b, N)).view(nb * b, N)[:d]
    out = torch.empty_like(v)
    out[pi] = y
    return out


def _block_grad(u, v, pi, nb, b):
    d, N = u.shape
    uu, vv = (torch.zeros((nb * b, N), dtype=u.dtype, device=u.device) for _ in range(2))
    uu[:d], vv[:d] = u[pi], v[pi]
    return torch.bmm(uu.view(nb, b, N), vv.view(nb, b, N).transpose(1, 2).contiguous())


def _series_grad(theta, dG, b, d, k):
    th = theta.detach().clone().requires_grad_(True)
    return torch.autograd.grad(_residual(_skew(th, b, d), k), th, dG)[0]


def exact(case, seed):
    d = _draws(case, seed)
    f = lambda t: t.double()
    b, k = case["b"], case["k"]
    if case["kind"] == "series":
        dd = case["nb"] * b
        e = _residual(_skew(f(d["theta"]), b, dd), k)
        return {"E": torch.stack((e, e.transpose(1, 2)), 1), "dtheta": _series_grad(f(d["theta"]), f(d["dG"]), b, dd, k)}
    n, m = case["n"], case["m"]
    tm = case["layout"] == "token"
    nbR, nbP = _nblk(m, b), _nblk(n, b)
    piR, piP = d["pi_R"].long(), d["pi_P"].long()
    thR, thP = f(d["theta"][:nbR]), f(d["theta"][nbR:])
    eye = torch.eye(b, dtype=torch.float64, device="cuda")
    W = f(d["W"])
    X = f(d["X"].t() if tm else d["X"])
    back = lambda t: t.t().contiguous() if tm else t
    out = {}
    if case["kind"] == "step":
        E = {"R": _residual(_skew(thR, b, m), k), "P": _residual(_skew(thP, b, n), k)}
        GR, GP = E["R"] + eye, E["P"] + eye
        if case["dtype"] == "f32":
            out["blocks"] = torch.cat((GR, GP), 0)
        else:
            e = torch.cat((E["R"], E["P"]), 0)
            out["blocks"] = torch.stack((e, e.transpose(1, 2)), 1)
    elif case["dtype"] == "f32":
        GR, GP = f(d["blk_R"]), f(d["blk_P"])
    else:
        GR, GP = f(d["blk_R"][:, 0]) + eye, f(d["blk_P"][:, 0]) + eye
    keep = case["variant"] == "fast"
    if "B" in d:
        B = f(d["B"])
    else:
        B = W @ _apply(X, piR, GR, True)
    if case["kind"] != "bwd":
        out["Z"] = back(_apply(B, piP, GP, True))
        if keep:
            out["B"] = B
    if case["kind"] != "fwd":
        dZ = f(d["dZ"].t() if tm else d["dZ"])
        dA = W.t().contiguous() @ _apply(dZ, piP, GP)
        out["dX"] = back(_apply(dA, piR, GR))
        out["dtheta"] = torch.cat((_series_grad(thR, _block_grad(X, dA, piR, nbR, b), b, m, k),
                                   _series_grad(thP, _block_grad(B, dZ, piP, nbP, b), b, n, k)), 0)
    return out
