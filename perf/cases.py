"""Performance cases of the library's public entry points.

Each listed case is a call that a user makes: one layer's gradient at the sizes it is trained at
(full and truncated, with and without the projections), the forward alone, the K-layer stack, the
language head with its loss, the unstructured SSM, the explicit pair formulation, the projection
gradients on their own, and the smallest and a ragged call, where launches and latency count.  The
sizes are those of ``paper_2501_00692_amd/synth.py`` and ``bench.py`` or ragged ones of the same
order; ``draw`` spreads over the same ranges.
"""
import math

import torch

import paper_2501_00692_amd as ssm
from paper_2501_00692_amd import synth

DEV = "cuda"


def listed():
    return [
        # the parity-sized call: a handful of launches, latency only
        {"name": "scan_small_f32", "kind": "scan", "b": 1, "T": 256, "D": 64, "N": 16, "bf16": False, "proj": False,
         "h0": False, "tbar": 0, "variant": 0},
        # nothing a multiple of anything: gate and softplus, an initial state, a window inside the chunk
        {"name": "scan_ragged_f32", "kind": "scan", "b": 3, "T": 1021, "D": 203, "N": 13, "bf16": False, "proj": True,
         "h0": True, "tbar": 100, "variant": 0},
        # very long context, scan only, truncated
        {"name": "scan_vlong_trunc", "kind": "scan", "b": 1, "T": 262144, "D": 3072, "N": 16, "bf16": True,
         "proj": False, "h0": False, "tbar": 8192, "variant": 0},
        # one training layer at an ordinary context length, full gradient
        {"name": "layer", "kind": "layer", "b": 2, "T": 4096, "D": 1536, "N": 16, "dm": 768, "tbar": 0, "du": False},
        # the same layer at long context, truncated window
        {"name": "layer_long_trunc", "kind": "layer", "b": 2, "T": 65536, "D": 1536, "N": 16, "dm": 768, "tbar": 2048,
         "du": False},
        # the benchmark's layer, full gradient (the largest case)
        {"name": "layer_slice", "kind": "layer", "b": 1, "T": 262144, "D": 4096, "N": 16, "dm": 2048, "tbar": 0,
         "du": False},
        # the forward alone (evaluation), with gate, softplus and the final state
        {"name": "forward_long", "kind": "forward", "b": 2, "T": 65536, "D": 1536, "N": 16, "bf16": True,
         "proj": True, "h0": False},
        # two residual layers, forward and backpropagation (bf16 activations: in deeper stacks their rounding,
        # carried through the layers, hides everything else)
        {"name": "stack_exact", "kind": "stack", "K": 2, "b": 2, "T": 4096, "D": 1536, "N": 16, "tbar": 0,
         "exact": True},
        # the language head with its loss
        {"name": "head", "kind": "head", "M": 32768, "P": 2048, "V": 32000, "norm": True},
        # the unstructured row of the paper's table, truncated
        {"name": "unstructured_trunc", "kind": "unstructured", "b": 8, "T": 16384, "P": 64, "tbar": 256},
        # the paper's explicit VJPs at the layer's scan shape
        {"name": "pairs", "kind": "pairs", "b": 2, "T": 4096, "D": 1536, "N": 16, "bf16": True, "tbar": 256},
        # both projection gradients on their own, at sizes no tile divides
        {"name": "proj", "kind": "proj", "M": 8191, "K": 1528, "Nout": 1560},
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["scan", "scan", "layer", "layer", "forward", "stack", "head", "unstructured", "pairs", "proj"])
    if kind in ("scan", "forward"):
        b = rng.choice([1, 1, 2, 3])
        T = _logint(rng, 64, 65536)
        D = min(_logint(rng, 24, 3072), (1 << 27) // (b * T))
        c = {"kind": kind, "b": b, "T": T, "D": max(D, 8), "N": rng.choice([16, 16, 16, 8, rng.randint(1, 16)]),
             "bf16": rng.random() < 0.6, "proj": rng.random() < 0.6, "h0": rng.random() < 0.3}
        if kind == "scan":
            c["tbar"] = rng.choice([0, _logint(rng, 1, T)])
            c["variant"] = rng.choice([0, 0, 0, 1, 2, 3])
        return c
    if kind == "layer":
        T = _logint(rng, 512, 65536)
        D = 8 * _logint(rng, 16, 256)
        D = max(64, min(D, (1 << 27) // T // 8 * 8))
        return {"kind": kind, "b": rng.choice([1, 2]), "T": T, "D": D, "N": rng.choice([16, 16, 16, 8, 4]),
                "dm": max(64, D * rng.choice([4, 4, 8]) // 8 // 8 * 8), "tbar": rng.choice([0, _logint(rng, 16, T)]),
                "du": rng.random() < 0.4}
    if kind == "stack":
        return {"kind": kind, "K": rng.randint(1, 2), "b": rng.choice([1, 2]), "T": _logint(rng, 256, 4096),
                "D": 8 * rng.randint(32, 192), "N": 16, "tbar": rng.choice([0, 256]), "exact": rng.random() < 0.5}
    if kind == "head":
        return {"kind": kind, "M": _logint(rng, 300, 32768), "P": 8 * rng.randint(16, 256),
                "V": 8 * _logint(rng, 125, 4000), "norm": rng.random() < 0.8}
    if kind == "unstructured":
        return {"kind": kind, "b": rng.randint(1, 8), "T": _logint(rng, 300, 16384), "P": 16 * rng.randint(1, 8),
                "tbar": rng.choice([0, _logint(rng, 16, 299)])}
    if kind == "pairs":
        b, T = rng.choice([1, 2]), _logint(rng, 256, 4096)
        return {"kind": kind, "b": b, "T": T, "D": _logint(rng, 64, 1536), "N": rng.choice([16, 16, 8]),
                "bf16": rng.random() < 0.6, "tbar": _logint(rng, 16, 256)}
    return {"kind": "proj", "M": _logint(rng, 200, 65536), "K": 8 * _logint(rng, 16, 512),
            "Nout": 8 * _logint(rng, 16, 512)}


def prepare(case, seed):
    c = dict(case)
    k = c["kind"]
    if k in ("scan", "forward", "pairs"):
        w = synth.Workload(k, c["b"], c["T"], c["D"], c["N"], 0, c.get("tbar", 0), False, c["bf16"], seed)
        inp = synth.make_inputs(w, DEV, seed=seed, h0=c.get("h0", False))
        if c.get("proj"):  # softplus inside and the output gate: Delta_pre and z from their marginals
            g = torch.Generator(device=DEV)
            g.manual_seed(seed + 1)
            for n in ("delta", "z"):
                inp[n] = torch.randn(c["b"], c["T"], c["D"], generator=g, device=DEV).to(inp["x"].dtype)
        if c.get("variant", 0) & 1:
            inp["A_log"] = inp["A_log"][:, 0].contiguous()
    elif k == "layer":
        w = synth.Workload(k, c["b"], c["T"], c["D"], c["N"], c["dm"], c["tbar"], True, True, seed)
        inp = synth.make_inputs(w, DEV, seed=seed)
    elif k == "stack":
        inp = synth.make_stack_inputs(c["K"], c["b"], c["T"], c["D"], c["N"], seed, DEV)
    elif k == "head":
        inp = synth.make_head_inputs(c["M"], c["P"], c["V"], seed, DEV)
    elif k == "unstructured":
        inp = synth.make_unstructured_inputs(c["b"], c["T"], c["P"], seed, device=DEV, h0=True)
    else:
        g = torch.Generator(device=DEV)
        g.manual_seed(seed)

        def rnd(*shape, std=1.0):
            return (torch.randn(*shape, generator=g, device=DEV) * std).to(torch.bfloat16)
        inp = {"X": rnd(c["M"], c["K"]), "dZ": rnd(c["M"], c["Nout"]),
               "W": rnd(c["K"], c["Nout"], std=1.0 / math.sqrt(c["K"]))}
    return c, inp


def run(state):
    c, i = state
    k = c["kind"]
    if k == "scan":
        return ssm.ssm_adjoint_grad(i["x"], i["delta"], i["A_log"], i["B"], i["C"], i["dy"], h0=i.get("h0"),
                                    z=i.get("z"), softplus=c["proj"], tbar=c["tbar"], b_delta=bool(c["variant"] & 2))
    if k == "forward":
        return ssm.ssm_adjoint_forward(i["x"], i["delta"], i["A_log"], i["B"], i["C"], h0=i.get("h0"), z=i.get("z"),
                                       softplus=c["proj"], want_h_last=True)
    if k == "pairs":
        return ssm.ssm_adjoint_grad_pairs(i["x"], i["delta"], i["A_log"], i["B"], i["C"], i["dy"], tbar=c["tbar"])
    if k == "layer":
        return ssm.ssm_layer_grad(i["u"], i["x"], i["z"], i["delta"], i["B"], i["C"], i["W_x"], i["W_in"], i["A_log"],
                                  i["dy"], tbar=c["tbar"], want_du=c["du"])
    if k == "stack":
        return ssm.ssm_stack_grad(i["y0"], i["W_in"], i["W_x"], i["A_log"], i["gK"], c["N"], exact=c["exact"],
                                  tbar=c["tbar"], want_yK=True)
    if k == "head":
        return ssm.ssm_lm_head_grad(i["y"], i["omega"], i["targets"], norm=c["norm"])
    if k == "unstructured":
        return ssm.ssm_unstructured_grad(i["A"], i["B"], i["C"], i["x"], i["dy"], h0=i["h0"], tbar=c["tbar"])
    return ssm.ssm_proj_grad(i["X"], i["dZ"], i["W"], want_dX=True)


def work(case):
    c = case
    k = c["kind"]
    if k in ("scan", "forward", "pairs"):
        M, D, N = c["b"] * c["T"], c["D"], c["N"]
        el = 2 if c["bf16"] else 4
        gate = 1 if c.get("proj") else 0
        if k == "forward":
            return {"bytes": M * (D * el * (3 + gate) + 2 * N * el), "flops": 7 * M * D * N}
        full = {"bytes": M * (D * (el * (3 + gate) + 4 * (2 + gate)) + N * (2 * el + 8)),
                "flops": (29 if c["tbar"] else 22) * M * D * N}
        if k == "pairs":  # each adjoint state of the window formed (one product) and weighted and summed (two)
            W = min(c["tbar"] or c["T"], c["T"])
            pairs = c["b"] * (W * c["T"] - W * (W - 1) // 2)
            full["flops"] += 4 * pairs * D * N
        return full
    if k == "layer":
        M, D, N, dm = c["b"] * c["T"], c["D"], c["N"], c["dm"]
        nx = D + 2 * N
        flops = (29 if c["tbar"] else 22) * M * D * N + 2 * M * (D * nx + dm * 2 * D)
        flops += 2 * M * nx * D if c["du"] else 2 * M * nx * min(D, dm)
        flops += 2 * M * dm * 2 * D if c["du"] else 0
        by = 2 * M * (4 * D + dm + 2 * N) + 6 * (D * nx + dm * 2 * D) + (4 * M * dm if c["du"] else 0)
        return {"bytes": by, "flops": flops}
    if k == "stack":
        M, D, N, K = c["b"] * c["T"], c["D"], c["N"], c["K"]
        nx = D + 2 * N
        gemm = 2 * M * D * (2 * D + nx)  # one product with each projection
        flops = K * (2 * gemm + 2 * M * nx * D + (22 + 7) * M * D * N)
        if c["exact"]:
            flops += (K - 1) * 2 * M * D * 2 * D
        return {"bytes": 12 * M * D + K * 6 * D * (2 * D + nx), "flops": flops}
    if k == "head":
        M, P, V = c["M"], c["P"], c["V"]
        return {"bytes": 8 * M * P + 6 * V * P + 8 * M, "flops": 6 * M * P * V}
    if k == "unstructured":
        M, P = c["b"] * c["T"], c["P"]
        return {"bytes": 4 * M * (2 * 256 + 4 * 16 * P + 3 * P), "flops": M * (2 * 4 * 256 + 2 * 5 * 16 * P)}
    M, K, Nout = c["M"], c["K"], c["Nout"]
    return {"bytes": 2 * (M * K + M * Nout + K * Nout) + 4 * (K * Nout + M * K), "flops": 4 * M * K * Nout}


def tolerance(case):
    """About four times the error against 64 bits that the listed cases show."""
    k = case["kind"]
    if k in ("scan", "pairs"):  # 2e-7 to 5e-7 (the dA_log sums)
        return {"rel": 2e-6, "max": 1e-4}
    if k == "forward":  # y is stored in the input type (1.7e-3 in bf16)
        return {"rel": 7e-3, "max": 2e-2} if case["bf16"] else {"rel": 1e-6, "max": 5e-5}
    if k == "layer":  # the scan's gradients enter the products in bf16 (1.7e-3)
        return {"rel": 7e-3, "max": 0.1}
    if k == "stack":  # bf16 activations from layer to layer: a changed rounding travels through all that follow
        return {"rel": 2.5e-2, "max": 0.9}
    if k == "head":  # the logit gradients enter the products in bf16 (1.7e-3)
        return {"rel": 7e-3, "max": 0.1}
    if k == "unstructured":  # 2e-7
        return {"rel": 1e-6, "max": 5e-5}
    return {"rel": 1.5e-6, "max": 6e-5}  # proj: 3e-7


# ---- the same results in 64 bits, by plain torch ----------------------------------------------------------------

def _scan64(x, delta, A_log, B, C, dy, h0, z, softplus, tbar, b_delta=False, grad=True):
    """Forward (y, h_last) and, with grad, all gradients of one scan layer; inputs of any type, blocks of channels."""
    f = torch.float64
    b, T, D = x.shape
    N = B.shape[-1]
    L = max(16, min(512, 1 << math.ceil(math.log2(max(2.0, math.sqrt(T))))))
    nc = -(-T // L)
    Tp, bn = nc * L, b * nc
    w_all = -torch.exp(A_log.to(f))
    if w_all.dim() == 1:
        w_all = w_all[:, None].expand(D, N)

    def chunked(t):  # [b, T, ...] -> [L, b nc, ...], padded with zeros
        t = torch.cat([t, t.new_zeros(b, Tp - T, *t.shape[2:])], 1) if Tp > T else t
        return t.reshape(bn, L, *t.shape[2:]).transpose(0, 1).contiguous()

    def flat(t):  # back to [b, T, ...]
        return t.transpose(0, 1).reshape(b, Tp, *t.shape[2:])[:, :T]
    Bc, Cc = chunked(B.to(f)), chunked(C.to(f))
    out = {"y": torch.empty(b, T, D, dtype=f, device=x.device), "h_last": torch.empty(b, D, N, dtype=f, device=x.device)}
    if grad:
        for n in ("dx", "ddelta") + (("dz",) if z is not None else ()):
            out[n] = torch.empty(b, T, D, dtype=f, device=x.device)
        out["dA_log"] = torch.empty(D, N, dtype=f, device=x.device)
        dBc, dCc = torch.zeros_like(Bc), torch.zeros_like(Cc)
    step = max(1, min(D, (1 << 28) // (b * Tp * N)))
    for d0 in range(0, D, step):
        s = slice(d0, min(D, d0 + step))
        w = w_all[s]
        pre = delta[:, :, s].to(f)
        dl = torch.nn.functional.softplus(pre, threshold=1e9) if softplus else pre
        xr = x[:, :, s].to(f)
        xin = chunked(xr * dl if b_delta else xr)
        dlc = chunked(dl)
        cum = dlc.cumsum(0)
        nd = w.shape[0]
        h = torch.empty(L, bn, nd, N, dtype=f, device=x.device)
        cur = torch.zeros(bn, nd, N, dtype=f, device=x.device)
        for t in range(L):
            cur = torch.exp(dlc[t][..., None] * w).mul_(cur).add_(xin[t][..., None] * Bc[t][:, None, :])
            h[t] = cur
        P = torch.exp(cum[-1][..., None] * w).view(b, nc, nd, N)
        H = torch.empty(b, nc, nd, N, dtype=f, device=x.device)
        H0 = h0[:, s].to(f) if h0 is not None else torch.zeros(b, nd, N, dtype=f, device=x.device)
        cur = H0
        end = h[-1].view(b, nc, nd, N)
        for q in range(nc):
            H[:, q] = cur
            cur = P[:, q] * cur + end[:, q]
        out["h_last"][:, s] = cur
        Hf = H.view(bn, nd, N)
        for t in range(L):
            h[t].addcmul_(torch.exp(cum[t][..., None] * w), Hf)
        y = flat(torch.stack([(h[t] * Cc[t][:, None, :]).sum(-1) for t in range(L)]))
        sg = None
        if z is not None:
            zz = z[:, :, s].to(f)
            sg = torch.sigmoid(zz)
            out["y"][:, :, s] = y * zz * sg
        else:
            out["y"][:, :, s] = y
        if not grad:
            continue
        gy = dy[:, :, s].to(f)
        gc = chunked(gy * zz * sg if z is not None else gy)
        if z is not None:
            out["dz"][:, :, s] = gy * y * sg * (1 + zz * (1 - sg))
        mu = torch.empty_like(h)
        cur = torch.zeros(bn, nd, N, dtype=f, device=x.device)
        for t in range(L - 1, -1, -1):
            mu[t] = torch.addcmul(cur, gc[t][..., None], Cc[t][:, None, :])
            cur = torch.exp(dlc[t][..., None] * w) * mu[t]
        R = cur.view(b, nc, nd, N)
        Kc = torch.empty_like(H)
        cur = torch.zeros(b, nd, N, dtype=f, device=x.device)
        for q in range(nc - 1, -1, -1):
            Kc[:, q] = cur
            cur = P[:, q] * cur + R[:, q]
        if "dh0" not in out:
            out["dh0"] = torch.empty(b, D, N, dtype=f, device=x.device)
        out["dh0"][:, s] = cur
        Kf = Kc.view(bn, nd, N)
        for t in range(L):
            mu[t].addcmul_(torch.exp((cum[-1] - cum[t])[..., None] * w), Kf)
        if 0 < tbar < T:  # mubar_i = mu_i - P(i, i + tbar) mu_{i + tbar}
            m = mu.view(L, b, nc, nd, N).permute(1, 2, 0, 3, 4).reshape(b, Tp, nd, N)
            S = dl.cumsum(1)
            blk = max(1, (1 << 26) // (b * nd * N))
            for i0 in range(0, T - tbar, blk):  # in order: what is read lies ahead of what is written
                i1 = min(T - tbar, i0 + blk)
                Pw = torch.exp((S[:, i0 + tbar:i1 + tbar] - S[:, i0:i1])[..., None] * w)
                m[:, i0:i1] -= Pw * m[:, i0 + tbar:i1 + tbar].clone()
            mu = m.view(b, nc, L, nd, N).permute(2, 0, 1, 3, 4).reshape(L, bn, nd, N)
            del m
        dA = torch.zeros(nd, N, dtype=f, device=x.device)
        dxs, dds = [], []
        for t in range(L):
            hp = h[t - 1] if t else Hf
            sv = mu[t] * torch.exp(dlc[t][..., None] * w) * hp
            dds.append((sv * w).sum(-1))
            dA += (sv * dlc[t][..., None]).sum(0)
            dxs.append((mu[t] * Bc[t][:, None, :]).sum(-1))
            dBc[t] += (mu[t] * xin[t][..., None]).sum(1)
            dCc[t] += (gc[t][..., None] * h[t]).sum(1)
        dx, dd = flat(torch.stack(dxs)), flat(torch.stack(dds))
        if b_delta:
            dd = dd + dx * xr
            dx = dx * dl
        out["dx"][:, :, s] = dx
        out["ddelta"][:, :, s] = dd * torch.sigmoid(pre) if softplus else dd
        out["dA_log"][s] = dA * w
        del h, mu
    if grad:
        out["dB"], out["dC"] = flat(dBc).contiguous(), flat(dCc).contiguous()
        if A_log.dim() == 1:
            out["dA_log"] = out["dA_log"].sum(-1)
    return out


def _layer64(u, x, z, delta, B, C, W_x, W_in, A_log, dy, tbar, du=False):
    f = torch.float64
    D = x.shape[-1]
    s = _scan64(x, delta, A_log, B, C, dy, None, z, True, tbar)
    dzx = torch.cat([s["ddelta"], s["dB"], s["dC"]], -1).reshape(-1, W_x.shape[1])
    o = {"dA_log": s["dA_log"], "dW_x": x.reshape(-1, D).to(f).t().contiguous() @ dzx}
    dxt = s["dx"].reshape(-1, D) + dzx @ W_x.to(f).t().contiguous()
    dxz = torch.cat([dxt, s["dz"].reshape(-1, D)], -1)
    o["dW_in"] = u.reshape(-1, u.shape[-1]).to(f).t().contiguous() @ dxz
    if du:
        o["du"] = (dxz @ W_in.to(f).t().contiguous()).view(u.shape)
    return o


def _stack64(c, i):
    f = torch.float64
    y, D, N, K = i["y0"].to(f), c["D"], c["N"], c["K"]
    kept = []
    for k in range(K):
        r = torch.rsqrt(y.square().mean(-1, keepdim=True) + 1e-6)
        u = y * r
        xz = u @ i["W_in"][k].to(f)
        x, z = xz[..., :D].contiguous(), xz[..., D:].contiguous()
        p = x @ i["W_x"][k].to(f)
        d, B, C = p[..., :D].contiguous(), p[..., D:D + N].contiguous(), p[..., D + N:].contiguous()
        kept.append((r, u, x, z, d, B, C))
        y = y + _scan64(x, d, i["A_log"][k], B, C, None, None, z, True, 0, grad=False)["y"]
    o = {"dW_in": [None] * K, "dW_x": [None] * K, "dA_log": [None] * K, "yK": y}
    g = i["gK"].to(f)
    for k in range(K - 1, -1, -1):
        r, u, x, z, d, B, C = kept[k]
        want = c["exact"] and k > 0
        l = _layer64(u, x, z, d, B, C, i["W_x"][k], i["W_in"][k], i["A_log"][k], g, c["tbar"], du=want)
        for n in ("dW_in", "dW_x", "dA_log"):
            o[n][k] = l[n]
        if want:
            g = g + (l["du"] - u * (l["du"] * u).mean(-1, keepdim=True)) * r
    return o


def _head64(c, i):
    f = torch.float64
    om = i["omega"].to(f)
    y = i["y"].to(f)
    r = torch.rsqrt(y.square().mean(-1, keepdim=True) + 1e-6)
    u = y * r if c["norm"] else y
    loss = torch.empty(c["M"], dtype=f, device=y.device)
    du = torch.empty_like(y)
    dom = torch.zeros_like(om)
    omt = om.t().contiguous()
    for m0 in range(0, c["M"], 4096):
        s = slice(m0, min(c["M"], m0 + 4096))
        o = u[s] @ omt
        t = i["targets"][s].long()[:, None]
        lse = torch.logsumexp(o, -1, keepdim=True)
        loss[s] = (lse - o.gather(1, t))[:, 0]
        g = torch.exp(o - lse)
        g.scatter_add_(1, t, torch.full_like(lse, -1.0))
        du[s] = g @ om
        dom += g.t().contiguous() @ u[s]
    dy = (du - u * (du * u).mean(-1, keepdim=True)) * r if c["norm"] else du
    return {"loss": loss, "dy": dy, "domega": dom}


def _unstructured64(c, i):
    f = torch.float64
    A, B, C, x, dy, h = (i[n].to(f) for n in ("A", "B", "C", "x", "dy", "h0"))
    b, T = x.shape[:2]
    bx = (B * x[:, :, None, :]).sum(-1)
    v = (C * dy[..., None]).sum(-2)
    hs = torch.empty(T + 1, b, 16, dtype=f, device=x.device)
    hs[0] = h
    At = A.transpose(0, 1).contiguous()
    bxt = bx.transpose(0, 1).contiguous()
    for t in range(T):
        hs[t + 1] = (At[t] * hs[t][:, None, :]).sum(-1).add_(bxt[t])
    if 0 < c["tbar"] < T:  # the vectors of all windows, carried back a step at a time
        tb = c["tbar"]
        w = v[:, tb:].clone()
        n = T - tb
        for s in range(tb, 0, -1):
            w = (A[:, s:s + n] * w[..., None]).sum(-2)
        v = v.clone()
        v[:, :n] -= w
    vt = v.transpose(0, 1).contiguous()
    mu = torch.empty(T, b, 16, dtype=f, device=x.device)
    mu[T - 1] = vt[T - 1]
    for t in range(T - 2, -1, -1):
        mu[t] = (At[t + 1] * mu[t + 1][:, :, None]).sum(-2).add_(vt[t])
    mu, hp, hc = mu.transpose(0, 1), hs[:-1].transpose(0, 1), hs[1:].transpose(0, 1)
    return {"dA": mu[..., None] * hp[:, :, None, :], "dB": mu[..., None] * x[:, :, None, :],
            "dC": dy[..., None] * hc[:, :, None, :], "dx": (B * mu[..., None]).sum(-2)}


def exact(case, seed):
    c, i = prepare(case, seed)
    k = c["kind"]
    if k in ("scan", "pairs"):
        o = _scan64(i["x"], i["delta"], i["A_log"], i["B"], i["C"], i["dy"], i.get("h0"), i.get("z"),
                    bool(c.get("proj")), c["tbar"], bool(c.get("variant", 0) & 2))
        return {n: o[n] for n in ("dx", "ddelta", "dA_log", "dB", "dC", "dz") if n in o}
    if k == "forward":
        o = _scan64(i["x"], i["delta"], i["A_log"], i["B"], i["C"], None, i.get("h0"), i.get("z"), bool(c["proj"]), 0,
                    grad=False)
        return o["y"], o["h_last"]
    if k == "layer":
        return _layer64(i["u"], i["x"], i["z"], i["delta"], i["B"], i["C"], i["W_x"], i["W_in"], i["A_log"], i["dy"],
                        c["tbar"], c["du"])
    if k == "stack":
        return _stack64(c, i)
    if k == "head":
        return _head64(c, i)
    if k == "unstructured":
        return _unstructured64(c, i)
    f = torch.float64
    X, dZ, W = (i[n].to(f) for n in ("X", "dZ", "W"))
    return X.t().contiguous() @ dZ, dZ @ W.t().contiguous()
