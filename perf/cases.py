"""What a program that serves a model with clustered heads asks of this library, one layer at a time: decode steps
over bf16, fp32 and quantised caches, prompt attention, the projections that feed both, and the membership step.

A case is a plain dict.  "path" names the call; sizes are B batch rows, H heads, k clusters, T cached tokens (the new
one included), cap the capacity of the caches, Tq prompt positions from q_start on, Tn projected tokens, D model width.
All tensors are drawn on the GPU from the seed alone.
"""
import math
import random

import numpy as np
import torch

import paper_2403_08058_amd as C

D_HEAD = 128
SCALE = float(np.float32(1.0 / math.sqrt(D_HEAD)))
N_TOK = 5                          # tokens whose attention scores decide the membership
MAX_PASSES = 50                    # bound of the k-means passes, the entry point's default


def listed():
    return [
        # one request, short context, fp32: the smallest call, nothing but latency
        {"name": "decode_fp32_small", "path": "attention", "B": 1, "H": 32, "k": 8, "T": 256, "cap": 256, "dtype": "f32"},
        # the ordinary decode step of a full batch, cache growth included
        {"name": "decode_step_16x32", "path": "step", "B": 16, "H": 32, "k": 8, "T": 2048, "cap": 2048, "dtype": "bf16"},
        # a small batch soon after a 512-token prompt: many heads, short ragged context inside a larger cache
        {"name": "decode_step_4x72_short", "path": "step", "B": 4, "H": 72, "k": 16, "T": 577, "cap": 2048, "dtype": "bf16"},
        # long documents, one dominant cluster: the largest decode call
        {"name": "decode_step_long", "path": "step", "B": 4, "H": 32, "k": 4, "T": 32768, "cap": 32768, "dtype": "bf16",
         "skewed": True},
        # an unclustered layer of a single request
        {"name": "decode_dense_single", "path": "dense", "B": 1, "H": 52, "k": 52, "T": 1777, "cap": 2048, "dtype": "bf16"},
        # a full batch over 8-bit caches: the new rows quantised into the caches, then attention
        {"name": "decode_q8_16x32", "path": "q8", "B": 16, "H": 32, "k": 8, "T": 2048, "cap": 2048, "dtype": "bf16"},
        # a batch of full-length prompts in one block, after the membership decision on the first five positions
        {"name": "prefill_16x2043", "path": "prefill", "B": 16, "H": 32, "k": 8, "Tq": 2043, "q_start": 5},
        # a small batch of short prompts
        {"name": "prefill_4x507", "path": "prefill", "B": 4, "H": 72, "k": 16, "Tq": 507, "q_start": 5},
        # a prompt that is processed in blocks: 256 positions behind 1792 that are cached already
        {"name": "prefill_block_behind", "path": "prefill", "B": 4, "H": 52, "k": 8, "Tq": 256, "q_start": 1792},
        # query and key projections of the representatives over a batch of prompts
        {"name": "project_prompt", "path": "project", "B": 16, "H": 32, "k": 8, "Tn": 2043, "D": 4096, "pos0": 5},
        # the same for the one new token of every request: a decode step's projections
        {"name": "project_token", "path": "project", "B": 16, "H": 32, "k": 8, "Tn": 1, "D": 4096, "pos0": 1023},
        # the membership decision and the pruning of the key cache after a prompt
        {"name": "membership_4x72", "path": "membership", "B": 4, "H": 72, "k": 16, "T": 512, "cap": 512, "quantise": False},
    ]


# cost of the largest listed calls: no drawn case passes it
MOST_BYTES = 1.2e9
MOST_FLOPS = 3.4e11


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng: random.Random):
    while True:
        path = rng.choice(["attention", "step", "step", "dense", "q8", "prefill", "prefill", "project", "project",
                           "membership"])
        H = rng.choice([32, 52, 72])
        case = {"path": path, "B": _log_int(rng, 1, 16), "H": H, "k": rng.choice([4, 8, 16])}
        if path in ("attention", "step", "dense", "q8"):
            T = _log_int(rng, 64, 32768)
            case.update(T=T, cap=T + rng.choice([0, rng.randrange(1, 512)]),
                        dtype="f32" if path != "q8" and rng.random() < 0.25 else "bf16", skewed=rng.random() < 0.3)
            if path == "dense":
                case["k"] = H
        elif path == "prefill":
            case.update(Tq=_log_int(rng, 24, 4096), q_start=rng.choice([0, N_TOK, _log_int(rng, 64, 4096)]))
            if rng.random() < 0.2:
                case["k"] = H                           # an unclustered layer
        elif path == "project":
            case.update(Tn=rng.choice([1, _log_int(rng, 2, 2043)]), D=H * D_HEAD, pos0=rng.randrange(0, 512))
        else:
            T = _log_int(rng, 64, 2048)
            case.update(T=T, cap=T + rng.choice([0, rng.randrange(1, 512)]), quantise=rng.random() < 0.5)
        w = work(case)
        if w["bytes"] <= MOST_BYTES and w["flops"] <= MOST_FLOPS:
            return case


# ------------------------------------------------------------------------------------------------- inputs
def _normal(g, shape, dtype, sigma=1.0):
    x = torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)
    if sigma != 1.0:
        x *= sigma
    return x.to(dtype)


def _maps(case, seed):
    """Head -> cluster maps with no empty cluster, a partition of its own per batch row; representative = lowest member,
    slots numbered by it.  Skewed: one cluster holds most heads."""
    B, H, k = case["B"], case["H"], case["k"]
    g = np.random.default_rng(seed)
    share = np.full(k, 1.0 / k) if not case.get("skewed") else 0.4 ** np.arange(k) / (0.4 ** np.arange(k)).sum()
    h2c, rep = np.empty((B, H), np.int32), np.empty((B, k), np.int32)
    for b in range(B):
        raw = np.concatenate([np.arange(k), g.choice(k, size=H - k, p=share)])[g.permutation(H)]
        first = np.array([np.flatnonzero(raw == j)[0] for j in range(k)])
        order = np.argsort(first)
        label = np.empty(k, np.int64)
        label[order] = np.arange(k)
        h2c[b], rep[b] = label[raw], first[order]
    return torch.from_numpy(h2c).cuda(), torch.from_numpy(rep).cuda()


def _inputs(case, seed):
    path, B, H, k = case["path"], case["B"], case["H"], case["k"]
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    x = {}
    if path in ("attention", "step", "dense", "q8"):
        dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
        x["h2c"], x["rep"] = _maps(case, seed)
        x["q"] = _normal(g, (B, H, D_HEAD), dt)
        x["k"] = _normal(g, (B, k, case["cap"], D_HEAD), dt)
        x["v"] = _normal(g, (B, H, case["cap"], D_HEAD), dt)
        if path in ("step", "q8"):
            x["k_new"], x["v_new"] = _normal(g, (B, H, D_HEAD), dt), _normal(g, (B, H, D_HEAD), dt)
    elif path == "prefill":
        n = case["q_start"] + case["Tq"]
        x["h2c"], x["rep"] = _maps(case, seed)
        x["q"] = _normal(g, (B, H, case["Tq"], D_HEAD), torch.bfloat16)
        x["k"] = _normal(g, (B, k, n, D_HEAD), torch.bfloat16)
        x["v"] = _normal(g, (B, H, n, D_HEAD), torch.bfloat16)
    elif path == "project":
        _, x["rep"] = _maps(case, seed)
        x["x"] = _normal(g, (B, case["Tn"], case["D"]), torch.bfloat16)
        x["w_q"] = _normal(g, (H * D_HEAD, case["D"]), torch.bfloat16, 0.05)
        x["w_k"] = _normal(g, (H * D_HEAD, case["D"]), torch.bfloat16, 0.05)
    else:
        x["q5"] = _normal(g, (B, H, N_TOK, D_HEAD), torch.bfloat16)
        x["k"] = _normal(g, (B, H, case["cap"], D_HEAD), torch.bfloat16)
        x["v"] = _normal(g, (B, H, case["cap"], D_HEAD), torch.bfloat16) if case["quantise"] else None
        starts = np.random.default_rng(seed)
        x["init"] = torch.from_numpy(np.stack([starts.choice(H, size=k, replace=False) for _ in range(B)]).astype(np.int32)).cuda()
    return x


def prepare(case, seed):
    """The tensors, and the buffers that a serving loop keeps from call to call."""
    path, B, H, k = case["path"], case["B"], case["H"], case["k"]
    s = _inputs(case, seed)
    s["case"] = case
    new = lambda shape, dt: torch.zeros(shape, dtype=dt, device="cuda")  # noqa: E731
    if path in ("attention", "step", "dense"):
        s["out"] = new((B, H, D_HEAD), torch.float32)
        s["ws"] = C.alloc_workspace(B, H, k, case["T"], D_HEAD, C.CHAI_F32 if case["dtype"] == "f32" else C.CHAI_BF16)
    elif path == "q8":
        s["out"] = new((B, H, D_HEAD), torch.float32)
        s["k8"], s["ks"] = C.chai_quantize_rows(s.pop("k"))
        s["v8"], s["vs"] = C.chai_quantize_rows(s.pop("v"))
        s["ws"] = new((max(256, C.chai_decode_q8_workspace_bytes(B, H, k, case["T"])),), torch.uint8)
    elif path == "prefill":
        s["out"] = new((B, H, case["Tq"], D_HEAD), torch.float32)
        s["ws"] = new((C.chai_prefill_workspace_bytes(B, H, k, case["q_start"] + case["Tq"]),), torch.uint8)
    elif path == "project":
        s["q_out"] = new((B, H, case["Tn"], D_HEAD), torch.bfloat16)
        s["kc"] = new((B, k, case["pos0"] + case["Tn"], D_HEAD), torch.bfloat16)
    else:
        s["feat"] = new((B, H, N_TOK * N_TOK), torch.float32)
        s["h2c"], s["rep"] = new((B, H), torch.int32), new((B, k), torch.int32)
        s["ncl"], s["iters"] = new((B,), torch.int32), new((B,), torch.int32)
        s["kc"] = new((B, k, case["cap"], D_HEAD), torch.bfloat16)
        if case["quantise"]:
            s["k8"], s["ks"] = new(s["kc"].shape, torch.uint8), new(s["kc"].shape[:3], torch.float32)
            s["v8"], s["vs"] = new(s["v"].shape, torch.uint8), new(s["v"].shape[:3], torch.float32)
    return s


def run(s):
    case = s["case"]
    path = case["path"]
    if path == "attention":
        return C.chai_decode_attention(s["q"], s["k"], s["v"], s["h2c"], s["rep"], case["T"], SCALE, s["out"], s["ws"])
    if path == "step":
        C.chai_decode_step(s["q"], s["k_new"], s["v_new"], s["k"], s["v"], s["h2c"], s["rep"], case["T"], SCALE, s["out"],
                           s["ws"])
        return {"out": s["out"], "k": s["k"], "v": s["v"]}
    if path == "dense":
        return C.chai_dense_decode_attention(s["q"], s["k"], s["v"], case["T"], SCALE, s["out"], s["ws"])
    if path == "q8":
        C.chai_append_kv_q8(s["k_new"], s["v_new"], s["rep"], s["k8"], s["ks"], s["v8"], s["vs"], case["T"] - 1)
        C.chai_decode_attention_q8(s["q"], s["k8"], s["ks"], s["v8"], s["vs"], s["h2c"], s["rep"], case["T"], SCALE, s["out"],
                                   s["ws"])
        return {"out": s["out"], "k8": s["k8"], "ks": s["ks"], "v8": s["v8"], "vs": s["vs"]}
    if path == "prefill":
        if case["k"] == case["H"]:
            return C.chai_dense_prefill_attention(s["q"], s["k"], s["v"], case["q_start"], SCALE, s["out"], s["ws"])
        return C.chai_prefill_attention(s["q"], s["k"], s["v"], s["h2c"], s["rep"], case["q_start"], SCALE, s["out"], s["ws"])
    if path == "project":
        C.chai_project_qk(s["x"], s["w_q"], s["w_k"], s["rep"], s["q_out"], s["kc"], case["pos0"])
        return {"q": s["q_out"], "k": s["kc"]}
    C.chai_score_features(s["q5"], s["k"], N_TOK, SCALE, s["feat"])
    C.chai_assign_clusters(s["feat"], s["init"], MAX_PASSES, s["h2c"], s["rep"], s["ncl"], s["iters"])
    C.chai_compact_kcache(s["k"], s["rep"], s["kc"], case["T"])
    got = {"feat": s["feat"], "h2c": s["h2c"], "rep": s["rep"], "ncl": s["ncl"], "iters": s["iters"], "kc": s["kc"]}
    if case["quantise"]:
        C.chai_quantize_rows(s["kc"], s["k8"], s["ks"])
        C.chai_quantize_rows(s["v"], s["v8"], s["vs"])
        got.update(k8=s["k8"], ks=s["ks"], v8=s["v8"], vs=s["vs"])
    return got


def work(case):
    path, B, H, k = case["path"], case["B"], case["H"], case["k"]
    if path in ("attention", "step", "dense", "q8"):
        T = case["T"]
        e = 4 if case["dtype"] == "f32" else 2
        row = D_HEAD + 4 if path == "q8" else D_HEAD * e                   # one cached row: codes and scale, or elements
        b = B * (k + H) * T * row + B * k * D_HEAD * e + 2 * B * H * 4 + B * H * D_HEAD * 4
        if path in ("step", "q8"):
            b += B * (k + H) * D_HEAD * e                                  # the new token's rows
        return {"bytes": b, "flops": 2 * B * (k + H) * T * D_HEAD}
    if path == "prefill":
        Tq, n = case["Tq"], case["q_start"] + case["Tq"]
        pairs = Tq * case["q_start"] + Tq * (Tq + 1) // 2
        return {"bytes": B * (k + H) * n * D_HEAD * 2 + B * k * Tq * D_HEAD * 2 + B * H * Tq * D_HEAD * 4,
                "flops": 2 * D_HEAD * (k + H) * B * pairs}
    if path == "project":
        Tn, D = case["Tn"], case["D"]
        heads = H * (1.0 - (1.0 - k / H) ** B)                             # heads that represent some row's cluster
        return {"bytes": B * Tn * D * 2 + 2 * heads * D_HEAD * D * 2 + 2 * B * k * Tn * D_HEAD * 2,
                "flops": 2.0 * B * Tn * D * 2 * k * D_HEAD}
    T = case["T"]
    b = 2 * B * H * N_TOK * D_HEAD * 2 + B * H * N_TOK * N_TOK * 4 + 2 * B * k * T * D_HEAD * 2
    if case["quantise"]:
        b += B * (k + H) * case["cap"] * (2 * D_HEAD + D_HEAD + 4)
    return {"bytes": b, "flops": 2 * B * H * N_TOK * (N_TOK + 1) // 2 * D_HEAD}


def tolerance(case):
    path = case["path"]
    if path in ("attention", "step", "dense", "q8"):
        return {"rel": 1e-5, "max": 1e-4}          # fp32 sums in another order; grown caches are copies
    if path == "prefill":
        return {"rel": 1e-3, "max": 2e-2}          # probabilities carry 11 bits into the second product
    if path == "project":
        return {"rel": 2e-3, "max": 1e-2}          # one rounding to bf16
    return {"rel": 1e-6, "max": 1e-5}              # features rounded once to fp32; labels, counts and copies the same


# ------------------------------------------------------------------------------------------------- 64 bits
def _quantised(x):
    """Rows as the 8-bit caches hold them, dequantised: nearest E4M3 of x * (448 / max) with scale max / 448."""
    f = x.float()
    top = f.abs().amax(-1, keepdim=True)
    full = torch.full_like(top, 448.0)                 # tensor by tensor: rounded divisions, not a reciprocal's product
    inv = torch.where(top > 0, full / top, torch.zeros_like(top))
    return (f * inv).clamp(-448, 448).to(torch.float8_e4m3fn).double() * (top / full).double()


def exact(case, seed):
    x = _inputs(case, seed)
    path, B, H, k = case["path"], case["B"], case["H"], case["k"]
    if path in ("attention", "step", "dense", "q8"):
        T = case["T"]
        out = torch.empty((B, H, D_HEAD), dtype=torch.float64, device="cuda")
        for b in range(B):
            rep = torch.arange(H, device="cuda") if path == "dense" else x["rep"][b].long()
            lab = rep if path == "dense" else x["h2c"][b].long()
            kk, vv = x["k"][b, :, :T], x["v"][b, :, :T]
            if path in ("step", "q8"):
                kk, vv = kk.clone(), vv.clone()
                kk[:, T - 1], vv[:, T - 1] = x["k_new"][b, rep], x["v_new"][b]
            if path == "q8":
                kk, vv = _quantised(kk), _quantised(vv)
            p = torch.softmax(SCALE * (kk.double() * x["q"][b, rep].double()[:, None, :]).sum(-1), -1)
            for h in range(H):
                out[b, h] = p[lab[h]] @ vv[h].double()
        if path in ("attention", "dense"):
            return out
        if path == "step":
            return {"out": out, "k": None, "v": None}
        return {"out": out, "k8": None, "ks": None, "v8": None, "vs": None}
    if path == "prefill":
        Tq, n, q0 = case["Tq"], case["q_start"] + case["Tq"], case["q_start"]
        dense = k == H
        out = torch.empty((B, H, Tq, D_HEAD), dtype=torch.float64, device="cuda")
        pos = torch.arange(q0, n, device="cuda")[:, None]
        hidden = torch.arange(n, device="cuda")[None, :] > pos
        for b in range(B):
            rep = range(H) if dense else x["rep"][b].tolist()
            lab = range(H) if dense else x["h2c"][b].tolist()
            for j, r in enumerate(rep):
                s = SCALE * (x["q"][b, r].double() @ x["k"][b, j].double().t().contiguous())
                p = torch.softmax(s.masked_fill_(hidden, -math.inf), -1)
                for h in range(H):
                    if lab[h] == j:
                        out[b, h] = p @ x["v"][b, h].double()
        return out
    if path == "project":
        Tn, pos0 = case["Tn"], case["pos0"]
        q = torch.zeros((B, H, Tn, D_HEAD), dtype=torch.float64, device="cuda")
        kc = torch.zeros((B, k, pos0 + Tn, D_HEAD), dtype=torch.float64, device="cuda")
        for b in range(B):
            xb = x["x"][b].double()
            for j, r in enumerate(x["rep"][b].tolist()):
                rows = slice(r * D_HEAD, (r + 1) * D_HEAD)
                q[b, r] = xb @ x["w_q"][rows].double().t().contiguous()
                kc[b, j, pos0:] = xb @ x["w_k"][rows].double().t().contiguous()
        return {"q": q, "k": kc}
    s = SCALE * (x["q5"].double()[:, :, :, None, :] * x["k"][:, :, None, :N_TOK].double()).sum(-1)
    hidden = torch.ones((N_TOK, N_TOK), dtype=torch.bool, device="cuda").triu(1)
    feat = torch.softmax(s.masked_fill(hidden, -math.inf), -1).reshape(B, H, N_TOK * N_TOK)
    got = {"feat": feat, "h2c": None, "rep": None, "ncl": None, "iters": None, "kc": None}
    if case["quantise"]:
        got.update(k8=None, ks=None, v8=None, vs=None)
    return got
