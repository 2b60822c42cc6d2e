"""The work that a user of this framework has it do, as cases that can be timed
and compared: scoring batches of candidate programs, the distillation steps,
the progressive forward and what consumes the scores.

  listed()            the cases, dicts of plain values
  draw(rng)           one more case of the same ranges
  prepare(case, seed) inputs, models and workspaces, as a program holds them
  run(state)          one pass through the public entry points; its outputs
  work(case)          bytes and operations that one pass cannot do without
  tolerance(case)     how far another correct implementation may be off
  exact(case, seed)   the same outputs in 64 bits, in plain torch

Features are log1p(lognormal(0, 1)) per entry (zero past a program's length),
lengths uniform, weights U(+-1/sqrt(fan_in)) with jittered gains, A_log, D
and dt biases, as a trained model's differ per channel.
"""
from __future__ import annotations

import math

import numpy as np
import torch
import torch.nn.functional as F

from paper_2604_12891_amd import binding as tb

# The models of this repository's workloads: the small one, the 256-wide one
# that its scoring workloads use, the distillation student and the paper's own
# model on 41 x 20 inputs (three-layer encoder and decoder, d_state 8).
MODELS = {
    "tiny": dict(F=164, d_model=64, d_inner=128, d_state=16, d_conv=4, dt_rank=4, n_layers=2, head_hidden=64),
    "d256": dict(F=164, d_model=256, d_inner=512, d_state=16, d_conv=4, dt_rank=16, n_layers=4, head_hidden=256),
    "student": dict(F=164, d_model=128, d_inner=256, d_state=16, d_conv=4, dt_rank=8, n_layers=2, head_hidden=128),
    "paper": dict(F=20, d_model=128, d_inner=128, d_state=8, d_conv=4, dt_rank=8, n_layers=1, head_hidden=64,
                  enc_hidden=(64, 128), dec_hidden2=32),
}
EPS = 1e-5
LR, BETA1, BETA2, ADAM_EPS = 1e-3, 0.9, 0.999, 1e-8
KD = dict(beta=0.5, phi=0.7, sigma=1.0, ewc_lambda=1e4)  # the paper's beta and lambda


def listed():
    return [
        # the smallest call: a handful of candidates looked at again, latency only
        dict(name="score_few_f32", kind="score", model="d256", dtype="f32", B=8, L=25, lo=5),
        # a small model on a small batch
        dict(name="score_small_model_f32", kind="score", model="tiny", dtype="f32", B=64, L=25, lo=5),
        # one tuning round, the headline workload
        dict(name="score_round_f32", kind="score", model="d256", dtype="f32", B=4096, L=25, lo=5),
        # long programs, the largest fp32 call
        dict(name="score_long_f32", kind="score", model="d256", dtype="f32", B=8192, L=256, lo=64),
        # a whole pool at once in bf16
        dict(name="score_pool_bf16", kind="score", model="d256", dtype="bf16", B=65536, L=25, lo=5),
        # odd sizes, below the two-halves limit
        dict(name="score_ragged_bf16", kind="score", model="d256", dtype="bf16", B=1531, L=77, lo=3),
        # the paper's own model on its GPU traces' input shape
        dict(name="score_paper_f32", kind="score", model="paper", dtype="f32", B=4096, L=41, lo=8),
        # continual learning: the active column beside the frozen knowledge base
        dict(name="progressive_f32", kind="progressive", model="paper", dtype="f32", B=4096, L=41, lo=8, adapter=8),
        # one teacher -> student training step, two mean squared errors
        dict(name="distill_step", kind="distill", model="d256", dtype="bf16", B=1024, L=25, lo=5),
        # the paper's distillation objective (two LambdaRank terms, gate, EWC) on an odd batch
        dict(name="distill_kd_ragged", kind="distill_kd", model="d256", dtype="bf16", B=509, L=61, lo=7),
        # the RDU sampler over one platform's dataset
        dict(name="rdu_dataset", kind="rdu", N=8_650_000, n_ops=20, n_initial=1024, n_select=64),
        # the best candidates of each of a round's tasks
        dict(name="topk_tasks", kind="topk", n_seg=16, seg=4096, K=64),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["score"] * 6 + ["progressive", "distill", "distill_kd", "rdu", "topk"])
    if kind == "rdu":
        N = _log(rng, 4000, 8_650_000)
        return dict(kind=kind, N=N, n_ops=rng.randint(1, 64), n_initial=_log(rng, 1, min(2048, N // 4)),
                    n_select=_log(rng, 8, 128))
    if kind == "topk":
        n_seg = _log(rng, 1, 512)
        return dict(kind=kind, n_seg=n_seg, seg=_log(rng, 32, min(65536, 2_000_000 // n_seg)), K=_log(rng, 1, 512))
    if kind == "progressive":
        L = rng.randint(4, 96)
        B = _log(rng, 1, min(32768, 400_000 // L))
        return dict(kind=kind, model="paper", dtype="f32", B=B, L=L, lo=max(1, L // 5), adapter=rng.choice([4, 8, 12, 16]))
    if kind.startswith("distill"):
        L = rng.randint(9, 130)
        return dict(kind=kind, model="d256", dtype="bf16", B=_log(rng, 32, min(2048, 40_000 // L)), L=L,
                    lo=max(1, L // 5))
    model = rng.choice(["tiny", "d256", "d256", "student", "paper"])
    L = _log(rng, 8, 256)
    B = _log(rng, 1, min(65536, 1_600_000 // L))
    dtype = "f32" if model == "paper" else rng.choice(["f32", "bf16"])
    return dict(kind=kind, model=model, dtype=dtype, B=B, L=L, lo=max(1, L // 5))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _layout(m):
    """Names and shapes of a model's parameters in the blob's order."""
    d, E, N, K, R, h = (m[k] for k in ("d_model", "d_inner", "d_state", "d_conv", "dt_rank", "head_hidden"))
    dims = [m["F"], *m.get("enc_hidden", ()), d]
    out = []
    for i in range(len(dims) - 1):
        out += [(f"enc{i}.W", (dims[i + 1], dims[i])), (f"enc{i}.b", (dims[i + 1],))]
    for i in range(m["n_layers"]):
        out += [(f"{i}.g", (d,)), (f"{i}.W_in", (2 * E, d)), (f"{i}.conv_w", (E, K)), (f"{i}.conv_b", (E,)),
                (f"{i}.W_x", (R + 2 * N, E)), (f"{i}.W_dt", (E, R)), (f"{i}.b_dt", (E,)), (f"{i}.A_log", (E, N)),
                (f"{i}.D", (E,)), (f"{i}.W_out", (d, E))]
    dec = [d, h, *([m["dec_hidden2"]] if m.get("dec_hidden2") else []), 1]
    out += [("g_f", (d,))]
    for i in range(len(dec) - 1):
        out += [(f"dec{i}.W", (dec[i + 1], dec[i])), (f"dec{i}.b", (dec[i + 1],))]
    return out


def _widths(m):
    """(inputs, outputs) of every layer after the first, in forward order."""
    d = m["d_model"]
    enc = [*m.get("enc_hidden", ()), d]
    dec = [d, m["head_hidden"], *([m["dec_hidden2"]] if m.get("dec_hidden2") else []), 1]
    return list(zip(enc[:-1], enc[1:])) + [(d, d)] * m["n_layers"] + list(zip(dec[:-1], dec[1:]))


def _blob(m, rng, dtype):
    parts, fan = [], 1
    for name, shape in _layout(m):
        base = name.split(".")[-1]
        if base.startswith("W"):
            fan = shape[1]
            a = rng.uniform(-1, 1, shape) / math.sqrt(fan)
        elif base == "b":
            a = rng.uniform(-1, 1, shape) / math.sqrt(fan)
        elif base.startswith("conv"):
            a = rng.uniform(-1, 1, shape) / math.sqrt(m["d_conv"])
        elif base in ("g", "g_f"):
            a = 1.0 + 0.2 * rng.standard_normal(shape)
        elif base == "A_log":
            a = np.log(np.arange(1, m["d_state"] + 1)) + 0.3 * rng.standard_normal(shape)
        elif base == "D":
            a = 1.0 + 0.5 * rng.standard_normal(shape)
        else:  # b_dt: softplus(b_dt) log-uniform in [1e-3, 1e-1]
            t = np.exp(rng.uniform(math.log(1e-3), math.log(1e-1), shape))
            a = t + np.log(-np.expm1(-t))
        parts.append(np.asarray(a, np.float32).reshape(-1))
    blob = np.concatenate(parts)
    # a bf16 model's weights are bf16 values
    return torch.from_numpy(blob).bfloat16().float().numpy() if dtype == "bf16" else blob


def _lateral(m, a, rng):
    parts = []
    for n_in, n_out in _widths(m):
        bv, bu = 1 / math.sqrt(n_in), 1 / math.sqrt(a)
        parts += [rng.uniform(-bv, bv, a * n_in), rng.uniform(-bv, bv, a), rng.uniform(-bu, bu, n_out * a),
                  rng.uniform(0.5, 1.5, n_out)]
    return np.concatenate(parts).astype(np.float32)


def _programs(case, seed, n_feat):
    g = torch.Generator(device="cuda").manual_seed(seed)
    B, L = case["B"], case["L"]
    lengths = torch.randint(case["lo"], L + 1, (B,), generator=g, device="cuda", dtype=torch.int32)
    X = torch.randn(B, L, n_feat, generator=g, device="cuda").exp_().log1p_()
    X.masked_fill_((torch.arange(L, device="cuda")[None, :] >= lengths[:, None])[:, :, None], 0.0)
    return X, lengths, g


def _inputs(case, seed):
    """Everything a pass reads, from the seed alone."""
    kind = case["kind"]
    if kind in ("rdu", "topk"):
        g = torch.Generator(device="cuda").manual_seed(seed)
        if kind == "rdu":
            N = case["N"]
            share = torch.rand(case["n_ops"], generator=g, device="cuda") + 0.2
            op = torch.bucketize(torch.rand(N, generator=g, device="cuda"), (share / share.sum()).cumsum(0)[:-1])
            first = torch.randperm(N, generator=g, device="cuda")[:case["n_initial"]]
            return dict(scores=0.3 * torch.randn(N, generator=g, device="cuda"), op=op.int(), initial=first.int())
        # segments of uneven length around case["seg"]
        size = (case["seg"] * (0.5 + torch.rand(case["n_seg"], generator=g, device="cuda"))).int().clamp_(min=1)
        offs = torch.zeros(case["n_seg"] + 1, dtype=torch.int32, device="cuda")
        offs[1:] = size.cumsum(0)
        return dict(scores=0.3 * torch.randn(int(offs[-1]), generator=g, device="cuda"), offs=offs)
    m, rng = MODELS[case["model"]], np.random.default_rng(seed)
    X, lengths, g = _programs(case, seed, m["F"])
    d = dict(X=X, lengths=lengths, blob=_blob(m, rng, case["dtype"]))
    if kind == "progressive":
        d.update(kb=_blob(m, rng, "f32"), lat=_lateral(m, case["adapter"], rng))
    if kind.startswith("distill"):
        d["student"] = _blob(MODELS["student"], rng, "bf16")
        # labels that depend on the program, with measurement noise
        w = torch.randn(m["F"], generator=g, device="cuda")
        y = (X.sum(1) / lengths[:, None]) @ w
        d["labels"] = 0.1 * (y - y.mean()) + 0.05 * torch.randn(case["B"], generator=g, device="cuda")
        n = d["student"].size
        d["fisher"] = 1e-5 * torch.rand(n, generator=g, device="cuda") ** 2
        prev = torch.from_numpy(d["student"]).cuda()
        d["theta_prev"] = prev + 1e-3 * torch.randn(n, generator=g, device="cuda")
    return d


def _config(name, dtype):
    m = dict(MODELS[name])
    return tb.make_config(**m, final_norm=1, norm_eps=EPS, dtype=dtype)


def prepare(case, seed):
    s = dict(_inputs(case, seed), case=case)
    kind = case["kind"]
    if kind == "rdu":
        need = tb.lib().tcl_rdu_workspace_bytes(case["N"], case["n_ops"])
        s["ws"] = torch.empty(max(need, 256), dtype=torch.uint8, device="cuda")
    elif kind != "topk":
        B, L = case["B"], case["L"]
        s["net"] = tb.CostModel(_config(case["model"], case["dtype"]), s["blob"])
        if kind == "score":
            s["net"].workspace(B, L)
        elif kind == "progressive":
            s["prog"] = tb.Progressive(tb.CostModel(_config(case["model"], "f32"), s["kb"]), s["net"],
                                       case["adapter"], s["lat"])
            s["prog"].workspace(B, L)
        else:
            learner = tb.CostModel(_config("student", "bf16"), s["student"])
            s["trainer"] = tb.Trainer(s["net"], learner, lr=LR, betas=(BETA1, BETA2), eps=ADAM_EPS, max_B=B, max_L=L)
            s["trainer"].workspace(B, L)
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "score":
        return s["net"].score(s["X"], s["lengths"])
    if kind == "progressive":
        return s["prog"].score(s["X"], s["lengths"])
    if kind == "distill":
        loss = s["trainer"].step(s["X"], s["lengths"], s["labels"])
        return dict(loss=loss, grads=s["trainer"].grads())
    if kind == "distill_kd":
        loss = s["trainer"].step_kd(s["X"], s["lengths"], s["labels"], **KD, fisher=s["fisher"],
                                    theta_prev=s["theta_prev"])
        return dict(loss=loss, grads=s["trainer"].grads())
    if kind == "rdu":
        selected, count = tb.rdu_select(s["scores"], s["op"], case["n_ops"], s["initial"], case["n_select"],
                                        workspace=s["ws"])
        return dict(selected=selected, count=count)
    return tb.topk(s["scores"], s["offs"], case["K"])


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def _params(m):
    return sum(int(np.prod(shape)) for _, shape in _layout(m))


def _forward_flops(m, tokens, B):
    d, E, N, K, R = (m[k] for k in ("d_model", "d_inner", "d_state", "d_conv", "dt_rank"))
    dims = [m["F"], *m.get("enc_hidden", ()), d]
    per_token = sum(2 * a * b for a, b in zip(dims[:-1], dims[1:]))
    # in_proj, conv, x_proj, dt_proj, the scan (five operations and one
    # exponential per state), out_proj
    per_token += m["n_layers"] * (2 * d * 2 * E + 2 * E * K + 2 * E * (R + 2 * N) + 2 * R * E + 6 * E * N + 2 * E * d)
    dec = [d, m["head_hidden"], *([m["dec_hidden2"]] if m.get("dec_hidden2") else []), 1]
    return per_token * tokens + B * sum(2 * a * b for a, b in zip(dec[:-1], dec[1:]))


def work(case):
    kind = case["kind"]
    if kind == "rdu":  # every selection weighs every candidate: t = f d + u, about ten operations
        return dict(bytes=8.0 * case["N"] + 4.0 * (case["n_initial"] + case["n_select"]),
                    flops=10.0 * case["N"] * case["n_select"])
    if kind == "topk":
        n = case["n_seg"] * case["seg"]
        return dict(bytes=4.0 * n + 4.0 * case["n_seg"] * case["K"], flops=1.0 * n)
    m, B = MODELS[case["model"]], case["B"]
    tokens = B * (case["lo"] + case["L"]) / 2
    flops = _forward_flops(m, tokens, B)
    size = 2 if case["dtype"] == "bf16" else 4
    nbytes = 4 * m["F"] * tokens + 8 * B + size * _params(m)
    if kind == "progressive":
        a = case["adapter"]
        widths = _widths(m)
        token_layers = len(m["enc_hidden"]) + m["n_layers"]
        flops = 2 * flops + sum(2 * a * (i + o) * (tokens if j < token_layers else B)
                                for j, (i, o) in enumerate(widths))
        nbytes += 4 * _params(m) + 4 * sum(a * (i + o + 1) + o for i, o in widths)
    elif kind.startswith("distill"):
        st = MODELS["student"]
        flops += 3 * _forward_flops(st, tokens, B)
        # the student's parameters and moments read and written, its gradient written
        nbytes += 4 * B + 28 * _params(st) + (8 * _params(st) if kind == "distill_kd" else 0)
    return dict(bytes=float(nbytes), flops=float(flops))


def tolerance(case):
    """About four times the largest error against exact() that was measured over
    several seeds of every listed case."""
    kind = case["kind"]
    if kind in ("rdu", "topk"):
        return "exact"
    if kind == "distill_kd":  # two scores within rounding may be ranked either way: 2.9e-2 measured
        return dict(rel=3e-2, max=0.9)
    if kind == "distill":  # 1.7e-3 in norm, 8e-2 at one entry
        return dict(rel=1e-2, max=0.35)
    if case["dtype"] == "bf16":  # 3.3e-3, 1.3e-2
        return dict(rel=1.3e-2, max=6e-2)
    return dict(rel=1.5e-5, max=6e-5)  # 3.5e-6, 1.5e-5


# ---------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------

def _unpack(blob, m, grad=False):
    v = torch.as_tensor(blob).cuda().double().requires_grad_(grad)
    out, at = {}, 0
    for name, shape in _layout(m):
        n = int(np.prod(shape))
        out[name] = v[at:at + n].view(shape)
        at += n
    return out, v


def _rmsnorm(h, g):
    return h * torch.rsqrt(h.square().mean(-1, keepdim=True) + EPS) * g


def _block(P, i, h, m):
    E, N, K, R = (m[k] for k in ("d_inner", "d_state", "d_conv", "dt_rank"))
    B, L, _ = h.shape
    x, z = (_rmsnorm(h, P[f"{i}.g"]) @ P[f"{i}.W_in"].t()).split(E, -1)
    pad = F.pad(x, (0, 0, K - 1, 0))
    u = F.silu(P[f"{i}.conv_b"] + sum(P[f"{i}.conv_w"][:, k] * pad[:, k:k + L] for k in range(K)))
    r, Bm, Cm = (u @ P[f"{i}.W_x"].t()).split([R, N, N], -1)
    dt = F.softplus(r @ P[f"{i}.W_dt"].t() + P[f"{i}.b_dt"], threshold=1000.0)
    A = -P[f"{i}.A_log"].exp()
    s, ys = torch.zeros(B, E, N, dtype=h.dtype, device=h.device), []
    for t in range(L):
        s = torch.exp(dt[:, t, :, None] * A) * s + (dt[:, t] * u[:, t])[:, :, None] * Bm[:, t, None, :]
        ys.append((s * Cm[:, t, None, :]).sum(-1))
    y = torch.stack(ys, 1) + P[f"{i}.D"] * u
    return h + (y * F.silu(z)) @ P[f"{i}.W_out"].t()


def _column(P, X, lengths, m, lat=None, kb=None):
    """One column's scores, and every layer's input; with lat and kb (the other
    column's layer inputs) each layer after the first adds its adapter's term."""
    seen = []

    def layer(h, f):
        j = len(seen)
        seen.append(h)
        out = f(h)
        if lat is not None and j:
            V, c, U, alpha = lat[j - 1]
            out = out + alpha * (torch.relu(kb[j] @ V.t() + c) @ U.t())
        return out

    n_enc, n_dec = len(m.get("enc_hidden", ())) + 1, 3 if m.get("dec_hidden2") else 2
    h = X
    for i in range(n_enc):
        h = layer(h, lambda v: v @ P[f"enc{i}.W"].t() + P[f"enc{i}.b"])
        h = torch.relu(h) if i < n_enc - 1 else h
    for i in range(m["n_layers"]):
        h = layer(h, lambda v: _block(P, i, v, m))
    valid = torch.arange(X.shape[1], device=X.device)[None, :] < lengths[:, None]
    v = (_rmsnorm(h, P["g_f"]) * valid[:, :, None]).sum(1) / lengths[:, None]
    for i in range(n_dec):
        v = layer(v, lambda q: q @ P[f"dec{i}.W"].t() + P[f"dec{i}.b"])
        v = torch.relu(v) if i < n_dec - 1 else v
    return v[:, 0], seen


def _in_parts(f, X, lengths):
    """f over groups of programs, so that the widest activation stays small."""
    step = max(1, 600_000 // X.shape[1])
    return torch.cat([f(X[i:i + step].double(), lengths[i:i + step]) for i in range(0, X.shape[0], step)])


def _lambdarank(s, labels, sigma):
    """The LambdaRank loss of scores s, its weights held constant."""
    rel = (labels - labels.min()) / (labels.max() - labels.min())
    rank = torch.empty_like(rel)
    rank[torch.sort(s.detach(), descending=True, stable=True).indices] = torch.arange(
        1, len(rel) + 1, dtype=rel.dtype, device=rel.device)
    ideal = rel.sort(descending=True).values
    gain = (torch.exp2(rel) - 1)
    place = torch.arange(1, len(rel) + 1, dtype=rel.dtype, device=rel.device)
    gain = gain / ((torch.exp2(ideal) - 1) / torch.log2(1 + place)).sum()
    inv = 1 / torch.log2(1 + rank)
    w = (gain[:, None] - gain[None, :]).abs() * (inv[:, None] - inv[None, :]).abs() * (rel[:, None] > rel[None, :])
    return (w * F.softplus(-sigma * (s[:, None] - s[None, :]), threshold=1000.0)).sum() / math.log(2.0)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("rdu", "topk"):
        return None  # whole numbers
    d, m = _inputs(case, seed), MODELS[case["model"]]
    X, lengths = d["X"], d["lengths"]
    P, _ = _unpack(d["blob"], m)
    with torch.no_grad():
        if kind == "progressive":
            K, _ = _unpack(d["kb"], m)
            lat, at, a = [], 0, case["adapter"]
            v = torch.from_numpy(d["lat"]).cuda().double()
            for n_in, n_out in _widths(m):
                one = []
                for shape in ((a, n_in), (a,), (n_out, a), (n_out,)):
                    one.append(v[at:at + math.prod(shape)].view(shape))
                    at += math.prod(shape)
                lat.append(one)
            return _in_parts(lambda x, n: _column(P, x, n, m, lat, _column(K, x, n, m)[1])[0], X, lengths)
        scores = _in_parts(lambda x, n: _column(P, x, n, m)[0], X, lengths)
    if kind == "score":
        return scores
    S, v = _unpack(d["student"], MODELS["student"], grad=True)
    s, y = _column(S, X.double(), lengths, MODELS["student"])[0], d["labels"].double()
    if kind == "distill":
        terms = [(s - scores).square().mean(), (s - y).square().mean()]
        total = terms[0] + terms[1]
    else:
        by_teacher, by_label = (_lambdarank(s, r, KD["sigma"]) for r in (scores, y))
        penalty = KD["ewc_lambda"] / 2 * (d["fisher"].double() * (v - d["theta_prev"].double()).square()).sum()
        terms = [by_teacher, by_label, penalty]
        total = KD["beta"] * by_label + (1 - KD["beta"]) * KD["phi"] * by_teacher + penalty
    total.backward()
    return dict(loss=torch.stack([total, *terms]).detach(), grads=v.grad)
