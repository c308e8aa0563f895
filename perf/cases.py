"""Performance cases of the TSP per-rank library: the calls one rank of a group makes
for one transformer layer, through the Python binding of the C ABI.

Operations (``op``)
  layer     the rank's layer forward: prefill, inference, the forward of an evaluation
            pass (``noalloc``: the entry point for callers that cannot allocate)
  attn      the attention block forward that keeps A and the log-sum-exp (training)
  mlp       the gated MLP block forward
  attn_bwd  first stage of the attention backward, from the kept activations (training)
            or (``recompute``) recomputing them (activation recomputation)
  mlp_bwd   the MLP backward
  kv        the K/V projections around the sequence-wise exchange: the rank's rows of the
            all-gather (forward), and the backward of those projections for its
            reduce-scattered gradients

A case names the shape (the fields of tsp_shape) and the standard deviation of the
weights.  The sizes are the layer shapes of the library's own workloads (7B, 13B and 70B
class and the tiny one) and of its parity tests, and between them generic ones.
"""
import math

import torch

from paper_2604_26294_amd import tsp as T

OPS = ("layer", "attn", "mlp", "attn_bwd", "mlp_bwd", "kv")


def _case(name, op, batch, seq, hidden, ffn, n_heads, n_kv, head_dim, degree, rank, w_std,
          layout=0, group_steps=0, noalloc=False, recompute=False):
    c = dict(op=op, batch=batch, seq=seq, hidden=hidden, ffn=ffn, n_heads=n_heads,
             n_kv_heads=n_kv, head_dim=head_dim, degree=degree, rank=rank, w_std=w_std,
             layout=layout, group_steps=group_steps, noalloc=noalloc, recompute=recompute)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # The smallest call: a layer of a few microseconds of work, where launches and
        # latency count (the shape of the smoke test).
        _case("layer tiny", "layer", 1, 256, 256, 688, 4, 4, 64, 2, 1, 0.02),
        # A short prompt of the 7B class: 1024 tokens per rank, through the entry point
        # of serving loops that cannot allocate.
        _case("layer 7b s8k noalloc", "layer", 1, 8192, 4096, 11008, 32, 32, 128, 8, 7, 0.02,
              noalloc=True),
        # The long-context prefill of the benchmark (the heaviest contiguous rank).
        _case("layer 7b s64k", "layer", 1, 65536, 4096, 11008, 32, 32, 128, 8, 7, 0.02),
        # The 70B class with grouped-query attention, one kv head per shard.
        _case("layer 70b s32k", "layer", 1, 32768, 8192, 28672, 64, 8, 128, 8, 7, 0.015),
        # A micro-batch of 4 of the 13B class in the balanced (zigzag) layout.
        _case("layer 13b s16k b4 zigzag", "layer", 4, 16384, 5120, 13824, 40, 40, 128, 4, 0,
              0.02, layout=1),
        # The training forward of a small grouped-query layer: head dim 64, ragged tiles
        # (192 rows per rank), two batch entries, zigzag rows.
        _case("attn train gqa d64 zigzag", "attn", 2, 768, 512, 1376, 8, 4, 64, 4, 0, 0.05,
              layout=1),
        # Attention backward of a training step at the benchmark's long context and at a
        # short sequence, from the kept activations.
        _case("attn_bwd 7b s64k", "attn_bwd", 1, 65536, 4096, 11008, 32, 32, 128, 8, 7, 0.02),
        _case("attn_bwd 7b s8k", "attn_bwd", 1, 8192, 4096, 11008, 32, 32, 128, 8, 7, 0.02),
        # The same with activation recomputation on a small layer with ragged tiles (640
        # rows per rank).
        _case("attn_bwd mid recompute", "attn_bwd", 1, 1280, 1024, 2768, 8, 8, 128, 2, 1, 0.03,
              recompute=True),
        # MLP backward of a training step, long and short.
        _case("mlp_bwd 7b s64k", "mlp_bwd", 1, 65536, 4096, 11008, 32, 32, 128, 8, 7, 0.02),
        _case("mlp_bwd 7b s8k", "mlp_bwd", 1, 8192, 4096, 11008, 32, 32, 128, 8, 7, 0.02),
        # Both sides of the K/V exchange of a training step.
        _case("kv 7b s64k", "kv", 1, 65536, 4096, 11008, 32, 32, 128, 8, 7, 0.02),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_once(rng):
    op = rng.choice(OPS)
    kind = rng.choice(("small", "small", "mid", "7b", "13b", "70b"))
    layout = rng.choice((0, 1))
    batch = rng.choice((1, 1, 1, 2, 4))
    if kind in ("small", "mid"):
        d = rng.choice((64, 128))
        degree = rng.choice((1, 2, 3, 4, 8))
        group = rng.choice((1, 1, 2, 4))
        top = 1024 if kind == "small" else 3072
        kv_per_shard = rng.choice((1, 2))
        while kv_per_shard * group * degree * d > top:
            degree, group, kv_per_shard = max(1, degree // 2), max(1, group // 2), 1
        n_kv = kv_per_shard * degree
        n_heads = n_kv * group
        hidden = n_heads * d
        ffn = degree * 8 * max(8, int(hidden * rng.uniform(2.5, 4.0) / degree / 8))
        w_std = round(1.28 / math.sqrt(hidden), 4)
    else:
        d = 128
        hidden, ffn, n_heads, n_kv, w_std, degrees = {
            "7b": (4096, 11008, 32, 32, 0.02, (4, 8)),
            "13b": (5120, 13824, 40, 40, 0.02, (4, 8)),
            "70b": (8192, 28672, 64, 8, 0.015, (4, 8)),
        }[kind]
        degree = rng.choice(degrees)
    s_loc = _log_int(rng, 96, 8192)
    if layout == 1:
        s_loc += s_loc % 2
    if op == "attn_bwd":  # training sequences: whole 64-token blocks, S a multiple of 256
        step = 64 * max(1 + layout, 4 // math.gcd(4, degree))
        s_loc = max(1, s_loc // step) * step
    rank = rng.randrange(degree)
    return _case(None, op, batch, s_loc * degree, hidden, ffn, n_heads, n_kv, d, degree, rank,
                 w_std, layout=layout, group_steps=rng.choice((0, 0, 0, 0, 1, 2)),
                 noalloc=op == "layer" and kind == "small" and batch * s_loc <= 2048 and
                 rng.random() < 0.5,
                 recompute=op == "attn_bwd" and rng.random() < 0.3)


def draw(rng):
    most = max(work(c)["flops"] for c in listed())
    while True:
        c = _draw_once(rng)
        # (the size limit of the library's 32-bit operand offsets is far above these)
        if work(c)["flops"] <= 0.7 * most and c["batch"] * c["seq"] <= 65536:
            return c


# ------------------------------------------------------------------ shapes and inputs


def _segments(c):
    """The rank's rows as (first local row, rows, first position) pieces."""
    s_loc = c["seq"] // c["degree"]
    if c["layout"] == 0:
        return [(0, s_loc, c["rank"] * s_loc)]
    s_c = s_loc // 2
    return [(0, s_c, c["rank"] * s_c), (s_c, s_c, (2 * c["degree"] - 1 - c["rank"]) * s_c)]


def _shape(c):
    return T.make_shape(c["batch"], c["seq"], c["hidden"], c["ffn"], c["n_heads"],
                        c["n_kv_heads"], c["head_dim"], c["degree"], c["rank"], c["layout"], 0.0,
                        c["group_steps"])


def _inputs(c, seed):
    """The bf16 tensors of a case, from the seed: what the caller has in hand."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)

    def normal(*shape, std=1.0):
        t = torch.empty(shape, dtype=torch.bfloat16, device="cuda")
        return t.normal_(0.0, std, generator=g)

    D, h, d, w = c["degree"], c["hidden"], c["head_dim"], c["w_std"]
    qd, kd, fs = c["n_heads"] // D * d, c["n_kv_heads"] // D * d, c["ffn"] // D
    B, s_loc, op = c["batch"], c["seq"] // D, c["op"]
    i = {"x": normal(B, s_loc, h)}
    if op in ("layer", "attn", "attn_bwd", "kv"):
        i["wa"] = [normal(2 * qd + 2 * kd, h, std=w) for _ in range(D)]
    if op in ("layer", "attn", "attn_bwd"):
        # the other ranks' K and V rows (projections of unit-variance tokens)
        i["k"] = normal(B, c["seq"], c["n_kv_heads"], d, std=w * math.sqrt(h))
        i["v"] = normal(B, c["seq"], c["n_kv_heads"], d, std=w * math.sqrt(h))
    if op in ("layer", "mlp", "mlp_bwd"):
        for k in ("w1", "w3", "w2"):
            i[k] = [normal(fs, h, std=w) for _ in range(D)]
    if op in ("attn_bwd", "mlp_bwd"):
        i["dy"] = normal(B, s_loc, h)
    if op == "kv":
        i["dk"] = normal(B, s_loc, c["n_kv_heads"], d)
        i["dv"] = normal(B, s_loc, c["n_kv_heads"], d)
    return i


def prepare(case, seed):
    s = _inputs(case, seed)
    op, D, h = case["op"], case["degree"], case["hidden"]
    B, s_loc = case["batch"], case["seq"] // D
    nh, nkv, d, fs = case["n_heads"], case["n_kv_heads"], case["head_dim"], case["ffn"] // D
    s["case"], s["shape"] = case, _shape(case)

    def f32(*shape):
        return torch.zeros(shape, dtype=torch.float32, device="cuda")

    def workspace(*ops):
        n = max(T.workspace_bytes(s["shape"], o) for o in ops)
        return torch.empty(max(n, 256), dtype=torch.uint8, device="cuda")

    if op in ("layer", "attn", "mlp"):
        s["y"] = f32(B, s_loc, h)
        if not case["noalloc"]:
            s["ws"] = workspace({"layer": T.OP_LAYER, "attn": T.OP_ATTN, "mlp": T.OP_MLP}[op])
    if op in ("attn", "attn_bwd"):
        s["a"] = torch.empty(B, s_loc, nh, d, dtype=torch.bfloat16, device="cuda")
        s["lse"] = f32(B, nh, s_loc)
    if op in ("attn_bwd", "kv"):
        s["dx"] = f32(B, s_loc, h)
        s["dw"] = f32(D, 2 * (nh + nkv) // D * d, h)
        s["dws"] = list(s["dw"])
    if op == "attn_bwd":
        s["dk"], s["dv"] = f32(B, case["seq"], nkv, d), f32(B, case["seq"], nkv, d)
        # the step's forward: its own K/V rows, and what it keeps for the backward
        s["ws"] = workspace(T.OP_ATTN)
        T.tsp_attn_rank_fwd_train(s["shape"], s["x"], s["wa"], s["k"], s["v"], f32(B, s_loc, h),
                                  False, s["a"], s["lse"], s["ws"])
        s["ws"] = workspace(T.OP_ATTN_BWD)
    if op == "mlp_bwd":
        s["dx"] = f32(B, s_loc, h)
        s["dw"] = [f32(D, fs, h) for _ in range(3)]
        s["dws"] = [list(t) for t in s["dw"]]
        s["ws"] = workspace(T.OP_MLP_BWD)
    if op == "kv":
        s["k"] = torch.zeros(B, case["seq"], nkv, d, dtype=torch.bfloat16, device="cuda")
        s["v"] = torch.zeros_like(s["k"])
        s["ws"] = workspace(T.OP_ATTN_KV_BWD)
    return s


def _own_rows(c, buf):
    """The rank's rows of a [B, S, n_kv, d] buffer, as views (one per segment)."""
    return [buf[:, p0:p0 + n] for _, n, p0 in _segments(c)]


def run(state):
    s = state
    c, sh = s["case"], s["shape"]
    op = c["op"]
    qd, kd = c["n_heads"] // c["degree"] * c["head_dim"], \
        c["n_kv_heads"] // c["degree"] * c["head_dim"]
    if op == "layer":
        if c["noalloc"]:
            T.tsp_layer_rank_fwd_noalloc(sh, s["x"], s["wa"], s["w1"], s["w3"], s["w2"], s["k"],
                                         s["v"], s["y"])
        else:
            T.tsp_layer_rank_fwd(sh, s["x"], s["wa"], s["w1"], s["w3"], s["w2"], s["k"], s["v"],
                                 s["y"], s["ws"])
        return {"y": s["y"], "k": _own_rows(c, s["k"]), "v": _own_rows(c, s["v"])}
    if op == "attn":
        T.tsp_attn_rank_fwd_train(sh, s["x"], s["wa"], s["k"], s["v"], s["y"], False, s["a"],
                                  s["lse"], s["ws"])
        return {"y": s["y"], "a": s["a"], "lse": s["lse"], "k": _own_rows(c, s["k"]),
                "v": _own_rows(c, s["v"])}
    if op == "mlp":
        T.tsp_mlp_rank_fwd(sh, s["x"], s["w1"], s["w3"], s["w2"], s["y"], False, s["ws"])
        return {"y": s["y"]}
    if op == "attn_bwd":
        if c["recompute"]:
            T.tsp_attn_rank_bwd(sh, s["x"], s["dy"], s["wa"], s["k"], s["v"], s["dx"], False,
                                s["dws"], s["dk"], s["dv"], s["ws"])
        else:
            T.tsp_attn_rank_bwd_saved(sh, s["x"], s["dy"], s["wa"], s["k"], s["v"], s["a"],
                                      s["lse"], s["dx"], False, s["dws"], s["dk"], s["dv"],
                                      s["ws"])
        return {"dx": s["dx"], "dwq": s["dw"][:, :qd], "dwo": s["dw"][:, qd + 2 * kd:],
                "dk": s["dk"], "dv": s["dv"]}
    if op == "mlp_bwd":
        T.tsp_mlp_rank_bwd(sh, s["x"], s["dy"], s["w1"], s["w3"], s["w2"], s["dx"], False,
                           s["dws"][0], s["dws"][1], s["dws"][2], s["ws"])
        return {"dx": s["dx"], "dw1": s["dw"][0], "dw3": s["dw"][1], "dw2": s["dw"][2]}
    T.tsp_kv_rank_fwd(sh, s["x"], s["wa"], s["k"], s["v"])
    T.tsp_attn_kv_rank_bwd(sh, s["x"], s["wa"], s["dk"], s["dv"], s["dx"], False, s["dws"],
                           s["ws"])
    return {"k": _own_rows(c, s["k"]), "v": _own_rows(c, s["v"]), "dx": s["dx"],
            "dwkv": s["dw"][:, qd:qd + 2 * kd]}


# ------------------------------------------------------------------------ work and error


def work(case):
    """Bytes: every weight, token row and visible K/V row read once, every output written
    once.  FLOPs: the products of the method, the causal core at the visible keys only (the
    backwards form again what their interface does not hand them: Q, G and U, and with
    ``recompute`` the forward core)."""
    c, op = case, case["op"]
    B, h, d, D = c["batch"], c["hidden"], c["head_dim"], c["degree"]
    M = B * (c["seq"] // D)
    kvw, F = c["n_kv_heads"] * d, c["ffn"]
    pairs = sum(n * p0 + n * (n + 1) // 2 for _, n, p0 in _segments(c))  # per head and entry
    core = 4.0 * B * c["n_heads"] * d * pairs
    seen = B * max(p0 + n for _, n, p0 in _segments(c))  # K/V rows read
    w_attn, w_mlp = (2 * h + 2 * kvw) * h, 3 * F * h     # weights, in elements
    proj, mlp = 4.0 * M * h * (h + kvw), 6.0 * M * h * F
    if op == "layer":
        return {"bytes": 2 * (w_attn + w_mlp) + 2 * M * h + 4 * M * h + 2 * 2 * kvw * (seen + M),
                "flops": proj + mlp + core}
    if op == "attn":
        return {"bytes": 2 * w_attn + 2 * M * h + 4 * M * h + 2 * M * h +
                4 * M * c["n_heads"] + 2 * 2 * kvw * (seen + M), "flops": proj + core}
    if op == "mlp":
        return {"bytes": 2 * w_mlp + 2 * M * h + 4 * M * h, "flops": mlp}
    if op == "attn_bwd":
        # in: x, dY, (A, lse), W_Q, W_O, K, V; out: dX, dW_Q, dW_O, dK, dV
        kept = 0 if c["recompute"] else 2 * M * h + 4 * M * c["n_heads"]
        return {"bytes": 2 * 2 * M * h + kept + 2 * 2 * h * h + 2 * 2 * kvw * seen +
                4 * M * h + 4 * 2 * h * h + 4 * 2 * B * c["seq"] * kvw,
                "flops": 10.0 * M * h * h + (3.5 if c["recompute"] else 2.5) * core}
    if op == "mlp_bwd":
        return {"bytes": 2 * 2 * M * h + 2 * w_mlp + 4 * M * h + 4 * w_mlp,
                "flops": 16.0 * M * h * F}
    # kv: in x, W_K, W_V (both directions), dK, dV; out K, V rows, dX, dW_K, dW_V
    return {"bytes": 2 * (2 * M * h + 2 * 2 * kvw * h) + 2 * 2 * M * kvw * 2 + 4 * M * h +
            4 * 2 * kvw * h, "flops": 12.0 * M * h * kvw}


def tolerance(case):
    """About four times the error measured against 64-bit values: one bf16 rounding of an
    intermediate or result in the MLP and the K/V projections (rel 0.0017, max 0.011), the
    roundings of Q, K, V, P and A in the attention forward (0.0036, 0.068), and those of
    dA, dS and dQ too in its backward (0.005, 0.18: the dK / dV rows of late keys, which
    few queries see, are small beside the first keys' rows)."""
    if case["op"] in ("mlp", "mlp_bwd", "kv"):
        return {"rel": 0.007, "max": 0.05}
    if case["op"] == "attn_bwd":
        return {"rel": 0.018, "max": 0.7}
    return {"rel": 0.015, "max": 0.27}


# ------------------------------------------------------------------------ 64-bit values


def _attention(c, i, wa, x, k, v, grads=None):
    """Attention of the rank in 64 bits, head by head: A [B, S_loc, n_h, d] and the base-2
    log-sum-exp [B, n_h, S_loc]; with ``grads`` = dA also (dQ, dK, dV)."""
    B, s_loc, nh, d = c["batch"], x.shape[1], c["n_heads"], c["head_dim"]
    D, nkv = c["degree"], c["n_kv_heads"]
    qd = nh // D * d
    scale = 1.0 / math.sqrt(d)
    q = torch.cat([x @ w[:qd].T for w in wa], dim=2).view(B, s_loc, nh, d)
    a, lse = torch.empty_like(q), q.new_empty(B, nh, s_loc)
    if grads is not None:
        dq, dk, dv = torch.empty_like(q), torch.zeros_like(k), torch.zeros_like(v)
    for b in range(B):
        for r0, n, p0 in _segments(c):
            keys = p0 + n
            late = torch.arange(keys, device=x.device)[None, :] > \
                p0 + torch.arange(n, device=x.device)[:, None]
            for j in range(nh):
                e = j // (nh // nkv)
                qq, kk, vv = q[b, r0:r0 + n, j], k[b, :keys, e], v[b, :keys, e]
                s = (qq @ kk.T).mul_(scale).masked_fill_(late, -math.inf)
                ls = torch.logsumexp(s, dim=1)
                lse[b, j, r0:r0 + n] = ls / math.log(2.0)
                p = s.sub_(ls[:, None]).exp_()
                o = p @ vv
                a[b, r0:r0 + n, j] = o
                if grads is not None:
                    do = grads[b, r0:r0 + n, j]
                    dv[b, :keys, e] += p.T @ do
                    ds = (do @ vv.T).sub_((do * o).sum(1, keepdim=True)).mul_(p).mul_(scale)
                    dq[b, r0:r0 + n, j] = ds @ kk
                    dk[b, :keys, e] += ds.T @ qq
                    del ds
                del s, p
    return (a, lse) if grads is None else (a, lse, dq, dk, dv)


def exact(case, seed):
    c, op = case, case["op"]
    i = {k: [t.double() for t in v] if isinstance(v, list) else v.double()
         for k, v in _inputs(c, seed).items()}
    x, D, h, d = i["x"], c["degree"], c["hidden"], c["head_dim"]
    qd, kd = c["n_heads"] // D * d, c["n_kv_heads"] // D * d
    B, s_loc = x.shape[:2]
    M = B * s_loc
    wa = i.get("wa")

    def own_kv():
        heads = (B, s_loc, c["n_kv_heads"], d)
        return (torch.cat([x @ w[qd:qd + kd].T for w in wa], dim=2).view(heads),
                torch.cat([x @ w[qd + kd:qd + 2 * kd].T for w in wa], dim=2).view(heads))

    def mlp(t):
        return sum((torch.nn.functional.silu(t @ g.T) * (t @ u.T)) @ w
                   for g, u, w in zip(i["w1"], i["w3"], i["w2"]))

    if op == "mlp":
        return {"y": mlp(x)}
    if op == "mlp_bwd":
        dy, xm = i["dy"], x.view(M, h)
        dym, dx = dy.view(M, h), torch.zeros_like(x.view(M, h))
        dw = [[], [], []]
        for g, u, w in zip(i["w1"], i["w3"], i["w2"]):
            gg, uu, dh = xm @ g.T, xm @ u.T, dym @ w.T
            sg = torch.sigmoid(gg)
            sl = gg * sg
            dg, du = dh * uu * sg * (1 + gg * (1 - sg)), dh * sl
            dx += dg @ g + du @ u
            dw[0].append(dg.T @ xm)
            dw[1].append(du.T @ xm)
            dw[2].append((sl * uu).T @ dym)
        return {"dx": dx.view(B, s_loc, h), "dw1": torch.stack(dw[0]), "dw3": torch.stack(dw[1]),
                "dw2": torch.stack(dw[2])}
    ko, vo = own_kv()
    if op == "kv":
        gk, gv = i["dk"].view(M, D, kd), i["dv"].view(M, D, kd)
        dx, dw, xm = torch.zeros_like(x.view(M, h)), [], x.view(M, h)
        for r, w in enumerate(wa):
            dx += gk[:, r] @ w[qd:qd + kd] + gv[:, r] @ w[qd + kd:qd + 2 * kd]
            dw.append(torch.cat([gk[:, r].T @ xm, gv[:, r].T @ xm]))
        rows = [(r0, n) for r0, n, _ in _segments(c)]
        return {"k": [ko[:, r0:r0 + n] for r0, n in rows],
                "v": [vo[:, r0:r0 + n] for r0, n in rows],
                "dx": dx.view(B, s_loc, h), "dwkv": torch.stack(dw)}
    k, v = i["k"], i["v"]
    for r0, n, p0 in _segments(c):
        k[:, p0:p0 + n], v[:, p0:p0 + n] = ko[:, r0:r0 + n], vo[:, r0:r0 + n]
    if op == "attn_bwd":
        dy = i["dy"]
        da = torch.cat([dy @ w[qd + 2 * kd:].T for w in wa], dim=2).view(B, s_loc, -1, d)
        a, _, dq, dk, dv = _attention(c, i, wa, x, k, v, da)
        xm, dym = x.view(M, h), dy.view(M, h)
        dq, a = dq.view(M, D, qd), a.view(M, D, qd)
        return {"dx": sum(dq[:, r] @ wa[r][:qd] for r in range(D)).view(B, s_loc, h),
                "dwq": torch.stack([dq[:, r].T @ xm for r in range(D)]),
                "dwo": torch.stack([a[:, r].T @ dym for r in range(D)]), "dk": dk, "dv": dv}
    a, lse = _attention(c, i, wa, x, k, v)
    am = a.view(B, s_loc, D, qd)
    y = sum(am[:, :, r] @ wa[r][qd + 2 * kd:] for r in range(D))
    out = {"k": _own_rows(c, k), "v": _own_rows(c, v)}
    if op == "attn":
        return dict(out, y=y, a=a, lse=lse)
    u = x + y
    return dict(out, y=u + mlp(u))
