"""The work a program that decodes with this library has it do, as cases to be timed and checked.

A case is one decode step's worth of calls on the public entry points: the fused attention block (plain, with RMSNorm
and residual, with rows of different lengths, as a stack), the feed-forward block, the latent-attention (MLA) block and
the team collectives.  Shapes are those of cf_inputs.py, with the batches and cached lengths its configurations and
benchmarks use, and for drawn cases any other of the same ranges.  Decoding walks through the layers of a model, so
that weights and caches come from memory and not from a cache: where one layer is small a case has several, each with
weights and caches of its own.  Outputs are what the calls write: the block's output and the appended cache rows (the
whole of the updated state; every other cache row stays as it was).
"""
import math

import torch

import cf_inputs
from paper_2508_18850_amd import binding

DEV = "cuda"
EPS = 1e-5
TEAM_MODES = {"rounds": 0, "two_kernels": 1, "direct": 2, "two_hops": 3}


# ---- the cases -------------------------------------------------------------------------------------------------

def _block(name, shape, batch, kv, call, layers):
    s = cf_inputs.SHAPES[shape]
    return {"name": name, "kind": "block", "call": call, "d_model": s.d_model, "n_q": s.n_q_heads, "n_kv": s.n_kv_heads,
            "head_dim": s.head_dim, "rope_base": s.rope_base, "batch": batch, "kv": kv, "layers": layers}


def _ffn(name, shape, batch, layers):
    s = cf_inputs.FFN_SHAPES[shape]
    return {"name": name, "kind": "ffn", "d_model": s.d_model, "d_ff": s.d_ff, "batch": batch, "activation": "silu",
            "layers": layers}


def _mla(name, batch, kv, layers):
    s = cf_inputs.MLA_SHAPES["deepseek_v2_lite"]
    return {"name": name, "kind": "mla", "d_model": s.d_model, "n_heads": s.n_heads, "nope": s.nope_dim,
            "v_dim": s.v_head_dim, "rope_base": s.rope_base, "batch": batch, "kv": kv, "layers": layers}


def listed():
    return [
        # the smallest call: one small layer, where launch and hand-over latency are all there is
        _block("block tiny b1", "tiny", 1, 256, "row_major", 1),
        # a small grouped-query layer of odd sizes: nothing divides evenly, weights as a checkpoint has them
        {"name": "block odd sizes b3", "kind": "block", "call": "row_major", "d_model": 2056, "n_q": 14, "n_kv": 7,
         "head_dim": 64, "rope_base": 10000.0, "batch": 3, "kv": 777, "layers": 2},
        # one user's chat on a 7B model: the benchmark's headline
        _block("block 7b b1 kv4096", "llama2_7b", 1, 4096, "packed", 4),
        # continuous batching of a few users: rows of different lengths, norm and residual taken into the kernel
        _block("layer rows 8b b4 kv8192", "llama3_8b", 4, 8192, "rows", 2),
        # a full batch of a serving engine
        _block("block 8b b16 kv8192", "llama3_8b", 16, 8192, "packed", 1),
        # one user with a long context on the largest model
        _block("block 70b b1 kv32768", "llama2_70b", 1, 32768, "packed", 1),
        # all attention layers of a pass enqueued by one call, as a pre-norm decoder has them
        _block("stack 8b b1 kv2048", "llama3_8b", 1, 2048, "stack_norm", 8),
        # the other half of a layer, for one user and for a full batch
        _ffn("ffn 7b b1", "llama2_7b", 1, 2),
        _ffn("ffn 8b b16", "llama3_8b", 16, 1),
        # latent attention, for one user and for a full batch
        _mla("mla b1 kv4096", 1, 4096, 8),
        _mla("mla b16 kv4096", 16, 4096, 4),
        # the exchange primitive by itself: the attention vectors of a team of 8 workgroups per head, summed in one hop
        {"name": "team reduce 32x8 4KB", "kind": "team", "call": "reduce", "teams": 32, "team_size": 8, "elems": 1024,
         "op": "sum", "mode": "direct"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


MOST_BYTES = 620e6      # of a drawn pass: the largest listed one has 621 MB
MOST_BATCH = 16         # batch limit of the library


def draw(rng):
    while True:
        kind = rng.choice(["block", "block", "block", "ffn", "mla", "team"])
        if kind == "block":
            head_dim = rng.choice([64, 128, 128])
            n_kv = rng.choice([rng.randint(1, 32), 8, 32])
            group = rng.choice([1, 2, 4, 8])
            case = {"kind": kind, "call": rng.choice(["packed", "packed", "row_major", "norm", "rows", "stack", "stack_norm"]),
                    "d_model": 8 * _log(rng, 32, 1024), "n_q": n_kv * group, "n_kv": n_kv, "head_dim": head_dim,
                    "rope_base": rng.choice([10000.0, 500000.0]), "batch": _log(rng, 1, MOST_BATCH), "kv": _log(rng, 1, 32768),
                    "layers": rng.randint(1, 4)}
            if case["call"] == "stack":   # the bare stack stands for whole models: widths and head counts as they have them
                case["d_model"] = 256 * _log(rng, 1, 32)
                case["n_kv"] = rng.choice([1, 2, 4, 8, 16, 32])
                case["n_q"] = case["n_kv"] * group
            if case["n_q"] * head_dim > 8192:
                continue
            if case["call"] == "rows":   # every row's appended key and value is an output of its own
                case["layers"] = min(case["layers"], 64 // (1 + 2 * case["batch"]))
        elif kind == "ffn":
            case = {"kind": kind, "d_model": 8 * _log(rng, 64, 1024), "d_ff": _log(rng, 1376, 28672),
                    "batch": _log(rng, 1, MOST_BATCH), "activation": rng.choice(["silu", "gelu"]), "layers": rng.randint(1, 3)}
        elif kind == "mla":
            heads = rng.choice([16, 16, rng.randint(4, 16)])
            case = {"kind": kind, "d_model": 32 * rng.randint(8, 4 * heads) if heads < 16 else 32 * rng.randint(32, 64),
                    "n_heads": heads, "nope": rng.choice([128, 8 * rng.randint(4, 16)]), "v_dim": rng.choice([128, 8 * rng.randint(4, 16)]),
                    "rope_base": 10000.0, "batch": _log(rng, 1, MOST_BATCH), "kv": _log(rng, 1, 16384), "layers": rng.randint(2, 8)}
        else:
            size = rng.choice([2, 4, 8, 16])
            elems = _log(rng, 64, 16384)
            case = {"kind": kind, "call": rng.choice(["reduce", "reduce", "gather"]), "teams": rng.randint(1, 256 // size),
                    "team_size": size, "elems": elems, "op": rng.choice(["sum", "max"]),
                    "mode": rng.choice(["rounds", "direct", "two_kernels", "two_hops"])}
            if case["call"] == "gather":
                if case["mode"] == "two_hops" or size * elems > 65536:
                    continue
        if work(case)["bytes"] <= MOST_BYTES:
            return case


# ---- inputs ----------------------------------------------------------------------------------------------------

def _generator(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _normal(g, shape, std=1.0):
    t = torch.randn(shape, generator=g, device=DEV, dtype=torch.float16)
    return t if std == 1.0 else t.mul_(std)


def _row_lengths(case):
    """Cached tokens of every batch row: one length, or spread between half of it and all of it."""
    B, L = case["batch"], case["kv"]
    return [L - (b * L) // (2 * B) for b in range(B)] if case.get("call") == "rows" else [L] * B


def _has_norm(case):
    return case["call"] in ("norm", "rows", "stack_norm")


def _is_stack(case):
    return case["call"].startswith("stack")


def _layer_inputs(case, g):
    """One layer's tensors, with the distributions of cf_inputs.py."""
    B, D = case["batch"], case["d_model"]
    if case["kind"] == "block":
        nq, nkv, d, L = case["n_q"], case["n_kv"], case["head_dim"], case["kv"]
        S = cf_inputs.default_max_seq(L)
        t = {"x": _normal(g, (B, D)), "w_qkv": _normal(g, (D, (nq + 2 * nkv) * d), 0.02), "w_o": _normal(g, (nq * d, D), 0.02)}
        for name in ("k", "v"):
            t[name] = _normal(g, (B, nkv, S, d))
            for b, n in enumerate(_row_lengths(case)):
                t[name][b, :, n:] = 0
        if _has_norm(case):
            t["gamma"] = _normal(g, (D,), 0.1).add_(1.0)
        return t
    if case["kind"] == "ffn":
        F = case["d_ff"]
        return {"z": _normal(g, (B, D)), "w1": _normal(g, (F, D), 0.02), "w2": _normal(g, (F, D), 0.02), "w3": _normal(g, (F, D), 0.02)}
    nh, n, v, lat, r, L = case["n_heads"], case["nope"], case["v_dim"], 512, 64, case["kv"]
    t = {"x": _normal(g, (B, D)), "w_q": _normal(g, (D, nh * (n + r)), D ** -0.5), "w_kv": _normal(g, (D, lat + r), D ** -0.5),
         "w_up": _normal(g, (nh, n, lat), n ** -0.5), "w_down": _normal(g, (nh, lat, v), lat ** -0.5),
         "w_o": _normal(g, (nh * v, D), (nh * v) ** -0.5), "kv": _normal(g, (B, cf_inputs.default_max_seq(L), lat + r))}
    t["kv"][:, L:] = 0
    return t


def _team_input(case, g):
    return torch.randn((case["teams"], case["team_size"], case["elems"]), generator=g, device=DEV, dtype=torch.float32)


# ---- prepare and run -------------------------------------------------------------------------------------------

class State:
    pass


def _prepare_block(case, seed):
    st, g = State(), _generator(seed)
    B, D, nq, nkv, d, L, n = (case[k] for k in ("batch", "d_model", "n_q", "n_kv", "head_dim", "kv", "layers"))
    st.handle = binding.DecodeBlock(D, nq, nkv, d, B, cf_inputs.default_max_seq(L), case["rope_base"])
    stream = torch.cuda.current_stream().cuda_stream
    packed = case["call"] != "row_major"
    sizes = st.handle.packed_sizes()
    lengths = _row_lengths(case)
    st.rows = torch.tensor(lengths, dtype=torch.int32, device=DEV)
    st.keep, st.outputs = [], []
    args = []
    for _ in range(n):
        t = _layer_inputs(case, g)
        if packed:
            wq, wo = (torch.empty(size // 2, dtype=torch.float16, device=DEV) for size in sizes)
            st.handle.pack_weights(t["w_qkv"].data_ptr(), t["w_o"].data_ptr(), wq.data_ptr(), wo.data_ptr(), stream)
            t["w_qkv"], t["w_o"] = wq, wo
        t["out"] = torch.empty((B, D), dtype=torch.float16, device=DEV)
        st.keep.append(t)
        if len(set(lengths)) == 1:
            new = [t[c][:, :, lengths[0]] for c in ("k", "v")]
        else:
            new = [t[c][b, :, m] for c in ("k", "v") for b, m in enumerate(lengths)]
        st.outputs += ([] if _is_stack(case) else [t["out"]]) + new
        args.append({k: v.data_ptr() for k, v in t.items()})
    h, out = st.handle, st.outputs
    if _is_stack(case):
        st.outputs.append(st.keep[-1]["out"])
        lists = [[a[k] for a in args] for k in ("w_qkv", "w_o", "k", "v")]
        gammas = [a["gamma"] for a in args] if _has_norm(case) else None
        first, last, residual = args[0]["x"], args[-1]["out"], 1 if _has_norm(case) else 0

        def call(stream):
            h.decode_stack(B, first, gammas, EPS, residual, 1, *lists, L, last, stream)
    elif case["call"] == "rows":
        rows = st.rows.data_ptr()

        def call(stream):
            for a in args:
                h.decode_layer_rows(B, a["x"], a["gamma"], EPS, 1, 1, a["w_qkv"], a["w_o"], a["k"], a["v"], rows, L, a["out"], stream)
    elif case["call"] == "norm":
        def call(stream):
            for a in args:
                h.decode_layer(B, a["x"], a["gamma"], EPS, 1, 1, a["w_qkv"], a["w_o"], a["k"], a["v"], L, a["out"], stream)
    else:
        one = h.decode_block_packed if packed else h.decode_block

        def call(stream):
            for a in args:
                one(B, a["x"], a["w_qkv"], a["w_o"], a["k"], a["v"], L, a["out"], stream)
    st.call, st.outputs = call, out
    return st


def _prepare_ffn(case, seed):
    st, g = State(), _generator(seed)
    B, D = case["batch"], case["d_model"]
    act = binding.FFN_GELU if case["activation"] == "gelu" else binding.FFN_SILU
    st.handle = h = binding.FfnBlock(D, case["d_ff"], B, act)
    st.keep = [_layer_inputs(case, g) for _ in range(case["layers"])]
    st.outputs = [torch.empty((B, D), dtype=torch.float16, device=DEV) for _ in st.keep]
    args = [[t[k].data_ptr() for k in ("z", "w1", "w2", "w3")] + [o.data_ptr()] for t, o in zip(st.keep, st.outputs)]

    def call(stream):
        for a in args:
            h.decode(B, *a, stream)
    st.call = call
    return st


def _prepare_mla(case, seed):
    st, g = State(), _generator(seed)
    B, D, L = case["batch"], case["d_model"], case["kv"]
    st.handle = h = binding.MlaBlock(D, case["n_heads"], case["nope"], 64, 512, case["v_dim"], B, cf_inputs.default_max_seq(L), case["rope_base"])
    st.keep = [_layer_inputs(case, g) for _ in range(case["layers"])]
    outs = [torch.empty((B, D), dtype=torch.float16, device=DEV) for _ in st.keep]
    st.outputs = [x for t, o in zip(st.keep, outs) for x in (o, t["kv"][:, L])]
    args = [([t[k].data_ptr() for k in ("x", "w_q", "w_kv", "w_up", "w_down", "w_o", "kv")], o.data_ptr()) for t, o in zip(st.keep, outs)]

    def call(stream):
        for a, o in args:
            h.decode(B, *a, L, o, stream)
    st.call = call
    return st


def _prepare_team(case, seed):
    st = State()
    T, N, E = case["teams"], case["team_size"], case["elems"]
    gather = case["call"] == "gather"
    st.handle = h = binding.TeamCollectives(T * N, N * E if gather else E)
    st.keep = src = _team_input(case, _generator(seed))
    dst = torch.empty((T, N, N, E) if gather else (T, N, E), dtype=torch.float32, device=DEV)
    st.outputs = [dst]
    a, b, mode, op = src.data_ptr(), dst.data_ptr(), TEAM_MODES[case["mode"]], 1 if case["op"] == "max" else 0
    st.call = (lambda stream: h.gather(T, N, a, b, E, mode, stream)) if gather else (lambda stream: h.reduce(T, N, op, a, b, E, mode, stream))
    return st


def prepare(case, seed):
    return {"block": _prepare_block, "ffn": _prepare_ffn, "mla": _prepare_mla, "team": _prepare_team}[case["kind"]](case, seed)


def run(state):
    state.call(torch.cuda.current_stream().cuda_stream)
    return state.outputs


# ---- what a pass cannot do without -----------------------------------------------------------------------------

def work(case):
    if case["kind"] == "team":
        T, N, E = case["teams"], case["team_size"], case["elems"]
        gather = case["call"] == "gather"
        return {"bytes": 4 * T * N * E * (1 + (N if gather else 1)), "flops": 0 if gather else T * (N - 1) * E}
    B, D, n = case["batch"], case["d_model"], case["layers"]
    if case["kind"] == "ffn":
        w = 3 * D * case["d_ff"]
        return {"bytes": n * (2 * w + 4 * B * D), "flops": n * 2 * B * w}
    if case["kind"] == "mla":
        nh, q, v, lat, r, L = case["n_heads"], case["nope"], case["v_dim"], 512, 64, case["kv"]
        w = D * nh * (q + r) + D * (lat + r) + nh * q * lat + nh * lat * v + nh * v * D
        return {"bytes": n * (2 * w + 2 * B * (L + 1) * (lat + r) + 4 * B * D),
                "flops": n * (2 * B * w + 2 * B * nh * (L + 1) * (2 * lat + r))}
    nq, nkv, d = case["n_q"], case["n_kv"], case["head_dim"]
    keys = sum(_row_lengths(case)) + B
    w = D * (nq + 2 * nkv) * d + nq * d * D
    return {"bytes": n * (2 * w + 4 * keys * nkv * d + (2 * D if _has_norm(case) else 0) + (0 if _is_stack(case) else 4 * B * D))
            + (4 * B * D if _is_stack(case) else 0),
            "flops": n * (2 * B * w + 4 * keys * nq * d)}


def tolerance(case):
    """About four times the error of the path against exact() (2.1e-4): the rounding of the 16-bit results.  In a stack the
    rounding of every layer's hidden state travels on (measured 3e-4 after two layers, 6e-4 after eight)."""
    if case["kind"] == "team":
        return "exact" if case["call"] == "gather" or case["op"] == "max" else {"rel": 1e-6}
    return {"rel": 1e-3 * (1.0 + 0.25 * case["layers"]) if case["kind"] == "block" and _is_stack(case) else 1e-3}


# ---- the same in 64 bits ---------------------------------------------------------------------------------------

def _rope(v, pos, base, pairs_of):
    """Pairs (i, i + pairs_of / 2) of the last dimension turned by pos * base^(-2i / pairs_of)."""
    half = pairs_of // 2
    angle = pos * base ** (-2.0 * torch.arange(half, device=DEV, dtype=torch.float64) / pairs_of)
    c, s, lo, hi = torch.cos(angle), torch.sin(angle), v[..., :half], v[..., half:]
    return torch.cat([lo * c - hi * s, hi * c + lo * s], -1)


def _exact_block(case, t, x):
    B, D, nq, nkv, d = (case[k] for k in ("batch", "d_model", "n_q", "n_kv", "head_dim"))
    h = x
    if _has_norm(case):
        h = x / torch.sqrt(x.square().mean(-1, keepdim=True) + EPS) * t["gamma"].double()
    qkv = h @ t["w_qkv"].double()
    heads, new_k, new_v = [], [], []
    for b, n in enumerate(_row_lengths(case)):
        q = _rope(qkv[b, :nq * d].reshape(nq, d), n, case["rope_base"], d)
        k1 = _rope(qkv[b, nq * d:(nq + nkv) * d].reshape(nkv, d), n, case["rope_base"], d)
        v1 = qkv[b, (nq + nkv) * d:].reshape(nkv, d)
        new_k.append(k1)
        new_v.append(v1)
        for g in range(nkv):
            keys = torch.cat([t["k"][b, g, :n].double(), k1[g:g + 1]])
            values = torch.cat([t["v"][b, g, :n].double(), v1[g:g + 1]])
            own = q[g * (nq // nkv):(g + 1) * (nq // nkv)]
            heads.append(torch.softmax(own @ keys.T / math.sqrt(d), -1) @ values)
    out = torch.cat(heads).reshape(B, nq * d) @ t["w_o"].double()
    return (out + x if _has_norm(case) else out), new_k, new_v


def _exact_mla(case, t):
    B, nh, n, lat, r, L, base = (case["batch"], case["n_heads"], case["nope"], 512, 64, case["kv"], case["rope_base"])
    x = t["x"].double()
    q = (x @ t["w_q"].double()).reshape(B, nh, n + r)
    kv = x @ t["w_kv"].double()
    row = torch.cat([kv[:, :lat], _rope(kv[:, lat:], L, base, r)], -1)
    a = []
    for b in range(B):
        keys = torch.cat([t["kv"][b, :L].double(), row[b:b + 1]])
        q_lat = torch.stack([q[b, i, :n] @ t["w_up"][i].double() for i in range(nh)])
        query = torch.cat([q_lat, _rope(q[b, :, n:], L, base, r)], -1)
        z = torch.softmax(query @ keys.T / math.sqrt(n + r), -1) @ keys[:, :lat]
        a.append(torch.cat([z[i] @ t["w_down"][i].double() for i in range(nh)]))
    return torch.stack(a) @ t["w_o"].double(), row


def exact(case, seed):
    g = _generator(seed)
    if case["kind"] == "team":
        src = _team_input(case, g)
        N = case["team_size"]
        if case["call"] == "gather":  # out[k][b][j] = in[k][(b - j) mod N]
            return [torch.stack([torch.stack([src[:, (b - j) % N] for j in range(N)], 1) for b in range(N)], 1).double()]
        all_of = src.double().sum(1, keepdim=True) if case["op"] == "sum" else src.double().amax(1, keepdim=True)
        return [all_of.expand(-1, N, -1).contiguous()]
    outputs, x = [], None
    for _ in range(case["layers"]):
        t = _layer_inputs(case, g)
        if case["kind"] == "ffn":
            z = t["z"].double()
            h, u = z @ t["w1"].double().T, z @ t["w2"].double().T
            act = h * torch.sigmoid(h) if case["activation"] == "silu" else 0.5 * h * (1.0 + torch.erf(h / math.sqrt(2.0)))
            outputs.append((act * u) @ t["w3"].double())
        elif case["kind"] == "mla":
            outputs += _exact_mla(case, t)
        else:
            x, k, v = _exact_block(case, t, x if _is_stack(case) and x is not None else t["x"].double())
            if not _is_stack(case):
                outputs.append(x)
            outputs += [torch.stack(k), torch.stack(v)] if len(set(_row_lengths(case))) == 1 else k + v
    return outputs + ([x] if case["kind"] == "block" and _is_stack(case) else [])
