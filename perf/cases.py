"""Performance cases of the sketch-and-walk attention path.

Each case is one pass through the public calls of ``paper_2602_07397_amd.binding``
as a program that serves or evaluates a model makes them: a prefill layer
(sketch, walk, selection, attention), its single calls, a decode step over all
layers, and the decode calls of one layer.

    listed()            the named cases
    draw(rng)           one more case of the same ranges
    prepare(case, seed) what the program holds before the call, on the GPU
    run(state)          one pass; returns its outputs
    work(case)          bytes and operations one pass cannot do without
    tolerance(case)     how far two correct implementations may differ
    exact(case, seed)   the outputs in 64 bits, plain torch
"""
import math

import numpy as np
import torch

from paper_2602_07397_amd import binding as sw

R_DIM = 64       # sketch dimension (capped at the head dimension)
POWER = 8        # walk exponent

_PREFILL = {"kind": "prefill", "dtype": "bf16", "h_q": 32, "h_kv": 8, "d": 128, "B": 128, "pct": 20}
_ATTN = {"kind": "attn", "pct": 20, "lse": False}
_DECODE = {"kind": "decode_step", "dtype": "bf16", "h_q": 32, "h_kv": 8, "d": 128, "B": 64, "pct": 20}


def listed():
    return [
        # the smallest whole layer: one fp32 head of 2048 tokens; launches and latency
        {**_PREFILL, "name": "prefill_2k_1head_f32", "dtype": "f32", "h_q": 1, "h_kv": 1, "d": 64,
         "B": 64, "lens": "2048"},
        # a short prompt (ragged end) of a Llama-3-8B-shaped layer
        {**_PREFILL, "name": "prefill_4k_bf16", "lens": "4000"},
        # the long prompt of the same layer
        {**_PREFILL, "name": "prefill_32k_bf16", "lens": "32768"},
        # a batch of prompts of different lengths, 28 query heads over 4 key heads
        {**_PREFILL, "name": "prefill_varlen_bf16", "h_q": 28, "h_kv": 4,
         "lens": "14336,9001,12800,3333,8192"},
        # the sketch alone (with the block means a decode state starts from)
        {"kind": "sketch", "name": "sketch_32k_bf16", "dtype": "bf16", "h_q": 32, "h_kv": 8,
         "d": 128, "B": 128, "lens": "32768"},
        # walk and selection of a 131072-token prompt: 1024 blocks
        {"kind": "walk", "name": "walk_select_128k", "blocks": "1024", "variant": "power",
         "first": False, "pct": 20},
        # fp32 attention of an evaluation run: grouped heads, log-sum-exp asked for
        {**_ATTN, "name": "attn_8k_f32", "dtype": "f32", "h_q": 8, "h_kv": 2, "d": 128, "B": 64,
         "lens": "8192", "lse": True},
        # a model without grouped heads and with a head dimension of 64
        {**_ATTN, "name": "attn_8k_mha_d64_bf16", "dtype": "bf16", "h_q": 16, "h_kv": 16, "d": 64,
         "B": 64, "lens": "8000"},
        # serving: 16 sequences of 65536 cached tokens, one step over the layers
        {**_DECODE, "name": "decode_step_b16_64k", "batch": 16, "ctx": 65536, "layers": 8,
         "ragged": False},
        # one user: batch 1, every layer of the model, 32768 cached tokens
        {**_DECODE, "name": "decode_step_b1_32k", "batch": 1, "ctx": 32768, "layers": 32,
         "ragged": False},
        # a model that calls layer by layer, sequences of different lengths
        {**_DECODE, "kind": "decode_layer", "name": "decode_layer_b4_16k", "batch": 4, "ctx": 16000,
         "layers": 1, "ragged": True},
        # fp32 decode attention of an evaluation run
        {"kind": "decode_attn", "name": "decode_attn_b4_32k_f32", "dtype": "f32", "h_q": 32,
         "h_kv": 8, "d": 128, "B": 64, "batch": 4, "ctx": 32768, "pct": 20, "ragged": False},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


_HEADS = ((32, 8), (28, 4), (16, 16), (8, 2), (8, 8), (4, 1), (1, 1))
_HEADS_DECODE = ((32, 8), (16, 16), (8, 2), (8, 1), (16, 8))


def draw(rng):
    kind = rng.choice(["prefill", "prefill", "sketch", "walk", "attn", "attn", "decode_step",
                       "decode_step", "decode_layer", "decode_attn"])
    dtype = rng.choice(["bf16", "bf16", "f32"])
    pct = rng.choice([10, 20, 20, 30])
    if kind == "walk":
        blocks = _log_int(rng, 16, 1000)
        many = rng.random() < 0.3
        return {"kind": "walk", "blocks": "%d,%d,%d" % (blocks // 3 + 1, blocks // 2 + 1, blocks // 4 + 1)
                if many else str(blocks),
                "variant": rng.choice(["power", "power", "relu", "softmax", "matpow"]) if blocks <= 512
                else "power", "first": rng.random() < 0.2, "pct": pct}
    if kind in ("prefill", "sketch", "attn"):
        h_q, h_kv = rng.choice(_HEADS)
        d, B = rng.choice([64, 128, 128]), rng.choice([64, 128, 128])
        top = 20000 if dtype == "bf16" else 6000
        n = _log_int(rng, 700, min(40000, top * 32 // max(8, h_q)))
        lens = str(n)
        if rng.random() < 0.3:
            a, b = n // 2 + rng.randrange(1, 60), n // 3 + 1
            lens = "%d,%d,%d" % (a, b, n // 5 + 17)
        case = {"kind": kind, "dtype": dtype, "h_q": h_q, "h_kv": h_kv, "d": d, "B": B, "lens": lens}
        if kind != "sketch":
            case["pct"] = pct
        if kind == "attn":
            case["lse"] = rng.random() < 0.3
        return case
    h_q, h_kv = rng.choice(_HEADS_DECODE)
    batch = _log_int(rng, 1, 24)
    case = {"kind": kind, "dtype": dtype, "h_q": h_q, "h_kv": h_kv, "d": rng.choice([64, 128, 128]),
            "B": rng.choice([64, 64, 128]), "pct": pct, "batch": batch,
            "ctx": _log_int(rng, 500, 400000 // max(8, batch)) + rng.randrange(64),
            "ragged": rng.random() < 0.5}
    if kind != "decode_attn":
        layers = _log_int(rng, 2, 24 if batch <= 4 else 8) if kind == "decode_step" else 1
        # a pass stays below the largest listed one
        per_layer = work({**case, "layers": 1})["bytes"]
        case["layers"] = max(1, min(layers, int(3.5e9 // per_layer)))
    return case


# --------------------------------------------------------------------------- inputs


def _gen(seed, *salt):
    g = torch.Generator(device="cuda")
    s = int(seed) * 1000003 + 17
    for x in salt:
        s = (s * 7919 + int(x) + 1) % (1 << 62)
    g.manual_seed(s)
    return g


def _dtype(case):
    return torch.bfloat16 if case.get("dtype") == "bf16" else torch.float32


def _lens(case):
    return [int(x) for x in case["lens"].split(",")]


def _cu(lens):
    return [0] + [int(x) for x in np.cumsum(lens)]


def _srht(d, seed):
    rng = np.random.default_rng(seed + 999)
    signs = rng.choice(np.array([-1, 1], dtype=np.int8), size=d)
    cols = rng.choice(d, size=min(R_DIM, d), replace=False).astype(np.int32)
    return torch.from_numpy(signs).cuda(), torch.from_numpy(cols).cuda()


def _qk(case, lens, g):
    """Queries and keys N(0, 1) with a sink in block 0, a local window and two
    needle blocks per sequence, rounded to the case's type."""
    N, h_q, h_kv, d, B = sum(lens), case["h_q"], case["h_kv"], case["d"], case["B"]
    dt = _dtype(case)
    Q = torch.randn((h_q, N, d), generator=g, device="cuda", dtype=dt)
    K = torch.randn((h_kv, N, d), generator=g, device="cuda", dtype=dt)
    a = 0
    for n in lens:
        u = torch.randn((h_kv, 1, d), generator=g, device="cuda")
        u = u / u.norm(dim=-1, keepdim=True)
        e = a + n
        K[:, a:a + min(B, n)] += (3.0 * u).to(dt)
        if n > B:
            K[:, a:e - B] += 0.5 * Q[::h_q // h_kv, a + B:e]
        for f in (0.31, 0.62):
            j = a + int(f * n) // B * B
            p = a + min(n - 1, int(f * n) + 2 * B)
            w = min(B, e - j)
            K[:, j:j + w] = Q[::h_q // h_kv, p:p + 1] + 0.1 * K[:, j:j + w]
        a = e
    return Q, K


def _walk_state(blocks, g):
    """A walk state of an earlier layer: lower triangular rows of (a / c)^8
    divided by their largest value, sequences back to back."""
    parts = []
    for b in blocks:
        a = torch.tril(torch.randn((b, b), generator=g, device="cuda", dtype=torch.float64))
        w = (a / a.abs().max().clamp_min(1e-300)) ** POWER
        parts.append((w / w.amax(dim=1, keepdim=True).clamp_min(1e-300)).reshape(-1))
    return torch.cat(parts)


def _budget(avail, pct):
    return max(min(2, avail), min(avail, (avail * pct + 99) // 100))


def _random_selection(blocks, pct, g):
    """A selection as sw.select_topk_blocks lays it out: first, own and random
    earlier blocks of every row."""
    kmax = max(_budget(i + 1, pct) for b in blocks for i in range(b))
    rows, cnts = [], []
    for b in blocks:
        v = torch.rand((b, b), generator=g, device="cuda", dtype=torch.float64)
        m = _select_mask(v, pct)
        rows.append(_mask_to_idx(m, kmax))
        cnts.append(m.sum(dim=1).to(torch.int32))
    return torch.cat(rows).contiguous(), torch.cat(cnts).contiguous(), kmax


def _select_mask(R, pct):
    """Selected blocks of every row of a square walk state (forced first and
    own block, then the largest values, lower index first among equals)."""
    b = R.shape[0]
    i = torch.arange(b, device=R.device)
    v = R.masked_fill(i[None, :] > i[:, None], -math.inf)
    v[:, 0] = math.inf
    v[i, i] = math.inf
    order = torch.sort(v, dim=1, descending=True, stable=True).indices
    tau = ((i + 1) * pct + 99) // 100
    tau = torch.minimum(torch.maximum(tau, torch.clamp(i + 1, max=2)), i + 1)
    rank = torch.empty_like(order)
    rank.scatter_(1, order, i[None, :].expand(b, b).contiguous())
    return rank < tau[:, None]


def _mask_to_idx(mask, kmax):
    b = mask.shape[1]
    j = torch.arange(b, device=mask.device)
    x = torch.where(mask, j[None, :].expand_as(mask), b)
    x = torch.sort(x, dim=1).values
    if x.shape[1] < kmax:
        x = torch.cat([x, x.new_full((x.shape[0], kmax - x.shape[1]), b)], dim=1)
    x = x[:, :kmax]
    return torch.where(x < b, x, -1).to(torch.int32)


def _positions(case):
    """Position of the new token of every sequence (= tokens cached before it)."""
    ctx = case["ctx"]
    if not case["ragged"]:
        return [ctx] * case["batch"]
    return [max(1, ctx - (b * 977 + 41 * b * b) % (ctx // 2 + 1)) for b in range(case["batch"])]


def _decode_prompt(case, seed, layer, seq, n):
    g = _gen(seed, 11, layer, seq)
    Q, K = _qk(case, [n], g)
    V = torch.randn((case["h_kv"], n, case["d"]), generator=g, device="cuda", dtype=_dtype(case))
    return Q, K, V


def _decode_tokens(case, seed, L):
    g = _gen(seed, 12)
    dt, b = _dtype(case), case["batch"]
    q = torch.randn((L, b, case["h_q"], case["d"]), generator=g, device="cuda", dtype=dt)
    k = torch.randn((L, b, case["h_kv"], case["d"]), generator=g, device="cuda", dtype=dt)
    v = torch.randn((L, b, case["h_kv"], case["d"]), generator=g, device="cuda", dtype=dt)
    return q, k, v


def _decode_sel(case, seed):
    g = _gen(seed, 13)
    B, pos = case["B"], _positions(case)
    kmax = max(_budget(p // B + 1, case["pct"]) for p in pos)
    idx = torch.full((len(pos), kmax), -1, dtype=torch.int32, device="cuda")
    cnt = torch.zeros((len(pos),), dtype=torch.int32, device="cuda")
    for b, p in enumerate(pos):
        nb = p // B + 1
        t = _budget(nb, case["pct"])
        v = torch.rand((nb,), generator=g, device="cuda")
        v[0] = v[nb - 1] = 2.0
        idx[b, :t] = torch.sort(torch.topk(v, t).indices).values.to(torch.int32)
        cnt[b] = t
    return idx, cnt, kmax


def prepare(case, seed):
    kind = case["kind"]
    st = {"case": case}
    if kind == "walk":
        blocks = [int(x) for x in case["blocks"].split(",")]
        g = _gen(seed, 1)
        A, c = _score_input(blocks, g)
        st.update(cu=_cu([128 * b for b in blocks]), A=A, c=c,
                  R=None if case["first"] else _walk_state(blocks, g))
        return st
    if kind in ("prefill", "sketch", "attn"):
        lens = _lens(case)
        g = _gen(seed, 2)
        Q, K = _qk(case, lens, g)
        st.update(cu=_cu(lens), Q=Q, K=K)
        st["signs"], st["cols"] = _srht(case["d"], seed)
        blocks = [-(-n // case["B"]) for n in lens]
        if kind != "sketch":
            st["V"] = torch.randn(K.shape, generator=g, device="cuda", dtype=_dtype(case))
        if kind == "prefill":
            st["R"] = _walk_state(blocks, g)
        if kind == "attn":
            st["idx"], st["cnt"], st["kmax"] = _random_selection(blocks, case["pct"], g)
        return st
    # decode
    L, batch, B, d = case.get("layers", 1), case["batch"], case["B"], case["d"]
    pos = _positions(case)
    b_max = max(pos) // B + 1
    T = b_max * B
    dt = _dtype(case)
    q, k, v = _decode_tokens(case, seed, L)
    Kc = torch.zeros((L, batch, case["h_kv"], T, d), dtype=dt, device="cuda")
    Vc = torch.zeros_like(Kc)
    st.update(q=q, k=k, v=v, Kc=Kc, Vc=Vc, b_max=b_max,
              pos=torch.tensor(pos, dtype=torch.int32, device="cuda"))
    if kind == "decode_attn":
        g = _gen(seed, 14)
        Kc.normal_(generator=g)
        Vc.normal_(generator=g)
        st["idx"], st["cnt"], st["kmax"] = _decode_sel(case, seed)
        st["O"] = torch.empty_like(q[0])
        st["ws"] = torch.empty((sw.decode_attn_workspace_bytes(batch, case["h_q"], case["h_kv"], d),),
                               dtype=torch.uint8, device="cuda")
        return st
    st["signs"], st["cols"] = _srht(d, seed)
    r = int(st["cols"].numel())
    state = torch.zeros((L, sw.decode_state_bytes(batch, d, r, b_max)), dtype=torch.uint8, device="cuda")
    for l in range(L):
        for b, n in enumerate(pos):
            Q, K, V = _decode_prompt(case, seed, l, b, n)
            sk = sw.sketch_scores(Q, K, [0, n], B, st["signs"], st["cols"], want_means=True)
            sw.decode_state_init(state[l], batch, d, r, b_max, b, n, B, sk)
            Kc[l, b, :, :n] = K
            Vc[l, b, :, :n] = V
    st["state"] = state
    kmax = sw.select_max_count_decode(b_max, density_pct=case["pct"])
    st["kmax"] = kmax
    if kind == "decode_step":
        st["out"] = {"rows": torch.zeros((L, batch, b_max), dtype=torch.float64, device="cuda"),
                     "idx": torch.zeros((L, batch, kmax), dtype=torch.int32, device="cuda"),
                     "cnt": torch.zeros((L, batch), dtype=torch.int32, device="cuda"),
                     "O": torch.zeros_like(q)}
        st["ws"] = torch.empty((sw.load().sw_decode_step_workspace_bytes(batch, case["h_q"], case["h_kv"], d),),
                               dtype=torch.uint8, device="cuda")
    else:
        st["r_prev"] = _decode_row(case, seed)
        st["r_out"] = torch.zeros_like(st["r_prev"])
        st["idx"] = torch.zeros((batch, kmax), dtype=torch.int32, device="cuda")
        st["cnt"] = torch.zeros((batch,), dtype=torch.int32, device="cuda")
        st["O"] = torch.zeros_like(q[0])
        st["ws"] = torch.empty((sw.decode_attn_workspace_bytes(batch, case["h_q"], case["h_kv"], d),),
                               dtype=torch.uint8, device="cuda")
    return st


def _score_input(blocks, g):
    """Block scores as a sketch gives them: causal inner products of 64-dim
    rows with a heavy first column."""
    parts, scale = [], []
    for b in blocks:
        q = torch.randn((b, R_DIM), generator=g, device="cuda", dtype=torch.float64)
        k = torch.randn((b, R_DIM), generator=g, device="cuda", dtype=torch.float64)
        k[0] += 0.5 * q.mean(dim=0) + 0.1
        a = torch.tril(q @ k.T) / math.sqrt(R_DIM)
        parts.append(a.reshape(-1))
        scale.append(a.abs().max())
    return torch.cat(parts).contiguous(), torch.stack(scale)


def _decode_row(case, seed):
    """The walk row an earlier layer left for every sequence."""
    pos = _positions(case)
    b_max = max(pos) // case["B"] + 1
    g = _gen(seed, 15)
    w = torch.randn((len(pos), b_max), generator=g, device="cuda", dtype=torch.float64).abs() ** 4
    bc = torch.tensor([p // case["B"] for p in pos], device="cuda")
    w = torch.where(torch.arange(b_max, device="cuda")[None, :] <= bc[:, None], w, 0.0)
    return (w / w.amax(dim=1, keepdim=True)).contiguous()


# --------------------------------------------------------------------------- one pass

_VARIANT = {"power": sw.WALK_POWER, "relu": sw.WALK_RELU, "softmax": sw.WALK_SOFTMAX,
            "matpow": sw.WALK_MATPOW}


def run(state):
    c = state["case"]
    kind = c["kind"]
    if kind == "prefill":
        cu, B = state["cu"], c["B"]
        sk = sw.sketch_scores(state["Q"], state["K"], cu, B, state["signs"], state["cols"])
        R = sw.walk_update(sk["A"], sk["A_scale"], POWER, cu, B, R_prev=state["R"])
        idx, cnt, kmax = sw.select_topk_blocks(R, cu, B, density_pct=c["pct"])
        O = sw.sparse_attn_prefill(state["Q"], state["K"], state["V"], cu, B, idx, cnt, kmax)
        return {"R": R, "idx": idx, "cnt": cnt, "O": O}
    if kind == "sketch":
        return sw.sketch_scores(state["Q"], state["K"], state["cu"], c["B"], state["signs"],
                                state["cols"], want_means=True)
    if kind == "walk":
        if c["variant"] == "power":
            R = sw.walk_update(state["A"], state["c"], POWER, state["cu"], 128, R_prev=state["R"])
        else:
            R = sw.walk_update_variant(_VARIANT[c["variant"]], state["A"], state["c"], POWER,
                                       state["cu"], 128, R_prev=state["R"], logit_scale=0.7)
        idx, cnt, _ = sw.select_topk_blocks(R, state["cu"], 128, density_pct=c["pct"])
        return {"R": R, "idx": idx, "cnt": cnt}
    if kind == "attn":
        return sw.sparse_attn_prefill(state["Q"], state["K"], state["V"], state["cu"], c["B"],
                                      state["idx"], state["cnt"], state["kmax"], want_lse=c["lse"])
    if kind == "decode_attn":
        return sw.sparse_attn_decode(state["q"][0], state["Kc"][0], state["Vc"][0], c["B"],
                                     state["pos"], state["idx"], state["cnt"], state["kmax"],
                                     O=state["O"], workspace=state["ws"])
    if kind == "decode_step":
        return sw.decode_step(state["q"], state["k"], state["v"], state["Kc"], state["Vc"],
                              state["state"], state["pos"], state["signs"], state["cols"], c["B"],
                              state["b_max"], s=POWER, density_pct=c["pct"], kmax=state["kmax"],
                              out=state["out"], workspace=state["ws"])
    q, k, v = state["q"][0], state["k"][0], state["v"][0]
    Kc, Vc, stt, pos = state["Kc"][0], state["Vc"][0], state["state"][0], state["pos"]
    batch, d, b_max = c["batch"], c["d"], state["b_max"]
    sw.kv_append(k, v, Kc, Vc, pos)
    sw.sketch_scores_decode(q, k, c["B"], pos, state["signs"], state["cols"], b_max, stt)
    row = sw.walk_update_decode(stt, batch, d, int(state["cols"].numel()), b_max, c["B"], pos, POWER,
                                r_prev=state["r_prev"], r_out=state["r_out"])
    idx, cnt, kmax = sw.select_topk_blocks_decode(row, c["B"], pos, density_pct=c["pct"],
                                                  kmax=state["kmax"], idx=state["idx"],
                                                  cnt=state["cnt"])
    O = sw.sparse_attn_decode(q, Kc, Vc, c["B"], pos, idx, cnt, kmax, O=state["O"],
                              workspace=state["ws"])
    return {"rows": row, "idx": idx, "cnt": cnt, "O": O}


# --------------------------------------------------------------------------- work and tolerance


def _prefill_pairs(n, B, pct):
    """(query, key) pairs one head attends to in one sequence."""
    b, pairs = -(-n // B), 0
    for i in range(b):
        rows = min(B, n - i * B)
        pairs += (_budget(i + 1, pct) - 1) * B * rows + rows * (rows + 1) // 2
    return pairs


def work(case):
    kind = case["kind"]
    es = 2 if case.get("dtype") == "bf16" else 4
    nbytes = flops = 0
    if kind in ("prefill", "walk"):
        blocks = ([int(x) for x in case["blocks"].split(",")] if kind == "walk"
                  else [-(-n // case["B"]) for n in _lens(case)])
        for b in blocks:
            # A and R_prev read, R written (triangles), the selection written
            nbytes += 8 * 3 * b * (b + 1) // 2 + 4 * sum(_budget(i + 1, case["pct"]) for i in range(b))
            if kind == "prefill" or not case["first"]:
                flops += b * (b + 1) * (b + 2) // 3
            if case.get("variant") == "matpow":
                flops += 3 * b * (b + 1) * (b + 2) // 3
    if kind in ("prefill", "sketch", "attn"):
        N, h_q, h_kv, d, B = sum(_lens(case)), case["h_q"], case["h_kv"], case["d"], case["B"]
        nbytes += (h_q + h_kv) * N * d * es
        if kind != "attn":
            flops += (h_q + h_kv) * N * d
        if kind == "sketch":
            for n in _lens(case):
                b = -(-n // B)
                nbytes += 8 * (b * b + 2 * b * (R_DIM + d))
                flops += b * b * R_DIM
        if kind != "sketch":
            nbytes += (h_q + h_kv) * N * d * es
            flops += 4 * d * h_q * sum(_prefill_pairs(n, B, case["pct"]) for n in _lens(case))
    if kind.startswith("decode"):
        L, h_q, h_kv, d, B = case.get("layers", 1), case["h_q"], case["h_kv"], case["d"], case["B"]
        for p in _positions(case):
            nb = p // B + 1
            tok = (_budget(nb, case["pct"]) - 1) * B + p - (nb - 1) * B + 1
            nbytes += L * (2 * h_kv * tok * d * es + 2 * h_q * d * es)
            flops += L * 4 * d * h_q * tok
            if kind != "decode_attn":
                # score cache (fp32 triangle), both sketches, token rows
                nbytes += L * (2 * nb * (nb + 1) + 16 * nb * min(R_DIM, d) + 4 * h_kv * d * es + 16 * nb)
                flops += L * (2 * nb * (nb + 1) // 2 + 4 * nb * min(R_DIM, d))
    return {"bytes": int(nbytes), "flops": int(flops)}


def tolerance(case):
    kind = case["kind"]
    if kind in ("sketch", "walk"):
        # fp64 throughout: about 1e-15 from the 64-bit result; the signed sums
        # of a matrix power cancel
        return {"rel": 1e-11, "max": 1e-9} if case.get("variant") == "matpow" else {"rel": 1e-13, "max": 1e-11}
    # decode: scores cached in fp32 (walk rows about 1e-7 from 64 bits), so a
    # near tie of two blocks may fall either way
    if case["dtype"] == "f32":
        return {"rel": 2.5e-6, "max": 2e-4, "differ": 2e-3 if kind.startswith("decode_") else 0.0}
    return {"rel": 1e-2, "max": 0.1, "differ": 2e-3 if kind.startswith("decode_") else 0.0}


# --------------------------------------------------------------------------- 64-bit results


def _hadamard(d):
    H = torch.ones((1, 1), dtype=torch.float64)
    while H.shape[0] < d:
        H = torch.cat([torch.cat([H, H], 1), torch.cat([H, -H], 1)], 0)
    return H.cuda()


def _pool(x, B):
    """Block means of the head mean of x [h][n][d], in 64 bits."""
    n, d = x.shape[1], x.shape[2]
    m = torch.zeros((n, d), dtype=torch.float64, device=x.device)
    for h in range(x.shape[0]):
        m += x[h].double()
    m /= x.shape[0]
    b = -(-n // B)
    full = n // B
    out = torch.empty((b, d), dtype=torch.float64, device=x.device)
    out[:full] = m[:full * B].reshape(full, B, d).mean(dim=1)
    if full < b:
        out[full] = m[full * B:].mean(dim=0)
    return out


def _project(m, signs, cols):
    H = _hadamard(m.shape[-1])
    return ((m * signs.double()) @ H)[..., cols.long()] / math.sqrt(cols.numel())


def _weights(a, c, variant="power"):
    c = c if float(c) > 0 else 1.0
    if variant == "softmax":
        x = (0.7 * a).masked_fill(torch.triu(torch.ones_like(a), 1) > 0, -math.inf)
        return torch.softmax(x, dim=1)
    w = a / c
    if variant == "matpow":
        w = w @ w
        w = w @ w
        return w @ w
    return (w.clamp_min(0.0) if variant == "relu" else w) ** POWER


def _norm_rows(R):
    mx = R.abs().amax(dim=-1, keepdim=True)
    return R / torch.where(mx > 0, mx, 1.0)


def _attend(Q, K, V, mask, B, out, lse=None):
    """out[h][n][d] of one sequence in 64 bits; mask [b][b] of selected blocks."""
    h_q, n, d = Q.shape
    G = h_q // K.shape[0]
    t = torch.arange(n, device=Q.device)
    for g in range(K.shape[0]):
        k, v = K[g].double(), V[g].double()
        kt = k.T.contiguous()
        for a in range(0, n, 1024):
            e = min(n, a + 1024)
            keep = mask[t[a:e] // B][:, t[:e] // B] & (t[None, :e] <= t[a:e, None])
            for u in range(g * G, (g + 1) * G):
                s = (Q[u, a:e].double() @ kt[:, :e]) / math.sqrt(d)
                s.masked_fill_(~keep, -math.inf)
                if lse is not None:
                    lse[u, a:e] = torch.logsumexp(s, dim=1)
                out[u, a:e] = torch.softmax(s, dim=1) @ v[:e]


def exact(case, seed):
    kind = case["kind"]
    if kind in ("prefill", "sketch", "attn"):
        lens, B = _lens(case), case["B"]
        st = prepare(case, seed)
        Q, K, cu = st["Q"], st["K"], st["cu"]
        res = {n: [] for n in ("Qs", "Ks", "A", "A_scale", "Qbar", "Kbar", "R", "idx", "cnt")}
        O = torch.empty(Q.shape, dtype=torch.float64, device="cuda") if kind != "sketch" else None
        lse = (torch.empty(Q.shape[:2], dtype=torch.float64, device="cuda")
               if kind == "attn" and case["lse"] else None)
        mo = ro = 0
        blocks = [-(-n // B) for n in lens]
        kmax = max(_budget(i + 1, case.get("pct", 20)) for b in blocks for i in range(b))
        for s, n in enumerate(lens):
            b, a, e = blocks[s], cu[s], cu[s + 1]
            if kind == "attn":
                ix = st["idx"][ro:ro + b].long()
                mask = torch.zeros((b, b + 1), dtype=torch.bool, device="cuda")
                mask.scatter_(1, torch.where(ix < 0, b, ix), True)
                _attend(Q[:, a:e], K[:, a:e], st["V"][:, a:e], mask[:, :b], B, O[:, a:e],
                        None if lse is None else lse[:, a:e])
                ro += b
                continue
            qb, kb = _pool(Q[:, a:e], B), _pool(K[:, a:e], B)
            qs, ks = _project(qb, st["signs"], st["cols"]), _project(kb, st["signs"], st["cols"])
            A = torch.tril(qs @ ks.T) / math.sqrt(qs.shape[1])
            c = A.abs().max()
            for name, x in (("Qs", qs), ("Ks", ks), ("A", A.reshape(-1)), ("A_scale", c.reshape(1)),
                            ("Qbar", qb), ("Kbar", kb)):
                res[name].append(x)
            if kind == "prefill":
                R = _norm_rows(torch.tril(st["R"][mo:mo + b * b].reshape(b, b) @ _weights(A, c)))
                mask = _select_mask(R, case["pct"])
                res["R"].append(R.reshape(-1))
                res["idx"].append(_mask_to_idx(mask, kmax))
                res["cnt"].append(mask.sum(dim=1).to(torch.int32))
                _attend(Q[:, a:e], K[:, a:e], st["V"][:, a:e], mask, B, O[:, a:e])
                mo += b * b
        if kind == "sketch":
            return {n: torch.cat(res[n]) for n in ("Qs", "Ks", "A", "A_scale", "Qbar", "Kbar")}
        if kind == "prefill":
            return {**{n: torch.cat(res[n]) for n in ("R", "idx", "cnt")}, "O": O}
        return (O, lse) if lse is not None else O
    if kind == "walk":
        st = prepare(case, seed)
        blocks = [int(x) for x in case["blocks"].split(",")]
        kmax = max(_budget(i + 1, case["pct"]) for b in blocks for i in range(b))
        Rs, idx, cnt, mo = [], [], [], 0
        for s, b in enumerate(blocks):
            W = _weights(st["A"][mo:mo + b * b].reshape(b, b), st["c"][s], case["variant"])
            if st["R"] is not None:
                W = st["R"][mo:mo + b * b].reshape(b, b) @ W
            R = _norm_rows(torch.tril(W))
            mask = _select_mask(R, case["pct"])
            Rs.append(R.reshape(-1))
            idx.append(_mask_to_idx(mask, kmax))
            cnt.append(mask.sum(dim=1).to(torch.int32))
            mo += b * b
        return {"R": torch.cat(Rs), "idx": torch.cat(idx), "cnt": torch.cat(cnt)}
    return _exact_decode(case, seed)


def _exact_decode(case, seed):
    kind, L, batch, B, d = case["kind"], case.get("layers", 1), case["batch"], case["B"], case["d"]
    pos, h_q, h_kv = _positions(case), case["h_q"], case["h_kv"]
    G = h_q // h_kv
    b_max = max(pos) // B + 1
    q, k, v = _decode_tokens(case, seed, L)
    O = torch.zeros((L, batch, h_q, d), dtype=torch.float64, device="cuda")

    def attend(l, b, blocks, Kb, Vb):
        tok = (torch.as_tensor(blocks, device="cuda").long()[:, None] * B
               + torch.arange(B, device="cuda")[None, :]).reshape(-1)
        tok = tok[tok <= pos[b]]
        for g in range(h_kv):
            s = q[l, b, g * G:(g + 1) * G].double() @ Kb[g, tok].double().T.contiguous() / math.sqrt(d)
            O[l, b, g * G:(g + 1) * G] = torch.softmax(s, dim=1) @ Vb[g, tok].double()

    if kind == "decode_attn":
        st = prepare(case, seed)
        for b in range(batch):
            attend(0, b, st["idx"][b, :int(st["cnt"][b])], st["Kc"][0, b], st["Vc"][0, b])
        return O[0]
    signs, cols = _srht(d, seed)
    r = int(cols.numel())
    rows = torch.zeros((L, batch, b_max), dtype=torch.float64, device="cuda")
    first = _decode_row(case, seed) if kind == "decode_layer" else None
    kmax = max(_budget(i + 1, case["pct"]) for i in range(b_max))
    idx = torch.full((L, batch, kmax), -1, dtype=torch.int32, device="cuda")
    cnt = torch.zeros((L, batch), dtype=torch.int32, device="cuda")
    for l in range(L):
        for b, n in enumerate(pos):
            Q, K, V = _decode_prompt(case, seed, l, b, n)
            qb, kb = _pool(Q, B), _pool(K, B)
            bc = n // B
            A = torch.zeros((bc + 1, bc + 1), dtype=torch.float64, device="cuda")
            nb = qb.shape[0]
            Qs, Ks = _project(qb, signs, cols), _project(kb, signs, cols)
            A[:nb, :nb] = torch.tril(Qs @ Ks.T) / math.sqrt(r)
            c = A.abs().max()
            have = n - bc * B
            qn, kn = q[l, b].double().mean(dim=0), k[l, b].double().mean(dim=0)
            qm = (qb[bc] * have + qn) / (have + 1) if have else qn
            km = (kb[bc] * have + kn) / (have + 1) if have else kn
            qt, qo, ko = (_project(x, signs, cols) for x in (qn, qm, km))
            A[bc, :bc] = Ks[:bc] @ qt / math.sqrt(r)
            A[:bc, bc] = Qs[:bc] @ ko / math.sqrt(r)
            A[bc, bc] = qo @ ko / math.sqrt(r)
            W = _weights(A, c)
            prev = first[b, :bc + 1] if kind == "decode_layer" else rows[l - 1, b, :bc + 1] if l else None
            row = _norm_rows(W[bc] if prev is None else prev @ W)
            rows[l, b, :bc + 1] = row
            t = _budget(bc + 1, case["pct"])
            ranked = row.clone()
            ranked[0] = ranked[bc] = math.inf
            sel = torch.sort(torch.sort(ranked, descending=True, stable=True).indices[:t]).values
            idx[l, b, :t] = sel.to(torch.int32)
            cnt[l, b] = t
            attend(l, b, sel, torch.cat([K, k[l, b][:, None]], 1), torch.cat([V, v[l, b][:, None]], 1))
    if kind == "decode_layer":
        return {"rows": rows[0], "idx": idx[0], "cnt": cnt[0], "O": O[0]}
    return {"rows": rows, "idx": idx, "cnt": cnt, "O": O}
