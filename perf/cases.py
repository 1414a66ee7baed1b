"""The work that a program built on this library has it do, as measurable cases.

Three kinds of pass, each through the public entry points:

  decode     `layers` FFN blocks for `tokens` new tokens, each block with its own weights, in the
             overlapped form (halo_ffn_forward_ahead / _ahead_q4: the FFN of a block with the mask predicted
             one block earlier, predictor + mask of the next block beside it), captured once into a
             HIP graph and replayed per pass -- how a serving loop runs the blocks of a model.  Every block
             gets a hidden state of its own (N(0, 1), as after a norm) instead of the previous block's output,
             so that a rounding difference in one block cannot move the masks of the following ones.
  forward    one FFN block, predictor -> mask -> FFN back to back (halo_ffn_forward / _q4), called
             directly: a prompt's tokens at once (prefill), or a few tokens without the overlap.
  attention  `layers` attention blocks for one new token over a KV cache of `context` rows
             (halo_mha_forward_ahead), captured and replayed like `decode`.

Shapes are the LLaMA-7B / 13B / 2-70B FFN and attention shapes and the tiny float32 block that the
workloads of this repository use, and ragged ones around them.
"""
import math

import numpy as np
import torch

import paper_2601_11676_amd as H

DEV = "cuda"
GS = 128                                             # neurons per group
PLR = (0.0, 0.05, 0.1, 0.2)                          # loss rates of the simulated devices


def _ffn(name, kind, d, groups, rank, tokens, keep, weights, layers=1):
    return {"name": name, "kind": kind, "d": d, "groups": groups, "rank": rank, "tokens": tokens, "keep": keep,
            "weights": weights, "layers": layers}


def listed():
    return [
        # the smallest block: 16 tokens in float32 -- a few launches of almost no work, called from Python
        _ffn("tiny_f32", "forward", 256, 8, 64, 16, 0.5, "f32"),
        # one sequence being generated on a 7B model in bf16 (the headline): one token, half the groups
        _ffn("decode_7b", "decode", 4096, 86, 256, 1, 0.5, "bf16", 8),
        # a small batch of sequences on a 13B model, few groups kept
        _ffn("decode_13b_4tok", "decode", 5120, 108, 256, 4, 0.3, "bf16", 6),
        # a batch of sequences on a 70B model: the largest decode
        _ffn("decode_70b_8tok", "decode", 8192, 224, 512, 8, 0.5, "bf16", 2),
        # the same three over the 4-bit weights the paper's models are stored in, one sequence on 7B and 13B
        _ffn("decode_7b_q4", "decode", 4096, 86, 256, 1, 0.5, "q4", 8),
        _ffn("decode_13b_q4", "decode", 5120, 108, 256, 1, 0.5, "q4", 6),
        _ffn("decode_70b_q4_8tok", "decode", 8192, 224, 512, 8, 0.5, "q4", 4),
        # a prompt of 512 tokens through a 7B block, in bf16 and over 4-bit weights
        _ffn("prefill_7b_512", "forward", 4096, 86, 256, 512, 0.5, "bf16"),
        _ffn("prefill_7b_q4_512", "forward", 4096, 86, 256, 512, 0.5, "q4"),
        # the paper's request: a prompt of 128 tokens on a 4-bit 13B model
        _ffn("prefill_13b_q4_128", "forward", 5120, 108, 256, 128, 0.5, "q4"),
        # the largest: a long prompt, not a multiple of any tile, through a 70B block
        _ffn("prefill_70b_1000", "forward", 8192, 224, 512, 1000, 0.5, "bf16"),
        # one sequence being generated: the attention block of a 7B model with 2048 cached positions
        {"name": "attention_7b_2048", "kind": "attention", "d": 4096, "heads": 32, "rank": 256, "context": 2048,
         "keep": 0.5, "layers": 8},
    ]


def draw(rng):
    def spread(lo, hi):                              # over the logarithm
        return math.exp(rng.uniform(math.log(lo), math.log(hi)))

    kind = rng.choice(["decode", "decode", "forward", "forward", "attention", "f32"])
    keep = round(rng.uniform(0.3, 0.7), 2)
    rank = rng.choice([64, 128, 256, 512])
    if kind == "f32":
        d = 8 * round(spread(128, 1024) / 8)
        return _drop_name(_ffn("", "forward", d, rng.randint(4, 24), rng.choice([40, 64, 128]),
                               round(spread(1, 64)), keep, "f32"))
    # half of the time a hidden size of the model family, else any multiple of 128
    d = rng.choice([2048, 4096, 5120, 8192]) if rng.random() < 0.5 else 128 * round(spread(1024, 8192) / 128)
    if kind == "attention":
        return {"kind": "attention", "d": d, "heads": d // 128, "rank": rank, "context": round(spread(100, 16000)),
                "keep": keep, "layers": rng.randint(2, 6)}
    groups = max(8, min(224, round(d / GS * rng.uniform(2.5, 3.5))))
    weights = rng.choice(["bf16", "q4"])
    if kind == "decode":
        return _drop_name(_ffn("", "decode", d, groups, rank, round(spread(1, 16)), keep, weights, rng.randint(2, 4)))
    return _drop_name(_ffn("", "forward", d, groups, rank, round(spread(1, 900)), keep, weights))


def _drop_name(case):
    return {k: v for k, v in case.items() if k != "name"}


# --------------------------------------------------------------------------
# inputs: plain torch, from the seed alone
# --------------------------------------------------------------------------
def _keep_count(case, n):
    return max(1, min(n, math.floor(case["keep"] * n + 0.5)))


def _normal(g, shape, sigma, dtype):
    return torch.empty(shape, dtype=dtype, device=DEV).normal_(0.0, sigma, generator=g)


def _codes(g, words):
    """Packed 4-bit codes, bell-shaped around 8 like rounded normal weights: element 2i of a word's eight in
    bits 4i.., element 2i+1 in bits 16+4i.."""
    q = torch.special.ndtri((torch.arange(4096, dtype=torch.float64) + 0.5) / 4096)
    table = torch.clamp(torch.floor(q * 2.5 + 8.5), 0, 15).to(torch.int32).to(DEV)
    out = torch.zeros(words, dtype=torch.int32, device=DEV)
    for shift in (0, 16, 4, 20, 8, 24, 12, 28):
        out |= table[torch.randint(0, 4096, (words,), generator=g, device=DEV)] << shift
    return out


def _scales(g, n):
    return ((1.0 + torch.randint(0, 128, (n,), generator=g, device=DEV) / 128.0) * 2.0 ** -8).to(torch.bfloat16)


def _layer_inputs(case, g):
    """One FFN block: weights in the library's layouts, predictor, hidden states, loss outcomes."""
    d, G, r, T = case["d"], case["groups"], case["rank"], case["tokens"]
    ffn = G * GS
    dt = torch.float32 if case["weights"] == "f32" else torch.bfloat16
    lay = {"x": _normal(g, (T, d), 1.0, dt), "At": _normal(g, (r, d), 0.02, dt), "Bt": _normal(g, (G, r), 0.02, dt),
           "drop": (torch.rand((T, len(PLR)), generator=g, device=DEV)
                    < torch.tensor(PLR, device=DEV)).to(torch.uint8)}
    if case["weights"] == "q4":
        lay["w"] = (_codes(g, ffn * d // 8).view(ffn, d // 8), _scales(g, ffn * d // 128).view(ffn, d // 128),
                    _codes(g, ffn * d // 8).view(ffn, d // 8), _scales(g, ffn * d // 128).view(ffn, d // 128),
                    _codes(g, ffn * d // 8).view(G, d, GS // 8), _scales(g, G * d).view(G, d))
    else:
        lay["w"] = (_normal(g, (ffn, d), 0.02, dt), _normal(g, (ffn, d), 0.02, dt), _normal(g, (G, d, GS), 0.02, dt))
    return lay


def _mha_layer_inputs(case, g):
    d, n, r, pos = case["d"], case["heads"], case["rank"], case["context"]
    dt, rows = torch.bfloat16, case["context"] + 256
    return {"x": _normal(g, (1, d), 1.0, dt), "At": _normal(g, (r, d), 0.02, dt), "Bt": _normal(g, (n, r), 0.02, dt),
            "drop": (torch.rand((1, len(PLR)), generator=g, device=DEV)
                     < torch.tensor(PLR, device=DEV)).to(torch.uint8),
            "Wq": _normal(g, (n * GS, d), 0.02, dt), "Wk": _normal(g, (n * GS, d), 0.02, dt),
            "Wv": _normal(g, (n * GS, d), 0.02, dt), "Wo": _normal(g, (n, d, GS), 0.02, dt),
            "k": _normal(g, (n, rows, GS), 1.0, dt), "v": _normal(g, (n, rows, GS), 1.0, dt), "pos": pos}


def _inputs(case, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    make = _mha_layer_inputs if case["kind"] == "attention" else _layer_inputs
    return [make(case, g) for _ in range(case["layers"])]


# --------------------------------------------------------------------------
# the passes
# --------------------------------------------------------------------------
def _prediction_buffers(T, G, K):
    return {"scores": torch.zeros((T, G), dtype=torch.float32, device=DEV),
            "mask": torch.zeros((T, G), dtype=torch.uint8, device=DEV),
            "surv_idx": torch.zeros((T, K), dtype=torch.int32, device=DEV),
            "n_surv": torch.zeros((T,), dtype=torch.int32, device=DEV)}


def _captured(enqueue):
    enqueue()                                        # once outside the capture, as a program warms up
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        enqueue()
    torch.cuda.synchronize()
    return graph.replay


def prepare(case, seed):
    layers = _inputs(case, seed)
    attention = case["kind"] == "attention"
    G, r, T, d = case["heads" if attention else "groups"], case["rank"], case.get("tokens", 1), case["d"]
    K = _keep_count(case, G)
    prio = torch.from_numpy(H.halo_build_schedule(K, PLR)).to(DEV)
    dt = torch.float32 if case.get("weights") == "f32" else torch.bfloat16
    ys = [torch.zeros((T, d), dtype=dt, device=DEV) for _ in layers]
    state = {"layers": layers, "prio": prio, "ys": ys}

    if case["kind"] == "forward":
        lay, q4 = layers[0], case["weights"] == "q4"
        shape = H.Shape(d, G * GS, GS, r, "f32" if case["weights"] == "f32" else "bf16")
        size = H.halo_workspace_bytes_q4 if q4 else H.halo_workspace_bytes
        ws = torch.zeros(size(shape, T, K), dtype=torch.uint8, device=DEV)
        out = _prediction_buffers(T, G, K)
        call = H.halo_ffn_forward_q4 if q4 else H.halo_ffn_forward

        def go():
            w = (lay["w"],) if q4 else lay["w"]
            call(shape, lay["x"], lay["At"], lay["Bt"], *w, K, prio, len(PLR), lay["drop"], ys[0], ws, **out)
        state.update(go=go, out={"y": ys[0], **out})
        return state

    # overlapped forms: block l runs with masks[l] and predicts masks[l + 1] from its own input
    preds = [_prediction_buffers(T, G, K) for _ in range(len(layers) + 1)]
    nxt = [{k + "_next": v for k, v in p.items()} for p in preds]
    if attention:
        shape, rows = H.MhaShape(d, G, GS, r), layers[0]["k"].shape[1]
        pos = case["context"]
        ws = torch.zeros(H.halo_mha_workspace_bytes(shape, rows), dtype=torch.uint8, device=DEV)
        as_ffn = H.Shape(d, G * GS, GS, r, "bf16")
    else:
        shape = as_ffn = H.Shape(d, G * GS, GS, r, "bf16")
        size = H.halo_workspace_bytes_q4 if case["weights"] == "q4" else H.halo_workspace_bytes
        ws = torch.zeros(size(shape, T, K), dtype=torch.uint8, device=DEV)
    # the first block's mask, from the block before the first
    ws0 = torch.zeros(H.halo_workspace_bytes(as_ffn, T, K), dtype=torch.uint8, device=DEV)
    first = layers[-1]
    H.halo_predict_scores(as_ffn, first["x"], layers[0]["At"], layers[0]["Bt"], preds[0]["scores"], ws0)
    H.halo_build_group_mask(preds[0]["scores"], K, prio, len(PLR), layers[0]["drop"], preds[0]["mask"])

    def enqueue():
        for l, lay in enumerate(layers):
            after = layers[(l + 1) % len(layers)]
            args = (preds[l]["mask"], ys[l], lay["x"], after["At"], after["Bt"], K, prio, len(PLR), after["drop"],
                    nxt[l + 1]["mask_next"], ws)
            rest = {k: v for k, v in nxt[l + 1].items() if k != "mask_next"}
            if attention:
                H.halo_mha_forward_ahead(shape, lay["x"], lay["Wq"], lay["Wk"], lay["Wv"], lay["Wo"], lay["k"],
                                         lay["v"], pos, *args, **rest)
            elif case["weights"] == "q4":
                H.halo_ffn_forward_ahead_q4(shape, lay["x"], lay["w"], *args, **rest)
            else:
                H.halo_ffn_forward_ahead(shape, lay["x"], *lay["w"], *args, **rest)

    out = {"y": ys, "scores": [p["scores"] for p in preds[1:]], "mask": [p["mask"] for p in preds[1:]]}
    if attention:                                    # the cache rows that the pass adds
        out["k_row"] = [lay["k"][:, pos] for lay in layers]
        out["v_row"] = [lay["v"][:, pos] for lay in layers]
    state.update(go=_captured(enqueue), out=out, ws=ws, preds=preds)
    return state


def run(state):
    state["go"]()
    return state["out"]


# --------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------
def _expected_union(G, keep, T):
    """Groups read for T tokens.  The hidden layer of the predictor is non-negative, so two tokens' scores of a
    group share 1/pi of their variance; given that shared part, tokens keep the group independently."""
    z = math.sqrt(2.0) * float(torch.erfinv(torch.tensor(1.0 - 2.0 * keep, dtype=torch.float64)))
    u = torch.linspace(-5.0, 5.0, 401, dtype=torch.float64)
    weight = torch.exp(-u * u / 2.0)
    rho = 1.0 / math.pi
    p = 0.5 * torch.erfc((z - math.sqrt(rho) * u) / math.sqrt(2.0 * (1.0 - rho))) * (1.0 - sum(PLR) / len(PLR))
    return G * float((weight * (1.0 - (1.0 - p) ** T)).sum() / weight.sum())


def work(case):
    d, r, L = case["d"], case["rank"], case["layers"]
    alive = case["keep"] * (1.0 - sum(PLR) / len(PLR))
    if case["kind"] == "attention":
        n, ctx = case["heads"], case["context"]
        rows = 2 * n * GS + alive * n * GS
        by = 2 * (rows * d + alive * n * GS * d + alive * n * 2 * ctx * GS + 2 * n * GS + r * d + n * r + 2 * d)
        fl = 2 * (rows * d + alive * n * GS * d + alive * n * 2 * ctx * GS + r * d + n * r)
        return {"bytes": L * by, "flops": L * fl}
    G, T = case["groups"], case["tokens"]
    w = {"f32": 4.0, "bf16": 2.0, "q4": 0.5 + 2.0 / 128}[case["weights"]]
    io = 4.0 if case["weights"] == "f32" else 2.0
    by = _expected_union(G, case["keep"], T) * 3 * GS * d * w + io * (2 * T * d + r * d + G * r) + T * G * 5
    fl = 2 * T * (alive * G * 3 * GS * d + r * d + G * r)
    return {"bytes": L * by, "flops": L * fl}


def tolerance(case):
    # float32: sums of up to a few thousand terms, in another order (seen against 64 bits: 1.5e-7).  bf16: the output and the
    # activation between the projections are rounded to bf16 (2^-9 each), and so are 4-bit weights where they
    # are expanded; seen against 64 bits: 2.4e-3, and 3.3e-3 over expanded weights.
    return {"rel": 2e-6} if case.get("weights") == "f32" else {"rel": 1e-2}


# --------------------------------------------------------------------------
# the same in 64 bits, plain torch
# --------------------------------------------------------------------------
def _schedule(n):
    """Device of each priority index: devices by ascending loss rate take equal runs, cuts rounded half up."""
    order = sorted(range(len(PLR)), key=lambda i: (PLR[i], i))
    cuts = [(2 * n * (k + 1) + len(PLR)) // (2 * len(PLR)) for k in range(len(PLR))]
    return np.array([order[next(k for k, c in enumerate(cuts) if p < c)] for p in range(n)])


def _predict64(x, At, Bt):
    return torch.relu(x.double() @ At.double().T) @ Bt.double().T


def _mask64(scores, K, drop):
    rank = torch.argsort(torch.argsort(-scores, dim=1, stable=True), dim=1)
    dev = torch.from_numpy(_schedule(K)).to(DEV)[rank.clamp(max=K - 1)]
    return (rank < K) & (torch.gather(drop.long(), 1, dev) == 0)


def _dequant64(codes, scales, rows, cols):
    w = codes.reshape(-1, 1) >> torch.tensor([0, 16, 4, 20, 8, 24, 12, 28], dtype=torch.int32, device=DEV)
    v = ((w & 15) - 8).reshape(-1, 128).double() * scales.reshape(-1, 1).double()
    return v.reshape(rows, cols)


def _ffn64(case, lay, mask):
    d, G = case["d"], case["groups"]
    x = lay["x"].double()
    q4 = case["weights"] == "q4"

    def matrix(i, rows, cols):
        return _dequant64(lay["w"][2 * i], lay["w"][2 * i + 1], rows, cols) if q4 else lay["w"][i].double().view(rows, cols)
    act = x @ matrix(0, G * GS, d).T
    act = act * torch.sigmoid(act)
    act = act * (x @ matrix(1, G * GS, d).T)
    act = act * mask.double().repeat_interleave(GS, dim=1)
    down = matrix(2, G * d, GS).view(G, d, GS)
    y = torch.zeros((x.shape[0], d), dtype=torch.float64, device=DEV)
    for g in range(G):
        y += act[:, g * GS:(g + 1) * GS] @ down[g].T
    return y


def _mha64(case, lay, mask):
    n, pos = case["heads"], case["context"]
    x = lay["x"].double()[0]
    q, k, v = ((lay[w].double() @ x).view(n, GS) for w in ("Wq", "Wk", "Wv"))
    keys = torch.cat([lay["k"][:, :pos].double(), k[:, None]], dim=1)
    values = torch.cat([lay["v"][:, :pos].double(), v[:, None]], dim=1)
    p = torch.softmax((keys * q[:, None]).sum(-1) / math.sqrt(GS), dim=1)
    o = (p[:, :, None] * values).sum(1) * mask.double()[0][:, None]
    y = torch.zeros(case["d"], dtype=torch.float64, device=DEV)
    for h in range(n):
        y += lay["Wo"][h].double() @ o[h]
    return y[None], k, v


def exact(case, seed):
    layers = _inputs(case, seed)
    attention = case["kind"] == "attention"
    K = _keep_count(case, case["heads" if attention else "groups"])
    if case["kind"] == "forward":
        lay = layers[0]
        scores = _predict64(lay["x"], lay["At"], lay["Bt"])
        y = _ffn64(case, lay, _mask64(scores, K, lay["drop"]))
        return {"y": y, "scores": scores, "mask": None, "surv_idx": None, "n_surv": None}
    L = len(layers)
    out = {"y": [], "scores": [], "mask": [None] * L}
    if attention:
        out.update(k_row=[], v_row=[])
    mask = _mask64(_predict64(layers[-1]["x"], layers[0]["At"], layers[0]["Bt"]), K, layers[0]["drop"])
    for l, lay in enumerate(layers):
        after = layers[(l + 1) % L]
        if attention:
            y, k, v = _mha64(case, lay, mask)
            out["k_row"].append(k)
            out["v_row"].append(v)
        else:
            y = _ffn64(case, lay, mask)
        out["y"].append(y)
        scores = _predict64(lay["x"], after["At"], after["Bt"])
        out["scores"].append(scores)
        mask = _mask64(scores, K, after["drop"])
    return out
