"""GPU parity of the FFN over 4-bit block-quantised weights (paper Sec. V-A) against the CPU
oracle, whose view of such weights is the dequantised matrices.  Same bars as the other
parity tests: bit-exact scores / ranking / masks, relative L2 <= 1e-5 (f32) or 2e-2 (bf16)."""
import dataclasses

import numpy as np
import pytest
import torch

import halo_synth as hs
import paper_2601_11676_amd as H
from oracle import ref
from tests import harness as hz

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-5, "bf16": 2e-2}


def _say(msg):
    print("[case] " + msg, flush=True)


def test_q4_generator_bits_identical_on_cpu_and_gpu():
    _say("q4 generator cpu/gpu")
    w = hs.small_variant(hs.LLAMA7B_DECODE, 384, 3, 64)
    for a, b in zip(hs.ffn_weights_q4(w, 1, "cpu"), hs.ffn_weights_q4(w, 1, hz.DEV)):
        b = b.cpu()
        if a.dtype == torch.bfloat16:
            a, b = a.view(torch.int16), b.view(torch.int16)
        assert torch.equal(a, b)


@pytest.mark.parametrize("dtype,T,d,G,r", [
    ("f32", 16, 256, 8, 64),       # the tiny shape
    ("f32", 5, 640, 7, 72),
    ("bf16", 3, 384, 9, 40),       # (these four run on the tuned kernels)
    ("bf16", 1, 1024, 5, 264),
    ("bf16", 7, 4096, 6, 256),
    ("bf16", 40, 512, 70, 64),
    ("bf16", 20, 8320, 3, 40),     # rows longer than they take
    ("bf16", 40, 128, 260, 64),    # more groups
])
def test_q4_plain_path_whole_pass(dtype, T, d, G, r):
    w = dataclasses.replace(hs.TINY, name="case", d=d, ffn=G * 128, rank=r, T=T, dtype=dtype, seed=12)
    _say(f"q4 plain {dtype} T={T} d={d} G={G} r={r}")
    L = hz.Q4Layer(w)
    x = hs.hidden_states(w, 0, hz.DEV)
    K = max(1, G // 2)
    pd = H.halo_build_schedule(K, w.device_plr())
    drop = hs.drop_outcomes(w, T=T)
    g = hz.gpu_forward_q4(w, L, x, K, pd, drop)
    c = hz.oracle_forward(w, L, x, K, pd, drop)
    hz.assert_parity(g, c, TOL[dtype], "q4 plain")


@pytest.mark.parametrize("d,G,K", [(4096, 7, 4), (8192, 6, 6), (4096, 200, 150), (4096, 9, 1)])
def test_q4_one_token_streaming_path(d, G, K):
    w = dataclasses.replace(hs.LLAMA7B_DECODE, name="case", d=d, ffn=G * 128, rank=256, seed=22)
    _say(f"q4 one-token path d={d} G={G} K={K}")
    L = hz.Q4Layer(w)
    pd = H.halo_build_schedule(K, w.device_plr())
    for step in range(3):
        x = hs.hidden_states(w, step, hz.DEV)
        drop = hs.drop_outcomes(w, 0, step)
        g = hz.gpu_forward_q4(w, L, x, K, pd, drop)
        c = hz.oracle_forward(w, L, x, K, pd, drop)
        hz.assert_parity(g, c, TOL["bf16"], f"q4 t1 d={d} step {step}")


@pytest.mark.parametrize("T,d,G,r", [
    (2, 1024, 5, 64),
    (4, 5120, 9, 256),       # LLaMA-13B row length (ten 512-element chunks: the last code buffer is half full)
    (8, 8192, 7, 512),       # LLaMA-2-70B row length
    (16, 4096, 6, 256),
    (5, 4096, 20, 256),      # union larger than any token's set; ragged neuron runs per wave
    (3, 512, 3, 40),         # a single chunk per row
    (6, 5120, 90, 256),      # more 16-row tiles than workgroups: a workgroup walks several
    (16, 8192, 40, 256),     # x larger than its LDS space: staged a range of columns at a time, per tile
    (17, 1024, 9, 64),       # more than 16 tokens: tiles of tokens, here 15 + 2 (no tile of one token)
    (33, 2048, 12, 64),      # 16 + 15 + 2
    (100, 1024, 20, 40),     # six tiles of 16 and one of 4
])
def test_q4_few_tokens_matrix_core_path(T, d, G, r):
    w = dataclasses.replace(hs.LLAMA13B_STACK, name="case", d=d, ffn=G * 128, rank=r, T=T, layers=1, seed=18)
    _say(f"q4 few tokens T={T} d={d} G={G}")
    L = hz.Q4Layer(w)
    x = hs.hidden_states(w, 0, hz.DEV)
    for K in (max(1, G // 2), G):
        pd = H.halo_build_schedule(K, w.device_plr())
        drop = hs.drop_outcomes(w, T=T)
        if K < G:
            drop[T - 1] = 1                    # one token loses every device: exact zeros expected
        g = hz.gpu_forward_q4(w, L, x, K, pd, drop)
        c = hz.oracle_forward(w, L, x, K, pd, drop)
        hz.assert_parity(g, c, TOL["bf16"], f"q4 few tokens K={K}")


def test_q4_llama7b_decode_full_size_steps():
    w = hs.LLAMA7B_DECODE
    _say("q4 llama7b decode full size")
    L = hz.Q4Layer(w)
    K = w.k_keep()
    pd = H.halo_build_schedule(K, w.device_plr())
    for step in (0, 1, 2, 3, 7, 100, 500, 1023):
        x = hs.hidden_states(w, step, hz.DEV)
        drop = hs.drop_outcomes(w, 0, step)
        g = hz.gpu_forward_q4(w, L, x, K, pd, drop)
        c = hz.oracle_forward(w, L, x, K, pd, drop)
        hz.assert_parity(g, c, TOL["bf16"], f"q4 7b step {step}")


def test_q4_ffn_entry_point_with_handmade_masks_and_errors():
    w = dataclasses.replace(hs.LLAMA7B_DECODE, name="case", ffn=10 * 128, rank=64, seed=23)
    _say("q4 ffn entry point, handmade masks")
    L = hz.Q4Layer(w)
    s = hz.shape_of(w)
    _, _, Wg, Wu, WdT = L.host()
    ws = torch.empty(H.halo_workspace_bytes(s, 1, 0), dtype=torch.uint8, device=hz.DEV)
    x = hs.hidden_states(w, 3, hz.DEV)
    xn = hz.to_np32(x)
    for bits in ([0] * 10, [1] * 10, [1, 0, 0, 0, 0, 0, 0, 0, 0, 1], [0, 0, 0, 0, 1, 0, 0, 0, 0, 0]):
        mask_np = np.array([bits], np.uint8)
        y = torch.full((1, w.d), float("nan"), dtype=torch.bfloat16, device=hz.DEV)
        H.halo_group_sparse_ffn_q4(s, x, L.q4, torch.from_numpy(mask_np).to(hz.DEV), y, ws)
        torch.cuda.synchronize()
        yg = hz.to_np32(y).astype(np.float64)
        yc = ref.group_sparse_ffn(xn, Wg, Wu, WdT, 128, mask_np)
        if not any(bits):
            assert not yg.any()
        else:
            assert np.linalg.norm(yg - yc) / np.linalg.norm(yc) <= TOL["bf16"]
    # a group size other than the quantisation block is refused before anything is enqueued
    bad = H.Shape(w.d, 20 * 64, 64, w.rank, "bf16")
    y = torch.zeros((1, w.d), dtype=torch.bfloat16, device=hz.DEV)
    with pytest.raises(H.HaloError):
        H.halo_group_sparse_ffn_q4(bad, x, L.q4, torch.zeros((1, 20), dtype=torch.uint8, device=hz.DEV), y, ws)
    # no tokens: nothing to do
    H.halo_group_sparse_ffn_q4(s, x[:0], L.q4, torch.zeros((0, 10), dtype=torch.uint8, device=hz.DEV), y[:0], ws)
    torch.cuda.synchronize()


@pytest.mark.parametrize("T,d,G", [(2, 8192, 6), (4, 5120, 10), (16, 4096, 5), (3, 1024, 70)])
def test_q4_few_tokens_with_handmade_masks(T, d, G):
    # the matrix-core kernels on masks no schedule would give: no group at all (exact zeros), one group of one
    # token, every group of every token, a different single group per token, the last group only
    w = dataclasses.replace(hs.LLAMA13B_STACK, name="case", d=d, ffn=G * 128, rank=64, T=T, layers=1, seed=31)
    _say(f"q4 few tokens, handmade masks T={T} d={d} G={G}")
    L = hz.Q4Layer(w)
    s = hz.shape_of(w)
    _, _, Wg, Wu, WdT = L.host()
    ws = torch.empty(H.halo_workspace_bytes(s, T, G), dtype=torch.uint8, device=hz.DEV)
    x = hs.hidden_states(w, 1, hz.DEV)
    xn = hz.to_np32(x)
    masks = [np.zeros((T, G), np.uint8), np.zeros((T, G), np.uint8), np.ones((T, G), np.uint8),
             np.zeros((T, G), np.uint8), np.zeros((T, G), np.uint8)]
    masks[1][T - 1, G // 2] = 1
    for t in range(T):
        masks[3][t, (3 * t + 1) % G] = 1
    masks[4][:, G - 1] = 1
    for mask_np in masks:
        y = torch.full((T, d), float("nan"), dtype=torch.bfloat16, device=hz.DEV)
        H.halo_group_sparse_ffn_q4(s, x, L.q4, torch.from_numpy(mask_np).to(hz.DEV), y, ws)
        torch.cuda.synchronize()
        yg = hz.to_np32(y).astype(np.float64)
        yc = ref.group_sparse_ffn(xn, Wg, Wu, WdT, 128, mask_np)
        for t in range(T):
            if not mask_np[t].any():
                assert not yg[t].any(), t
            else:
                assert np.linalg.norm(yg[t] - yc[t]) / np.linalg.norm(yc[t]) <= TOL["bf16"], t


@pytest.mark.parametrize("q4", [True, False])
@pytest.mark.parametrize("T,d,G,r", [
    (2, 128, 3, 40),           # 4-bit: half a unit, seven of eight waves without one; bf16: two units
    (8, 1152, 27, 264),        # an odd number of blocks
    (9, 2176, 5, 64),          # the last wave's second unit is half a unit
    (16, 3200, 40, 512),       # four passes of two predictor rows
    (3, 5248, 200, 256),       # three rows of eight outputs to a workgroup
    (13, 6784, 6, 64),         # bf16: thirteen or fourteen units to a wave
    (5, 7936, 9, 256),         # ... fifteen or sixteen
    (16, 8064, 256, 64),       # the most groups: every neuron of a workgroup's run in one group
    (2, 8320, 3, 40),          # rows longer than the streaming kernels take: the other gate/up, and the plain path over codes
    (16, 8320, 5, 72),
    (7, 256, 260, 64),         # more groups than they take: a list of groups in memory
    (16, 640, 257, 40),
])
def test_few_tokens_of_any_row_length(q4, T, d, G, r):
    # against the oracle, and the overlapped form equal to the serial one bit for bit
    w = dataclasses.replace(hs.LLAMA13B_STACK, name="case", d=d, ffn=G * 128, rank=r, T=T, layers=1, seed=28)
    _say(f"few tokens, any row length q4={q4} T={T} d={d} G={G}")
    s, L = hz.shape_of(w), (hz.Q4Layer if q4 else hz.Layer)(w)
    forward = hz.gpu_forward_q4 if q4 else hz.gpu_forward
    x, xn = hs.hidden_states(w, 0, hz.DEV), hs.hidden_states(w, 1, hz.DEV)
    for K in sorted({max(1, G // 2), G}):
        pd = H.halo_build_schedule(K, w.device_plr())
        drop, dn = hs.drop_outcomes(w, 0, 0, T=T), hs.drop_outcomes(w, 0, 1, T=T)
        if K < G:
            drop[T - 1] = 1                    # one token loses every device: exact zeros expected
        g = forward(w, L, x, K, pd, drop)
        if G < 200 or K < G:
            hz.assert_parity(g, hz.oracle_forward(w, L, x, K, pd, drop), TOL["bf16"], f"K={K}")
        gn = forward(w, L, xn, K, pd, dn)
        y = torch.full((T, d), float("nan"), dtype=torch.bfloat16, device=hz.DEV)
        mn = torch.zeros((T, G), dtype=torch.uint8, device=hz.DEV)
        ws = torch.empty(H.halo_workspace_bytes(s, T, K), dtype=torch.uint8, device=hz.DEV)
        rest = (torch.from_numpy(g["mask"]).to(hz.DEV), y, xn, L.At, L.Bt, K, torch.from_numpy(pd).to(hz.DEV), w.n_dev,
                torch.from_numpy(dn).to(hz.DEV), mn, ws)
        if q4:
            H.halo_ffn_forward_ahead_q4(s, x, L.q4, *rest)
        else:
            H.halo_ffn_forward_ahead(s, x, L.Wg, L.Wu, L.Wd, *rest)
        torch.cuda.synchronize()
        assert np.array_equal(hz.to_np32(y).astype(np.float64), g["y"]) and np.array_equal(mn.cpu().numpy(), gn["mask"])


def _pack_codes(k):
    """integers -8 .. 7 [..., n] -> words [..., n / 8] of codes k + 8 in the storage order"""
    c = (np.asarray(k, np.int64) + 8).reshape(*k.shape[:-1], -1, 8)
    shift = [4 * (e // 2) + 16 * (e % 2) for e in range(8)]
    return sum(c[..., e] << shift[e] for e in range(8)).astype(np.uint32).view(np.int32)


@pytest.mark.parametrize("what", ["sums", "activations"])
@pytest.mark.parametrize("T,d", [(2, 384), (8, 1152), (16, 5248), (37, 640), (4, 1152), (2, 5248), (7, 5248)])
def test_q4_few_tokens_of_any_row_length_keep_float32(what, T, d):
    # Rows that are no multiple of 1024: sums over c - 8 in float32, the activation in float32.  y is bf16, so results are made
    # small beside what they are summed from.  sums: the tokens' values have a mean of 1, and a row's products cancel (to a few
    # hundredths of the largest); y is a neuron's activation.  activations: y is the difference of two that share 12 leading bits.
    _say(f"q4 precision {what} T={T} d={d}")
    rng = np.random.default_rng(17)
    G = 2
    kg, ku, kd = np.zeros((G * 128, d), np.int64), np.zeros((G * 128, d), np.int64), np.zeros((G, d, 128), np.int64)
    m = np.arange(G * 128)
    if what == "sums":
        x = torch.from_numpy(rng.normal(1, 1, d).astype(np.float32)).to(torch.bfloat16).float().numpy().astype(np.float64)
        kg[m, rng.choice(np.flatnonzero(np.abs(x) > 0.5), G * 128)] = 4
        ku[:] = rng.integers(-1, 2, ku.shape)
        for _ in range(40):                        # the code whose change by one brings each row's sum nearest to 0
            u = ku @ x
            step = np.abs(np.stack([np.where(ku < 1, u[:, None] + x, np.inf), np.where(ku > -1, u[:, None] - x, np.inf)]))
            best = step.transpose(1, 0, 2).reshape(G * 128, -1)
            at = best.argmin(1)
            better = best.min(1) < np.abs(u)
            ku[m[better], at[better] % d] += np.where(at[better] < d, 1, -1)
        kd[m // 128, m, m % 128] = 1
    else:
        x = np.zeros(d)
        x[[3, 130, 258]] = 1.0, 2.0 ** -10, 2.0 ** -13
        kg[:, 3] = np.repeat(rng.integers(1, 8, G), 128)
        ku[:, 3], ku[:, 130], ku[:, 258] = 7, rng.integers(-7, 8, G * 128), rng.integers(-7, 8, G * 128)
        j = np.arange(G * 64)
        kd[j // 64, j, j % 64], kd[j // 64, j, 64 + j % 64] = 1, -1
    xs = np.stack([x * 2.0 ** -(t % 3) for t in range(T)])
    ones = lambda *n: torch.ones(n, dtype=torch.bfloat16, device=hz.DEV)
    q4 = tuple(w for k in (kg, ku) for w in (torch.from_numpy(_pack_codes(k)).to(hz.DEV), ones(G * 128, d // 128)))
    q4 += (torch.from_numpy(_pack_codes(kd)).to(hz.DEV), ones(G, d))
    s = H.Shape(d, G * 128, 128, 64, "bf16")
    ws = torch.empty(H.halo_workspace_bytes(s, T, G), dtype=torch.uint8, device=hz.DEV)
    y = torch.full((T, d), float("nan"), dtype=torch.bfloat16, device=hz.DEV)
    H.halo_group_sparse_ffn_q4(s, torch.from_numpy(xs).to(torch.bfloat16).to(hz.DEV), q4,
                               torch.ones((T, G), dtype=torch.uint8, device=hz.DEV), y, ws)
    torch.cuda.synchronize()
    yg = hz.to_np32(y).astype(np.float64)
    yc = ref.group_sparse_ffn(xs, *ref.dequant_ffn_q4([q.float().cpu().numpy() if q.dtype == torch.bfloat16 else q.cpu().numpy() for q in q4]),
                              128, np.ones((T, G), np.uint8))
    # y's own rounding, 2^-8; the activation function's, well below 2^-18; and 2^-24 of what a sum is made of at each of its
    # roundings: in gate/up at most 20 (four steps of a block, eight blocks of a wave, eight waves), of an activation two and its sums
    gate = xs @ kg.T
    silu = np.abs(gate / (1 + np.exp(-gate)))
    part = 20 * silu * (np.abs(xs) @ np.abs(ku).T) if what == "sums" else 6 * silu * np.abs(xs @ ku.T)
    bound = (2.0 ** -8 + 2.0 ** -18) * np.abs(yc)
    for g in range(G):
        bound += 2.0 ** -24 * part[:, g * 128:(g + 1) * 128] @ np.abs(kd[g]).T
    worst = (np.abs(yg - yc)[bound > 0] / bound[bound > 0]).max()
    assert worst <= 1 and not yg[bound == 0].any(), f"worst error {worst:.3f} of the bound"


@pytest.mark.parametrize("d,T,r,G,K", [
    (4096, 1, 256, 20, 10), (8192, 1, 256, 20, 10), (512, 3, 256, 20, 10), (5120, 4, 256, 20, 10),
    (8192, 8, 256, 20, 10), (384, 3, 256, 20, 10),
    (4096, 1, 256, 86, 43),      # enough surviving neurons for the runs to be cut by weight around the predictor rows
    (4096, 1, 512, 86, 60),      # two predictor rows per gate/up workgroup
    (4096, 1, 128, 20, 10),      # a predictor size that is not dealt evenly: workgroups of its own
    (1024, 20, 64, 12, 6),       # more than 16 tokens: tiles of tokens, the prediction enqueued after the FFN
])
def test_q4_one_step_ahead_overlap_equals_the_serial_pass(d, T, r, G, K):
    # predictor + mask of step s+1 beside (or, for shapes without spare workgroups, after) the FFN of step s
    w = dataclasses.replace(hs.LLAMA7B_DECODE, name="case", d=d, ffn=G * 128, rank=r, T=T, seed=9)
    _say(f"halo_ffn_forward_ahead_q4 vs halo_ffn_forward_q4 d={d} T={T} r={r} G={G} K={K}")
    s = hz.shape_of(w)
    L = hz.Q4Layer(w)
    n = 5
    pd = H.halo_build_schedule(K, w.device_plr())
    xs = [hs.hidden_states(w, i, hz.DEV) for i in range(n + 1)]
    drops = [hs.drop_outcomes(w, 0, i, T=T) for i in range(n + 1)]
    serial = [hz.gpu_forward_q4(w, L, xs[i], K, pd, drops[i]) for i in range(n)]
    ws = torch.empty(H.halo_workspace_bytes(s, T, K), dtype=torch.uint8, device=hz.DEV)
    pdd = torch.from_numpy(pd).to(hz.DEV)
    dd = [torch.from_numpy(x).to(hz.DEV) for x in drops]
    masks = torch.zeros((n + 1, T, G), dtype=torch.uint8, device=hz.DEV)
    ys = torch.zeros((n, T, w.d), dtype=torch.bfloat16, device=hz.DEV)
    sc = torch.empty((T, G), dtype=torch.float32, device=hz.DEV)
    H.halo_predict_scores(s, xs[0], L.At, L.Bt, sc, ws)
    H.halo_build_group_mask(sc, K, pdd, w.n_dev, dd[0], masks[0])

    def run(ys_, masks_):
        for i in range(n):
            H.halo_ffn_forward_ahead_q4(s, xs[i], L.q4, masks_[i], ys_[i], xs[i + 1], L.At, L.Bt, K, pdd,
                                        w.n_dev, dd[i + 1], masks_[i + 1], ws)

    run(ys, masks)
    torch.cuda.synchronize()
    for i in range(n):
        assert np.array_equal(masks[i].cpu().numpy(), serial[i]["mask"]), i
        assert np.array_equal(hz.to_np32(ys[i]).astype(np.float64), serial[i]["y"]), i
    g = torch.cuda.CUDAGraph()
    ys2 = torch.zeros_like(ys)
    masks2 = masks.clone()
    with torch.cuda.graph(g):
        run(ys2, masks2)
    for _ in range(2):
        ys2.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(ys2, ys) and torch.equal(masks2, masks)


@pytest.mark.parametrize("wl", [hs.LLAMA13B_STACK, hs.LLAMA70B_STACK])
def test_q4_full_size_single_layer_of_the_stacks(wl):
    # 4 / 8 tokens at the 13B / 70B layer shapes (the plain 4-bit path); y for every token
    _say(f"q4 {wl.name} one full-size layer")
    L = hz.Q4Layer(wl, layer=2)
    x = hs.hidden_states(wl, 0, hz.DEV)
    K = wl.k_keep(0.5)
    pd = H.halo_build_schedule(K, wl.device_plr())
    drop = hs.drop_outcomes(wl, 2, 0)
    g = hz.gpu_forward_q4(wl, L, x, K, pd, drop)
    c = hz.oracle_forward(wl, L, x, K, pd, drop)
    hz.assert_parity(g, c, TOL["bf16"], "q4 " + wl.name)


@pytest.mark.parametrize("big_workspace", [False, True])
def test_q4_llama7b_prefill_all_tokens(big_workspace):
    # 512 tokens over 4-bit weights: with the plain workspace the few-token kernels walk the tokens 16 at a
    # time; with room for a block's weights as bf16 the many-token kernels run on weights rounded to bf16
    w = hs.LLAMA7B_PREFILL
    _say(f"q4 7B prefill, 512 tokens, every token, big workspace {big_workspace}")
    s = hz.shape_of(w)
    K = w.k_keep()
    small, big = H.halo_workspace_bytes(s, w.T, K), H.halo_workspace_bytes_q4(s, w.T, K)
    assert big == small + 3 * w.ffn * w.d * 2 and H.halo_workspace_bytes_q4(s, 16, K) == H.halo_workspace_bytes(s, 16, K)
    L = hz.Q4Layer(w)
    x = hs.hidden_states(w, 0, hz.DEV)
    pd = H.halo_build_schedule(K, w.device_plr())
    drop = hs.drop_outcomes(w)
    g = hz.gpu_forward_q4(w, L, x, K, pd, drop, big_workspace=big_workspace)
    c = hz.oracle_forward(w, L, x, K, pd, drop)
    hz.assert_parity(g, c, TOL["bf16"], "q4 7B prefill")


@pytest.mark.parametrize("T,d,G", [(17, 128, 9), (64, 128, 12), (65, 1024, 9), (140, 2048, 12), (300, 1024, 20)])
def test_q4_many_tokens_on_expanded_weights(T, d, G):
    # small shapes on weights rounded to bf16 (workspace of halo_workspace_bytes_q4)
    w = dataclasses.replace(hs.LLAMA13B_STACK, name="case", d=d, ffn=G * 128, rank=64, T=T, layers=1, seed=19)
    _say(f"q4 many tokens, expanded weights T={T} d={d} G={G}")
    L = hz.Q4Layer(w)
    x = hs.hidden_states(w, 0, hz.DEV)
    K = max(1, G // 2)
    pd = H.halo_build_schedule(K, w.device_plr())
    drop = hs.drop_outcomes(w, T=T)
    g = hz.gpu_forward_q4(w, L, x, K, pd, drop, big_workspace=True)
    c = hz.oracle_forward(w, L, x, K, pd, drop)
    hz.assert_parity(g, c, TOL["bf16"], "q4 many tokens expanded")


@pytest.mark.parametrize("wl,keep,layers", [(hs.LLAMA13B_STACK, 0.3, None), (hs.LLAMA70B_STACK, 0.5, 6)])
def test_q4_stack_teacher_forced(wl, keep, layers):
    # the free-running stack over 4-bit weights, predictor one layer ahead (layer 0 dense: every group of
    # every token, so the few-token kernels walk several tiles per workgroup); checked layers are compared
    # with the oracle fed the GPU's own layer inputs
    n = wl.layers if layers is None else layers
    check = sorted({0, 1, 2, n // 2, n - 1})
    _say(f"q4 {wl.name} stack of {n} layers, checked {check}")
    seen = []

    def on_layer(l, rec, pd_np, K):
        hz.check_stack_layer(wl, l, rec, pd_np, K, TOL["bf16"])
        seen.append(l)
        print(f"  layer {l} ok", flush=True)
    h = hz.run_stack_gpu(wl, keep, layers=layers, check_layers=check, on_layer=on_layer, q4=True)
    assert torch.isfinite(h).all() and seen == check



@pytest.mark.parametrize("d,G,K,r", [(128, 3, 2, 40), (1152, 9, 9, 256), (2048, 70, 33, 64), (2560, 7, 4, 512), (5120, 86, 43, 256),
                                     (6272, 6, 3, 256), (8064, 40, 30, 128)])
def test_q4_one_token_of_any_row_length(d, G, K, r):
    # rows that are not whole 2048-element parts; the activation stays in float32 there: serial and overlapped form,
    # the second equal to the first bit for bit
    w = dataclasses.replace(hs.LLAMA7B_DECODE, name="case", d=d, ffn=G * 128, rank=r, seed=24)
    _say(f"q4 one token, any row length d={d} G={G} r={r}")
    s = hz.shape_of(w)
    L = hz.Q4Layer(w)
    pd = H.halo_build_schedule(K, w.device_plr())
    pdd = torch.from_numpy(pd).to(hz.DEV)
    ws = torch.empty(H.halo_workspace_bytes(s, 1, K), dtype=torch.uint8, device=hz.DEV)
    x, xn = hs.hidden_states(w, 0, hz.DEV), hs.hidden_states(w, 1, hz.DEV)
    drop, dn = hs.drop_outcomes(w, 0, 0), hs.drop_outcomes(w, 0, 1)
    g = hz.gpu_forward_q4(w, L, x, K, pd, drop)
    hz.assert_parity(g, hz.oracle_forward(w, L, x, K, pd, drop), TOL["bf16"], f"q4 any d={d}")
    gn = hz.gpu_forward_q4(w, L, xn, K, pd, dn)
    y = torch.full((1, d), float("nan"), dtype=torch.bfloat16, device=hz.DEV)
    mn = torch.zeros((1, G), dtype=torch.uint8, device=hz.DEV)
    H.halo_ffn_forward_ahead_q4(s, x, L.q4, torch.from_numpy(g["mask"]).to(hz.DEV), y, xn, L.At, L.Bt, K, pdd, w.n_dev,
                                torch.from_numpy(dn).to(hz.DEV), mn, ws)
    torch.cuda.synchronize()
    assert np.array_equal(hz.to_np32(y).astype(np.float64), g["y"]) and np.array_equal(mn.cpu().numpy(), gn["mask"])


@pytest.mark.parametrize("T,d,G,K", [
    (17, 128, 3, 2),           # one block of codes per row
    (128, 640, 5, 2),          # an odd number of blocks per row: the scales' words straddle rows
    (200, 384, 70, 60),        # half tiles in gate/up, many groups of three blocks
    (129, 1152, 24, 12),       # two half tiles in both, one token in the second
    (129, 4096, 40, 20),       # half tiles in gate/up, a whole tile with half of it empty in down
    (257, 1024, 6, 6),         # dense: no token needs a row of zeros
    (257, 1152, 9, 5),         # three half tiles in down, one token in the last
    (300, 256, 300, 30),       # more groups than the few-token kernels take
    (515, 4224, 9, 4),         # whole tiles in gate/up, five half tiles in down, one range
    (515, 4224, 40, 10),       # three whole tiles in down, the last with three tokens
])
def test_q4_many_token_rings(T, d, G, K):
    # the codes expanded on their way into LDS give what the bf16 kernels give on the expanded weights, bit for bit (where those
    # are the same kernels: with many groups the bf16 call runs on 256 x 256 tiles, which add a row up in one chain)
    w = dataclasses.replace(hs.LLAMA7B_PREFILL, name="case", d=d, ffn=G * 128, rank=64, T=T, seed=82)
    _say(f"q4 many-token rings T={T} d={d} G={G} K={K}")
    s = hz.shape_of(w)
    L = hz.Q4Layer(w)
    x = hs.hidden_states(w, 0, hz.DEV)
    pd = H.halo_build_schedule(K, w.device_plr())
    drop = hs.drop_outcomes(w, T=T)
    drop[0] = 1
    g = hz.gpu_forward_q4(w, L, x, K, pd, drop, big_workspace=True)
    hz.assert_parity(g, hz.oracle_forward(w, L, x, K, pd, drop), TOL["bf16"], f"q4 rings T={T}")
    if G * (T + 256) > 512 * 150:
        return
    Wg, Wu, WdT = (torch.from_numpy(np.ascontiguousarray(a)).to(torch.bfloat16).to(hz.DEV) for a in L.host()[2:])
    y = torch.full((T, d), float("nan"), dtype=torch.bfloat16, device=hz.DEV)
    ws = torch.empty(H.halo_workspace_bytes(s, T, K), dtype=torch.uint8, device=hz.DEV)
    H.halo_group_sparse_ffn(s, x, Wg, Wu, H.pack_down_proj(WdT, 128), torch.from_numpy(g["mask"]).to(hz.DEV), y, ws)
    torch.cuda.synchronize()
    assert np.array_equal(hz.to_np32(y).astype(np.float64), g["y"])


@pytest.mark.parametrize("q4", [True, False])
@pytest.mark.parametrize("T,d,G,K", [
    (17, 256, 3, 2),           # the fewest tokens, the shortest rows: one full block of eight token rows of a wave's, four stages
    (33, 640, 9, 9),           # dense, one token past half of the tile; an odd number of blocks per row
    (64, 1152, 20, 10),        # the full tile
    (65, 768, 8, 6),           # down projection: a second quarter tile of one token
    (193, 1024, 24, 12),       # ... a fourth of one token
    (520, 896, 9, 4),          # ... nine of them, more than two (the other numbering of the work)
])
def test_quarter_tiles_of_tokens(q4, T, d, G, K):
    w = dataclasses.replace(hs.LLAMA7B_PREFILL, name="case", d=d, ffn=G * 128, rank=64, T=T, seed=87)
    _say(f"quarter tiles q4={q4} T={T} d={d} G={G} K={K}")
    L = (hz.Q4Layer if q4 else hz.Layer)(w)
    x = hs.hidden_states(w, 0, hz.DEV)
    pd = H.halo_build_schedule(K, w.device_plr())
    drop = hs.drop_outcomes(w, T=T)
    drop[T - 1] = 1                            # one token loses every device: exact zeros expected
    g = hz.gpu_forward_q4(w, L, x, K, pd, drop, big_workspace=True) if q4 else hz.gpu_forward(w, L, x, K, pd, drop)
    hz.assert_parity(g, hz.oracle_forward(w, L, x, K, pd, drop), TOL["bf16"], f"quarter tiles T={T}")


@pytest.mark.parametrize("G,K", [(2, 1), (3, 2)])
def test_q4_more_tokens_than_the_row_table_holds(G, K):
    # 32768 tokens: the codes are expanded into the workspace and the bf16 kernels run on them
    T, d = 32768, 128
    w = dataclasses.replace(hs.LLAMA7B_PREFILL, name="case", d=d, ffn=G * 128, rank=8, T=T, seed=86)
    _say(f"q4 past the row table G={G}")
    L = hz.Q4Layer(w)
    x = hs.hidden_states(w, 0, hz.DEV)
    pd = H.halo_build_schedule(K, w.device_plr())
    drop = hs.drop_outcomes(w, T=T)
    g = hz.gpu_forward_q4(w, L, x, K, pd, drop, big_workspace=True)
    rows = np.r_[0:130, 16300:16500, T - 130:T]
    c = hz.oracle_forward(w, L, x[torch.from_numpy(rows).to(hz.DEV)], K, pd, drop[rows])
    hz.assert_parity({k: v[rows] for k, v in g.items()}, c, TOL["bf16"], "q4 past the row table")
    assert np.isfinite(g["y"]).all()


@pytest.mark.parametrize("mean", [0, 1])
@pytest.mark.parametrize("T,d,G,K", [
    (17, 256, 1, 1),           # one group: half a pair of groups in down, one pair of blocks in gate/up
    (18, 384, 5, 3),           # three blocks: some dies start their walk at half a pair
    (32, 256, 7, 7),           # dense, two full 16-token tiles
    (33, 640, 9, 4),           # an odd number of blocks per row: the scales' words straddle rows; three tiles in down
    (49, 1024, 12, 6),         # four tiles
    (64, 768, 33, 20),         # the full tile, ranges of an odd number of groups
    (64, 2176, 9, 9),          # dense, 17 blocks
])
def test_q4_17_to_64_tokens_scale_in_float(T, d, G, K, mean):
    # nothing is rounded but the activation and y, 2^-9 of a value at most each (relative L2 2.8e-3 together, 3.3e-3 with rounded
    # weights); the offset that the codes carry cancels also where the tokens' values do not sum to about nothing
    w = dataclasses.replace(hs.LLAMA7B_PREFILL, name="case", d=d, ffn=G * 128, rank=64, T=T, seed=91)
    _say(f"q4 17 to 64 tokens T={T} d={d} G={G} K={K} mean={mean}")
    L = hz.Q4Layer(w)
    x = (hs.hidden_states(w, 0, hz.DEV).float() + mean).to(torch.bfloat16)
    pd = H.halo_build_schedule(K, w.device_plr())
    drop = hs.drop_outcomes(w, T=T)
    drop[T - 1] = 1                            # a token that loses every device: exact zeros expected
    g = hz.gpu_forward_q4(w, L, x, K, pd, drop, big_workspace=True)
    c = hz.oracle_forward(w, L, x, K, pd, drop)
    hz.assert_parity(g, c, TOL["bf16"], f"q4 17 to 64 tokens T={T}")
    assert np.linalg.norm(g["y"] - c["y"]) <= 2 ** 0.5 * 2.0 ** -9 * np.linalg.norm(c["y"])


@pytest.mark.parametrize("T,d", [(17, 256), (37, 640), (64, 1152), (40, 2048)])
def test_q4_17_to_64_tokens_keep_sums_that_cancel(monkeypatch, T, d):
    # the same sums over c - 8 in float32 as with fewer tokens and as in the smaller workspace
    monkeypatch.setattr(H, "halo_workspace_bytes", H.halo_workspace_bytes_q4)
    test_q4_few_tokens_of_any_row_length_keep_float32("sums", T, d)


@pytest.mark.parametrize("T,d,G", [(17, 256, 2), (33, 640, 3), (64, 384, 5)])
def test_q4_17_to_64_tokens_zeros_range_and_infinities(T, d, G):
    # what the float32 sums of s (c - 8) x give where nothing is added to the codes: exact zeros over codes of 8, finite results of
    # values near the largest, infinities (token 0) that stay infinities and stay with their token
    _say(f"q4 zeros, range and infinities T={T} d={d} G={G}")
    rng = np.random.default_rng(T)
    x = rng.normal(1, 1, (T, d)) * np.where(rng.random((T, d)) < 0.01, 1e3, 1)
    x[1, :], x[1, 7], x[1, 9], x[1:, 3], x[0, 3] = 0, 2.0 ** 123, 1, 0, np.inf
    x = torch.from_numpy(x).to(torch.bfloat16).to(hz.DEV)
    kg, ku, kd = (np.zeros(n, np.int64) for n in ((G * 128, d), (G * 128, d), (G, d, 128)))
    kg[:, 3] = kg[:, 7] = ku[:, 3] = ku[:, 9] = 1
    idle = np.arange(G * 128) % 128 // 8 == 8
    ku[idle, 9] = 0                                              # neurons that are 0 whatever their gate (column 3 is token 0's alone)
    kd[:, ::2] = rng.integers(1, 8, (G, d // 2, 128))
    kd[:, 1::4, 64:72] = 3                                       # odd outputs: those neurons, or codes of 8 alone
    full = lambda v, *n: torch.full(n, v, dtype=torch.bfloat16, device=hz.DEV)
    scale = 2.0 ** -8
    q4 = tuple(w for k in (kg, ku) for w in (torch.from_numpy(_pack_codes(k)).to(hz.DEV), full(scale, G * 128, d // 128)))
    q4 += (torch.from_numpy(_pack_codes(kd)).to(hz.DEV), full(scale, G, d))
    s = H.Shape(d, G * 128, 128, 64, "bf16")
    ws = torch.empty(H.halo_workspace_bytes_q4(s, T, G), dtype=torch.uint8, device=hz.DEV)
    y = full(float("nan"), T, d)
    H.halo_group_sparse_ffn_q4(s, x, q4, torch.ones((T, G), dtype=torch.uint8, device=hz.DEV), y, ws)
    torch.cuda.synchronize()
    yg = hz.to_np32(y).astype(np.float64)
    assert (yg[1:, 1::2] == 0).all() and (yg[0, ::2] == np.inf).all()
    want = 2.0 ** 123 * scale ** 3 * np.delete(kd, np.arange(64, 72), axis=2)[:, ::2].sum(axis=(0, 2))
    assert (np.abs(yg[1, ::2] - want) <= 2.0 ** -7 * want).all() and np.isfinite(yg[1:]).all()


@pytest.mark.parametrize("T,d,G", [(65, 256, 2), (65, 128, 2), (129, 1152, 24), (257, 1152, 9), (300, 1024, 20), (200, 4096, 12)])
def test_q4_many_tokens_large_scales(T, d, G):
    # scales up to 2^120 in gate and up, to 2^105 in down, tokens' values and y the smaller and larger by the same power of two: the
    # same bits, whatever the tiles
    _say(f"q4 large scales T={T} d={d} G={G}")
    g = torch.Generator(device=hz.DEV)
    g.manual_seed(T + d)
    code = lambda *n: torch.randint(-2 ** 31, 2 ** 31, n, generator=g, device=hz.DEV, dtype=torch.int64).to(torch.int32)
    scale = lambda *n: ((1 + torch.randint(0, 128, n, generator=g, device=hz.DEV) / 128.0) * 2.0 ** -8).to(torch.bfloat16)
    q4 = [code(G * 128, d // 8), scale(G * 128, d // 128), code(G * 128, d // 8), scale(G * 128, d // 128), code(G, d, 16), scale(G, d)]
    x = (torch.rand((T, d), generator=g, device=hz.DEV) * 24 + 8).to(torch.bfloat16)
    x = torch.where(torch.rand((T, d), generator=g, device=hz.DEV) < 0.5, x, -x)
    mask = (torch.rand((T, G), generator=g, device=hz.DEV) < 0.7).to(torch.uint8)
    s = H.Shape(d, G * 128, 128, 64, "bf16")
    ws = torch.empty(H.halo_workspace_bytes_q4(s, T, G), dtype=torch.uint8, device=hz.DEV)
    ys = []
    for up, down in ((0, 0), (127, 112)):
        w = [t.float().mul(2.0 ** (down if i == 5 else up)).to(torch.bfloat16) if i % 2 else t for i, t in enumerate(q4)]
        y = torch.full((T, d), float("nan"), dtype=torch.bfloat16, device=hz.DEV)
        H.halo_group_sparse_ffn_q4(s, (x.float() * 2.0 ** -up).to(torch.bfloat16), w, mask, y, ws)
        ys.append(y.double() * 2.0 ** -down)
    torch.cuda.synchronize()
    assert torch.isfinite(ys[0]).all() and torch.equal(*ys)
