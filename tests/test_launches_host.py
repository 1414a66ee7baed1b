"""What the entry points launch, checked without a GPU (tests/launches.py)."""
import numpy as np

from tests.launches import record

BF16, F32 = 1, 0


def test_staged_and_fused_ffn_launch_the_same():
    # the ranges of the down projection, and with them the order of its sums, follow the shape and T, not the room that the
    # rest of a workspace leaves: T around the most tokens that the fixed scratch array takes
    rng = np.random.default_rng(9)
    cases = [(1152, 23, T, 256) for T in range(617, 650, 4)]
    for _ in range(60):
        d, G = 128 * int(rng.integers(1, 33)), int(rng.integers(8, 97))
        line = (8 << 20) / (G * 128 * 4 + G * 25 + 64)
        cases += [(d, G, max(17, int(line * f)), 64) for f in (0.5, 0.9, 0.95, 0.98, 1.0, 1.05)]
    calls = []
    for d, G, T, r in cases:
        shape = (d, G, 128, r, BF16)
        calls += [dict(fn="group_sparse_ffn", shape=shape, T=T)]
        calls += [dict(fn="ffn_forward", shape=shape, T=T, K=K) for K in (1, G // 2, G)]
        calls += [dict(fn="group_sparse_ffn_q4", shape=shape, T=T), dict(fn="ffn_forward_q4", shape=shape, T=T, K=G)]
    got = iter(record(calls))
    for case in cases:
        for n in (4, 2):                                         # the bf16 calls, the 4-bit calls
            runs = [next(got) for _ in range(n)]
            assert all(rc == 0 for rc, _, _ in runs), case
            staged = runs[0][2]
            for _, _, launches in runs[1:]:
                assert launches[-len(staged):] == staged, case


def test_grids_of_very_many_tokens_stay_within_the_limits():
    # the recorder refuses more than 65535 workgroups in y, as a device may
    scores, ffn = [1048560, 1048561, 1048576, 5000000], [2097121, 2100000, 4194304, 4200000]
    calls = [dict(fn="predict_scores", shape=(8, 8, 128, 8, BF16), T=T) for T in scores]
    calls += [dict(fn="group_sparse_ffn", shape=(8, 2, gs, 8, F32), T=T) for T in ffn for gs in (16, 128)]
    for c, (rc, _, launches) in zip(calls, record(calls)):
        assert rc == 0, (c, launches)
        # every token is covered: rows per workgroup of the kernels
        for name, rows in [("scores_mfma", 16), ("gate_up_f32", 64), ("down_f32", 32)]:
            runs = [y for n, _, y, _, _ in launches if name in n]
            assert not runs or (sum(runs) - 1) * rows < c["T"] <= sum(runs) * rows, (c, launches)


def test_more_lds_is_allowed_on_each_device():
    # kernels with more than 64 KiB of dynamic LDS, launched with one device current and then with another
    calls = [dict(fn="predict_scores", shape=(4096, 8, 128, 512, BF16), T=40, device=dev) for dev in (0, 1, 0, 7)]
    calls += [dict(fn=fn, shape=(d, 20, 128, 64, BF16), T=T, K=4, device=dev) for dev in (0, 1, 0, 7)
              for fn in ("ffn_forward", "ffn_forward_q4") for d in (8192, 3200) for T in (4, 16, 40, 300)]
    for c, (rc, _, launches) in zip(calls, record(calls)):
        assert rc == 0 and launches, (c, rc, launches)


def test_prediction_in_one_launch_by_shape():
    for T, G, d, r, one in [(64, 128, 256, 128, True), (64, 129, 256, 128, False), (64, 128, 240, 136, False)]:
        (rc, _, launches), = record([dict(fn="ffn_forward", shape=(d, G, 128, r, F32), T=T, K=4)])
        assert rc == 0 and ("predict_mask_kernel" in launches[0][0]) == one, (T, G, d, r, launches)
    for T, d, r, dtype, one in [(64, 1024, 64, BF16, True), (65, 1024, 64, BF16, False), (16, 1032, 64, BF16, False), (4, 1000, 64, BF16, True),
                                (5, 1000, 64, BF16, False), (64, 504, 64, F32, True), (64, 512, 64, F32, True), (64, 520, 64, F32, False)]:
        # (33 groups of float32: up to 32 the prediction has no launch of its own)
        (rc, _, launches), = record([dict(fn="ffn_forward", shape=(d, 33 if dtype == F32 else 8, 128, r, dtype), T=T, K=4)])
        assert rc == 0 and ("predict_mask_kernel" in launches[0][0]) == one, (T, d, r, launches)


def test_few_token_gate_up_by_shape():
    # the streaming kernel up to rows of 8192 and 256 groups, past either the one that walks its rows in chunks
    for T, d, G, name in [(2, 8192, 256, "gate_up_ft"), (5, 8192, 256, "gate_up_streamILNS_7WeightsE0E"), (16, 128, 3, "gate_up_streamILNS_7WeightsE0E"),
                          (2, 8320, 3, "gate_up_mtILb1E"), (16, 8320, 256, "gate_up_mtILb1E"), (7, 256, 260, "gate_up_mtILb0E"),
                          (16, 640, 257, "gate_up_mtILb0E")]:
        serial, ahead = record([dict(fn=fn, shape=(d, G, 128, 64, BF16), T=T, K=G // 2) for fn in ("group_sparse_ffn", "ffn_forward_ahead")])
        for rc, _, launches in (serial, ahead):
            assert rc == 0 and sum(name in n for n, *_ in launches) == 1, (T, d, G, launches)
    # over 4-bit weights: codes with an offset, codes as they are, and past the streaming kernels the plain path
    for T, d, G, names in [(2, 8192, 256, ["gate_up_streamILNS_7WeightsE1E", "down_q4_mt"]), (16, 1024, 3, ["gate_up_streamILNS_7WeightsE1E", "down_q4_mt"]),
                           (2, 8064, 256, ["gate_up_streamILNS_7WeightsE2E", "down_q4_f32ILi2ELi1E"]), (4, 128, 3, ["gate_up_streamILNS_7WeightsE2E", "down_q4_f32ILi1ELi2E"]),
                           (8, 4224, 9, ["gate_up_streamILNS_7WeightsE2E", "down_q4_f32ILi2ELi4E"]), (9, 3968, 9, ["gate_up_streamILNS_7WeightsE2E", "down_q4_f32ILi1ELi0E"]),
                           (2, 8320, 3, ["union_kernel", "gate_up_q4_generic", "down_q4_generic"]), (16, 640, 257, ["union_kernel", "gate_up_q4_generic", "down_q4_generic"])]:
        (rc, _, launches), = record([dict(fn="group_sparse_ffn_q4", shape=(d, G, 128, 64, BF16), T=T)])
        assert rc == 0 and len(launches) == len(names) and all(a in b[0] for a, b in zip(names, launches)), (T, d, G, launches)


def test_float32_projections_by_the_number_of_tokens():
    # groups of 128: what is asked for before the mask is known, and the form of the down projection
    for T, d, G, ask, down in [(1, 1024, 24, True, "down_f32ILi1E"), (5, 256, 8, True, "down_f32ILi1E"), (6, 256, 9, False, "down_f32_128"),
                               (8, 256, 8, False, "down_f32ILi1E"), (9, 256, 8, False, "down_f32_128"), (64, 8192, 64, False, "down_f32_128"),
                               (65, 816, 24, False, "down_f32_128"), (65, 824, 24, False, "down_f32ILi2E"), (512, 128, 8, False, "down_f32_128"),
                               (512, 256, 8, False, "down_f32ILi2E")]:
        (rc, _, launches), = record([dict(fn="group_sparse_ffn", shape=(d, G, 128, 64, F32), T=T)])
        assert rc == 0 and len(launches) == 2 and down in launches[1][0], (T, d, G, launches)
        assert ("gate_up_f32ILi1ELb1E" in launches[0][0]) == ask, (T, d, G, launches)


def test_first_predictor_layer_by_the_number_of_results():
    # few results (T * rank below 14 Ki), or fewer than 16 tokens, are a wave each; the others go to tiles
    cases = [(16, 64, False), (16, 512, False), (100, 128, False), (256, 48, False), (15, 1024, False), (28, 512, True), (64, 256, True),
             (300, 64, True)]
    calls = [dict(fn="predict_scores", shape=(d, 32, 128, r, BF16), T=T) for T, r, _ in cases for d in (128, 1024, 8192)]
    got = iter(record(calls))
    for T, r, tiles in cases:
        for _ in range(3):
            rc, _, launches = next(got)
            assert rc == 0 and ("hidden_mfma" in launches[0][0]) == tiles, (T, r, launches)


def test_kernels_past_the_row_table():
    shape = (128, 3, 128, 8, BF16)
    for T, q4, names in [(32767, False, ["group_tokens", "gate_up_pf_big", "down_pf_ring"]),
                         (32768, False, ["group_tokens", "gate_up_pf_ring", "7down_pf"]),
                         (32767, True, ["group_tokens", "gate_up_pf_ring", "down_pf_ring"]),
                         (32768, True, ["expand_q4"] * 3 + ["group_tokens", "gate_up_pf_ring", "7down_pf"])]:
        (rc, _, launches), = record([dict(fn="group_sparse_ffn" + ("_q4" if q4 else ""), shape=shape, T=T)])
        kernels = [n for n, *_ in launches if "reduce" not in n]
        assert rc == 0 and len(kernels) == len(names) and all(a in b for a, b in zip(names, kernels)), (T, q4, launches)


def test_many_token_cases_run_on_the_kernels_they_are_for():
    # the forms of the ring kernels that the parity cases are chosen to reach: tokens per tile, in gate/up and down
    for T, d, G, gate_up, down in [(17, 128, 3, 128, 128), (129, 640, 40, 128, 64), (129, 1152, 24, 128, 128), (129, 4096, 40, 128, 256),
                                   (257, 1024, 6, 256, 64), (257, 1152, 9, 256, 128), (515, 4224, 9, 256, 128), (515, 4224, 40, 256, 256)]:
        for q4 in (0, 1):
            (rc, _, launches), = record([dict(fn="ffn_forward" + ("_q4" if q4 else ""), shape=(d, G, 128, 64, BF16), T=T, K=G // 2)])
            names = [n for n, *_ in launches]
            for kernel, tokens in (("gate_up_pf_ring", gate_up), ("down_pf_ring", down)):
                assert rc == 0 and sum(f"{kernel}ILb{q4}ELi{tokens}E" in n for n in names) == 1, (T, d, G, q4, names)
    for T, d, G in [(300, 256, 300), (1100, 384, 180), (520, 128, 100), (300, 1152, 150), (2050, 256, 97)]:
        (rc, _, launches), = record([dict(fn="ffn_forward", shape=(d, G, 128, 64, BF16), T=T, K=G // 3)])
        assert rc == 0 and any("gate_up_pf_big" in n for n, *_ in launches), (T, d, G, launches)


def test_quarter_tiles_of_tokens():
    # tokens per tile in gate/up over codes and in down (gate/up over bf16 weights has no quarter tiles)
    for T, d, G, gate_up, down in [(17, 128, 3, 128, 128), (17, 256, 3, 64, 64), (33, 640, 9, 64, 64), (64, 1152, 20, 64, 64),
                                   (65, 768, 8, 128, 64), (193, 1024, 24, 128, 64), (520, 896, 9, 256, 64),
                                   (65, 640, 9, 128, 64), (65, 768, 7, 128, 64), (400, 256, 2, 256, 64), (65, 128, 9, 128, 128),
                                   (65, 2048, 24, 128, 128), (128, 5120, 108, 128, 128)]:
        for q4 in (0, 1):
            (rc, _, launches), = record([dict(fn="ffn_forward" + ("_q4" if q4 else ""), shape=(d, G, 128, 64, BF16), T=T, K=G // 2)])
            names = [n for n, *_ in launches]
            for kernel, tokens in (("gate_up_pf_ring", gate_up if q4 else max(gate_up, 128)), ("down_pf_ring", down)):
                assert rc == 0 and sum(f"{kernel}ILb{q4}ELi{tokens}E" in n for n in names) == 1, (T, d, G, q4, names)
            # the scale in float where gate/up has it so: codes of up to 64 tokens, rows of 256 and more
            assert sum(f"down_pf_ringILb{q4}ELi{down}ELb{int(q4 and gate_up == 64)}E" in n for n in names) == 1, (T, d, G, q4, names)


def test_small_float32_blocks_by_shape():
    # the whole pass in two launches: up to 64 tokens, rows of 4096, groups of 128, a wave of sixteen to a row (pair of rows) of Bt, few weights
    for T, d, G, gs, r, two in [(1, 1024, 24, 128, 64, True), (3, 1032, 24, 128, 64, False), (4, 1024, 32, 128, 256, True), (4, 1032, 32, 128, 256, False),
                                (64, 256, 8, 128, 64, True), (65, 256, 8, 128, 64, False), (16, 4096, 8, 128, 512, True), (16, 4104, 2, 128, 64, False), (8, 64, 33, 128, 256, False), (8, 64, 16, 128, 512, True),
                                (8, 64, 17, 128, 264, False), (8, 64, 4, 128, 520, False), (8, 64, 8, 64, 64, False)]:
        (rc, _, launches), = record([dict(fn="ffn_forward", shape=(d, G, gs, r, F32), T=T, K=G // 2)])
        names = [n for n, *_ in launches]
        assert rc == 0 and (len(names) == 2 and "hidden_gate_up_f32" in names[0] and "predict_down_f32" in names[1]) == two, (T, d, G, gs, r, names)
