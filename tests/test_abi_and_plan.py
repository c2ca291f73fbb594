"""CPU-only checks of the boundary: the library loads, exports every symbol the headers declare, and its
pure-host planner (ordering rules + list-order memory accounting) agrees bit for bit with the oracle."""
import ctypes
from dataclasses import replace
import os
import random
import re

import pytest

from oracle import schedule as S
from paper_2510_05186_amd import binding as B
from stage_inputs import configs as CFG
from stage_inputs import schedules as G

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_symbols():
    names = set()
    for hdr in ("optstage.h", "optstage_ops.h"):
        text = open(os.path.join(ROOT, "include", hdr)).read()
        text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
        names |= set(re.findall(r"\b(optstage_[a-z_0-9]+)\s*\(", text))
    return names


def test_library_exports_every_declared_symbol():
    names = declared_symbols()
    assert len(names) >= 30
    L = ctypes.CDLL(B.LIB_PATH)
    for n in sorted(names):
        assert hasattr(L, n), n
    assert names == set(B.EXPORTS)


def test_matrix_unit_attention_takes_what_its_grid_and_offsets_reach():
    """attn_mfma_applies(dtype, d, seq, n_q, n_kv, four pointers): row blocks of 128 are the grid's third dimension, at most 65535
    of them; one query and one kv head of 64 columns stay within 32-bit offsets up to 10.4 million rows."""
    f = ctypes.CDLL(B.LIB_PATH)["_Z17attn_mfma_appliesiiiiiPKvS0_S0_S0_"]
    f.restype, f.argtypes = ctypes.c_bool, [ctypes.c_int] * 5 + [ctypes.c_void_p] * 4
    takes = lambda d, seq, nq, nkv, at=4096: f(1, d, seq, nq, nkv, at, 4096, 4096, 4096)  # noqa: E731
    assert takes(64, 65535 * 128, 1, 1) and not takes(64, 65535 * 128 + 1, 1, 1)
    assert takes(128, 5_000_000, 1, 1) and not takes(128, 5_500_000, 1, 1)
    assert takes(128, 4096, 32, 8) and not takes(128, 4096, 32, 8, 4098) and not takes(64, 4096, 32, 8, 4104) and not takes(96, 4096, 32, 8)


def test_activation_epilogues_leave_weights_in_slabs_alone():
    """gemm_bf16_act_applies(M, N, K) chooses the activation's epilogue, which reads a plain weight, gemm_bf16_slab_applies(M, N, K, lda) keeps the
    weight in slabs: never both.  At hidden 8192 the two reach their 32-bit limits one ffn apart (959 row tiles)."""
    lib = ctypes.CDLL(B.LIB_PATH)
    act, slab = lib["_Z21gemm_bf16_act_appliesiii"], lib["_Z22gemm_bf16_slab_appliesiiii"]
    for f in (act, slab):
        f.restype = ctypes.c_bool
    assert act(320, 1792, 1024) and not slab(320, 1792, 1024, 1024) and slab(4096, 11008, 4096, 4096)
    assert slab(4096, 245504, 8192, 8192) and not slab(4096, 245512, 8192, 8192)
    rng = random.Random(3)
    sizes = [(4096, n, 8192) for n in range(245248, 245768, 8)] + [(int(2 ** rng.uniform(0, 17)), 8 * int(2 ** rng.uniform(3, 16)), 64 * int(2 ** rng.uniform(0, 7))) for _ in range(3000)]
    assert not any(act(*s) and slab(*s, s[2]) for s in sizes)


# us of an fp32 product in each form (tiles of 64 x 64, 64 x 32, 32 x 32, 16 x 32, 16 x 16, plain kernel), measured one after the other:
# (TN, 16-byte rows, epilogue, M, N, K, times).  Short contractions of many tiles are where a wrong form costs most, up to three times.
FP32_FORMS = [
    (0, 1, 0, 5168, 544, 4, (10.0, 11.5, 14.7, 25.0, 41.5, 8.8)), (0, 1, 0, 512, 4096, 4, (6.8, 8.3, 10.9, 19.0, 31.1, 7.5)),
    (0, 1, 0, 932, 1700, 8, (6.7, 8.4, 10.3, 16.1, 25.6, 7.6)), (0, 1, 0, 2048, 4096, 16, (19.3, 26.8, 37.2, 68.5, 117.6, 18.2)),
    (0, 1, 0, 512, 1024, 2048, (35.8, 22.9, 24.1, 38.2, 44.4, 333.2)), (0, 1, 0, 36, 3020, 4096, (66.3, 39.1, 29.0, 39.6, 33.1, 568.7)),
    (0, 1, 0, 200, 512, 2048, (35.4, 21.4, 13.1, 9.7, 11.7, 241.7)), (0, 0, 0, 932, 1700, 7, (5.7, 7.5, 7.1, 12.3, 15.3, 7.4)),
    (0, 0, 0, 756, 2056, 3, (5.5, 7.2, 6.8, 11.8, 14.7, 7.3)), (0, 0, 0, 1596, 876, 7, (5.6, 5.5, 6.2, 10.5, 13.7, 7.1)),
    (0, 0, 0, 1540, 3156, 407, (89.6, 126.4, 151.3, 219.0, 290.1, 112.4)), (0, 0, 0, 180, 1836, 1791, (74.2, 57.7, 71.0, 80.0, 99.5, 306.9)),
    (0, 0, 0, 272, 1788, 255, (15.5, 17.8, 12.9, 17.2, 21.3, 33.9)), (0, 0, 0, 200, 512, 1023, (41.7, 30.9, 21.6, 17.2, 21.7, 124.5)),
    (0, 0, 0, 8, 2284, 659, (21.4, 13.8, 11.1, 11.0, 7.3, 74.4)), (1, 1, 3, 3544, 232, 16, (5.0, 4.6, 5.7, 9.3, 13.0, 5.9)),
    (1, 1, 3, 132, 5372, 32, (5.0, 4.6, 5.9, 8.3, 11.5, 7.5)), (1, 1, 3, 3544, 232, 1024, (20.1, 20.3, 22.4, 31.4, 47.5, 196.6)),
    (1, 1, 3, 2304, 180, 1940, (32.2, 19.3, 20.2, 27.5, 36.3, 380.7)), (1, 1, 3, 36, 3020, 256, (7.7, 5.6, 4.8, 5.2, 5.2, 35.5)),
    (1, 1, 3, 744, 132, 1132, (20.4, 11.8, 7.7, 7.2, 9.1, 149.8)), (1, 1, 2, 512, 4096, 4, (6.5, 6.3, 9.4, 19.2, 27.5, 7.8)),
    (1, 1, 2, 1024, 1024, 8, (5.3, 4.7, 6.0, 10.6, 15.0, 6.9)), (1, 1, 2, 132, 5372, 48, (6.8, 5.4, 6.2, 8.9, 12.0, 12.4)),
    (1, 1, 2, 1024, 1024, 1024, (21.3, 21.3, 22.9, 36.0, 49.9, 225.2)), (1, 1, 2, 368, 2760, 100, (9.4, 8.8, 8.7, 12.6, 17.0, 20.6)),
    (1, 1, 2, 800, 800, 192, (7.5, 7.1, 5.7, 8.1, 11.6, 29.7)), (1, 1, 2, 60, 164, 496, (12.3, 7.8, 5.5, 5.1, 4.8, 69.4)),
    (1, 0, 3, 3543, 231, 24, (6.1, 5.8, 6.5, 11.9, 15.7, 7.5)), (1, 0, 3, 799, 799, 16, (6.1, 5.7, 5.1, 9.6, 12.1, 5.7)),
    (1, 0, 3, 2999, 2999, 256, (92.1, 97.3, 102.5, 139.8, 170.8, 119.7)), (1, 0, 3, 999, 1003, 128, (10.4, 9.7, 8.9, 15.6, 19.5, 20.2)),
    (1, 0, 3, 383, 255, 396, (17.5, 11.8, 6.9, 5.2, 5.5, 54.6)), (1, 0, 3, 311, 71, 1080, (34.9, 22.5, 12.0, 10.2, 7.4, 143.3)),
    (1, 0, 2, 931, 1699, 4, (12.0, 15.8, 15.5, 28.2, 38.9, 9.9)), (1, 0, 2, 1595, 875, 4, (11.6, 11.5, 9.3, 20.5, 34.7, 9.6)),
    (1, 0, 2, 807, 1059, 2924, (94.3, 113.0, 99.0, 122.9, 197.7, 614.7)), (1, 0, 2, 755, 2055, 128, (19.9, 21.3, 15.7, 26.6, 34.5, 25.2)),
    (1, 0, 2, 199, 511, 512, (23.3, 14.9, 9.3, 8.3, 8.7, 72.0)), (1, 0, 2, 63, 63, 192, (12.6, 10.0, 5.5, 5.5, 4.6, 29.1)),
    (0, 1, 0, 756, 2057, 4, (8.0, 9.9, 10.9, 17.2, 27.6, 7.3)), (0, 1, 1, 1032, 4149, 16, (29.0, 33.8, 38.0, 58.7, 105.5, 18.2)),
    (0, 1, 1, 2208, 2317, 16, (31.8, 35.8, 42.3, 69.3, 126.7, 20.7)),
]


@pytest.mark.parametrize("case", FP32_FORMS, ids=lambda c: "-".join(map(str, c[:6])))
def test_fp32_products_take_a_form_that_is_near_the_fastest(case):
    """The estimate by which a product picks its form (gemm_f32_form(tn, vec, epi, M, N, K, ldc)) is within 15 % of the fastest."""
    form = ctypes.CDLL(B.LIB_PATH)["_Z13gemm_f32_formbbiiiii"]
    form.argtypes = [ctypes.c_bool] * 2 + [ctypes.c_int] * 5
    tn, vec, epi, m, n, k, us = case
    assert us[form(tn, vec, epi, m, n, k, n)] <= 1.15 * min(us)


# us of the attention gradient, heads of 64, with one group of waves on a dK / dV workgroup's keys and with two: (tokens, sequences, n_q, n_kv, times)
D64_GROUPS = [(400, 4, 32, 8, (72.2, 62.1)), (1000, 4, 64, 8, (324.6, 281.2)), (1600, 4, 32, 8, (289.3, 251.8)), (4096, 2, 32, 8, (789.8, 688.4)), (256, 16, 32, 16, (62.1, 73.4)),
              (400, 16, 32, 16, (113.2, 127.1)), (640, 16, 32, 8, (175.0, 198.2)), (3000, 4, 32, 8, (745.9, 810.0)), (2048, 8, 64, 8, (1479.0, 1601.7)),
              (1300, 8, 16, 8, (171.2, 184.8)), (65, 8, 64, 8, (46.9, 39.2)), (640, 16, 8, 8, (56.6, 62.9)), (1000, 2, 8, 8, (48.0, 44.3))]


@pytest.mark.parametrize("case", D64_GROUPS, ids=lambda c: "-".join(map(str, c[:4])))
def test_attention_of_64_wide_heads_divides_its_keys_the_faster_way(case):
    groups = ctypes.CDLL(B.LIB_PATH)["_Z19attn_d64_key_groupsiiii"]
    assert case[4][groups(*case[:4]) - 1] <= 1.02 * min(case[4])


def oracle_table(cfg):
    return S.memory_table(cfg.family, cfg.hidden, cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim, cfg.ffn,
                          cfg.seq * cfg.micro_batch, cfg.elem_size)


@pytest.mark.parametrize("cfg", [CFG.CFG1, CFG.CFG2, CFG.CFG4, CFG.CFG5, CFG.CFG6], ids=lambda c: c.name)
def test_memory_table_matches_oracle(cfg):
    ws, act, kinds = B.query_sizes(cfg)
    t = oracle_table(cfg)
    assert kinds == t
    assert act == S.op_delta("F", cfg.n_layers, t)
    assert ws > 0


@pytest.mark.parametrize("hidden,tokens,norms", [(256, 128, 8), (1024, 320, 8), (2048, 300, 4), (4096, 300, 2), (8192, 4096, 1), (8192, 3, 8)])
def test_workspace_for_waiting_norm_sums_is_bounded(hidden, tokens, norms):
    """Partial sums of the norms of one launch (up to eight, of 2 hidden floats for each of up to 256 rows) stay within 16 MiB, or are one
    norm's: what a layer adds to the workspace beyond its weight copies, by layer."""
    sizes = [B.query_sizes(replace(CFG.shrunken(CFG.CFG4, hidden=hidden, n_q=2, n_kv=1, ffn=256, seq=tokens), n_layers=n))[0] for n in range(1, 8)]
    one = 2 * min(tokens, 256) * hidden * 4
    copies = sizes[-1] - sizes[-2]
    assert [s - sizes[0] - copies * i for i, s in enumerate(sizes)] == [(min(2 * (i + 1), norms) - min(2, norms)) * one for i in range(7)]


@pytest.mark.parametrize("cfg", [CFG.CFG1, CFG.CFG2, CFG.CFG4], ids=lambda c: c.name)
def test_recompute_memory_table_matches_oracle(cfg):
    _, act, kinds = B.query_sizes(cfg, recompute=1)
    t = oracle_table(cfg)
    assert kinds == t
    assert act == S.op_delta("F", cfg.n_layers, t, recompute=True) < S.op_delta("F", cfg.n_layers, t)


def test_recompute_plan_matches_oracle_accounting():
    cfg = small_cfg()
    t = oracle_table(cfg)
    p, m, L = 4, cfg.n_microbatches, cfg.n_layers
    lists = [G.one_f_one_b(p, m, i) for i in range(p)] + G.split_bw_greedy(p, m)
    more = [G.add_offload(base, L, ("X_IN", "QKV", "X_MID", "GU"), min_gap=gap, lead=1) for base in lists for gap in (1, 3)]
    for ev in lists + more:
        S.check_order(ev, m, L, recompute=True)
        peak, trace = S.account_memory(ev, L, t, recompute=True)
        st, bad, lib_peak, live = B.plan(cfg, ev, recompute=1)
        assert st == B.OK, B.lib().optstage_last_error()
        assert lib_peak == peak and live == trace
        assert peak < S.account_memory(ev, L, t)[0]
        st, bad, _, _ = B.plan(cfg, ev, budget=peak - 1, recompute=1)
        assert st == B.E_BUDGET
        with pytest.raises(S.ScheduleError) as ei:
            S.account_memory(ev, L, t, limit=peak - 1, recompute=True)
        assert ei.value.index == bad
    # a kind F does not keep cannot be offloaded: same event rejected on both sides
    ev = G.add_offload(lists[0], L, ("N2",), min_gap=1)
    with pytest.raises(S.ScheduleError) as ei:
        S.check_order(ev, m, L, recompute=True)
    st, bad, _, _ = B.plan(cfg, ev, recompute=1)
    assert st == B.E_ORDER and bad == ei.value.index


def test_plan_with_model_chunks_matches_oracle():
    """A stage that holds two model chunks: the planner's order rules and accounting are the oracle's."""
    cfg = small_cfg(m=4, L=4)
    t = oracle_table(cfg)
    m, L, v = cfg.n_microbatches, cfg.n_layers, 2
    for i in range(2):
        base = G.interleaved_one_f_one_b(2, m, i, v)
        for ev in (base, G.add_offload(base, L, ("X_IN", "QKV", "GU"), min_gap=2, lead=1)):
            S.check_order(ev, m, L, n_chunks=v)
            peak, trace = S.account_memory(ev, L, t, n_chunks=v)
            st, bad, lib_peak, live = B.plan(cfg, ev, n_chunks=v)
            assert st == B.OK, B.lib().optstage_last_error()
            assert lib_peak == peak and live == trace
            st, bad, _, _ = B.plan(cfg, ev, budget=peak - 1, n_chunks=v)
            assert st == B.E_BUDGET
            with pytest.raises(S.ScheduleError) as ei:
                S.account_memory(ev, L, t, limit=peak - 1, n_chunks=v)
            assert ei.value.index == bad
    kinds = ("QKV",)
    bad_lists = [
        [("F", 0, 0), ("B", 0, 1)],                                            # B of a chunk before its F
        [("F", 1, 1)],                                                         # chunk 1 starts at micro-batch 0
        [("F", 0, 0), ("F", 0, 1), ("O", 0, 3, kinds), ("OWAIT", 0, 3, kinds), ("B", 0, 1)],   # not reloaded
        [("F", 0, 0), ("O", 0, 2, kinds)],                                     # layer 2 belongs to chunk 1
    ]
    for ev in bad_lists:
        with pytest.raises(S.ScheduleError) as ei:
            S.check_order(ev, m, L, n_chunks=v)
        st, bad, _, _ = B.plan(cfg, ev, n_chunks=v)
        assert st == B.E_ORDER and bad == ei.value.index, (ev, st, bad, ei.value.index)
    assert B.plan(cfg, [("F", 0, 2)], n_chunks=v)[0] == B.E_ARG               # no such chunk
    d = B.make_desc(cfg, n_chunks=3)                                           # 4 layers do not split in three
    assert B.lib().optstage_query_sizes(d, None, None, None) == B.E_ARG


def small_cfg(m=6, L=3):
    return CFG.shrunken(CFG.CFG4, hidden=256, n_q=4, n_kv=2, ffn=384, seq=192, n_layers=L, n_microbatches=m)


def test_plan_matches_oracle_accounting_on_generated_schedules():
    cfg = small_cfg()
    t = oracle_table(cfg)
    p, m, L = 4, cfg.n_microbatches, cfg.n_layers
    lists = [G.one_f_one_b(p, m, i) for i in range(p)] + G.split_bw_greedy(p, m)
    more = []
    for base in lists:
        for gap in (1, 2, 4):
            for lead in (1, 2):
                more.append(G.add_offload(base, L, ("X_IN", "QKV", "X_MID"), min_gap=gap, lead=lead))
        more.append(G.add_offload(base, L, ("N1", "GU", "A", "LSE", "STATS", "O", "N2"), min_gap=1))
    for ev in lists + more:
        S.check_order(ev, m, L)
        peak, trace = S.account_memory(ev, L, t)
        st, bad, lib_peak, live = B.plan(cfg, ev)
        assert st == B.OK, B.lib().optstage_last_error()
        assert lib_peak == peak and live == trace
        # budget exactly at the peak passes, one byte less fails at the same event as the oracle
        assert B.plan(cfg, ev, budget=peak)[0] == B.OK
        st, bad, _, _ = B.plan(cfg, ev, budget=peak - 1)
        assert st == B.E_BUDGET
        with pytest.raises(S.ScheduleError) as ei:
            S.account_memory(ev, L, t, limit=peak - 1)
        assert ei.value.index == bad


def test_plan_rejects_what_the_oracle_rejects():
    cfg = small_cfg(m=2, L=2)
    q = ("QKV",)
    bad_lists = [
        [("B", 0), ("F", 0), ("W", 0), ("F", 1), ("B", 1), ("W", 1)],
        [("F", 0), ("W", 0), ("B", 0), ("F", 1), ("B", 1), ("W", 1)],
        [("F", 1), ("F", 0), ("B", 0), ("W", 0), ("B", 1), ("W", 1)],
        [("F", 0), ("F", 0), ("B", 0), ("W", 0)],
        [("F", 0), ("B", 0), ("W", 0)],
        [("O", 0, 0, q), ("F", 0), ("B", 0), ("W", 0), ("F", 1), ("B", 1), ("W", 1)],
        [("F", 0), ("O", 0, 0, q), ("OWAIT", 0, 0, q), ("B", 0), ("W", 0), ("F", 1), ("B", 1), ("W", 1)],
        [("F", 0), ("O", 0, 0, q), ("R", 0, 0, q), ("B", 0), ("W", 0), ("F", 1), ("B", 1), ("W", 1)],
        [("F", 0), ("O", 0, 0, q), ("O", 0, 0, q), ("B", 0), ("W", 0), ("F", 1), ("B", 1), ("W", 1)],
        [("F", 0), ("OWAIT", 0, 0, q), ("B", 0), ("W", 0), ("F", 1), ("B", 1), ("W", 1)],
        [("F", 0), ("B", 0), ("O", 0, 0, q), ("W", 0), ("F", 1), ("B", 1), ("W", 1)],
    ]
    for ev in bad_lists:
        with pytest.raises(S.ScheduleError) as ei:
            S.check_order(ev, 2, 2)
        st, bad, _, _ = B.plan(cfg, ev)
        assert st == B.E_ORDER, ev
        assert bad == ei.value.index, (ev, bad, ei.value.index)
    # argument errors: bad layer, non-offloadable kind, micro-batch out of range
    assert B.plan(cfg, [("F", 0), ("O", 0, 5, q)])[0] == B.E_ARG
    assert B.plan(cfg, [("F", 0), ("O", 0, 0, ("DY",))])[0] == B.E_ARG
    assert B.plan(cfg, [("F", 7)])[0] == B.E_ARG


def test_plan_random_valid_interleavings():
    rng = random.Random(7)
    cfg = small_cfg(m=4, L=2)
    t = oracle_table(cfg)
    m, L = 4, 2
    for _ in range(200):
        # random valid compute order
        nxt = {"F": 0, "B": 0, "W": 0}
        ev = []
        while nxt["W"] < m:
            cands = []
            if nxt["F"] < m:
                cands.append("F")
            if nxt["B"] < nxt["F"]:
                cands.append("B")
            if nxt["W"] < nxt["B"]:
                cands.append("W")
            c = rng.choice(cands)
            ev.append((c, nxt[c]))
            nxt[c] += 1
        ev = G.add_offload(ev, L, tuple(rng.sample(S.F_KINDS, rng.randint(1, 4))), min_gap=rng.randint(0, 3), lead=rng.randint(1, 3))
        S.check_order(ev, m, L)
        peak, trace = S.account_memory(ev, L, t)
        st, _, lib_peak, live = B.plan(cfg, ev)
        assert st == B.OK and lib_peak == peak and live == trace


@pytest.mark.parametrize("recompute", [False, True])
def test_planner_equals_oracle_accounting_on_random_valid_lists(recompute):
    """Property over the schedule grammar, host only: for random valid lists (compute order, offloaded items and
    transfer positions all drawn) the library's planner reports the oracle's live bytes after every event and the
    oracle's peak, accepts a budget equal to that peak and refuses one allocation granule less."""
    import numpy as np
    from stage_inputs import schedules as G
    cfg = replace(CFG.shrunken(CFG.CFG2, hidden=256, n_q=2, n_kv=2, ffn=512, seq=256, n_layers=3, n_microbatches=5), name="plan_random")
    t = S.memory_table(cfg.family, cfg.hidden, cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim, cfg.ffn, cfg.seq * cfg.micro_batch, cfg.elem_size)
    kinds = ("X_IN", "QKV", "X_MID", "O", "GU", "LSE") if recompute else ("X_IN", "N1", "QKV", "X_MID", "O", "GU", "A", "STATS")
    for seed in range(40):
        rng = np.random.default_rng(seed)
        ev = G.random_valid_list(rng, cfg.n_microbatches, cfg.n_layers, kinds, p_offload=0.5)
        S.check_order(ev, cfg.n_microbatches, cfg.n_layers, recompute=recompute)
        peak, trace = S.account_memory(ev, cfg.n_layers, t, recompute=recompute)
        code, bad, ppeak, live = B.plan(cfg, ev, budget=peak, recompute=int(recompute))
        assert code == B.OK and ppeak == peak and list(live[:len(ev)]) == trace, (seed, code, bad)
        assert B.plan(cfg, ev, budget=peak - S.ALIGN, recompute=int(recompute))[0] == B.E_BUDGET, seed
