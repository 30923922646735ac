"""Kernel variants at the sizes where they can go wrong: edges of their tiles, remainders, the smallest and the
largest of their range.  Everything goes through the C-ABI and is compared with the oracle."""
import math

import numpy as np
import pytest
import torch

from oracle import codecsight_oracle as oc
from tests import helpers as hp
from tests.test_gpu_parity import DEV, PLAN_HDR_INTS, _attention_plan, _attn_case, _pool, _project_gpu, _random_block_frames, _residual_gpu, cs, say   # noqa: F401  (cs is a fixture)
from tests.test_gpu_parity import test_attention_plan_is_a_valid_schedule as _plan_is_valid

pytestmark = pytest.mark.gpu


# fp32 attention: row tiles of 32 (token, head) rows, key tiles of 32 dealt to 8 waves
F32_ATTN = [
    # Hq, Hkv, d, kv_lens, n_qs
    (1, 1, 64, [1], [1]),
    (1, 1, 128, [31, 32, 33], [31, 32, 33]),                       # key and row tile edges
    (3, 1, 128, [255, 256, 257], [11, 10, 32]),                    # one turn of the eight waves, and one key more
    (16, 1, 64, [600, 16, 15, 17], [2, 3, 0, 5]),
    (28, 4, 128, [700], [77]),
    (2, 2, 64, [20] * 130, [2] * 130),                             # more streams than one turn of the row-tile search
]


@pytest.mark.parametrize("case", range(len(F32_ATTN)))
def test_f32_attention_tile_edges(cs, case):
    hq, hkv, d, kv_lens, n_qs = F32_ATTN[case]
    say(f"f32 attention edges {case}: heads={hq}/{hkv} d={d} kv={kv_lens[:4]} n_q={n_qs[:4]}")
    say(f"  -> {_attn_case(cs, np.random.default_rng(9100 + case), 'f32', hq, hkv, d, kv_lens, n_qs)}")


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_f32_attention_masked_rows_do_not_reach_earlier_queries(cs, bad):
    """A cache row that holds no finite number reaches the queries that see it and no other, also those that
    share its tile."""
    say(f"f32 attention: a {bad} row in the cache")
    rng = np.random.default_rng(9200)
    d, kv_len, at = 64, 90, 75
    kc, vc, q = _pool(rng, (96, 1, d), "f32"), _pool(rng, (96, 1, d), "f32"), _pool(rng, (kv_len, 1, d), "f32")
    ref = oc.window_attn(hp.f64(q), hp.f64(kc), hp.f64(vc), np.array([0, kv_len]), np.arange(kv_len),
                         np.arange(6)[None], 1, 1 / math.sqrt(d))
    vc[at] = bad
    kc[at] = bad
    out = torch.zeros_like(q, device=DEV)
    i32 = lambda v: torch.tensor(v, dtype=torch.int32, device=DEV)
    cs.cs_window_prefill_attn(q.to(DEV), kc.to(DEV), vc.to(DEV), i32([0, kv_len]), i32(list(range(kv_len))), i32([kv_len]),
                              i32([list(range(6))]), 6, 16, out, kv_len, 1, 1, 1, d, d, d, 1 / math.sqrt(d), cs.CS_F32)
    got = out.cpu()
    hp.check_attention(got[:at], ref[:at], "f32")
    assert not torch.isfinite(got[at:]).any()


# bf16 attention without a plan (head_dim 64, and head_dim 128 while the row tiles are few): key tiles of 64 shared by
# one, two or four key groups; 64- or 128-row tiles
TILE_ATTN = [
    # Hq, Hkv, d, kv_lens, n_qs
    (7, 1, 128, [63, 64, 65, 1], [9, 10, 65, 1]),                       # two key groups, one of them without a tile
    (28, 4, 128, [580, 577, 513], [40, 150, 3]),                        # four key groups, 9 and 10 key tiles
    (28, 4, 128, [1100], [470]),                                        # four key groups, row tiles of 64 with a remainder
    (28, 4, 128, [900, 1, 830, 128], [420, 1, 333, 0]),                 # two key groups, a stream without queries
    (32, 8, 128, [700 + 61 * i for i in range(7)], [190 + 17 * i for i in range(7)]),    # rows of 128
    (16, 2, 128, [1500, 400, 1400], [600, 300, 777]),                   # two key groups, 24 key tiles
    (4, 4, 64, [1, 63, 64, 65, 129], [1, 63, 30, 65, 2]),
    (16, 1, 64, [2300], [100]),                                         # two key groups, 36 key tiles
    (28, 4, 64, [300 + 7 * i for i in range(40)], [90 + i for i in range(40)]),   # one key group
    (2, 2, 64, [20] * 130, [2] * 130),
]


@pytest.mark.parametrize("case", range(len(TILE_ATTN)))
def test_unplanned_attention_tile_edges(cs, case):
    hq, hkv, d, kv_lens, n_qs = TILE_ATTN[case]
    say(f"unplanned attention {case}: heads={hq}/{hkv} d={d} kv={kv_lens[:4]} n_q={n_qs[:4]}")
    for mult in (1.0, 6.0):                                             # (wide scores: maxima far apart between key groups)
        say(f"  -> {_attn_case(cs, np.random.default_rng(9300 + case), 'bf16', hq, hkv, d, kv_lens, n_qs, scale_mult=mult)}")


# bf16 attention from a plan, head_dim 128: jobs of one or two 128-row tiles, four waves of 64 rows, 32 keys at a time
# (0 and 1 have at most 128 rows a stream on average, 3 to 5 few row tiles: these run without a plan)
PLANNED_ATTN = [
    # Hq, Hkv, kv_lens, n_qs
    (8, 8, [1 + 9 * i % 71 for i in range(132)], [1 + 5 * i % (1 + 9 * i % 71) for i in range(132)]),   # one head a group, jobs of one or two key tiles
    (32, 2, [40 + i % 90 for i in range(516)], [1 + i % 11 for i in range(516)]),                        # 16 heads a group
    (12, 4, [33 * (1 + i % 6) for i in range(260)], [22 * (1 + i % 6) for i in range(260)]),             # ends of half tiles, one to four row tiles
    (7, 1, [6100], [42]),                                                                                # split sweeps, three row tiles
    (8, 2, [7000, 64, 4200], [150, 64, 31]),                                                             # split and whole, frontiers far apart
    (28, 4, [4300], [19]),                                                                               # two row tiles, 5 rows in the second
    (8, 8, [400 if i % 2 else 1 + 9 * i % 71 for i in range(132)], [320 if i % 2 else 1 + 5 * i % (1 + 9 * i % 71) for i in range(132)]),   # one head a group, jobs of one key tile and more
    (32, 2, [40 + i % 90 for i in range(516)], [1 + i % 11 if i % 4 else 21 for i in range(516)]),        # 16 heads a group, one to three row tiles
    (14, 2, [8100], [640]),                                                                              # split sweeps, 35 row tiles a kv head
    (8, 2, [9000, 64, 7200], [750, 64, 431]),                                                            # split and whole, frontiers far apart
    (56, 4, [4300, 4250], [150, 10]),                                                                    # 140 rows: 12 in the second row tile
    (16, 16, [5105, 300, 110], [100, 100, 100]),                                                         # three streams of two row tiles, 81 key tiles
    # (6 and 7 again, with a window that is too long for jobs of one row tile each)
    (8, 8, [3100] + [400 if i % 2 else 1 + 9 * i % 71 for i in range(132)], [70] + [320 if i % 2 else 1 + 5 * i % (1 + 9 * i % 71) for i in range(132)]),
    (32, 2, [3100] + [40 + i % 90 for i in range(516)], [9] + [1 + i % 11 if i % 4 else 21 for i in range(516)]),
]


@pytest.mark.parametrize("case", range(len(PLANNED_ATTN)))
def test_planned_attention_job_edges(cs, case):
    hq, hkv, kv_lens, n_qs = PLANNED_ATTN[case]
    say(f"planned attention {case}: heads={hq}/{hkv} kv={kv_lens[:4]} n_q={n_qs[:4]} streams={len(kv_lens)}")
    for mult in (1.0, 6.0):                                             # (wide scores: the reference maximum is raised along the sweep)
        say(f"  -> {_attn_case(cs, np.random.default_rng(9350 + case), 'bf16', hq, hkv, 128, kv_lens, n_qs, scale_mult=mult)}")


# Lists of up to 72 units an XCD are dealt by length over the whole list, longer ones batch by batch.  (A unit is two row tiles
# but in the first two cases, where it is one.)
DEALT = [
    # Hq, Hkv, kv_lens, n_qs
    (8, 8, [180 + 7 * (i % 40) for i in range(72)], [130 + i % 20 for i in range(72)]),                 # 72 units, ties
    (8, 8, [180 + 7 * (i % 40) for i in range(73)], [130 + i % 20 for i in range(73)]),                 # 73
    (8, 8, [3100] + [180 + 7 * (i % 40) for i in range(71)], [130 + i % 20 for i in range(72)]),         # 72 units, ties
    (8, 8, [3100] + [180 + 7 * (i % 40) for i in range(72)], [130 + i % 20 for i in range(73)]),         # 73
    (28, 4, [900 + 31 * i for i in range(11)], [390 + 40 * (i % 4) for i in range(11)]),                 # pairs left over, odd row tiles
    (16, 1, [700 + 60 * i for i in range(17)], [520 + 20 * (i % 3) if i != 5 else 0 for i in range(17)]),  # one pair left over, a stream without rows
]


@pytest.mark.parametrize("case", range(len(DEALT)))
def test_planned_attention_dealt_by_length(cs, case):
    hq, hkv, kv_lens, n_qs = DEALT[case]
    n_qs = [min(n, k) for n, k in zip(n_qs, kv_lens)]
    _plan_is_valid(cs, hq, hkv, kv_lens, n_qs)
    say(f"  -> {_attn_case(cs, np.random.default_rng(9390 + case), 'bf16', hq, hkv, 128, kv_lens, n_qs)}")


# A stream's odd first row tile, a unit of its own, stands in a chain before a later unit of the same sweep that ends in the
# same key tile: the two are no job, since the keys of a job end with its first row tile's.
FIRST_TILE_ALONE = [
    # Hq, Hkv, kv_lens, n_qs
    (32, 8, [128, 5000], [70, 512]), (64, 8, [60, 8000], [40, 40]), (56, 8, [64, 8000], [41, 90]), (64, 4, [60, 4300], [40, 150]),
    (64, 8, [2072], [2064]),                                                                             # whole sweeps, ordered by length
]


@pytest.mark.parametrize("case", range(len(FIRST_TILE_ALONE)))
def test_planned_attention_first_row_tile_alone(cs, case):
    hq, hkv, kv_lens, n_qs = FIRST_TILE_ALONE[case]
    say(f"planned attention, first row tile alone {case}: heads={hq}/{hkv} kv={kv_lens} n_q={n_qs}")
    say(f"  -> {_attn_case(cs, np.random.default_rng(9420 + case), 'bf16', hq, hkv, 128, kv_lens, n_qs, last_queries=True)}")


# Both sides of the lines from which whole sweeps run from a plan: row tiles x kv heads, key tiles of the table's rows (a block
# more than the window has), and more than 128 rows a stream on average.
WHOLE_SWEEPS = [
    # Hq, Hkv, streams, rows of all streams, longest window, row tiles, key tiles, a BUILD call makes a plan
    (16, 4, 8, 3840, 700, 512, 12, True), (16, 4, 8, 3839, 700, 508, 12, False), (16, 4, 8, 3840, 496, 512, 8, False),
    (16, 4, 8, 3840, 497, 512, 9, True), (16, 4, 8, 3840, 2032, 512, 32, True), (16, 4, 8, 3840, 2033, 512, 33, False),
    (32, 8, 6, 2880, 700, 768, 12, True), (32, 8, 6, 2879, 700, 760, 12, False),
    (16, 4, 64, 6144, 400, 1024, 7, True), (16, 4, 64, 6143, 400, 1020, 7, False),
    (8, 4, 128, 8192, 300, 1024, 5, False), (8, 4, 128, 8193, 300, 1024, 5, True),
]


@pytest.mark.parametrize("hq,hkv,n_streams,rows,window,row_tiles,key_tiles,plans", WHOLE_SWEEPS)
def test_attention_at_the_lines_of_whole_sweeps(cs, hq, hkv, n_streams, rows, window, row_tiles, key_tiles, plans):
    n_qs = [rows // n_streams + (1 if i < rows % n_streams else 0) for i in range(n_streams)]
    kv_lens = [max(n, window - 3 * i % 200) for i, n in enumerate(n_qs)]
    assert (rows * (hq // hkv) // 128 + n_streams) * hkv == row_tiles
    assert -(-(-(-max(kv_lens) // 16) + 1) * 16 // 64) == key_tiles
    _plan_is_valid(cs, hq, hkv, kv_lens, n_qs)
    say(f"  -> {_attn_case(cs, np.random.default_rng(9400 + window + rows), 'bf16', hq, hkv, 128, kv_lens, n_qs, left=(left := []))}")
    assert (left[0] != left[1]) == plans                                  # the plan header's first bytes, before and after


# Whole sweeps whose row tiles are jobs of their own, two workgroups a CU: both sides of every line (row tiles, mean rows of a
# stream, key tiles), row tiles of all fillings, streams without rows, frontiers on tile edges.
ROW_TILE_JOBS = [
    # Hq, Hkv, kv_lens, n_qs, row tiles, key tiles, row tiles are jobs
    (32, 4, [300 - i for i in range(64)], [50] * 64, 1056, 5, True), (32, 4, [300 - i for i in range(62)], [50] * 62, 1020, 5, False),
    (32, 4, [3056] + [90] * 63, [50] * 64, 1056, 48, True), (32, 4, [3057] + [90] * 63, [50] * 64, 1056, 49, False),
    (32, 4, [1521] + [90] * 63, [50] * 64, 1056, 25, True), (32, 4, [1521] + [90] * 63, [51] + [50] * 63, 1056, 25, False),
    (28, 4, [1520] + [260] * 23, [200] * 24, 1144, 24, True), (28, 4, [1521] + [260] * 23, [200] * 24, 1144, 25, False),
    (28, 4, [1520] + [260] * 23, [201] + [200] * 23, 1144, 24, False),
    (8, 1, [90] * 360, [64] * 359 + [63], 1799, 2, True), (8, 1, [90] * 360, [64] * 360, 1800, 2, False),
    (8, 8, [321 + i % 70 for i in range(66)], [(0, 1, 31, 33, 127, 128, 129, 160, 255, 257, 321)[i % 11] for i in range(66)], 1064, 7, True),
    (16, 1, [63 + i % 4 for i in range(1100)], [(0, 1, 2, 8, 9, 16, 60)[i % 7] for i in range(1100)], 2984, 2, True),
]


@pytest.mark.parametrize("case", range(len(ROW_TILE_JOBS)))
def test_attention_whose_row_tiles_are_jobs(cs, case):
    hq, hkv, kv_lens, n_qs, row_tiles, key_tiles, jobs = ROW_TILE_JOBS[case]
    assert (sum(n_qs) * (hq // hkv) // 128 + len(n_qs)) * hkv == row_tiles
    assert -(-(-(-max(kv_lens) // 16) + 1) * 16 // 64) == key_tiles
    _plan_is_valid(cs, hq, hkv, kv_lens, n_qs, entries=(entries := []))
    if row_tiles >= 1024:
        assert entries[0][:, :32].all() and entries[0][:, 32:].any() == jobs      # the workgroups that have work
    for mult, outlier in ((1.0, 12.0), (6.0, 0.0)):
        r = _attn_case(cs, np.random.default_rng(9500 + case), "bf16", hq, hkv, 128, kv_lens, n_qs, scale_mult=mult, late_outlier=outlier, last_queries=mult > 1)
        say(f"  -> {r}")


# A BUILD call of whole sweeps below 1,024 row tiles makes the plan in a workgroup of the tile launch.
BUILD_BESIDE = [
    # Hq, Hkv, kv_lens, n_qs
    (16, 4, [700 - 3 * i for i in range(8)], [480] * 8),                                                # 512 row tiles, 32 pairs
    (28, 4, [1100, 900, 1201], [1090, 0, 1200]),                                                        # 12 pairs: ordered by length; a stream without rows
    (16, 1, [700 + 9 * i for i in range(23)], [250 + 3 * i for i in range(23)]),                         # pairs left over by whole rounds
    (8, 1, [520 + i % 40 for i in range(250)], [20 + i % 30 for i in range(250)]),                       # more streams than one turn of the workgroup's scan
    (32, 8, [1040, 1007, 1000], [1000] * 3),
]


@pytest.mark.parametrize("case", range(len(BUILD_BESIDE)))
def test_attention_plan_made_beside_the_first_layer(cs, case):
    """The BUILD call's results, the plan it leaves (that of an ONLY call), and a REUSE call that runs from it."""
    hq, hkv, kv_lens, n_qs = BUILD_BESIDE[case]
    say(f"attention, plan beside the first layer: heads={hq}/{hkv} kv={kv_lens[:4]} n_q={n_qs[:4]} streams={len(kv_lens)}")
    rng, d, n_streams = np.random.default_rng(9480 + case), 128, len(kv_lens)
    nb = [-(-k // 16) for k in kv_lens]
    bt, ids, at = np.zeros((n_streams, max(nb)), np.int32), rng.permutation(sum(nb)), 0
    for s in range(n_streams):
        bt[s, : nb[s]] = ids[at: at + nb[s]]
        at += nb[s]
    cu = np.concatenate([[0], np.cumsum(n_qs)]).astype(np.int32)
    q_pos = np.concatenate([np.sort(rng.choice(kv_lens[s], n_qs[s], replace=False)) for s in range(n_streams)]).astype(np.int32)
    n_q = int(cu[-1])
    assert 512 <= (n_q * (hq // hkv) // 128 + n_streams) * hkv < 1024 and n_q * (hq // hkv) > 128 * n_streams
    to = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    wsb = cs.cs_window_prefill_attn_workspace(n_q, n_streams, hq, hkv, d, max(nb), cs.CS_BF16)
    ws = torch.randint(0, 255, (wsb,), dtype=torch.uint8, device=DEV)
    lists = [to(cu), to(q_pos), to(np.asarray(kv_lens, np.int32)), to(bt)]
    for mode in (cs.CS_ATTN_PLAN_BUILD, cs.CS_ATTN_PLAN_REUSE):
        kc, vc = (_pool(rng, (sum(nb) * 16, hkv, d), "bf16") for _ in range(2))
        q = _pool(rng, (n_q, hq, d), "bf16")
        out = torch.full_like(q, 7.0, device=DEV)
        cs.cs_window_prefill_attn(q.to(DEV), kc.to(DEV), vc.to(DEV), *lists, max(nb), 16, out, n_q, n_streams, hq, hkv, d, hkv * d, d,
                                  1 / math.sqrt(d), cs.CS_BF16, ws, wsb, mode)
        ref = oc.window_attn(hp.f64(q), hp.f64(kc), hp.f64(vc), cu, q_pos, bt, hq, 1 / math.sqrt(d))
        say(f"  -> {hp.check_attention(out.cpu(), ref, 'bf16')}")
        assert cs.cs_attn_status(ws) == 0
    left = ws.clone()
    hdr, items = _attention_plan(cs, cu, q_pos, np.asarray(kv_lens), bt, hq, hkv)
    off = (((PLAN_HDR_INTS + 63) // 64 * 64 + 18 * 64) * 4 + 255) // 256 * 256
    got = left[off: off + items.nbytes].view(torch.int32).cpu().numpy().reshape(items.shape)
    assert np.array_equal(left[:36].view(torch.int32).cpu().numpy(), hdr[:9])
    if n_streams * hkv >= 16:
        assert np.array_equal(got, items)
    else:                                                                 # (equally long items in the order of arrival)
        part = lambda a: sorted(tuple(int(v) for v in (*i[:6], i[7])) for i in a)
        assert part(got) == part(items)


def test_fused_call_of_a_shape_whose_plan_is_made_beside(cs):
    """BUILD, then REUSE: the fused call against the two calls of the same mode, bit for bit, cache contents included."""
    rng, hq, hkv, d, n_streams, n_tok, window = np.random.default_rng(9485), 16, 4, 128, 8, 480, 700
    nb, n_q = -(-window // 16), n_streams * n_tok
    say(f"fused call, plan beside the first layer: heads={hq}/{hkv} streams={n_streams} rows={n_q * (hq // hkv)}")
    to = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    bt = rng.permutation(n_streams * nb).astype(np.int32).reshape(n_streams, nb)
    pos = np.stack([np.sort(rng.choice(window, n_tok, replace=False)) for _ in range(n_streams)])
    slot = to((np.take_along_axis(bt, pos // 16, 1) * 16 + pos % 16).astype(np.int32).reshape(-1))
    lists = [to((np.arange(n_streams + 1) * n_tok).astype(np.int32)), to(pos.astype(np.int32).reshape(-1)),
             to(np.full(n_streams, window, np.int32)), to(bt)]
    wsb = cs.cs_window_prefill_attn_workspace(n_q, n_streams, hq, hkv, d, nb, cs.CS_BF16)
    ws = [torch.randint(0, 255, (wsb,), dtype=torch.uint8, device=DEV) for _ in range(2)]
    for mode in (cs.CS_ATTN_PLAN_BUILD, cs.CS_ATTN_PLAN_REUSE):
        pool = [_pool(rng, (n_streams * nb * 16, hkv, d), "bf16").to(DEV) for _ in range(2)]
        new = [_pool(rng, (n_q, hkv, d), "bf16").to(DEV) for _ in range(2)]
        q = _pool(rng, (n_q, hq, d), "bf16").to(DEV)
        tail = lambda out, w: (*lists, nb, 16, out, n_q, n_streams, hq, hkv, d, hkv * d, d, 1 / math.sqrt(d), cs.CS_BF16, w, wsb, mode)
        k1, v1, k2, v2 = (t.clone() for t in pool + pool)
        out1, out2 = torch.zeros_like(q), torch.ones_like(q)
        cs.cs_refresh_prefill_attn(*new, slot, n_q, q, k1, v1, *tail(out1, ws[0]))
        cs.cs_kv_refresh_scatter(*new, slot, k2, v2, n_q, hkv, d, hkv * d, d, cs.CS_BF16)
        cs.cs_window_prefill_attn(q, k2, v2, *tail(out2, ws[1]))
        for a, b in ((k1, k2), (v1, v2), (out1, out2)):
            assert torch.equal(a.view(torch.int16), b.view(torch.int16))
        assert cs.cs_attn_status(ws[0]) == 0


def test_attention_plan_of_more_streams_than_are_searched_in_lds(cs):
    _plan_is_valid(cs, 2, 1, [20] * 4100, [2 + i % 3 for i in range(4100)])


# Many streams of at most one row tile: the search for a workgroup's row tile in one, two and three steps (64 streams; 64 for
# each thread of the workgroup), streams without rows at either end, and both sides of 128 rows a stream.
MANY_STREAMS = [
    # dtype, Hq, Hkv, d, streams, n_qs (repeated), window
    ("bf16", 32, 16, 128, 64, [64], 130), ("bf16", 32, 16, 128, 65, [0, 64, 128, 64], 130), ("bf16", 32, 16, 128, 65, [65, 64], 130),
    ("bf16", 20, 4, 128, 257, [0, 3, 25, 1], 90), ("bf16", 8, 1, 128, 1100, [16, 1, 0, 5], 40), ("bf16", 1, 1, 128, 16385, [0, 1, 2], 20),
    ("bf16", 2, 1, 64, 257, [0, 3, 90, 1], 90), ("bf16", 1, 1, 64, 32770, [0, 1], 17), ("f32", 2, 1, 64, 513, [0, 3, 20, 1], 40),
]


# Few row tiles with long sweeps: in pieces, each a workgroup.  Both sides of every line (pieces of a sweep, by the 64-row tiles;
# key tiles), rows at the edges of row tiles, streams that are shorter than others or have no rows.
FEW_ROW_TILES = [
    # Hq, Hkv, kv_lens, n_qs
    (28, 4, [750, 40], [17, 1]), (28, 4, [752, 40], [17, 1]), (28, 4, [753, 40], [17, 1]),               # 12 and 13 key tiles
    (28, 4, [5300, 1], [69, 1]), (16, 1, [1472, 64], [69, 1]), (8, 1, [17000], [8]), (8, 1, [17000], [9]),       # 64 and 72 rows
    (32, 4, [1900 - 60 * i for i in range(6)], [16, 0, 8, 17, 9, 0]),                                    # streams without rows, one to three row tiles
    (16, 16, [3000, 2990, 100, 3010], [64, 65, 64, 33]),                                                 # one head a group, two pieces
    (16, 16, [1230], [1]), (16, 1, [1100], [1]), (16, 1, [65, 15000], [3, 4]),
    (4, 1, [900 + 7 * i for i in range(66)], [1 + i % 16 for i in range(66)]),                           # more streams than a wave has lanes, three pieces
    (4, 1, [1300 + 7 * i for i in range(100)], [1 + i % 16 for i in range(100)]),                        # two
    (4, 1, [1300 + 7 * i for i in range(103)], [1 + i % 16 for i in range(103)]),                        # one
    (4, 1, [3100 + 9 * i for i in range(150)], [1 + i % 16 for i in range(150)]),                        # whole sweeps of up to 64 rows
    (16, 16, [5104, 300, 110], [100, 100, 100]),                                                         # two pieces, 80 key tiles
    (2, 1, [1700] * 100, [3] * 99 + [700]),                                                              # unlike streams: more row tiles than the rule counts
]


@pytest.mark.parametrize("case", range(len(FEW_ROW_TILES)))
def test_attention_of_few_row_tiles(cs, case):
    hq, hkv, kv_lens, n_qs = FEW_ROW_TILES[case]
    say(f"attention of few row tiles {case}: heads={hq}/{hkv} kv={kv_lens[:6]} n_q={n_qs[:6]} streams={len(kv_lens)}")
    for mult, last in ((1.0, False), (6.0, True)):
        r = _attn_case(cs, np.random.default_rng(9490 + case), "bf16", hq, hkv, 128, kv_lens, n_qs, scale_mult=mult, last_queries=last, left=(left := []))
        say(f"  -> {r}")
        assert left[0] == left[1]                                         # no plan


@pytest.mark.parametrize("case", range(len(MANY_STREAMS)))
def test_attention_of_many_streams(cs, case):
    dtype, hq, hkv, d, n_streams, n_qs, window = MANY_STREAMS[case]
    say(f"attention of many streams {case}: {dtype} heads={hq}/{hkv} d={d} streams={n_streams}")
    n_qs = [n_qs[i % len(n_qs)] for i in range(n_streams)]
    kv_lens = [max(n_qs[s], window - s % 13) for s in range(n_streams)]
    say(f"  -> {_attn_case(cs, np.random.default_rng(9470 + case), dtype, hq, hkv, d, kv_lens, n_qs)}")


# A key that is not finite, with finite values: on the routes of bf16 attention.  The early queries end in the half tile of
# keys 96-127, the late ones in the window's last 80 keys; 64 rows of a wave hold some of both.
NOT_FINITE = [
    # Hq, Hkv, d, streams, window
    (16, 8, 128, 64, 400),       # from a plan, whole sweeps, a row tile a job
    (64, 8, 128, 44, 400),       # from a plan, whole sweeps
    (16, 8, 128, 2, 4300),       # no plan, sweeps in pieces
    (16, 8, 128, 6, 7300),       # from a plan, split sweeps
    (16, 8, 128, 8, 400),        # no plan
    (8, 4, 64, 3, 400),
]


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), float("-inf")])
@pytest.mark.parametrize("case", range(len(NOT_FINITE)))
def test_bf16_attention_key_that_is_not_finite(cs, case, bad):
    """A key that is not finite reaches the queries that see it and no other: not those of an earlier frame in the same
    wave (keys 127, 200 and 250), nor those just before it (the window's end)."""
    hq, hkv, d, n_streams, window = NOT_FINITE[case]
    rng = np.random.default_rng(9450 + case)
    q_pos1 = np.concatenate([np.arange(100, 120), np.arange(window - 80, window)]).astype(np.int32)
    n_tok, nb = q_pos1.size, -(-window // 16)
    bt = rng.permutation(n_streams * nb).astype(np.int32).reshape(n_streams, nb)
    cu = (np.arange(n_streams + 1) * n_tok).astype(np.int32)
    q_pos = np.tile(q_pos1, n_streams)
    kc, vc = (_pool(rng, (n_streams * nb * 16, hkv, d), "bf16") for _ in range(2))
    q = _pool(rng, (cu[-1], hq, d), "bf16")
    ref = oc.window_attn(hp.f64(q), hp.f64(kc), hp.f64(vc), cu, q_pos, bt, hq, 1 / math.sqrt(d))
    to = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    wsb = cs.cs_window_prefill_attn_workspace(int(cu[-1]), n_streams, hq, hkv, d, nb, cs.CS_BF16)
    for at in (127, 200, 250, window - 41):
        say(f"bf16 attention, key {at} of {window} is {bad}: heads={hq}/{hkv} d={d} streams={n_streams}")
        k_bad = kc.clone()
        k_bad[bt[:, at // 16].astype(np.int64) * 16 + at % 16, :, 0] = bad
        out = torch.zeros_like(q, device=DEV)
        ws = torch.zeros((max(16, wsb),), dtype=torch.uint8, device=DEV)
        cs.cs_window_prefill_attn(q.to(DEV), k_bad.to(DEV), vc.to(DEV), to(cu), to(q_pos), to(np.full(n_streams, window, np.int32)),
                                  to(bt), nb, 16, out, int(cu[-1]), n_streams, hq, hkv, d, hkv * d, d, 1 / math.sqrt(d),
                                  cs.CS_BF16, ws, wsb)
        got, before = out.cpu(), q_pos < at
        hp.check_attention(got[before], ref[before], "bf16")
        if math.isnan(bad):
            assert not torch.isfinite(got[~before].float()).any()


@pytest.mark.parametrize("dtype,hq,hkv,d,kv_lens,n_qs", [
    ("bf16", 14, 2, 128, [300, 77], [40, 77]), ("bf16", 28, 4, 128, [1100], [300]), ("bf16", 8, 2, 64, [300, 77], [40, 77]),
    ("bf16", 28, 4, 128, [900, 700, 800, 640], [380, 500, 250, 400]), ("f32", 8, 2, 128, [300, 77], [40, 77])])
def test_unplanned_attention_head_major_pool_and_row_capacity(cs, dtype, hq, hkv, d, kv_lens, n_qs):
    """A head-major pool (slot stride d, head stride slots * d) and n_q beyond the rows the streams hold: rows past
    cu_q stay as they were."""
    say(f"unplanned attention, head-major pool: {dtype} heads={hq}/{hkv} d={d} kv={kv_lens}")
    rng = np.random.default_rng(9400 + d)
    n_streams, extra = len(kv_lens), 37
    nb = [-(-k // 16) for k in kv_lens]
    bt, ids, at = np.zeros((n_streams, max(nb)), np.int32), rng.permutation(sum(nb)), 0
    for s in range(n_streams):
        bt[s, : nb[s]] = ids[at: at + nb[s]]
        at += nb[s]
    slots = sum(nb) * 16
    kc, vc = _pool(rng, (slots, hkv, d), dtype), _pool(rng, (slots, hkv, d), dtype)
    cu = np.concatenate([[0], np.cumsum(n_qs)]).astype(np.int32)
    q_pos = np.concatenate([np.sort(rng.choice(kv_lens[s], n_qs[s], replace=False)) for s in range(n_streams)]).astype(np.int32)
    n_q = int(cu[-1])
    q = _pool(rng, (n_q + extra, hq, d), dtype)
    ref = oc.window_attn(hp.f64(q[:n_q]), hp.f64(kc), hp.f64(vc), cu, q_pos, bt, hq, 1 / math.sqrt(d))
    head_major = lambda t: t.permute(1, 0, 2).contiguous().to(DEV)
    to = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    kd, vd = head_major(kc), head_major(vc)
    out = torch.full((n_q + extra, hq, d), 7.0, dtype=q.dtype, device=DEV)
    code = cs.CS_BF16 if dtype == "bf16" else cs.CS_F32
    wsb = cs.cs_window_prefill_attn_workspace(n_q + extra, n_streams, hq, hkv, d, max(nb), code)
    ws = torch.randint(0, 255, (max(16, wsb),), dtype=torch.uint8, device=DEV)
    pos = to(np.concatenate([q_pos, np.full(extra, 2 ** 30, np.int32)]))
    cs.cs_window_prefill_attn(q.to(DEV), kd, vd, to(cu), pos, to(np.asarray(kv_lens, np.int32)), to(bt), max(nb), 16, out,
                              n_q + extra, n_streams, hq, hkv, d, d, slots * d, 1 / math.sqrt(d), code, ws, wsb)
    got = out.cpu()
    hp.check_attention(got[:n_q], ref, dtype)
    assert torch.all(got[n_q:] == 7.0)
    if wsb:
        assert cs.cs_attn_status(ws) == 0


@pytest.mark.parametrize("capacity", [130, 8200])                       # two key groups; one
@pytest.mark.parametrize("stride_slot", [2 ** 26 - 8, 2 ** 26])         # 32-bit byte offsets inside a block; 64-bit addresses
def test_head_dim_64_attention_of_far_apart_slots(cs, stride_slot, capacity):
    """A pool whose slots are 2^26 elements apart (K and V of all slots in one 18-GiB allocation)."""
    say(f"head_dim 64 attention, slot stride {stride_slot}, room for {capacity} tokens")
    rng = np.random.default_rng(9700)
    hq, hkv, d, kv_len, n_q = 16, 1, 64, 137, 130
    bt = rng.permutation(9)[None].astype(np.int32)
    q, kc, vc = _pool(rng, (capacity, hq, d), "bf16"), _pool(rng, (144, hkv, d), "bf16"), _pool(rng, (144, hkv, d), "bf16")
    q_pos = np.sort(rng.choice(kv_len, n_q, replace=False)).astype(np.int32)
    ref = oc.window_attn(hp.f64(q[:n_q]), hp.f64(kc), hp.f64(vc), np.array([0, n_q]), q_pos, bt, hq, 1 / math.sqrt(d))
    pool = torch.empty((143 * stride_slot + 2 * hkv * d,), dtype=torch.bfloat16, device=DEV)
    kd, vd = (pool[at:].as_strided((144, hkv, d), (stride_slot, d, 1)) for at in (0, hkv * d))
    kd.copy_(kc)
    vd.copy_(vc)
    out = torch.full((capacity, hq, d), 7.0, dtype=torch.bfloat16, device=DEV)
    i32 = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.int32)).to(DEV)
    pos = i32(np.concatenate([q_pos, np.zeros(capacity - n_q, np.int32)]))
    cs.cs_window_prefill_attn(q.to(DEV), kd, vd, i32([0, n_q]), pos, i32([kv_len]), i32(bt), 9, 16, out, capacity, 1, hq, hkv, d,
                              stride_slot, d, 1 / math.sqrt(d), cs.CS_BF16)
    got = out.cpu()
    hp.check_attention(got[:n_q], ref, "bf16")
    assert torch.all(got[n_q:] == 7.0)


# residual proxy: workgroups of whole patches with their rows in 1, 2 or 4 parts, and patches too large for that
RESIDUAL_RUNS = [
    # frames, h, w, cell, in_w, in_h, patch, gh, gw, pad
    (2, 64, 640, 4, 640, 64, 31, 2, 20, 0),            # 31 rows per patch: one part
    (2, 200, 636, 4, 448, 112, 28, 4, 16, 16),         # 50 rows: two parts; patch borders inside 4-pixel groups
    (1, 303, 500, 8, 140, 84, 28, 3, 5, 0),            # 101 rows: four parts
    (1, 128, 1030, 16, 1030, 128, 127, 1, 8, 0),       # the last patch cut off, 128 rows with the rounding
    (1, 290, 520, 4, 56, 28, 28, 1, 2, 0),             # 290 rows per patch: rows split among workgroups
    (1, 40, 1600, 4, 80, 40, 40, 1, 2, 0),             # 800 pixels wide
    (2, 48, 96, 4, 48, 24, 8, 5, 7, 0),                # patches past the frame: no pixel, score 0
    (2, 270, 500, 16, 140, 112, 28, 4, 5, 16),         # four parts that begin and end inside a cell row
    (49, 48, 1540, 4, 154, 128, 8, 16, 20, 0),         # 784 patch rows of 385 groups: a workgroup of 512 lanes per row
    (26, 45, 3100, 8, 160, 120, 8, 15, 20, 16),        # two runs of 10 patches per row, 780 workgroups
    (47, 48, 1540, 16, 154, 128, 8, 16, 20, 0),        # 752 patch rows: short runs
]


@pytest.mark.parametrize("case", range(len(RESIDUAL_RUNS)))
def test_residual_proxy_work_splits(cs, case):
    from oracle import residual_oracle as ro
    f, h, w, cell, in_w, in_h, patch, gh, gw, pad = RESIDUAL_RUNS[case]
    say(f"residual_proxy split {case}: {f} frames {w}x{h} cell {cell} -> grid {gh}x{gw}")
    rng = np.random.default_rng(9500 + case)
    cur, prev = (rng.integers(0, 256, size=(f, h, w), dtype=np.uint8) for _ in range(2))
    field = rng.integers(-60, 61, size=(f, -(-h // cell), -(-w // cell), 2)).astype(np.int16)
    field[:, ::3, ::5] *= 40                                        # some references leave the frame on every side
    want = ro.residual_proxy(cur, prev, field, cell, in_w, in_h, patch, gh, gw)
    assert np.array_equal(_residual_gpu(cs, cur, prev, field, cell, in_w, in_h, patch, gh, gw, pad), want)


@pytest.mark.parametrize("geom,counts", [
    ((640, 360, 448, 448, 28, 16, 16), [300] * 3),                  # few blocks and patches: one band
    ((640, 360, 1288, 728, 28, 26, 46), [700]),                     # eight bands of three or four
    ((640, 360, 448, 140, 28, 5, 16), [200, 0, 90]),
    ((640, 360, 448, 448, 28, 16, 16), [9] * 130),
    ((64, 48, 32, 24, 8, 3, 4), [5] * 520),                         # one band
    ((1280, 720, 448, 448, 28, 16, 16), [2000] * 2),                # 3,600 macroblocks: eight bands of two patch rows
    ((1280, 720, 448, 140, 28, 5, 16), [200, 0, 90]),               # as many bands as patch rows
    ((1280, 720, 448, 448, 28, 16, 16), [9] * 80),                  # three bands, five or six patch rows each
    ((1280, 720, 448, 448, 28, 16, 16), [9] * 128),                 # two bands
    ((1280, 720, 448, 448, 28, 16, 16), [9] * 129),                 # one band
])
def test_project_blocks_bands(cs, geom, counts):
    from oracle import projection_oracle as po
    say(f"project_blocks bands: geometry {geom}, {len(counts)} frames")
    blocks, cu = _random_block_frames(np.random.default_rng(9600 + len(counts)), counts, geom[0], geom[1], 64, 40)
    mv_w, intra_w = po.project_blocks(blocks, cu, *geom)
    mv_g, intra_g = _project_gpu(cs, blocks, cu, geom)
    assert np.array_equal(mv_g, mv_w) and np.array_equal(intra_g, intra_w)


@pytest.mark.parametrize("hq,hkv,kv_lens,n_qs", [
    (28, 4, [2300, 1900, 2100, 900, 2200], [900, 1000, 800, 300, 1100]),        # 20 pairs, below 1,024 row tiles: split sweeps
    (16, 1, [700 + 9 * i for i in range(23)], [480 + 3 * i for i in range(23)]),  # 23 pairs
    (8, 8, [900, 40, 1000], [6000, 0, 7000]),                                   # 24 pairs, a third of them empty, split sweeps
])
def test_attention_plan_pairs_left_over_by_whole_rounds(cs, hq, hkv, kv_lens, n_qs):
    kv_lens = [max(k, n) for k, n in zip(kv_lens, n_qs)]
    _plan_is_valid(cs, hq, hkv, kv_lens, n_qs)


@pytest.mark.parametrize("hq,hkv,kv_lens,n_qs", [
    (28, 4, [2300, 1900, 2100, 900, 2200], [1200, 1300, 1100, 600, 1500]),      # 20 pairs: two whole rounds of the XCDs, four left over
    (16, 1, [700 + 9 * i for i in range(23)], [480 + 3 * i for i in range(23)]),  # 23 pairs
    (12, 3, [2000 + 90 * i for i in range(7)], [1500, 1700, 1900, 2000, 1800, 1990, 0]),  # 21 pairs, three of those left over empty
    (16, 1, [300] * 2052, [20 + i % 9 for i in range(2052)]),                   # more streams than are sorted by work
])
def test_attention_plan_deals_the_left_over_pairs_in_order(cs, hq, hkv, kv_lens, n_qs):
    """The row tiles of the pairs beyond the last whole round of eight: on all XCDs in like numbers, behind the whole
    pairs, those nearest their stream's end first, and the same plan from one call to the next."""
    group, n_pairs = hq // hkv, len(kv_lens) * hkv
    say(f"attention plan, {n_pairs % 8} of {n_pairs} pairs left over")
    assert (sum(n_qs) * group // 128 + len(kv_lens)) * hkv >= 1024              # whole sweeps, not split ones
    _plan_is_valid(cs, hq, hkv, kv_lens, n_qs)
    cu = np.concatenate([[0], np.cumsum(n_qs)])
    q_pos = np.concatenate([np.arange(k - n, k) for k, n in zip(kv_lens, n_qs)])
    bt = np.arange(len(kv_lens) * (max(kv_lens) // 16 + 1)).reshape(len(kv_lens), -1)
    hdr, items = _attention_plan(cs, cu, q_pos, np.asarray(kv_lens), bt, hq, hkv)
    again = _attention_plan(cs, cu, q_pos, np.asarray(kv_lens), bt, hq, hkv)
    assert np.array_equal(hdr[:9], again[0][:9]) and np.array_equal(items, again[1])
    tiles = [-(-n * group // 128) for n in n_qs]
    work = [sum(int(q_pos[cu[s] + (min((t + 1) * 128, n_qs[s] * group) - 1) // group]) // 64 + 1 for t in range(tiles[s]))
            for s in range(len(kv_lens))]
    rank = np.argsort(np.argsort([-w for w in work], kind="stable"), kind="stable")
    if len(kv_lens) > 2048:
        rank = np.arange(len(kv_lens))
    counts = []
    for x in range(8):
        part = items[hdr[x]: hdr[x + 1]]
        stream, kvh = part[:, 3] >> 8, part[:, 3] & 255
        left = rank[stream] * hkv + kvh >= n_pairs // 8 * 8
        level = np.asarray(tiles)[stream] - 1 - part[:, 2] // 128
        assert not np.any(left[:-1] & ~left[1:]) and np.all(np.diff(level[left]) >= 0)
        counts.append(int(left.sum()))
    assert max(counts) - min(counts) <= n_pairs % 8                             # each pair's are shared evenly
