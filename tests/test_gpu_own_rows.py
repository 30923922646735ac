"""cs_refresh_prefill_attn with CS_ATTN_OWN_ROWS against the refresh write followed by attention: caches and results bit
for bit, on every route such a call can take (results where it takes another kernel than the separate call: against the oracle).  The slots of the new rows hold no number before the call, so a key read
from the cache in place of the caller's rows shows."""
import math

import numpy as np
import pytest
import torch

from oracle import codecsight_oracle as oc
from tests import helpers as hp
from tests.test_gpu_parity import DEV, _pool, cs, say   # noqa: F401  (cs is a fixture)

pytestmark = pytest.mark.gpu

CASES = [
    # Hq, Hkv, d, kv_lens, n_qs, pattern of the query positions
    (28, 4, 128, [915], [425], "runs"),                        # 64-row tiles, four key groups
    (28, 4, 128, [917], [425], "any"),
    (16, 8, 128, [300], [130], "runs"),                        # two key groups
    (28, 4, 128, [915, 1, 640, 77], [425, 1, 333, 0], "runs"),
    (28, 4, 128, [1000 + 7 * i for i in range(6)], [421 + i for i in range(6)], "runs"),      # plan, made beside the first layer
    (8, 2, 128, [3000, 700, 40], [257, 64, 40], "runs"),       # sweeps in pieces
    (28, 4, 128, [13700], [18], "any"),
    (32, 8, 128, [200 + i for i in range(66)], [31] * 66, "any"),       # one row tile of 128 a stream, more streams than lanes
    (32, 8, 128, [200 + i for i in range(66)], [64] * 66, "runs"),      # row tiles are jobs
    (28, 4, 128, [6033], [300], "runs"),                       # split sweeps and merge
    (28, 4, 128, [1100 + 13 * i for i in range(32)], [380 + 5 * i for i in range(32)], "runs"),      # whole sweeps
    (4, 4, 64, [200, 129, 16, 17, 15], [64, 129, 16, 1, 14], "any"),    # head_dim 64, few row tiles
    (16, 4, 64, [900 + 11 * i for i in range(12)], [370 + i for i in range(12)], "runs"),
    (16, 4, 64, [300 + 11 * i for i in range(40)], [250 + i % 7 for i in range(40)], "runs"),      # many
    (8, 1, 64, [70] * 130, [3] * 130, "any"),
    # other lines with own rows: 64-row tiles of longer sweeps up to 510 row tiles of 128, those up to 850, plan from there
    (28, 4, 128, [1500 + 7 * i for i in range(5)], [421 + i for i in range(5)], "runs"),
    (28, 4, 128, [1220 - 9 * i for i in range(5)], [420 - i for i in range(5)], "any"),
    (28, 4, 128, [1190 - 9 * i for i in range(5)], [420 - i for i in range(5)], "any"),
    (28, 4, 128, [900 + 7 * i for i in range(5)], [421 + i for i in range(5)], "runs"),
    (16, 4, 128, [1000 + 7 * i for i in range(9)], [440] * 8 + [436], "runs"),
    (16, 4, 128, [1000 + 7 * i for i in range(9)], [440] * 8 + [437 + 19], "any"),
    (28, 4, 128, [1100 - 50 * i for i in range(7)], [421 + i for i in range(7)], "any"),
    (8, 1, 128, [700 + i for i in range(33)], [395] * 33, "runs"),
    (8, 1, 128, [700 + i for i in range(33)], [397] * 33, "runs"),
    # row tiles by length: 300 (by stream), 301, the most streams of a list by length with some that have no rows, one more
    (8, 1, 64, [400] * 15, [320] * 15, "runs"),
    (8, 1, 64, [400] * 15, [321] + [320] * 14, "runs"),
    (16, 4, 64, [100 + 7 * i for i in range(64)], [33 if i % 9 else 0 for i in range(64)], "any"),
    (16, 4, 64, [100 + 7 * i for i in range(65)], [33 if i % 9 else 0 for i in range(65)], "any"),
    # ... one stream, two, streams whose tiles take several rounds of numbers to rank, of alike and of unlike streams
    (16, 1, 64, [2600], [2500], "runs"),
    (16, 1, 64, [1500, 1400], [1250, 1300], "any"),
    (16, 1, 64, [2600] + [40 + i for i in range(39)], [2500] + [i for i in range(39)], "runs"),
    (16, 2, 64, [340 + i for i in range(33)], [330 + i % 5 for i in range(33)], "runs"),
    # workgroups that bring keys into L2: three kv heads, two, more streams than such workgroups, windows that end in the first trip
    (12, 3, 128, [1100, 290, 333], [400, 133, 50], "any"),
    (16, 2, 128, [1030], [500], "runs"),
    (8, 1, 128, [900, 640, 500, 820, 930, 257], [200] * 6, "runs"),
    (28, 4, 128, [256], [256], "any"),
    (4, 1, 64, [129, 500], [100, 41], "any"),
    # long sweeps over many row tiles (by the longest window): as without the flag; just below the line
    (1, 1, 128, [6033] + [20 + i % 40 for i in range(1099)], [7] + [1 + i % 2 for i in range(1099)], "any"),
    (1, 1, 128, [5600] + [20 + i % 40 for i in range(1099)], [7] + [1 + i % 2 for i in range(1099)], "any"),
    (1, 1, 64, [16800] + [20 + i % 40 for i in range(1999)], [7] + [1] * 1999, "any"),
    (1, 1, 64, [16300] + [20 + i % 40 for i in range(1999)], [7] + [1] * 1999, "any"),
]


def _positions(rng, kv_len, n_q, pattern):
    """Strictly increasing window positions: a few runs, the last one up to the end of the window, or any."""
    if pattern == "any" or n_q < 8:
        return np.sort(rng.choice(kv_len, size=n_q, replace=False))
    first = n_q // 2
    start = int(rng.integers(0, kv_len - n_q + 1))
    return np.concatenate([np.arange(start, start + first), np.arange(kv_len - (n_q - first), kv_len)])


@pytest.mark.parametrize("case", range(len(CASES)))
def test_own_rows_equal_refresh_write_then_attention(cs, case):
    hq, hkv, d, kv_lens, n_qs, pattern = CASES[case]
    say(f"own rows case {case}: heads={hq}/{hkv} d={d} kv={kv_lens[:6]} n_q={n_qs[:6]} {pattern}")
    rng = np.random.default_rng(8200 + case)
    n_streams = len(kv_lens)
    nb = [-(-n // 16) for n in kv_lens]
    max_blocks = max(nb) + 1
    ids = rng.permutation(sum(nb) + 3)
    bt = np.full((n_streams, max_blocks), -5, np.int32)          # (entries past a stream's last: never looked at)
    at = 0
    for s in range(n_streams):
        bt[s, : nb[s]] = ids[at: at + nb[s]]
        at += nb[s]
    pos = [_positions(rng, kv_lens[s], n_qs[s], pattern) for s in range(n_streams)]
    cu = np.concatenate([[0], np.cumsum([p.size for p in pos])]).astype(np.int32)
    q_pos = np.concatenate(pos).astype(np.int32)
    slot = np.concatenate([bt[s, pos[s] // 16].astype(np.int64) * 16 + pos[s] % 16 for s in range(n_streams)]).astype(np.int32)
    n_q, pad = int(q_pos.size), 37
    n_all = n_q + pad
    dev = lambda a: torch.from_numpy(a).to(DEV)
    slot_p = dev(np.concatenate([slot, np.full(pad, -1, np.int32)]))
    meta = (dev(cu), dev(np.concatenate([q_pos, np.full(pad, 7, np.int32)])), torch.tensor(kv_lens, dtype=torch.int32, device=DEV), dev(bt))
    scale = 1.0 / math.sqrt(d)
    plain_bytes = cs.cs_window_prefill_attn_workspace(n_all, n_streams, hq, hkv, d, max_blocks, cs.CS_BF16)
    own_bytes = cs.cs_refresh_prefill_attn_workspace(n_all, n_streams, hq, hkv, d, max_blocks, cs.CS_BF16)
    dirty = lambda n: torch.randint(0, 255, (max(64, n),), dtype=torch.uint8, device=DEV)
    ws, ws_only, ws_two = dirty(own_bytes), dirty(own_bytes), dirty(plain_bytes)
    n_slots = ids.size * 16
    build, reuse, only = cs.CS_ATTN_PLAN_BUILD, cs.CS_ATTN_PLAN_REUSE, cs.CS_ATTN_PLAN_ONLY

    def rest(workspace, n_bytes, mode):
        return (n_all, n_streams, hq, hkv, d, hkv * d, d, scale, cs.CS_BF16, workspace, n_bytes, mode)

    def own(data, workspace, mode, out, k, v):
        kn, vn, q = data
        cs.cs_refresh_prefill_attn(kn, vn, slot_p, n_all, q, k, v, *meta, max_blocks, 16, out,
                                   *rest(workspace, own_bytes, mode | cs.CS_ATTN_OWN_ROWS))

    for rep, (workspace, mode) in enumerate(((ws, build), (ws, reuse), (ws, reuse), (ws_only, only), (ws_only, reuse))):
        if mode == only and d == 128:
            own((None, None, None), workspace, only, None, None, None)
            continue
        kc, vc = _pool(rng, (n_slots, hkv, d), "bf16"), _pool(rng, (n_slots, hkv, d), "bf16")
        kc[slot] = vc[slot] = float("nan")
        data = [t.to(DEV) for t in (_pool(rng, (n_all, hkv, d), "bf16"), _pool(rng, (n_all, hkv, d), "bf16"), _pool(rng, (n_all, hq, d), "bf16"))]
        k2, v2, k1, v1 = kc.to(DEV), vc.to(DEV), kc.to(DEV), vc.to(DEV)
        out2 = torch.full((n_all, hq, d), 7.0, dtype=torch.bfloat16, device=DEV)
        out1 = out2.clone()
        cs.cs_kv_refresh_scatter(data[0], data[1], slot_p, k2, v2, n_all, hkv, d, hkv * d, d, cs.CS_BF16)
        if rep == 4 and d == 128:
            cs.cs_window_prefill_attn(None, None, None, *meta, max_blocks, 16, None, *rest(ws_two, plain_bytes, only))
        cs.cs_window_prefill_attn(data[2], k2, v2, *meta, max_blocks, 16, out2, *rest(ws_two if plain_bytes else None, plain_bytes, mode))
        own(data, workspace, mode, out1, k1, v1)
        torch.cuda.synchronize()
        raw = torch.int16
        assert torch.equal(k1.view(raw), k2.view(raw)) and torch.equal(v1.view(raw), v2.view(raw)), f"cache, pass {rep}"
        row_tiles, key_tiles = hkv * (n_all * hq // hkv // 128 + n_streams), -(-max_blocks // 4)
        other_kernel = mode == reuse and d == 128 and n_streams <= 64 and (
            (440 < row_tiles <= 510 and 20 <= key_tiles <= 48) or ((768 if hkv > 4 else 512) <= row_tiles <= 850 and 8 < key_tiles <= 32))
        assert other_kernel or torch.equal(out1.view(raw), out2.view(raw)), f"results, pass {rep}"
        assert torch.all(out1[n_q:].float() == 7.0)
        if rep == 1 or other_kernel:
            ref = oc.window_attn(hp.f64(data[2][:n_q]), hp.f64(k2), hp.f64(v2), cu, q_pos, bt, hq, scale)
            say(f"  {hp.check_attention(out1[:n_q].cpu(), ref, 'bf16')}")


def test_own_rows_of_a_cache_in_another_layout(cs):
    """Slots further apart than a row: the flag changes nothing."""
    hq, hkv, d, kv_len, n_q = 28, 4, 128, 640, 200
    say(f"own rows: cache rows with a gap, heads={hq}/{hkv} kv={kv_len} n_q={n_q}")
    rng = np.random.default_rng(8301)
    pos = _positions(rng, kv_len, n_q, "runs")
    bt = rng.permutation(40).astype(np.int32)[None]
    slot = (bt[0, pos // 16].astype(np.int64) * 16 + pos % 16).astype(np.int32)
    dev = lambda a: torch.from_numpy(a).to(DEV)
    meta = (dev(np.array([0, n_q], np.int32)), dev(pos.astype(np.int32)), dev(np.array([kv_len], np.int32)), dev(bt))
    size = cs.cs_refresh_prefill_attn_workspace(n_q, 1, hq, hkv, d, 40, cs.CS_BF16)
    kn, vn, q = (_pool(rng, (n_q, h, d), "bf16").to(DEV) for h in (hkv, hkv, hq))
    pools = [_pool(rng, (640, hkv + 1, d), "bf16").to(DEV) for _ in range(2)]
    results = []
    for flag in (0, cs.CS_ATTN_OWN_ROWS):
        k, v = (t.clone() for t in pools)
        ws = torch.zeros(size, dtype=torch.uint8, device=DEV)
        out = torch.zeros((n_q, hq, d), dtype=torch.bfloat16, device=DEV)
        for mode in (cs.CS_ATTN_PLAN_BUILD, cs.CS_ATTN_PLAN_REUSE):
            cs.cs_refresh_prefill_attn(kn, vn, dev(slot), n_q, q, k, v, *meta, 40, 16, out, n_q, 1, hq, hkv, d, k.stride(0), k.stride(1),
                                       1.0 / math.sqrt(d), cs.CS_BF16, ws, size, mode | flag)
        results.append((k, v, out))
    torch.cuda.synchronize()
    for a, b in zip(*results):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))


@pytest.mark.parametrize("hq, hkv, d, n_streams", [(28, 4, 128, 1), (16, 4, 64, 1), (28, 4, 128, 5)])
def test_own_rows_past_a_block_table_row(cs, hq, hkv, d, n_streams):
    """Rows that the block-table row has no slot for (slot -1, position pulled back to the row's last, as cs_plan_refresh leaves
    them) do not stand in for that position's key: it is a reused row's, in the cache, or an earlier row's."""
    room, n_own = 640, 300
    say(f"own rows: rows past the block table, heads={hq}/{hkv} d={d} streams={n_streams}")
    rng = np.random.default_rng(8302)
    bt = rng.permutation(40 * n_streams).astype(np.int32).reshape(n_streams, 40)
    pos, slot = [], []
    for s in range(n_streams):
        p = np.sort(rng.choice(room - 1, size=n_own, replace=False))
        if s % 2:
            p[-1] = room - 1                                     # executed itself
        n_past = 21 + s
        pos += [p, np.full(n_past, room - 1)]
        slot += [bt[s, p // 16].astype(np.int64) * 16 + p % 16, np.full(n_past, -1)]
    cu = np.concatenate([[0], np.cumsum([a.size for a in pos])[1::2]]).astype(np.int32)
    n_q = int(cu[-1])
    dev = lambda a: torch.from_numpy(a).to(DEV)
    slot = dev(np.concatenate(slot).astype(np.int32))
    meta = (dev(cu), dev(np.concatenate(pos).astype(np.int32)), torch.full((n_streams,), room + 21, dtype=torch.int32, device=DEV), dev(bt))
    size = cs.cs_refresh_prefill_attn_workspace(n_q, n_streams, hq, hkv, d, 40, cs.CS_BF16)
    kn, vn, q = (_pool(rng, (n_q, h, d), "bf16").to(DEV) for h in (hkv, hkv, hq))
    pools = [_pool(rng, (640 * n_streams, hkv, d), "bf16").to(DEV) for _ in range(2)]
    results = []
    for flag in (0, cs.CS_ATTN_OWN_ROWS):
        ws = torch.zeros(size, dtype=torch.uint8, device=DEV)
        for mode in (cs.CS_ATTN_PLAN_BUILD, cs.CS_ATTN_PLAN_REUSE):
            k, v = (t.clone() for t in pools)
            out = torch.zeros((n_q, hq, d), dtype=torch.bfloat16, device=DEV)
            cs.cs_refresh_prefill_attn(kn, vn, slot, n_q, q, k, v, *meta, 40, 16, out, n_q, n_streams, hq, hkv, d, k.stride(0), k.stride(1),
                                       1.0 / math.sqrt(d), cs.CS_BF16, ws, size, mode | flag)
        results.append((k, v, out))
    torch.cuda.synchronize()
    for a, b in zip(*results):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))


def test_own_rows_step_under_capture(cs):
    """A step of own-row calls replayed from a HIP graph equals the step of separate calls, every time."""
    from paper_2604_06036_amd import engine, synth
    w = synth.small_variant(synth.CFG2, n_streams=1, n_layers=4)
    say(f"own rows: captured step, {w.name} streams={w.n_streams} layers={w.n_layers}")
    data = engine.assemble_step(w, engine.hip_scorer, device="cpu")
    caps = dict(reuse_cap=data.info["n_reuse"] + 64, q_cap=data.info["n_q"] + 64)
    two, one = engine.DeviceStep(data, own_rows=False, **caps), engine.DeviceStep(data, **caps)
    two.run()
    k0, v0 = data.k_pool.to(DEV), data.v_pool.to(DEV)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        one.run()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        one.run()
    for rep in range(3):
        one.k_pool.copy_(k0); one.v_pool.copy_(v0); one.out.zero_(); one.ws_d.fill_(0xA5)
        assert math.isfinite(torch.randn(1 << 20, device=DEV).sum().item())
        graph.replay()
        torch.cuda.synchronize()
        for name in ("k_pool", "v_pool", "out"):
            assert torch.equal(getattr(two, name).view(torch.int16), getattr(one, name).view(torch.int16)), (rep, name)


def test_public_calls_of_a_step_follow_any_call_that_plans(cs):
    """`refresh_and_attention` and `attention` of a step that runs own-row calls itself: behind a plan without own rows, and
    behind `run`, the same results as the step's."""
    from paper_2604_06036_amd import engine, synth
    for n_streams in (1, 7):
        w = synth.small_variant(synth.CFG2, n_streams=n_streams, n_layers=3)
        say(f"own rows: public calls, {w.name} streams={w.n_streams}")
        data = engine.assemble_step(w, engine.hip_scorer, device="cpu")
        caps = dict(reuse_cap=data.info["n_reuse"] + 64, q_cap=data.info["n_q"] + 64)
        two, one = engine.DeviceStep(data, own_rows=False, **caps), engine.DeviceStep(data, **caps)
        two.run()
        one.ws_d.fill_(0xA5)
        one.prepare()
        one.rerotate()
        for layer in range(w.n_layers):
            one.refresh_and_attention(layer, reuse_plan=layer > 0)
        torch.cuda.synchronize()
        assert torch.equal(two.out.view(torch.int16), one.out.view(torch.int16))
        one.run()
        one.out.zero_()
        for layer in range(w.n_layers):
            one.attention(layer, reuse_plan=True)
            two.attention(layer, reuse_plan=True)
        torch.cuda.synchronize()
        assert torch.equal(two.out.view(torch.int16), one.out.view(torch.int16))


@pytest.mark.parametrize("hq, hkv, d, n_streams", [(28, 4, 128, 1), (16, 4, 64, 1), (16, 4, 64, 12), (28, 4, 128, 7)])
def test_own_rows_step_reports_no_failed_barrier(cs, hq, hkv, d, n_streams):
    """The status word of a default step's workspace is 0 behind a good step, whatever the workspace held: for head_dim 64 too."""
    from dataclasses import replace
    from paper_2604_06036_amd import engine, synth
    w = replace(synth.small_variant(synth.CFG2, n_streams=n_streams, n_layers=2), n_q_heads=hq, n_kv_heads=hkv, head_dim=d)
    say(f"own rows: status word, heads={hq}/{hkv} d={d} streams={n_streams}")
    step = engine.DeviceStep(engine.assemble_step(w, engine.hip_scorer, device="cpu"))
    step.ws_d.fill_(0xA5)
    for _ in range(2):
        step.run()
        assert step.attention_status() == 0


def test_windows_that_share_a_cache_block(cs):
    """A window that holds another stream's new rows, under both step classes: they are written before anything attends."""
    from paper_2604_06036_amd import engine, synth
    w = synth.small_variant(synth.CFG2, n_streams=2, n_layers=4)
    say(f"own rows: shared cache block, {w.name} streams={w.n_streams} layers={w.n_layers}")
    data = engine.assemble_step(w, engine.hip_scorer, device="cpu")
    plan, table = data.plan, data.new_layout.block_table
    def whole_blocks(s, executed):
        rows = np.zeros(table.shape[1] * 16, bool)
        rows[plan.q_pos[plan.cu_q[s]: plan.cu_q[s + 1]]] = True
        rows = rows[: plan.kv_len[s] // 16 * 16].reshape(-1, 16)
        return np.flatnonzero((rows if executed else ~rows).all(axis=1))
    assert engine.DeviceStep(data).own_rows
    table[1, whole_blocks(1, False)[1]] = table[0, whole_blocks(0, True)[1]]
    data._plan = None
    two, step = engine.DeviceStep(data, own_rows=False), engine.DeviceStep(data)
    assert not step.own_rows
    for one in (two, step):
        one.run()
    torch.cuda.synchronize()
    for name in ("k_pool", "v_pool", "out"):
        assert torch.equal(getattr(two, name).view(torch.int16), getattr(step, name).view(torch.int16)), name

    front = engine.assemble_frontend_step(w, engine.hip_scorer, device="cpu")
    assert engine.FrontEndStep(front).own_rows
    front.bt_new[1, 3] = front.bt_new[0, 4]
    assert not engine.FrontEndStep(front).own_rows


def test_front_end_step_of_two_calls_a_layer(cs):
    """A front-end step without own rows against the default one (of few row tiles: the same kernels, so bit for bit)."""
    from paper_2604_06036_amd import engine, synth
    w = synth.small_variant(synth.CFG2, n_streams=1, n_layers=3)
    say(f"own rows: front-end step of two calls a layer, {w.name} streams={w.n_streams} layers={w.n_layers}")
    data = engine.assemble_frontend_step(w, engine.hip_scorer, device="cpu")
    steps = [engine.FrontEndStep(data, own_rows=own) for own in (False, True)]
    for one in steps:
        one.run()
    torch.cuda.synchronize()
    for name in ("k_pool", "v_pool", "out"):
        assert torch.equal(*(getattr(one, name).view(torch.int16) for one in steps)), name


@pytest.mark.parametrize("kv_len", [5, 16, 37, 48])
def test_a_full_block_of_own_rows_has_16_rows(cs, kv_len):
    """A window that is executed whole: the table's entry of its last, part-filled block names the rows that there are."""
    hq, hkv, d = 4, 1, 64
    say(f"own rows: last block of {kv_len} executed rows")
    dev = lambda a: torch.tensor(a, dtype=torch.int32, device=DEV)
    n_blocks = -(-kv_len // 16)
    kn, vn, q = (torch.randn((kv_len, h, d), device=DEV).to(torch.bfloat16) for h in (hkv, hkv, hq))
    k, v = (torch.zeros((n_blocks * 16, hkv, d), dtype=torch.bfloat16, device=DEV) for _ in range(2))
    size = cs.cs_refresh_prefill_attn_workspace(kv_len, 1, hq, hkv, d, n_blocks, cs.CS_BF16)
    ws = torch.zeros(size, dtype=torch.uint8, device=DEV)
    rows = list(range(kv_len))
    cs.cs_refresh_prefill_attn(kn, vn, dev(rows), kv_len, q, k, v, dev([0, kv_len]), dev(rows), dev([kv_len]), dev(list(range(n_blocks))),
                               n_blocks, 16, torch.zeros_like(q), kv_len, 1, hq, hkv, d, hkv * d, d, 0.125, cs.CS_BF16, ws, size,
                               cs.CS_ATTN_PLAN_BUILD | cs.CS_ATTN_OWN_ROWS)
    torch.cuda.synchronize()
    # (behind a header of 256 bytes two words a block, the rows in the low half of the second)
    table = ws[256: 256 + 8 * n_blocks].cpu().numpy().view(np.uint32).reshape(-1, 2)
    assert [bin(int(m) & 0xffff).count("1") for m in table[:, 1]] == [min(16, kv_len - 16 * b) for b in range(n_blocks)]


@pytest.mark.parametrize("head_dim", [64, 128])
def test_a_single_layer_makes_no_lists(cs, head_dim):
    """A step of one layer has no call that reads own rows: it takes the two calls, with no workspace for lists."""
    from dataclasses import replace
    from paper_2604_06036_amd import engine, synth
    for n_layers in (1, 2):
        w = replace(synth.small_variant(synth.CFG2, n_streams=1, n_layers=n_layers), n_q_heads=16, n_kv_heads=4, head_dim=head_dim)
        say(f"own rows: {n_layers} layers, d={head_dim}")
        steps = (engine.DeviceStep(engine.assemble_step(w, engine.hip_scorer, device="cpu")),
                 engine.FrontEndStep(engine.assemble_frontend_step(w, engine.hip_scorer, device="cpu")))
        for step in steps:
            shape = (step.q_cap, 1, 16, 4, head_dim, step.max_blocks, cs.CS_BF16)
            assert step.own_rows == (n_layers > 1)
            assert step.ws_d_bytes == (cs.cs_refresh_prefill_attn_workspace if step.own_rows else cs.cs_window_prefill_attn_workspace)(*shape)


@pytest.mark.parametrize("n_streams", [1, 32])
def test_refresh_write_does_not_wait_for_the_correction(cs, n_streams):
    """With the correction beside the layer loop, a step whose launches do not read own rows queues a layer's refresh write ahead of the
    wait for the layer's corrected rows; one whose launches do waits once a layer."""
    from paper_2604_06036_amd import engine, synth
    w = synth.small_variant(synth.CFG2, n_streams=n_streams, n_layers=3)
    say(f"own rows: correction beside the layer loop, streams={n_streams}")
    step = engine.DeviceStep(engine.assemble_step(w, engine.hip_scorer, device="cpu"), overlap=True, layers_per_rerotate=1)
    assert step.own_rows == (n_streams == 1)
    main, order = torch.cuda.current_stream(), []
    calls = ("cs_kv_refresh_scatter", "cs_window_prefill_attn", "cs_refresh_prefill_attn")

    class Recorded:
        def __getattr__(self, name):
            def call(*args):
                order.append(name)
                return getattr(cs, name)(*args)
            return call if name in calls else getattr(cs, name)
    step.cs = Recorded()
    wait = torch.cuda.Stream.wait_event

    def recorded_wait(stream, event):
        if stream == main:
            order.append("wait")
        return wait(stream, event)
    torch.cuda.Stream.wait_event = recorded_wait
    try:
        step.run()
    finally:
        torch.cuda.Stream.wait_event = wait
    torch.cuda.synchronize()
    layer = ["wait", calls[2]] if n_streams == 1 else [calls[0], "wait", calls[1]]
    assert order[: 3 * len(layer)] == 3 * layer
