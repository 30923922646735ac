"""Kernel variants at the sizes where they can go wrong: edges of their tiles, remainders, the smallest and the
largest of their range.  Everything goes through the C-ABI and is compared with the oracle."""
import math

import numpy as np
import pytest
import torch

from oracle import codecsight_oracle as oc
from tests import helpers as hp
from tests.test_gpu_parity import DEV, _attn_case, _pool, cs, say        # noqa: F401  (cs is a fixture)

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
