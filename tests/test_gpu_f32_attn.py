"""GPU parity of attn_f32 (fp32 caches) against the fp64 oracle at every step: query rows
around the 16-row blocks and the one- and two-block workgroups, key counts around the
16-key blocks, one to eight query heads per KV head, both head dims, a ring that wraps, a
kept region, forced and planned key splits, fused and separate append, decode rows, and
values that are not finite behind the causal mask.

Bar: 1e-4, as everywhere for fp32 caches.
"""
import dataclasses
import os

import numpy as np
import pytest

from synth.streams import CONFIGS, SEG_ACOUSTIC, SEG_DELIM, SEG_RESPONSE, SEG_TEXT, tiny_stream
from tests.harness import Lockstep, row_bounds

pytestmark = pytest.mark.gpu

F32_TOL = 1e-4


def _unit(n):
    return [SEG_TEXT if r % 9 == 4 else SEG_ACOUSTIC for r in range(n)]


SMALL = [SEG_ACOUSTIC] * 7 + [SEG_DELIM, SEG_TEXT, SEG_TEXT, SEG_DELIM]


@pytest.mark.parametrize("hq,hkv,d,rows,prefix,splits,fused,query_rows", [
    (1, 1, 64, 1, 0, None, True, None),          # one row, one head
    (8, 1, 128, 2, 15, None, False, None),       # 16 query rows: one block; 16 keys
    (4, 1, 64, 17, 64, "1", True, None),         # 68 query rows
    (16, 16, 128, 33, 700, None, True, None),    # two-block workgroups, an odd third block
    (32, 8, 64, 22, 900, None, False, None),     # planned splits, separate append
    (32, 8, 128, 22, 900, None, True, 5),        # the last 5 of 22 rows query
    (6, 3, 128, 40, 130, "5", True, None),       # forced splits of one to a few blocks
    (2, 2, 64, 90, 3, "128", True, None),        # more splits asked for than tiles
])
def test_f32_chunks(gpu, hq, hkv, d, rows, prefix, splits, fused, query_rows):
    cfg = dataclasses.replace(CONFIGS[0], n_q_heads=hq, n_kv_heads=hkv, head_dim=d)
    spec = tiny_stream([SMALL, _unit(rows), SMALL, _unit(rows), _unit(rows + 1), SMALL, _unit(rows)], prefix=prefix)
    bounds = row_bounds(spec)
    old = os.environ.get("A2T_SPLITS")
    if splits:
        os.environ["A2T_SPLITS"] = splits
    try:
        ls = Lockstep(cfg, 5, [spec], layers_checked=[0, 1], n_layers=2, budgets=[prefix + rows + 20], window=0,
                      unit_rows=max(2 * rows + 40 + prefix, 80), kept_rows=bounds[1] + 1,
                      max_step=max(bounds[2], rows + 1), tol=F32_TOL, dtype="f32", fused=fused, query_rows=query_rows)
    finally:
        if splits:
            if old is None:
                del os.environ["A2T_SPLITS"]
            else:
                os.environ["A2T_SPLITS"] = old
    try:
        ls.run()
    finally:
        ls.close()
    print(f"rows {rows}: max attention error {ls.max_err:.2e}, {ls.evictions} evictions", flush=True)


@pytest.mark.parametrize("d,rows,bad", [(64, 5, 4), (128, 22, 21), (128, 40, 17), (64, 33, 32)])
def test_masked_values_stay_out(gpu, d, rows, bad):
    """Row `bad` of the step holds infinite and NaN values: every query row before it, which
    does not see it, comes out as if they were finite; the rows that see it do not."""
    import torch
    import paper_2609_31224_amd as a2t
    hq, hkv = 4, 2
    g = torch.Generator(device="cuda").manual_seed(3)
    k, v, q = (torch.randn((rows, h, d), generator=g, device="cuda") for h in (hkv, hkv, hq))
    seg, pos = np.full(rows, SEG_ACOUSTIC, np.uint8), np.arange(rows)
    outs = []
    for spoil in (False, True):
        vv, kk = v.clone(), k.clone()
        if spoil:
            vv[bad, :, 0::2] = float("inf")
            vv[bad, :, 1::2] = float("nan")
            kk[bad, :, 3] = float("nan")
        c = a2t.a2t_cache_create(1, 1, hq, hkv, d, a2t.A2T_F32, 2 * rows, 8, rows)
        o = torch.zeros_like(q)
        a2t.a2t_append_attn(c, 0, [0], [rows], kk, vv, seg, pos, [0], [rows], q, o)
        a2t.a2t_sync(c)
        outs.append(o.cpu().numpy())
        a2t.a2t_cache_destroy(c)
    # the same sums in another order: a few roundings of a convex combination of |v| < 6
    assert np.abs(outs[0][:bad] - outs[1][:bad]).max(initial=0.0) < 1e-5
    assert np.isnan(outs[1][bad:]).all()


def _lockstep(monkeypatch, hq, hkv, d, rows, prefix, splits, fused, query_rows):
    """The long units of test_f32_chunks on workgroups of two query blocks (every launch of
    more than 16 query rows asks for them where one CU is counted)."""
    import paper_2609_31224_amd as a2t
    monkeypatch.setenv("A2T_TARGET_WGS", "1")
    monkeypatch.setenv("A2T_SPLITS", splits)
    cfg = dataclasses.replace(CONFIGS[0], n_q_heads=hq, n_kv_heads=hkv, head_dim=d)
    spec = tiny_stream([SMALL, _unit(rows), SMALL, _unit(rows), _unit(rows + 1), SMALL, _unit(rows), _unit(rows)], prefix=prefix)
    bounds = row_bounds(spec)
    ls = Lockstep(cfg, 5, [spec], layers_checked=[0, 1], n_layers=2, budgets=[prefix + rows + 20], window=0,
                  unit_rows=2 * rows + 40 + prefix, kept_rows=bounds[1] + 1,
                  max_step=max(bounds[2], rows + 1), tol=F32_TOL, dtype="f32", fused=fused, query_rows=query_rows)
    a2t.a2t_profile_enable(ls.cache, "attn_f32")
    try:
        ls.run()
        return ls, a2t.a2t_kernel_time(ls.cache, "attn_f32x2")[0], a2t.a2t_kernel_time(ls.cache, "attn_f32")[0]
    finally:
        ls.close()


@pytest.mark.parametrize("splits", ["1", "3", "5"])
@pytest.mark.parametrize("hq,hkv,d,rows,prefix,fused,query_rows", [
    (17, 17, 64, 17, 30, True, None),      # one query head: the second block holds one row
    (4, 1, 64, 33, 130, False, None),      # 132 query rows: an odd block, the last group half empty
    (8, 2, 128, 40, 200, True, None),      # 160: whole groups
    (8, 1, 128, 21, 70, True, 9),          # 72 of 168, the ring wraps between the queries' keys
    (3, 3, 128, 50, 0, False, 35),
])
def test_f32_two_blocks(gpu, monkeypatch, hq, hkv, d, rows, prefix, splits, fused, query_rows):
    """Groups of two query blocks over resident, wrapped and kept keys, with split partials."""
    ls, two, one = _lockstep(monkeypatch, hq, hkv, d, rows, prefix, splits, fused, query_rows)
    # two layers x the five long units (more than 16 query rows each) at least
    assert two >= 10 and ls.evictions >= 3, (two, one, ls.evictions)
    print(f"rows {rows}: max attention error {ls.max_err:.2e}, {two} of {two + one} launches of two blocks", flush=True)


@pytest.mark.parametrize("splits", ["1", "3"])
@pytest.mark.parametrize("d,rows,bad", [(64, 9, 5), (128, 22, 21), (128, 40, 17), (64, 33, 32)])
def test_masked_values_stay_out_of_two_blocks(gpu, monkeypatch, d, rows, bad, splits):
    """test_masked_values_stay_out on workgroups of two query blocks, onto resident rows."""
    import torch
    import paper_2609_31224_amd as a2t
    monkeypatch.setenv("A2T_TARGET_WGS", "1")
    monkeypatch.setenv("A2T_SPLITS", splits)
    hq, hkv, old = 4, 2, 70
    g = torch.Generator(device="cuda").manual_seed(3)
    k0, v0 = (torch.randn((old, hkv, d), generator=g, device="cuda") for _ in range(2))
    k, v, q = (torch.randn((rows, h, d), generator=g, device="cuda") for h in (hkv, hkv, hq))
    outs = []
    for spoil in (False, True):
        vv, kk = v.clone(), k.clone()
        if spoil:
            vv[bad, :, 0::2] = float("inf")
            vv[bad, :, 1::2] = float("nan")
            kk[bad, :, 3] = float("nan")
        c = a2t.a2t_cache_create(1, 1, hq, hkv, d, a2t.A2T_F32, old + 2 * rows, 8, max(old, rows))
        o = torch.zeros_like(q)
        a2t.a2t_append(c, 0, [0], [old], k0, v0, np.full(old, SEG_ACOUSTIC, np.uint8), np.arange(old), [0])
        a2t.a2t_evict(c, [0], [10 * old], 1)
        a2t.a2t_profile_enable(c, "attn_f32")
        a2t.a2t_append_attn(c, 0, [0], [rows], kk, vv, np.full(rows, SEG_ACOUSTIC, np.uint8), np.arange(old, old + rows), [1],
                            [rows], q, o)
        a2t.a2t_sync(c)
        assert a2t.a2t_kernel_time(c, "attn_f32x2")[0] == 1
        outs.append(o.cpu().numpy())
        a2t.a2t_cache_destroy(c)
    # as in test_masked_values_stay_out
    assert np.abs(outs[0][:bad] - outs[1][:bad]).max(initial=0.0) < 1e-5
    assert np.isnan(outs[1][bad:]).all()


@pytest.mark.parametrize("hkv,d,prefix,splits,target,valu", [
    (1, 64, 0, None, None, True), (1, 64, 60, None, None, True),      # one and two tiles
    (3, 128, 0, None, None, True), (3, 128, 200, None, None, False),  # four tiles
    (3, 128, 500, None, None, True), (3, 128, 500, "3", None, True),  # eight tiles of 128 dims
    (2, 64, 300, None, None, False),
    (2, 64, 300, None, "2", True), (2, 64, 300, "3", "2", True),      # two heads fill two CUs
    (2, 64, 1024, None, "2", False),                                  # 17 tiles of 64 dims
])
def test_f32_one_query_row(gpu, monkeypatch, hkv, d, prefix, splits, target, valu):
    """Decode rows with one query head per KV head: on the vector kernel where it is the faster
    one, on attn_f32 elsewhere, the oracle's results on both."""
    import paper_2609_31224_amd as a2t
    for name, value in (("A2T_SPLITS", splits), ("A2T_TARGET_WGS", target)):
        if value:
            monkeypatch.setenv(name, value)
    cfg = dataclasses.replace(CONFIGS[0], n_q_heads=hkv, n_kv_heads=hkv, head_dim=d)
    spec = tiny_stream([SMALL, [SEG_RESPONSE], [SEG_RESPONSE], SMALL, [SEG_RESPONSE], SMALL, [SEG_RESPONSE]], prefix=prefix)
    bounds = row_bounds(spec)
    ls = Lockstep(cfg, 5, [spec], layers_checked=[0, 1], n_layers=2, budgets=[prefix + 20], window=0,
                  unit_rows=prefix + 40, kept_rows=bounds[1] + 1, max_step=bounds[2], tol=F32_TOL, dtype="f32")
    a2t.a2t_profile_enable(ls.cache, "attn")
    try:
        ls.run()
        assert a2t.a2t_kernel_time(ls.cache, "attn_valu")[0] == (8 if valu else 0)
    finally:
        ls.close()
