"""What the fused append and attention calls refuse on a device cache: stream ids that are
missing, out of range or given twice, whatever the number of rows asks for.  A refused call
changes nothing.
"""
import ctypes as C

import numpy as np
import pytest

from synth.streams import SEG_ACOUSTIC

pytestmark = pytest.mark.gpu


def _i32(*x):
    return (C.c_int32 * len(x))(*x)


@pytest.mark.parametrize("call", ["a2t_append_attn", "a2t_append_attn_noalloc"])
@pytest.mark.parametrize("rows", [3, 80])      # 4 query heads per KV head: 12 and 320 query rows
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_stream_ids(gpu, dtype, rows, call):
    import torch
    import paper_2609_31224_amd as a2t
    S, hq, hkv, d = 2, 4, 1, 64
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    cache = a2t.a2t_cache_create(1, S, hq, hkv, d, a2t.A2T_F32 if dtype == "f32" else a2t.A2T_BF16, 4 * rows, 8, rows)
    kv = torch.randn((S * rows, hkv, d), device="cuda").to(t)
    q = torch.randn((S * rows, hq, d), device="cuda").to(t)
    o = torch.zeros_like(q)
    seg = np.full(S * rows, SEG_ACOUSTIC, np.uint8)
    pos = np.tile(np.arange(rows, dtype=np.int32), S)
    fn = getattr(a2t.raw_lib(), call)

    def step(ids, n):
        return fn(cache.ptr, 0, n, ids, _i32(*[rows] * n), kv.data_ptr(), kv.data_ptr(),
                  seg.ctypes.data_as(C.POINTER(C.c_uint8)), pos.ctypes.data_as(C.POINTER(C.c_int32)), _i32(*[0] * n),
                  _i32(*[rows] * n), q.data_ptr(), o.data_ptr())

    before = [a2t.a2t_stream_info_get(cache, s) for s in range(S)]
    for ids, n in ((None, 1), (_i32(-1), 1), (_i32(S), 1), (_i32(100_000_000), 1), (_i32(-2**31), 1), (_i32(0, S), 2),
                   (_i32(1, 1), 2)):
        assert step(ids, n) == a2t.A2T_ERR_INVALID, (list(ids) if ids else None, n)
    assert [a2t.a2t_stream_info_get(cache, s) for s in range(S)] == before
    a2t.a2t_sync(cache)
    assert not o.any()
    assert step(_i32(1, 0), 2) == a2t.A2T_OK
    a2t.a2t_sync(cache)
    assert o.any()
    a2t.a2t_cache_destroy(cache)
