"""How an append is cut up, over the whole range of calls (CPU: the library's
own choice, asked without a device).

The split-key attention fits its chunks to the call.  Whatever it picks, a
chunk is whole blocks and whole stages of keys, the chunks cover the keys, and
the plan kernel's LDS (the block ids of every member's chunk, beside 3080 bytes
of its own) fits in the 160 KiB of a CU.  The work area that kv_scratch_bytes
asks for holds every call that it is asked for in its fastest form, without
cutting it into layer groups.
"""
import ctypes

import pytest

from paper_2607_10987_amd import kvstate as kv

PORTABLE, PREFILL, PACKED, SPLIT = range(4)
CU_LDS = 160 * 1024
PLAN_STATIC = 3080


def query(cfg, batch, T, keys, scratch):
    out = (ctypes.c_int64 * 8)()
    f = kv.lib().kvs_query_append
    f.argtypes = [ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64, ctypes.c_int32, ctypes.c_size_t,
                  ctypes.c_void_p]
    st = f(ctypes.byref(cfg), batch, T, keys, scratch, out)
    assert st == 0, st
    return dict(zip(("layers", "bytes", "form", "path", "ck", "nch", "lists", "lds"), out))


def key_counts(top):
    """Key counts up to `top`: the smallest, the edges of blocks and chunks,
    and a spread whose step is not a divisor of any chunk size."""
    ks = {1, 2, 15, 16, 17, 63, 64, 65, 255, 256, 257, 511, 512, 513, 1023, 1024, 1025}
    n = 300
    while n < top:
        ks.add(n)
        n += max(97, n // 37)
    ks |= {m * 1024 + e for m in (2, 3, 4, 6, 8, 10, 16, 33) for e in (-1, 0, 1)}
    ks |= {9983, 9984, 9985, 10048, 10200, 10239, 10240, 10241, top}
    return sorted(k for k in ks if k <= top)


@pytest.mark.parametrize("L,hq,hkv", [(32, 32, 8), (80, 64, 8), (28, 28, 4), (2, 32, 8),
                                      (1, 4, 1), (40, 16, 16), (48, 48, 3), (16, 64, 4)])
def test_split_key_plan_fits(L, hq, hkv):
    for B in (16, 32, 64):
        cfg = kv.make_cfg(L, 4096, hq, hkv, 128, B, "bf16", 140000, 64)
        for T in (1, 2, 5, 32):
            for batch in (1, 2, 3, 4, 7, 8, 13, 16, 17, 24, 31, 32, 33, 47, 62, 63, 64):
                for keys in key_counts(140000 if batch < 4 else 40000):
                    if keys < T:
                        continue
                    q = query(cfg, batch, T, keys, 1 << 44)
                    what = (B, T, batch, keys, q)
                    assert q["layers"] == L, what
                    if q["path"] != SPLIT:
                        assert T > 1, what
                        continue
                    assert q["ck"] % 64 == 0 and q["ck"] % B == 0, what
                    assert (q["nch"] - 1) * q["ck"] < keys <= q["nch"] * q["ck"], what
                    assert q["lds"] >= batch * (q["ck"] // B) * 4, what
                    assert q["lds"] + PLAN_STATIC <= CU_LDS, what


def q_bytes(cfg, rows):
    return -(-rows * cfg.n_q_heads * cfg.head_dim * 2 // 256) * 256 * cfg.n_layers


@pytest.mark.parametrize("L,hq,hkv,B,batch,tokens,keys,factor", [
    (32, 32, 8, 16, 16, 16, 33792, 1.5), (80, 64, 8, 32, 4, 4, 16388, 1.7),
    (32, 32, 8, 16, 64, 64, 33792, 1.05), (32, 32, 8, 16, 32, 200, 6015, 1.05),
    (2, 32, 8, 16, 5, 40, 9001, 11), (28, 28, 4, 64, 7, 7, 20011, 2.1),
])
def test_work_area_holds_every_smaller_call(L, hq, hkv, B, batch, tokens, keys, factor):
    """A work area of kv_scratch_bytes runs every call of at most as many
    states, tokens and keys in the form that it would take in an unlimited one,
    in one layer group, and is at most `factor` times what the least layout takes
    to decode the whole batch (1024-key chunks; two layers over several tokens
    take many more chunks to fill the GPU)."""
    cfg = kv.make_cfg(L, 4096, hq, hkv, 128, B, "bf16", keys + 8, 64)
    area = kv.kv_scratch_bytes(cfg, tokens, batch, keys)
    for b in sorted({1, 2, 3, 5, batch // 3, batch // 2 + 1, batch - 1, batch} - {0}):
        for T in sorted({1, 2, 3, 5, 12, 31, 32, tokens // b}):
            if T * b > tokens or b > batch:
                continue
            for k in {*range(T, keys, max(61, keys // 90)), *range(max(T, keys - 70), keys + 1)}:
                want, got = query(cfg, b, T, k, 1 << 44), query(cfg, b, T, k, area)
                assert got == want and got["layers"] == L, (b, T, k, want, got)
    least = L * batch * hq * -(-keys // 1024) * 132 * 4
    assert area - q_bytes(cfg, tokens) <= factor * least + (1 << 20), (area, least)


@pytest.mark.parametrize("hq,hkv,keys,T,batch,path", [
    (32, 8, 8000, 4, 2, SPLIT), (64, 8, 8000, 4, 2, SPLIT),      # 4 and 8 query heads
    (32, 8, 8000, 64, 1, PREFILL), (32, 8, 8000, 16, 8, PACKED),
    (8, 8, 8000, 4, 2, PORTABLE), (16, 8, 8000, 4, 2, PORTABLE),
    (24, 8, 8000, 4, 2, PORTABLE), (48, 8, 8000, 2, 1, PORTABLE),
    (64, 4, 8000, 8, 1, PORTABLE), (24, 8, 8000, 64, 1, PORTABLE),
    (32, 8, 131072, 4, 2, SPLIT), (32, 8, 131073, 4, 2, PORTABLE),   # block tables above 32 KiB
    (24, 8, 8000, 1, 2, SPLIT), (32, 8, 139990, 1, 2, SPLIT),        # decode: any head group
])
def test_appends_keep_float32_probabilities(hq, hkv, keys, T, batch, path):
    """The split-key attention rounds probabilities to bf16, as the prefill
    attention does.  It takes appends from that one only: head groups and table
    sizes that run in the portable kernel (float32 throughout) stay there at
    every number of query vectors."""
    cfg = kv.make_cfg(32, 4096, hq, hkv, 128, 16, "bf16", 140000, 64)
    q = query(cfg, batch, T, keys, kv.kv_scratch_bytes(cfg, batch * T, batch, keys))
    assert q["path"] == path, q
