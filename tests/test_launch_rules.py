"""Which kernels a call takes, on the CPU: both sides of every line of the
launch rules, as the library answers them (no kernel runs here; the results on
both sides are compared with the oracle in the GPU tests)."""

import ctypes
import os

import pytest

from paper_2607_29591_amd import reskv as rk

HEAD, SPLIT, RANGES = "decode_head", "decode_split + decode_combine", "decode_ragged + decode_ragged_combine"


@pytest.fixture(scope="module", autouse=True)
def built():
    if not os.path.exists(rk.LIB_PATH):
        from paper_2607_29591_amd import build_lib
        build_lib.build()


def kernels(entry, dtype, d, G, pairs, C, Rcap=64):
    return rk.decode_kernels(rk.make_shape(pairs, G, 1, d, dtype, C, Rcap), entry)


@pytest.mark.parametrize("dtype,d,G,pairs,C,want", [
    # one round of slots: any count; bf16 two units more, but for few single heads (one pair x 640: 9.3 us split, 10.3)
    ("bf16", 128, 4, 1, 640, HEAD), ("bf16", 128, 4, 1, 641, SPLIT), ("bf16", 64, 1, 1, 640, HEAD),
    ("bf16", 128, 1, 7, 512, HEAD), ("bf16", 128, 1, 7, 513, SPLIT), ("bf16", 128, 1, 8, 640, HEAD),
    ("f32", 64, 4, 1, 512, HEAD), ("f32", 64, 4, 1, 513, SPLIT),
    # two rounds: fp32 rows need more pairs (64 x 768: 15.8 us split, 18.8 in one block)
    ("bf16", 128, 4, 63, 1024, SPLIT), ("bf16", 128, 4, 64, 1024, HEAD),
    ("f32", 64, 4, 79, 768, SPLIT), ("f32", 64, 4, 80, 768, HEAD),
    # three and four rounds: small groups need more pairs (96 x 1280, one query head: 15.9 and 18.9)
    ("bf16", 128, 1, 119, 1280, SPLIT), ("bf16", 128, 1, 120, 1280, HEAD), ("bf16", 128, 8, 96, 1280, HEAD),
    ("bf16", 128, 4, 143, 2048, SPLIT), ("bf16", 128, 4, 144, 2048, HEAD), ("bf16", 128, 16, 128, 2048, HEAD),
    ("bf16", 128, 4, 160, 2304, HEAD), ("bf16", 128, 4, 159, 2304, SPLIT),
    # long caches of small groups below 256 pairs (192 x 2560 with one long head: 18.4 and 29.0)
    ("bf16", 128, 4, 255, 2305, SPLIT), ("bf16", 128, 4, 256, 2305, HEAD), ("bf16", 128, 8, 160, 2560, HEAD),
    # fp32 rows of 128 always split
    ("f32", 128, 4, 256, 300, SPLIT),
])
def test_decode_one_block_per_head(dtype, d, G, pairs, C, want):
    assert kernels("attn", dtype, d, G, pairs, C) == want


@pytest.mark.parametrize("dtype,G,pairs,C,want", [
    ("bf16", 4, 64, 1024, HEAD), ("bf16", 4, 255, 2304, HEAD), ("bf16", 4, 512, 2304, HEAD),
    # long caches of small groups at any count (384 x 3072, few long heads: 35.0 us split, 77.9 in one block)
    ("bf16", 4, 256, 2305, SPLIT), ("bf16", 1, 512, 3072, SPLIT), ("bf16", 8, 256, 3072, HEAD),
])
def test_branches_one_block_per_head(dtype, G, pairs, C, want):
    assert kernels("branches", dtype, 128, G, pairs, C) == want


@pytest.mark.parametrize("dtype,d,G,pairs,C,want", [
    ("bf16", 128, 7, 256, 1152, HEAD), ("bf16", 128, 7, 256, 1536, HEAD), ("bf16", 128, 7, 256, 1537, RANGES),
    ("bf16", 128, 7, 257, 600, RANGES),
    # one block per head on longer caches: not with few query heads or fp32 rows
    ("bf16", 128, 4, 160, 2304, HEAD), ("bf16", 128, 2, 160, 1792, HEAD), ("bf16", 128, 2, 160, 1793, RANGES),
    ("f32", 64, 4, 192, 1792, HEAD), ("f32", 64, 4, 160, 2048, RANGES),
    # split-K blocks: short caches or few pairs, any with wide groups
    ("bf16", 128, 4, 96, 1280, SPLIT), ("bf16", 128, 4, 96, 1281, RANGES), ("bf16", 128, 8, 64, 2304, SPLIT),
    ("bf16", 128, 4, 64, 2304, SPLIT), ("bf16", 128, 4, 65, 2304, RANGES),
    ("f32", 64, 4, 48, 1024, SPLIT), ("f32", 64, 4, 48, 1025, RANGES), ("f32", 64, 4, 32, 2304, SPLIT),
    # bf16 rows of 64 at any
    ("bf16", 64, 1, 100, 2304, SPLIT), ("bf16", 64, 1, 170, 2304, HEAD), ("bf16", 64, 4, 100, 2305, RANGES),
])
def test_ragged_entry(dtype, d, G, pairs, C, want):
    assert kernels("ragged", dtype, d, G, pairs, C) == want


class BuildRules(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int32) for n in ("deal_rows", "key_groups", "select_blocks", "count_sel")]


def build_rules(dtype, d, G, heads, s, window, budget=512, res=0):
    """Launch rules of a construction of `heads` equal heads of s tokens."""
    i32 = lambda x: (ctypes.c_int32 * len(x))(*x)
    rules = BuildRules()
    fn = rk.lib().reskv_internal_build_rules
    fn.restype, fn.argtypes = ctypes.c_int, None
    assert fn(ctypes.byref(rk.make_shape(1, G * heads, heads, d, dtype, budget, max(1, res))),
              ctypes.byref(rk.BuildParams(s, window, window, 4, 0, 0)), i32([s]), i32([budget]), i32([res] * heads),
              ctypes.byref(rules)) == 0
    return rules


@pytest.mark.parametrize("dtype,heads,s,want", [
    ("f32", 2, 1024, 1), ("f32", 8, 16384, 1),   # 2 and 128 chunks of 1024 keys
    ("f32", 8, 16385, 0), ("f32", 8, 32768, 0),  # 136 and 256: 228 us of scoring undealt, 302 dealt
    ("bf16", 2, 1024, 0),
])
def test_lse_rows_dealt(dtype, heads, s, want):
    assert build_rules(dtype, 128, 4, heads, s, 32).deal_rows == want


@pytest.mark.parametrize("dtype,G,heads,s,want", [
    ("bf16", 4, 8, 32768, 1), ("bf16", 4, 8, 49152, 1), ("bf16", 4, 8, 49153, 4),   # 128 rows: 256, 384, 392 blocks
    ("bf16", 8, 8, 16384, 1), ("bf16", 8, 8, 16385, 4), ("bf16", 8, 8, 62000, 4),   # 256 rows: 144 us, 169 with one group
    ("f32", 8, 8, 49152, 1), ("f32", 8, 8, 62000, 4),
])
def test_score_pass_key_groups(dtype, G, heads, s, want):
    assert build_rules(dtype, 128, G, heads, s, 32).key_groups == want


@pytest.mark.parametrize("s,blocks,counted", [(8192, 1, 0), (65536, 8, 0), (65537, 9, 1), (1 << 20, 128, 1)])
def test_long_score_lists_are_counted(s, blocks, counted):
    """The placement rereads the scores before a block only on lists of up to 8 blocks (1M tokens, 8 heads: 979 us of
    construction counted, 1172 reread)."""
    rules = build_rules("bf16", 64, 4, 2, s, 8)
    assert (rules.select_blocks, rules.count_sel) == (blocks, counted)


class ProxyRules(ctypes.Structure):
    _fields_ = [("batched", ctypes.c_int32), ("least_bytes", ctypes.c_uint64)]


def proxy_rules(shape, params, proxy, seq_len, budget):
    i32 = lambda x: (ctypes.c_int32 * len(x))(*[int(v) for v in x])
    rules = ProxyRules()
    fn = rk.lib().reskv_internal_proxy_rules
    fn.restype, fn.argtypes = ctypes.c_int, None
    assert fn(ctypes.byref(shape), ctypes.byref(params), ctypes.byref(proxy), i32(seq_len), i32(budget),
              ctypes.byref(rules)) == 0
    return rules


@pytest.mark.parametrize("batch,ctx,want", [
    (8, 8192, 5), (9, 8192, 1),       # 64 and 72 pairs
    (8, 32768, 5), (8, 34000, 1),     # 64 pairs: up to 8192 assignment blocks of a candidate
    (4, 65536, 5), (4, 66000, 1),
])
def test_proxy_candidates_in_one_batch(batch, ctx, want):
    """The batch and its scratch per candidate stop with the context too, and the size query follows."""
    shape = rk.make_shape(batch, 32, 8, 128, "bf16", 256, 64)
    params, proxy = rk.BuildParams(ctx, 32, 32, 4, 0, 0), rk.make_proxy()
    rules = proxy_rules(shape, params, proxy, [ctx] * batch, [256] * batch)
    assert rules.batched == want
    size = rk.reskv_build_proxy_workspace_size(shape, params, proxy, [ctx] * batch, [256] * batch)
    assert size > rules.least_bytes if want > 1 else size == rules.least_bytes


def test_build_workspace_holds_what_is_read():
    """No partial sums without residual entries, no selection histograms where one block selects."""
    def size(s, r):
        return rk.reskv_build_workspace_size(rk.make_shape(1, 32, 8, 128, "bf16", 512, 256),
                                             rk.BuildParams(s, 32, 32, 4, 0, 0), [s], [512], [r] * 8)
    sums = 8 * 2 * (131072 // 256) * 2 * 128 * 8  # heads x slots x (keys, values) x d x fp64, about
    assert size(131072, 256) - size(131072, 0) > 0.9 * sums
    assert size(8193, 0) - size(8192, 0) > 8 * 32768
