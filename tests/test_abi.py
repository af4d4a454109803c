"""Host-side checks of the C ABI: the library loads, exports every entry
point declared in include/reskv.h, sizes workspaces, and rejects bad
arguments before launching anything (no GPU needed)."""

import ctypes
import os
import re

import numpy as np
import pytest

from paper_2607_29591_amd import reskv as rk

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def L():
    if not os.path.exists(rk.LIB_PATH):
        from paper_2607_29591_amd import build_lib
        build_lib.build()
    return rk.lib()


def declared_functions():
    text = open(os.path.join(ROOT, "include", "reskv.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(reskv_[a-z_]+)\s*\(", text)))


def test_every_declared_symbol_is_exported(L):
    names = declared_functions()
    assert {"reskv_build_cache", "reskv_decode_attn", "reskv_append_kv"} <= set(names)
    for n in names:
        assert hasattr(L, n), n
    assert set(rk._SIG) == set(names)


def test_status_strings(L):
    assert rk.status_string(0) == "ok"
    assert "workspace" in rk.status_string(3)


def shape(**kw):
    d = dict(batch=2, num_q_heads=8, num_kv_heads=2, head_dim=128, dtype="bf16", slot_cap=640, res_cap=64)
    d.update(kw)
    return rk.make_shape(**d)


def test_decode_workspace_size(L):
    s = shape()
    n = rk.reskv_decode_workspace_size(s)
    # 1 residual chunk + 3 main chunks of 256 slots, 4 heads, d + 2 floats each
    assert n >= 2 * 2 * 4 * 4 * (128 + 2) * 4
    assert rk.reskv_decode_workspace_size(shape(head_dim=96)) == 0
    assert rk.reskv_decode_workspace_size(shape(num_q_heads=7)) == 0


def test_ragged_workspace_counts_only_what_is_written(L):
    """A ragged call served by one block per head writes no split-K records: its workspace is that of the equal
    ranges, so a buffer sized for them takes it. Split-K records are counted where they are written."""
    s = shape(batch=64, num_kv_heads=4, num_q_heads=28, slot_cap=1152)
    past = shape(batch=65, num_kv_heads=4, num_q_heads=28, slot_cap=1152)  # 260 pairs: equal ranges
    assert rk.decode_kernels(s, "ragged") == "decode_head"
    assert rk.decode_kernels(past, "ragged") == "decode_ragged + decode_ragged_combine"
    n, n_past = rk.reskv_decode_ragged_workspace_size(s), rk.reskv_decode_ragged_workspace_size(past)
    assert n <= n_past < rk.reskv_decode_workspace_size(s)
    split = shape(batch=16, num_kv_heads=8, num_q_heads=56, slot_cap=2304, res_cap=1000)
    assert rk.decode_kernels(split, "ragged") == "decode_split + decode_combine"
    assert rk.reskv_decode_ragged_workspace_size(split) == rk.reskv_decode_workspace_size(split)


@pytest.mark.parametrize("kw,entry,kernels", [
    (dict(batch=32, num_kv_heads=8, num_q_heads=32, slot_cap=2304), "attn", "decode_head"),
    (dict(batch=8, num_kv_heads=8, num_q_heads=32, slot_cap=1024), "attn", "decode_head"),  # 64 pairs
    (dict(batch=1, num_kv_heads=8, num_q_heads=32, slot_cap=640), "attn", "decode_head"),   # one round of slots
    (dict(batch=4, num_kv_heads=8, num_q_heads=32, slot_cap=1088), "attn", "decode_split + decode_combine"),
    (dict(batch=64, num_kv_heads=4, num_q_heads=28, slot_cap=1152), "ragged", "decode_head"),
    (dict(batch=96, num_kv_heads=4, num_q_heads=28, slot_cap=2304), "ragged",
     "decode_ragged + decode_ragged_combine")])
def test_bench_labels_name_the_kernels_that_run(L, kw, entry, kernels):
    import bench
    assert rk.decode_kernels(shape(**kw), entry) == kernels
    assert kernels in bench.decode_label(rk, shape(**kw), entry)


class FakeTensor:
    """Stands in for a device tensor: a non-null pointer that is never
    dereferenced because validation fails first."""

    def __init__(self, nbytes=16):
        self._n = nbytes

    def is_contiguous(self):
        return True

    def data_ptr(self):
        return 0x1000

    def numel(self):
        return self._n

    def element_size(self):
        return 1


@pytest.mark.parametrize("bad,code", [
    (dict(head_dim=96), 2), (dict(num_q_heads=7), 1), (dict(num_q_heads=34), 2),
    (dict(batch=0), 1), (dict(slot_cap=0), 1), (dict(dtype=5), 2)])
def test_decode_rejects_bad_shapes(L, bad, code):
    t = FakeTensor()
    with pytest.raises(rk.ReskvError) as ei:
        rk.reskv_decode_attn(shape(**bad), rk.make_gate(), t, t, t, t, t, t, t, t, stream=FakeStream())
    assert ei.value.status == code
    assert rk.last_error()


class FakeStream:
    cuda_stream = 0


def test_decode_rejects_small_workspace_and_bad_gate(L):
    t = FakeTensor()
    with pytest.raises(rk.ReskvError) as ei:
        rk.reskv_decode_attn(shape(), rk.make_gate(), t, t, t, t, t, t, t, FakeTensor(8), stream=FakeStream())
    assert ei.value.status == 3
    with pytest.raises(rk.ReskvError) as ei:
        rk.reskv_decode_attn(shape(), rk.make_gate(g_min=1.5), t, t, t, t, t, t, t, t, stream=FakeStream())
    assert ei.value.status == 1
    with pytest.raises(rk.ReskvError) as ei:
        rk.reskv_decode_attn(shape(), rk.make_gate(), None, t, t, t, t, t, t, t, stream=FakeStream())
    assert ei.value.status == 1


def build_args(**kw):
    d = dict(S=300, w=16, recent=16, T=4, fit=0, seq=(300,), budget=(64,))
    d.update(kw)
    sh = rk.make_shape(1, 4, 2, 64, "f32", 64, 13)
    return sh, rk.BuildParams(d["S"], d["w"], d["recent"], d["T"], d["fit"]), d["seq"], d["budget"]


def test_build_workspace_and_fit_rows(L):
    sh, p, seq, bud = build_args()
    n_all = rk.reskv_build_workspace_size(sh, p, seq, bud, [13, 0])
    assert n_all > 0
    sh, p, seq, bud = build_args(fit=12)
    n_fit = rk.reskv_build_workspace_size(sh, p, seq, bud, [13, 0])
    assert 0 < n_fit <= n_all  # fewer scoring rows, no larger lse partials
    for fit in (-1, 17):
        sh, p, seq, bud = build_args(fit=fit)
        assert rk.reskv_build_workspace_size(sh, p, seq, bud, [13, 0]) == 0


GRID = (0.0, 0.05, 0.10, 0.15, 0.20)


@pytest.mark.parametrize("grid,val,delta,fit", [
    ((0.05, 0.1), 4, 0.01, 0),       # no zero fraction
    ((0.0, 1.0), 4, 0.01, 0),        # f >= 1
    ((0.0, float("nan")), 4, 0.01, 0),
    ((0.0, 0.5), 4, 0.01, 0),        # r = 32 above res_cap 13
    ((0.0, 0.1), 16, 0.01, 0),       # no fit rows left
    ((0.0, 0.1), 0, 0.01, 0),        # no validation rows
    ((0.0, 0.1), 4, 1.5, 0),         # delta outside [0, 1]
    ((0.0, 0.1), 4, 0.01, 10),       # fit rows disagree with w - val_rows
    ((0.0,) * 9, 4, 0.01, 0),        # more than 8 candidates
])
def test_proxy_rejects_bad_arguments(L, grid, val, delta, fit):
    sh, p, seq, bud = build_args(fit=fit)
    x = rk.make_proxy(grid, val, delta)
    assert rk.reskv_build_proxy_workspace_size(sh, p, x, seq, bud) == 0
    t = FakeTensor()
    with pytest.raises(rk.ReskvError) as ei:
        rk.reskv_build_cache_proxy(sh, p, x, rk.make_gate(), t, t, seq, t, bud, t, t, t, t, t, t, t,
                                   stream=FakeStream())
    assert ei.value.status == 1
    assert rk.last_error()


def test_proxy_workspace_holds_every_candidate(L):
    sh, p, seq, bud = build_args()
    x = rk.make_proxy(GRID, 4, 0.01)
    n = rk.reskv_build_proxy_workspace_size(sh, p, x, seq, bud)
    # at least the five candidate caches (K and V, 2 heads x 64 slots x 64 fp32)
    assert n >= 5 * 2 * 2 * 64 * 64 * 4
    sh2, p2, _, _ = build_args(fit=12)  # the fit rows may also be given explicitly
    assert rk.reskv_build_proxy_workspace_size(sh2, p2, x, seq, bud) == n
    t = FakeTensor(8)
    with pytest.raises(rk.ReskvError) as ei:
        rk.reskv_build_cache_proxy(sh, p, x, rk.make_gate(), t, t, seq, t, bud, t, t, t, t, t, t, t,
                                   stream=FakeStream())
    assert ei.value.status == 3


@pytest.mark.parametrize("pool,ok", [(0, True), (1, True), (3, True), (31, True), (2, False), (33, False), (-1, False)])
def test_build_pool_kernel_range(L, pool, ok):
    sh = rk.make_shape(1, 4, 2, 64, "f32", 64, 13)
    p = rk.BuildParams(300, 16, 16, 4, 0, pool)
    assert (rk.reskv_build_workspace_size(sh, p, (300,), (64,), [13, 0]) > 0) == ok


def test_merge_branches_rejects_bad_mode_and_alias(L):
    t = FakeTensor()
    with pytest.raises(rk.ReskvError) as ei:
        rk.reskv_merge_branches(shape(), 2, t, t, t, t, t, FakeTensor(), stream=FakeStream())
    assert ei.value.status == 1


def test_decode_branches_rejects_small_workspace(L):
    t = FakeTensor()
    with pytest.raises(rk.ReskvError) as ei:
        rk.reskv_decode_branches(shape(), rk.make_gate(), t, t, t, t, t, t, t, t, t, t, t, FakeTensor(8),
                                 stream=FakeStream())
    assert ei.value.status == 3


def test_adakv_workspace_covers_the_widest_allocation(L):
    """The cross-head build sizes its grids for every head holding up to
    min(s, C - r) main slots, so its workspace is at least the uniform one;
    safeguard 1 (the uniform split) keeps the evicted sets, and the main
    slots may still widen to the slot capacity."""
    sh = rk.make_shape(1, 4, 2, 64, "f32", 128, 13)
    p = rk.BuildParams(300, 16, 16, 4, 0, 0)
    uni = rk.reskv_build_workspace_size(sh, p, (300,), (64,), [13, 0])
    for g in (0.0, 0.2, 1.0):
        assert rk.reskv_build_adakv_workspace_size(sh, p, g, 0, (300,), (64,), [13, 0]) >= uni > 0
        assert rk.reskv_build_adakv_workspace_size(sh, p, g, 64, (300,), (64,), [13, 0]) >= uni


@pytest.mark.parametrize("reserve", [-1, 65])
def test_adakv_rejects_bad_decode_reserve(L, reserve):
    """budget + decode_reserve must fit the slot capacity (128 = 64 + 64)."""
    sh = rk.make_shape(1, 4, 2, 64, "f32", 128, 13)
    p = rk.BuildParams(300, 16, 16, 4, 0, 0)
    assert rk.reskv_build_adakv_workspace_size(sh, p, 0.2, reserve, (300,), (64,), [13, 0]) == 0
    t = FakeTensor()
    with pytest.raises(rk.ReskvError) as ei:
        rk.reskv_build_cache_adakv(sh, p, 0.2, reserve, t, t, (300,), t, (64,), [13, 0], t, t, t, t, t, t, t,
                                   stream=FakeStream())
    assert ei.value.status == 1 and "decode_reserve" in rk.last_error()


@pytest.mark.parametrize("safeguard,hkv,code", [(-0.1, 2, 1), (1.5, 2, 1), (float("nan"), 2, 1), (0.2, 33, 2)])
def test_adakv_rejects_bad_arguments(L, safeguard, hkv, code):
    sh = rk.make_shape(1, hkv, hkv, 64, "f32", 64, 13)
    p = rk.BuildParams(300, 16, 16, 4, 0, 0)
    res = [0] * hkv
    assert rk.reskv_build_adakv_workspace_size(sh, p, safeguard, 0, (300,), (64,), res) == 0
    t = FakeTensor()
    with pytest.raises(rk.ReskvError) as ei:
        rk.reskv_build_cache_adakv(sh, p, safeguard, 0, t, t, (300,), t, (64,), res, t, t, t, t, t, t, t,
                                   stream=FakeStream())
    assert ei.value.status == code
    assert rk.last_error()


def test_adakv_rejects_small_workspace(L):
    sh = rk.make_shape(1, 4, 2, 64, "f32", 128, 13)
    p = rk.BuildParams(300, 16, 16, 4, 0, 0)
    t = FakeTensor()
    with pytest.raises(rk.ReskvError) as ei:
        rk.reskv_build_cache_adakv(sh, p, 0.2, 0, t, t, (300,), t, (64,), [13, 0], t, t, t, t, t, t, FakeTensor(8),
                                   stream=FakeStream())
    assert ei.value.status == 3


def test_prepared_decode_call_reports_errors(L):
    """A prepared call validates like the direct call: a bad shape raises
    when it is issued, before anything is launched."""
    t = FakeTensor()
    call = rk.prepare_decode_attn(shape(head_dim=96), rk.make_gate(), t, t, t, t, t, t, t, t, stream=FakeStream())
    with pytest.raises(rk.ReskvError) as ei:
        call()
    assert ei.value.status == 2


def test_static_decode_rejects_shapes_above_its_scratch(L):
    """A shape whose split-K records exceed the 16 MiB static scratch is
    refused before anything is launched (no GPU needed)."""
    sh = rk.make_shape(1, 800, 200, 128, "bf16", 65536, 4096)
    assert rk.reskv_decode_workspace_size(sh) > 16 << 20
    t = FakeTensor()
    with pytest.raises(rk.ReskvError) as ei:
        rk.reskv_decode_attn_static(sh, rk.make_gate(), t, t, t, t, t, t, t, stream=FakeStream())
    assert ei.value.status == 3 and "static scratch" in rk.last_error()
