"""GPU parity at the edges of the launch rules: sizes where a call passes from
one kernel variant to another, each against the fp64 oracle."""

import numpy as np
import pytest

from paper_2607_29591_amd import reskv as rk
from paper_2607_29591_amd import synth
from tests.build_check import check_head, run_build
from tests.test_adakv_gpu import check_sequence, workload as ada_workload
from tests.test_build_gpu import host_copies
from tests.test_decode_branches_gpu import run_case as run_branches
from tests.test_decode_gpu import cache_case, check
from tests.test_decode_ragged_gpu import HEAD, RANGES, SPLIT, run_ragged
from tests.test_launch_rules import proxy_rules
from tests.test_proxy_gpu import GRID, check_proxy, run_proxy
from tests.test_graph_gpu import test_decode_step_graph_replays_match_eager as graph_replays

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d,G,C", [("bf16", 128, 16, 8192), ("bf16", 128, 7, 7937), ("bf16", 64, 5, 7681),
                                         ("f32", 128, 4, 7680), ("bf16", 64, 4, 8200)])
def test_combine_many_records(dtype, d, G, C):
    """31 to 34 split-K records per head, around the record count from which
    the merge of a call without an append is dealt to several blocks; heads
    that fill all, some and one of the records, with and without residuals."""
    Hkv, Rcap = 3, 200
    res = [[0, 200, 3]]
    main = [[C, 700, C - 3]]
    shape, q, kc, vc, logc = cache_case(40 + G, 1, G * Hkv, Hkv, d, dtype, C, Rcap, res, main)
    check(dtype, shape, q, kc, vc, logc, res, main)


@pytest.mark.parametrize("dtype,d,evicted,res,budget", [
    ("bf16", 128, 8192, (128, 3), 160),    # the sorting table of one block exactly full; groups of several pieces
    ("bf16", 64, 8193, (128, 127), 160),   # one token more: offsets and scatter launches
    ("bf16", 128, 1600, (600, 590), 640),  # 25 batches of 600 groups: 15000 of the table's 16384 entries
    ("f32", 64, 1025, (1, 2), 40),         # one and two groups, cut into pieces of 256 members
    ("f32", 128, 1100, (1030, 8), 1060),   # more than 1024 groups: offsets and scatter launches
])
def test_lloyd_sort_and_pieces(dtype, d, evicted, res, budget):
    """Evicted sets and group counts at the edges of the one-block counting
    sort and of the update's pieces (256 members each at these sizes)."""
    s = evicted + budget - max(res)
    wl = synth.tiny_workload(s=s, d=d, hq=4, hkv=2, budget=budget, res=0, window=8, dtype=dtype, n_heavy=6)
    wl.res = np.asarray(res, np.int64).reshape(1, 1, 2)
    x = host_copies(synth.gen_layer(wl, 0, seed=evicted, n_decode=1))
    got = run_build(wl, x)
    for h in range(2):
        check_head(wl, x, got, 0, h)


@pytest.mark.parametrize("dtype,d,G,window,s", [
    ("bf16", 128, 7, 19, 1100),   # 133 rows: the wide row chunk, a short last row tile
    ("bf16", 64, 8, 32, 1025),    # 256 rows: the wide chunk exactly full
    ("bf16", 128, 8, 33, 700),    # 264 rows: a second row chunk
    ("f32", 64, 8, 17, 1030),     # fp32: rows dealt to blocks 16 at a time, 136 rows
    ("f32", 128, 5, 27, 515),     # fp32 rows of 128: 135 rows, two row chunks in the score pass
])
def test_scoring_row_chunks(dtype, d, G, window, s):
    """Window row counts around the row chunks of the scoring passes, short
    contexts whose last chunk is ragged."""
    wl = synth.tiny_workload(s=s, d=d, hq=2 * G, hkv=2, budget=80, res=0, window=window, dtype=dtype, n_heavy=5)
    wl.res = np.asarray((16, 5), np.int64).reshape(1, 1, 2)
    x = host_copies(synth.gen_layer(wl, 0, seed=window, n_decode=1))
    got = run_build(wl, x)
    for h in range(2):
        check_head(wl, x, got, 0, h)


@pytest.mark.parametrize("s,budget,res,recent", [
    (8192 + 8, 200, (60, 0), 8),      # exactly one selection block of scores
    (8193 + 8, 4200, (100, 3), 8),    # one score in the second block, both thresholds deep
    (16385 + 8, 9000, (9, 800), 8),   # thresholds that cross the blocks
    (3 * 8192 - 5, 64, (63, 1), 70),  # all main slots protected: nothing selected, seeds only
    (5001, 5000, (1, 300), 4),        # nearly every score kept; unaligned rows of scores
    (8192, 700, (30, 699), 8),        # the longest list of the one-block selection
    (1024 + 8, 100, (20, 99), 8),     # one score per thread there, and two
    (1025 + 8, 100, (20, 0), 8),
    (65536, 900, (50, 3), 8),         # eight blocks, counted by the placement itself
    (65537, 900, (50, 3), 8),         # nine blocks (by context length): counts in a launch of their own
    (9 * 8192 + 9, 40000, (7, 600), 8),  # ten blocks, one score in the last, both thresholds deep
])
def test_selection_blocks(s, budget, res, recent):
    """Score lists at the edges of the selection's 8192-score blocks, with the
    thresholds high, low and absent; two heads (the second head's scores start
    unaligned where the context length is odd)."""
    wl = synth.tiny_workload(s=s, d=64, hq=4, hkv=2, budget=budget, res=0, window=8, dtype="bf16", n_heavy=6)
    wl.res = np.asarray(res, np.int64).reshape(1, 1, 2)
    x = host_copies(synth.gen_layer(wl, 0, seed=s, n_decode=1))
    got = run_build(wl, x, recent=recent, iters=1)
    for h in range(2):
        check_head(wl, x, got, 0, h, recent=recent, iters=1)


@pytest.mark.parametrize("s,budget", [(20000, 10100), (80000, 45000)])
def test_selection_tied_scores(s, budget):
    """Equal keys give equal scores over several blocks: the lowest positions
    are taken, counted over the blocks before (by the placement itself, and on
    the long list by a launch of its own)."""
    window = 8
    wl = synth.tiny_workload(s=s, d=64, hq=4, hkv=2, budget=budget, res=0, window=window, dtype="bf16", n_heavy=6)
    wl.res = np.asarray((40, 0), np.int64).reshape(1, 1, 2)
    x = synth.gen_layer(wl, 0, seed=3, n_decode=1)
    x["K"][:, :, 200:s - 1000] = x["K"][:, :, 200:201]
    got = run_build(wl, host_copies(x), iters=1)
    for h in range(2):
        check_head(wl, x, got, 0, h, iters=1)


@pytest.mark.parametrize("hkv,ctx,budget,alpha", [
    (5, [9000, 17001], [600, 301], 0.2),   # an odd head count, scores over several blocks, unaligned rows
    (32, [400], [60], 0.0),                # the most heads that share budgets
    (1, [8300], [64], 0.5),                # one head: the search runs against its own cap
])
def test_adakv_search_blocks(hkv, ctx, budget, alpha):
    """The cross-head search over several score blocks and head counts."""
    rng = np.random.default_rng(hkv)
    res = [[int(r) for r in rng.integers(0, b // 2, size=hkv)] for b in budget]
    wl, x = ada_workload(20 + hkv, "bf16", 64, ctx, budget, res, 2 * hkv, hkv)
    C = 2 * max(budget)
    got = run_build(wl, x, adakv=alpha, slot_cap=C)
    for b in range(len(ctx)):
        check_sequence(wl, x, got, b, alpha, C, wl.window, replay_heads=())


@pytest.mark.parametrize("dtype,d,B,Hkv,C,kernels", [
    ("bf16", 128, 1, 2, 640, HEAD), ("bf16", 128, 1, 2, 641, SPLIT),    # ten and eleven units of one head
    ("f32", 64, 1, 2, 512, HEAD), ("f32", 64, 1, 2, 513, SPLIT),
    ("bf16", 64, 16, 4, 1024, HEAD), ("bf16", 64, 16, 4, 1025, SPLIT),  # 64 pairs: two rounds of units, three
    ("bf16", 64, 15, 4, 1024, SPLIT),                                   # one pair count below
    ("f32", 64, 19, 4, 768, SPLIT), ("f32", 64, 20, 4, 768, HEAD),      # fp32 rows, two rounds
    ("bf16", 128, 30, 4, 1280, HEAD), ("bf16", 128, 40, 4, 2305, SPLIT),  # three rounds; past the longest capacity
])
def test_one_block_per_head_line(dtype, d, B, Hkv, C, kernels):
    """Both sides of the line between one block per head and split-K blocks,
    heads from nearly empty to full."""
    rng = np.random.default_rng(C)
    res = rng.integers(0, 200, size=(B, Hkv))
    main = np.array([[int(rng.integers(1, C - r + 1)) for r in row] for row in res])
    main[0, 0] = C - res[0, 0]
    main[0, 1] = 1
    shape, q, kc, vc, logc = cache_case(C, B, 4 * Hkv, Hkv, d, dtype, C, 200, res, main)
    assert rk.decode_kernels(shape) == kernels
    heads = [(0, 0), (0, 4)] + [(int(b), int(h)) for b, h in zip(rng.integers(0, B, 6), rng.integers(0, 4 * Hkv, 6))]
    check(dtype, shape, q, kc, vc, logc, res, main, heads=heads)


def test_split_decode_graph_replays():
    """Graph replays of the split-K path with its append: partial blocks that
    read and store the new token, then the combine, which advances the main
    lengths."""
    graph_replays(2, 2, 7, 900)


@pytest.mark.parametrize("dtype,d,B,Hkv,G,C,longest,appends,kernels", [
    ("bf16", 128, 64, 4, 7, 1536, 1500, True, HEAD),   # the per-head kernels' last capacity at 256 pairs
    ("bf16", 64, 3, 4, 7, 2304, 700, True, SPLIT),     # and their longest capacity, split-K
    ("bf16", 128, 3, 4, 7, 2305, 700, True, RANGES),   # one slot more: fewer units than blocks
    ("f32", 64, 2, 2, 2, 2400, 2390, True, RANGES),    # a head over many one-unit blocks
    ("bf16", 64, 65, 4, 4, 300, 290, True, RANGES),    # 260 pairs
    ("bf16", 64, 65, 4, 1, 300, 290, False, RANGES),   # one query head per KV head, no append
    ("bf16", 128, 24, 4, 4, 1281, 1200, True, RANGES),  # 96 pairs of small groups, a slot past their split-K line
    ("f32", 64, 12, 4, 2, 1025, 1000, False, RANGES),  # 48 pairs of fp32 rows
    ("bf16", 128, 40, 4, 2, 1793, 1700, False, RANGES),  # 160 pairs of up to two query heads
])
def test_ragged_schedule_line(dtype, d, B, Hkv, G, C, longest, appends, kernels):
    """Both sides of the line between the per-head kernels and the equal unit
    ranges of ragged calls."""
    rng = np.random.default_rng(C)
    res = rng.choice([0, 16, 40, 64], size=(B, Hkv))
    main = rng.integers(1, longest - 64, size=(B, Hkv))
    main[0, 0] = longest - res[0, 0]
    run_ragged(dtype, B, Hkv, G, d, C, 64, res, main, seed=C, appends=appends, compare_head=True, kernels=kernels)


@pytest.mark.parametrize("B", [8, 9])
def test_proxy_candidate_batches(B):
    """64 heads: every candidate in one batch; 72 heads: one after the other.
    Each candidate equal to the same construction alone either way."""
    wl = synth.tiny_workload(s=150, d=64, hq=8, hkv=8, budget=40, res=0, window=8, dtype="bf16", batch=B, n_heavy=3)
    wl.ctx = [150 - 7 * b for b in range(B)]
    wl.res = np.full((1, B, 8), 8)
    x = host_copies(synth.gen_layer(wl, 0, seed=B, n_decode=1))
    check_proxy(wl, x, GRID, 2, 0.01, full_heads=[(0, 0), (B - 1, 7)])


@pytest.mark.parametrize("B,Hkv", [(9, 8), (1, 3)])
def test_proxy_candidates_one_after_the_other(B, Hkv):
    """Candidates built one after the other on score lists of several selection
    blocks, whose histograms each candidate must find cleared: 72 heads by the
    rule; 3 heads through a workspace with scratch for one candidate only,
    bit for bit what the batch gives."""
    wl = synth.tiny_workload(s=8600, d=64, hq=Hkv, hkv=Hkv, budget=60, res=0, window=8, dtype="bf16", batch=B, n_heavy=3)
    wl.ctx = [8600 - 41 * b for b in range(B)]
    wl.res = np.full((1, B, Hkv), 12)
    x = host_copies(synth.gen_layer(wl, 0, seed=40 + B, n_decode=1))
    shape = rk.make_shape(B, wl.hq, Hkv, wl.d, "bf16", wl.slot_cap, wl.res_cap)
    params = rk.BuildParams(x["K"].shape[2], wl.window, wl.window, wl.lloyd_iters, 0)
    rules = proxy_rules(shape, params, rk.make_proxy(GRID, 2, 0.01), x["seq_len"], x["budget"])
    assert rules.batched == (1 if B == 9 else len(GRID))
    _, got = check_proxy(wl, x, GRID, 2, 0.01, full_heads=[(0, 0), (B - 1, Hkv - 1)])
    if rules.batched > 1:
        one = run_proxy(wl, x, GRID, 2, 0.01, nws=rules.least_bytes)
        for b in range(B):
            for h in range(Hkv):
                r, n = got["res_len"][b, h], got["main_len"][b, h]
                for k, m in (("kc", r + n), ("vc", r + n), ("logc", None), ("main_idx", n), ("val_loss", None)):
                    np.testing.assert_array_equal(one[k][b, h, :m], got[k][b, h, :m], err_msg=k)
        for k in ("res_len", "main_len"):
            np.testing.assert_array_equal(one[k], got[k])


@pytest.mark.parametrize("dtype,d,G,C,kernels", [("bf16", 128, 7, 600, HEAD), ("f32", 64, 4, 300, HEAD),
                                                 ("bf16", 128, 1, 600, SPLIT), ("bf16", 64, 16, 8300, SPLIT)])
def test_branches_paths(dtype, d, G, C, kernels):
    """Two-branch decode with one block per head, and through records (on the
    longest caches dealt to several merge blocks); a head without residual
    entries and one whose entries may all be empty."""
    assert rk.decode_kernels(rk.make_shape(1, 3 * G, 3, d, dtype, C, 130), "branches") == kernels
    run_branches(C, 1, 3 * G, 3, d, dtype, C, 130, [[0, 130, 1]], [[C - 4, 160, 1]])
