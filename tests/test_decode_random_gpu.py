"""GPU parity of the decode entry points on seeded random shapes (Sec. 5.4
shared-softmax decode, Sec. 5.5.2 gate, App. D Algorithm 2).

Each seed draws a cache geometry (group size, head dim, storage type, slot
capacity, residual capacity, per-head residual and main lengths), a gate, a
per-query or scalar threshold, and whether this step's token is appended in
the call. reskv_decode_attn, reskv_decode_attn_ragged (where its plan
applies: groups up to 8, bf16 or rows of 64) and reskv_decode_attn_static
(where the split records fit its 16 MiB) each run on fresh copies of the
same inputs; for each, every query head is compared with the oracle
decoding the same cache (after the append), to the bar of the other decode
tests, and the appended rows and lengths bit for bit. About half of the
first seeds have 256 (b, kv head) pairs (the one-block-per-head kernel), the
others a few pairs (one block per head or the split kernels, by capacity).
Ten more seeds draw 256 pairs of 520-1400-slot caches with up to 800 residual
entries, so the one-block-per-head kernel streams main blocks past its first
round in its staggered order, residual units run past the first round, and
the block holding slot r is split between the kinds. Twelve more are shapes
of the split kernels and twelve of the equal unit ranges of the ragged entry,
each held to be so.
"""

import numpy as np
import pytest
import torch

from oracle import reskv_oracle as orc
from paper_2607_29591_amd import reskv as rk
from tests.helpers import TOL, random_cache, rel_err_rows, to_dev

pytestmark = pytest.mark.gpu

STATIC_SCRATCH_BYTES = 16 << 20


def draw_case(seed, long_heads=False):
    rng = np.random.default_rng(1000 + seed + (500 if long_heads else 0))
    dtype = ["bf16", "f32"][seed % 2]
    d = [64, 128][(seed // 2) % 2]
    G = int(rng.choice([1, 2, 3, 4, 5, 7, 8, 12, 16]))
    whole = long_heads or ((seed // 4) % 2 == 0 and (dtype == "bf16" or d == 64))
    if long_heads:  # heads past the first round of eight 64-slot blocks
        dtype = "bf16" if d == 128 else dtype
        Hkv = int(rng.choice([1, 2, 4, 8]))
        B = 256 // Hkv
        C = int(rng.integers(520, 1400))
        Rcap = int(rng.integers(1, 800))
    elif whole:
        Hkv = int(rng.choice([1, 2, 4, 8]))
        B = 256 // Hkv
        C = int(rng.integers(8, 360))
        Rcap = int(rng.integers(1, 48))
    else:
        Hkv = int(rng.choice([1, 2, 4]))
        B = int(rng.integers(1, 6))
        C = int(rng.integers(8, 1400))
        Rcap = int(rng.integers(1, 300))
    return (rng, dtype, d, G, B, Hkv, C, Rcap) + draw_rest(rng, B, Hkv, C, Rcap)


def draw_kernels(seed, kernels):
    """Shapes of the split kernels (reskv_decode_attn) or of the equal ranges
    (reskv_decode_attn_ragged): few pairs of longer caches, or more pairs than
    one block per head serves at once."""
    rng = np.random.default_rng(3000 + seed + (100 if kernels == "ranges" else 0))
    dtype, d = [("bf16", 128), ("bf16", 64), ("bf16", 128), ("f32", 64)][seed % 4]
    Hkv = int(rng.choice([1, 2, 4]))
    if kernels == "split":
        G = int(rng.choice([1, 2, 4, 7, 8, 16]))
        B, C = int(rng.integers(1, 9)), int(rng.integers(700, 2600))
    else:
        G = int(rng.choice([1, 2, 3, 4, 7, 8]))
        if seed % 3 == 0:  # more than 256 pairs
            B, C = -(-int(rng.integers(257, 330)) // Hkv), int(rng.integers(64, 700))
        else:
            B, C = int(rng.integers(1, 9)), int(rng.integers(2305, 3400))
    Rcap = int(rng.integers(1, 400))
    return (rng, dtype, d, G, B, Hkv, C, Rcap) + draw_rest(rng, B, Hkv, C, Rcap)


def draw_rest(rng, B, Hkv, C, Rcap):
    res = rng.integers(0, min(Rcap, C - 1) + 1, size=(B, Hkv))
    main = np.array([[int(rng.integers(1, C - r + 1)) for r in row] for row in res])
    gate = dict(tau_scalar=float(rng.uniform(0.05, 0.6)), alpha=float(rng.choice([4.0, 12.0])),
                g_min=float(rng.choice([0.0, 0.2])), beta=float(rng.choice([0.5, 1.0])))
    per_query_tau = bool(rng.integers(0, 2))
    append = bool(rng.integers(0, 2))
    return res, main, gate, per_query_tau, append


@pytest.mark.parametrize("long_heads,seed", [(False, s) for s in range(40)] + [(True, s) for s in range(10)])
def test_decode_random_shape(long_heads, seed):
    check_case(*draw_case(seed, long_heads))


@pytest.mark.parametrize("kernels", ["split", "ranges"])
@pytest.mark.parametrize("seed", range(12))
def test_decode_random_shape_of(kernels, seed):
    case = draw_kernels(seed, kernels)
    _, dtype, d, G, B, Hkv, C, Rcap = case[:8]
    shape = rk.make_shape(B, G * Hkv, Hkv, d, dtype, C, Rcap)
    entry, names = {"split": ("attn", "decode_split + decode_combine"),
                    "ranges": ("ragged", "decode_ragged + decode_ragged_combine")}[kernels]
    assert rk.decode_kernels(shape, entry) == names
    check_case(*case)


def check_case(rng, dtype, d, G, B, Hkv, C, Rcap, res, main, gate, per_query_tau, append):
    Hq = G * Hkv
    kc, vc, logc = random_cache(rng, B, Hkv, C, Rcap, d, dtype, res, main)
    q = rng.normal(size=(B, Hq, d)) * 1.5
    q = np.asarray(torch.as_tensor(q, dtype=torch.float32).to(torch.bfloat16).double()) if dtype == "bf16" else \
        q.astype(np.float32).astype(np.float64)
    tau = rng.normal(0.3, 0.2, size=(B, Hq)) if per_query_tau else None
    shape = rk.make_shape(B, Hq, Hkv, d, dtype, C, Rcap)
    kn = vn = None
    if append:
        kn, vn = rng.normal(size=(B, Hkv, d)), rng.normal(size=(B, Hkv, d))

    # the expected caches and lengths after the call, and the oracle's outputs
    kc2, vc2, main2 = kc.copy(), vc.copy(), main.copy()
    if append:  # the token becomes main slot r + n wherever the cache has room
        knr = to_dev(kn, dtype).double().cpu().numpy()
        vnr = to_dev(vn, dtype).double().cpu().numpy()
        for b in range(B):
            for h in range(Hkv):
                slot = res[b, h] + main[b, h]
                if slot < C:
                    kc2[b, h, slot], vc2[b, h, slot] = knr[b, h], vnr[b, h]
                    main2[b, h] += 1
    t = gate["tau_scalar"] if tau is None else tau.astype(np.float32).astype(np.float64)
    ref, lse_m, lse_r, g = orc.decode(q, kc2, vc2, logc, res, main2, t, gate["alpha"], gate["g_min"], gate["beta"])
    fin = np.isfinite(lse_r)

    entries = ["workspace"]
    if rk.reskv_decode_ragged_workspace_size(shape) > 0:
        entries.append("ragged")
    if rk.reskv_decode_workspace_size(shape) <= STATIC_SCRATCH_BYTES:
        entries.append("static")
    for entry in entries:
        kcd, vcd = to_dev(kc, dtype), to_dev(vc, dtype)
        lcd = torch.as_tensor(logc.astype(np.float32)).cuda()
        rl = torch.as_tensor(res.astype(np.int32).reshape(-1)).cuda()
        ml = torch.as_tensor(main.astype(np.int32).reshape(-1)).cuda()
        out = torch.full((B, Hq, d), float("nan"), device="cuda")
        lm = torch.empty(B * Hq, device="cuda")
        lr = torch.empty(B * Hq, device="cuda")
        gt = torch.empty(B * Hq, device="cuda")
        taud = None if tau is None else torch.as_tensor(tau.astype(np.float32).reshape(-1)).cuda()
        knd = to_dev(kn, dtype) if append else None
        vnd = to_dev(vn, dtype) if append else None
        args = (shape, rk.make_gate(tau=taud, **gate), to_dev(q, dtype), kcd, vcd, lcd, rl, ml, out)
        if entry == "workspace":
            ws = torch.zeros(rk.reskv_decode_workspace_size(shape), dtype=torch.uint8, device="cuda")
            rk.reskv_decode_attn(*args, ws, lm, lr, gt, k_new=knd, v_new=vnd)
        elif entry == "ragged":
            ws = torch.zeros(rk.reskv_decode_ragged_workspace_size(shape), dtype=torch.uint8, device="cuda")
            rk.reskv_decode_attn_ragged(*args, ws, lm, lr, gt, k_new=knd, v_new=vnd)
        else:
            rk.reskv_decode_attn_static(*args, lm, lr, gt, k_new=knd, v_new=vnd)
        torch.cuda.synchronize()

        np.testing.assert_array_equal(ml.cpu().numpy().reshape(B, Hkv), main2, err_msg=entry)
        np.testing.assert_array_equal(kcd.double().cpu().numpy(), kc2, err_msg=entry)
        np.testing.assert_array_equal(vcd.double().cpu().numpy(), vc2, err_msg=entry)
        got = out.double().cpu().numpy()
        assert np.isfinite(got).all(), entry
        err = rel_err_rows(got, ref)
        assert err.max() <= TOL[dtype], f"{entry}: max rel err {err.max():.3e}"
        np.testing.assert_allclose(gt.double().cpu().numpy().reshape(B, Hq), g, rtol=1e-5, atol=1e-6, err_msg=entry)
        np.testing.assert_allclose(lm.double().cpu().numpy().reshape(B, Hq), lse_m, rtol=1e-5, atol=1e-5,
                                   err_msg=entry)
        got_lr = lr.double().cpu().numpy().reshape(B, Hq)
        assert (np.isfinite(got_lr) == fin).all(), entry
        np.testing.assert_allclose(got_lr[fin], lse_r[fin], rtol=1e-5, atol=1e-5, err_msg=entry)
