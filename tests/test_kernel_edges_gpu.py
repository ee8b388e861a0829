"""Kernels and dispatch branches at the sizes where they can go wrong (tile edges, remainders, ends of a range), against
the oracle.  Tolerances are those of the other parity tests: routing bit for bit, outputs TOL_BF16 / TOL_F32 of RMS."""
from dataclasses import replace

import pytest

import lexi_synth as S
from helpers import run_and_check_layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,k,d,F", [
    (1, 1, 128, 64),      # fewer K blocks than waves (down: 2), one row
    (15, 8, 128, 64), (16, 8, 128, 192), (17, 8, 256, 64),       # every expert: around one 16-row block
    (33, 8, 128, 320), (65, 8, 384, 64), (129, 8, 128, 64),      # 2 -> 4 -> 8 row blocks, a second tile of one row
    (300, 3, 128, 128),
])
@pytest.mark.parametrize("shared", [S.SHARED_NONE, S.SHARED_SIGMOID])
def test_fp32_layers_at_tile_edges(T, k, d, F, shared):
    cfg = replace(S.mini(S.C1, L=1, d=d, F=F, F_shared=0), F_shared=192 if shared else 0, shared_kind=shared)
    run_and_check_layer(cfg, 0, T, k)


@pytest.mark.parametrize("k_base,n_k,T", [(1, 1, 3), (3, 7, 40), (5, 8, 40), (6, 9, 40), (9, 17, 33), (64, 64, 17)])
def test_profile_list_lengths_around_a_group(k_base, n_k, T):
    """Listed k are taken eight at a time, slots four at a time: lists and baselines around multiples of both, the same
    k in several groups, against single-k calls (bit for bit: an entry does not depend on its neighbours) and the
    oracle's deltas (relative 5e-3, the bound derived in test_profile_gpu.py)."""
    import numpy as np
    import torch
    import oracle as O
    import paper_2509_02753_amd as P
    from helpers import device_and_host_layer
    cfg = S.mini(S.C2, L=1, d=256, F=128)
    dl, hl = device_and_host_layer(cfg, 0)
    x, xh = S.device_x(cfg, 0, T), S.host_x(cfg, 0, T)
    ks = [1 + (5 * i) % k_base for i in range(n_k)]
    got = P.lexi_moe_profile_layer(dl, x, k_base, ks)
    for i in {0, n_k // 2, n_k - 1}:
        assert torch.equal(got[i:i + 1], P.lexi_moe_profile_layer(dl, x, k_base, ks[i:i + 1]))
    ref = O.profile_layer(hl, xh, k_base, ks, round_act=True)
    scale = float(np.sqrt(np.sum(O.moe_layer(hl, xh, k_base, round_act=True).out ** 2)))
    for i, k in enumerate(ks):
        assert abs(float(got[i]) - ref[i]) <= 5e-3 * ref[i] + 1e-6 * scale
        assert k != k_base or float(got[i]) == 0.0


@pytest.mark.parametrize("T", [16, 17, 64, 65, 67, 1024, 1025, 1169])
@pytest.mark.parametrize("E,d,k,kind", [(1, 128, 1, "c1"), (8, 2176, 8, "c2"), (16, 256, 3, "c2"), (17, 1280, 5, "c2"),
                                        (60, 2048, 4, "c2"), (60, 640, 4, "c1"), (64, 384, 64, "c2")])
def test_router_at_block_and_segment_edges(T, E, d, k, kind):
    """Every router route at the ends of its range of T, one expert to 64 (the narrow form's last 16, and 17), segment
    counts around a pass of 16; bf16 (c2) and fp32 (c1) layers.  The routing is compared bit for bit.  (The fp32 layers stay
    below d = 1024: an expert GEMM is one chain of K fp32 fused multiply-adds, whose rounding is about 2^-24 * sqrt(K) / 2 of
    the result's RMS, five times that at the largest of 10^6 outputs: 7e-6 at K = 2048, and the product of two such values
    would exceed TOL_F32 = 1e-5 there.)"""
    cfg = replace(S.mini(S.C1 if kind == "c1" else S.C2, L=1, d=d, F=64, F_shared=0), E=E)
    run_and_check_layer(cfg, 0, T, k)


@pytest.mark.parametrize("T,E,d,k,kind", [
    (1030, 17, 128, 1, "c1"), (2048, 64, 2176, 8, "c2"), (2049, 33, 4224, 3, "c2"), (2055, 64, 640, 64, "c1"), (4111, 17, 2048, 4, "c2"),
    (12288, 40, 128, 2, "c2"), (12289, 40, 128, 2, "c2")])
def test_router_of_a_thousand_tokens_and_more_at_its_edges(T, E, d, k, kind):
    """Router and selection in one launch: 8 tokens per workgroup up to 2048, 16 above, partials through memory from 12289 on; a ragged last
    workgroup, one segment to 33 (two passes of 16 waves and one more), rows of W of 17 to 64 floats.  The routing is compared bit for bit."""
    cfg = replace(S.mini(S.C1 if kind == "c1" else S.C2, L=1, d=d, F=64, F_shared=0), E=E)
    run_and_check_layer(cfg, 0, T, k, tokens=[0, T // 2, T - 1])


def route(dl, T, k, gemm):
    """How a routed GEMM of a call is launched, as "<tile height> rows x<waves>" or "stream x<waves>"."""
    import paper_2509_02753_amd as P
    p = P.lexi_moe_gemm_plan(dl, T, k, gemm)
    if p["fused"]:
        return "fused"
    if p["streams"]:
        return f"stream x{p['waves']}"
    return f"{p['tile_rows']} rows x{p['waves']}" + (" cut" if p["ksplit"] > 1 else "") + (" direct" if p["direct"] else "")


@pytest.mark.parametrize("T,k,E,d,F,zipf,gate_up,down", [
    # few items: low tiles, four waves, whatever the sizes
    (161, 1, 1, 128, 64, 0.0, "64 rows x4", "64 rows x4 direct"), (160, 1, 1, 640, 192, 0.0, "64 rows x4", "64 rows x4 direct"),
    (320, 2, 2, 512, 128, 0.0, "64 rows x4", "64 rows x4"), (321, 2, 2, 1152, 128, 0.0, "64 rows x4", "64 rows x4"),
    (1100, 2, 8, 1152, 320, 0.0, "64 rows x4", "64 rows x4"),        # both column blocks of the last pair half empty
    (1030, 1, 8, 512, 128, 1.0, "64 rows x4", "64 rows x4 direct"),
    (1100, 3, 16, 256, 1024, 1.5, "128 rows x4", "64 rows x4"),       # skewed: tall experts, others with a handful of rows
    (700, 4, 64, 384, 2048, 2.0, "64 rows x4", "64 rows x4 cut"),     # more skewed, reduction cut in two
    (130, 2, 3, 256, 4096, 0.0, "64 rows x4", "64 rows x4 cut"),      # 87 rows per expert, few items
    (40, 2, 8, 256, 448, 0.0, "64 rows x4", "stream x8"),             # 10 rows per expert, few units
    (130, 3, 3, 512, 576, 0.0, "64 rows x4", "64 rows x4"), (65, 2, 2, 512, 576, 0.0, "96 rows x4", "96 rows x4"),
    # every expert: 15 whole tiles of 160 rows, one row more, and tiles of 9 and 10 blocks; the last of the eight-wave form's
    # column blocks of 512 holds 128 features
    (2400, 8, 8, 1664, 192, 0.0, "160 rows x4", "160 rows x8"), (2401, 8, 8, 1664, 192, 0.0, "160 rows x4", "160 rows x8"),
    (2380, 8, 8, 1664, 192, 0.0, "160 rows x4", "160 rows x8"), (2300, 8, 8, 1664, 192, 0.0, "160 rows x4", "128 rows x4"),
    (1280, 8, 8, 1152, 64, 0.0, "64 rows x4", "128 rows x8"), (1281, 8, 8, 1152, 64, 0.0, "64 rows x4", "128 rows x8"),
    # four waves at 160 rows, the last gate/up column block half empty
    (800, 8, 16, 1152, 448, 0.0, "160 rows x4", "160 rows x4"), (1999, 8, 16, 512, 192, 1.1, "160 rows x4", "64 rows x4"),
    # output rows stored directly: from eight waves (a ragged last column block), from four at 160 rows
    (4001, 1, 8, 3200, 64, 0.0, "64 rows x4", "128 rows x8 direct"), (4001, 1, 16, 3200, 128, 1.0, "64 rows x4", "160 rows x8 direct"),
    (4000, 1, 1, 2176, 64, 0.0, "64 rows x4", "160 rows x4 direct"),
])
def test_grouped_gemm_tiles(T, k, E, d, F, zipf, gate_up, down):
    """Every form of the tile schedule at the edges of its tiles and column blocks, against the oracle (routing bit for bit,
    TOL_BF16 of RMS; above 1100 tokens the outputs of 64 of them)."""
    import numpy as np
    from helpers import device_and_host_layer
    cfg = replace(S.mini(S.C5 if zipf else S.C2, L=1, d=d, F=F, F_shared=0), E=E, F_shared=0, shared_kind=S.SHARED_NONE)
    if zipf:
        cfg = replace(cfg, zipf_s=zipf)
    dl, _ = device_and_host_layer(cfg, 0)
    assert (route(dl, T, k, "gate_up"), route(dl, T, k, "down")) == (gate_up, down)
    del dl
    tokens = None
    if T > 1100:
        tokens = np.unique(np.concatenate([[0, 1, T - 2, T - 1], np.random.default_rng(T).integers(0, T, 60)])).astype(np.int32)
    run_and_check_layer(cfg, 0, T, k, tokens=tokens)


@pytest.mark.parametrize("T,k,E,d,F,gate_up,down", [
    (4, 4, 64, 2048, 1408, "stream x4", "fused"), (6, 1, 64, 2048, 1408, "stream x4", "fused"),
    (16, 4, 64, 256, 1408, "stream x4", "stream x4"), (20, 4, 64, 2048, 128, "stream x4", "stream x4"),
    (2, 6, 64, 1024, 2816, "stream x4", "fused"), (33, 2, 64, 2048, 1408, "stream x4", "stream x4"),
    (16, 1, 8, 2304, 8192, "stream x4", "stream x8"),        # a reduction of 8192: eight waves per unit
    (17, 8, 64, 256, 1408, "64 rows x4", "stream x4"),       # just above two rows per expert
    (33, 4, 64, 2048, 128, "64 rows x4", "64 rows x4"),
    (21, 3, 3, 640, 2624, "64 rows x4", "stream x8"), (64, 2, 2, 512, 576, "64 rows x4", "stream x8"),   # few units, 2 and 4 blocks
    (120, 2, 2, 384, 448, "64 rows x4", "stream x8"),        # 8 blocks, a short reduction
])
def test_decode_schedules_around_their_limits(T, k, E, d, F, gate_up, down):
    """Decode-sized calls on either side of the lines between weight streaming and tiles, against the oracle."""
    from helpers import device_and_host_layer
    cfg = replace(S.mini(S.C2, L=1, d=d, F=F, F_shared=0), E=E)
    dl, _ = device_and_host_layer(cfg, 0)
    assert (route(dl, T, k, "gate_up"), route(dl, T, k, "down")) == (gate_up, down)
    del dl
    run_and_check_layer(cfg, 0, T, k)


@pytest.mark.parametrize("T,k,d,F,Fs", [
    # the list of reduction steps dealt out over the waves: fewer steps than waves, parts of three experts in one share, a
    # shared expert longer and shorter than the routed ones, none; 8 features per workgroup up to d = 2048, 16 above
    (1, 1, 2048, 64, 0), (1, 1, 2176, 64, 64), (1, 2, 2048, 192, 64), (3, 6, 2048, 64, 2816), (8, 8, 2048, 64, 64),
    (8, 8, 2176, 128, 1408), (2, 3, 4096, 1408, 0), (1, 8, 2176, 1024, 128), (8, 1, 128, 704, 320), (7, 6, 2176, 64, 0),
])
def test_down_and_combine_in_one_launch_at_its_edges(T, k, d, F, Fs):
    """A handful of tokens: every way the reduction steps of the experts in use fall on the waves, against the oracle."""
    import paper_2509_02753_amd as P
    from helpers import device_and_host_layer
    cfg = replace(S.mini(S.C5, L=1, d=d, F=F), F_shared=Fs, shared_kind=S.SHARED_UNGATED if Fs else S.SHARED_NONE)
    dl, _ = device_and_host_layer(cfg, 0)
    assert route(dl, T, k, "down") == "fused"
    assert not Fs or P.lexi_moe_gemm_plan(dl, T, k, "down", shared=True)["waves"] == (8 if d <= 2048 else 16)
    del dl
    run_and_check_layer(cfg, 0, T, k)


def _with_router(cfg, w_scale, x, dtype):
    """The seeded layer of `cfg` with its router weights scaled, and x, on device and host."""
    import numpy as np
    import torch
    import oracle as O
    import paper_2509_02753_amd as P
    host = S.host_layer(cfg, 0)
    host["w_router"] = (host["w_router"] * np.float32(w_scale)).astype(np.float32)
    dev = S.device_layer(cfg, 0)
    dev["w_router"] = torch.from_numpy(host["w_router"]).cuda()
    xd = torch.from_numpy(x).cuda().to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    xh = xd.view(torch.int16).cpu().numpy().view(np.uint16) if dtype == "bf16" else xd.cpu().numpy()
    return P.Layer.from_tensors(dev, shared_kind=cfg.shared_kind), O.Layer.from_tensors(cfg, host), xd, xh


def _route(dl, xd, k, E):
    import torch
    import paper_2509_02753_amd as P
    T = xd.shape[0]
    rout = P.RoutingOut(T, k, E)
    P.lexi_moe_layer_forward(dl, xd, torch.empty((T, xd.shape[1]), dtype=torch.float32, device="cuda:0"), k,
                             P.alloc_workspace([dl], T, k), routing=rout)
    torch.cuda.synchronize()
    return rout


# one T in the range of every router kernel: whole segments per wave (64), router and top-k in one launch, partials through
# memory -- the last in its wide and its narrow form (up to 16 experts)
ROUTER_RANGES = [(64, 64), (65, 64), (1024, 17), (1025, 64), (1100, 17), (1100, 16), (1025, 5)]


@pytest.mark.parametrize("T,E", ROUTER_RANGES)
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_router_keeps_subnormal_products_and_sums(T, E, dtype):
    """Products around 2^-142 and sums of 256 of them around 2^-138: every multiply-add rounds to a multiple of 2^-149, and
    the order of the experts hangs on some thousand such steps.  Selection bit for bit as fmaf gives it; a kernel that
    flushed them would select experts 0..k-1 everywhere."""
    import numpy as np
    import oracle as O
    from helpers import check_routing
    cfg = replace(S.mini(S.C1 if dtype == "f32" else S.C2, L=1, d=256, F=64, F_shared=0), E=E)
    x = np.random.default_rng(T + E).standard_normal((T, cfg.d)).astype(np.float32) * np.float32(2.0 ** -56)
    dl, hl, xd, xh = _with_router(cfg, 2.0 ** -80, x, dtype)
    k = min(4, E)
    ref = O.moe_layer(hl, xh, k, routing_only=True)
    # (64 tokens that prefer one of 64 experts at random reach 40 of them)
    assert 0.0 < np.abs(ref.logits).max() < 2.0 ** -126 and len(np.unique(ref.topk_idx[:, 0])) >= E // 3
    check_routing(_route(dl, xd, k, E), ref)


@pytest.mark.parametrize("T,E", [(2049, 64), (12289, 17)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_router_of_many_tokens_keeps_subnormal_products_and_sums(T, E, dtype):
    test_router_keeps_subnormal_products_and_sums(T, E, dtype)


@pytest.mark.parametrize("T,E", ROUTER_RANGES)
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_router_with_infinite_and_nan_activations(T, E, dtype):
    """Two infinite activations leave a token's logits at +inf, -inf and NaN (both signs), one NaN all at NaN.  The logits are
    those of the fmaf chain and a NaN ranks as -inf; every other token is routed as usual."""
    import numpy as np
    import oracle as O
    from helpers import to_numpy
    cfg = replace(S.mini(S.C1 if dtype == "f32" else S.C2, L=1, d=256, F=64, F_shared=0), E=E)
    x = np.random.default_rng(T * E).standard_normal((T, cfg.d)).astype(np.float32)
    x[3, 5], x[3, 200] = np.inf, np.inf
    x[T - 1, 77] = np.nan
    dl, hl, xd, xh = _with_router(cfg, 1.0, x, dtype)
    k = min(6, E)
    logits = O.moe_layer(hl, xh, k, routing_only=True).logits
    assert np.isnan(logits[3]).any() and np.isinf(logits[3]).any() and np.isnan(logits[T - 1]).all()
    want = np.argsort(-np.where(np.isnan(logits), -np.inf, logits), axis=1, kind="stable")[:, :k]
    rout = _route(dl, xd, k, E)
    assert np.array_equal(to_numpy(rout.topk_idx), want)
    assert np.array_equal(np.sort(to_numpy(rout.perm)), np.arange(T * k))
    g = to_numpy(rout.gates)
    keep = ~np.isin(np.arange(T), (3, T - 1))
    assert np.isnan(g[~keep]).all() and np.abs(g[keep].sum(axis=1) - 1.0).max() <= 1e-5


@pytest.mark.parametrize("scale", [1.0, 2.0 ** -70])
def test_fp32_down_gemm_is_one_ascending_chain_of_fmaf(scale):
    """One expert, gate exactly 1: the output rows are the down GEMM's.  Token t is the unit vector e_t and the gate weights
    are all 64 (silu(64) is 64: 1 + exp(-64) rounds to 1), so its intermediate is 64 * W_up[:, t] exactly, and every output
    equals the chain of fmaf from the C library bit for bit -- with subnormal products and sums at the small scale."""
    import ctypes
    import numpy as np
    import torch
    import paper_2509_02753_amd as P
    T, d, F = 5, 128, 192
    rng = np.random.default_rng(7)
    w_up = (rng.standard_normal((F, d)) * scale).astype(np.float32)
    w_down = (rng.standard_normal((d, F)) * scale).astype(np.float32)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()
    dl = P.Layer.from_tensors(dict(w_router=dev(np.zeros((d, 1))), w_gate=dev(np.full((1, F, d), 64.0)), w_up=dev(w_up[None]),
                                   w_down=dev(w_down[None])))
    y = torch.empty((T, d), dtype=torch.float32, device="cuda:0")
    P.lexi_moe_layer_forward(dl, dev(np.eye(T, d)), y, 1, P.alloc_workspace([dl], T, 1))
    torch.cuda.synchronize()
    fmaf = ctypes.CDLL("libm.so.6").fmaf
    fmaf.restype, fmaf.argtypes = ctypes.c_float, [ctypes.c_float] * 3
    want = np.zeros((T, d), dtype=np.float32)
    for t in range(T):
        act = [float(v) for v in np.float32(64.0) * w_up[:, t]]
        for j in range(d):
            acc = 0.0
            for a, w in zip(act, w_down[j].tolist()):
                acc = fmaf(a, w, acc)
            want[t, j] = acc
    assert scale == 1.0 or 0.0 < np.abs(want).max() < 2.0 ** -126
    assert np.array_equal(y.cpu().numpy().view(np.int32), want.view(np.int32))


@pytest.mark.parametrize("T,k,E,d", [
    (1, 1, 1, 128), (1, 64, 64, 256), (2, 2, 16, 2048), (3, 5, 17, 2176), (4, 8, 60, 1920), (5, 1, 64, 4096), (7, 16, 64, 384),
    (8, 8, 60, 2048), (8, 16, 64, 2304), (9, 7, 64, 384), (12, 2, 17, 2176), (13, 1, 8, 128), (16, 8, 64, 2048),
])
@pytest.mark.parametrize("zipf", [0.0, 1.1])
def test_selection_inside_the_gate_up_launch(T, k, E, d, zipf):
    """Up to 16 tokens every workgroup of the gate/up launch selects for itself: one to 16 tokens, one to 64 experts, one
    segment of the router up to 32, around the 16 requested together; routing bit for bit, outputs, both as one layer and as a
    block of the chained stack (where the down GEMM reads the expert table too), against the oracle."""
    import torch
    import oracle as O
    import paper_2509_02753_amd as P
    from helpers import check_routing, device_and_host_layer, rel_err, TOL_BF16
    cfg = replace(S.mini(S.C5 if zipf else S.C2, L=1, d=d, F=128, F_shared=0), E=E, F_shared=0, shared_kind=S.SHARED_NONE)
    run_and_check_layer(cfg, 0, T, k)
    dl, hl = device_and_host_layer(cfg, 0)
    assert P.lexi_moe_gemm_plan(dl, T, k, "gate_up", chained=True)["streams"] == 1
    x = S.device_x(cfg, 0, T)
    y = torch.empty((T, d), dtype=torch.float32, device="cuda:0")
    rout = P.RoutingOut(T, k, E, moe_input=torch.empty_like(x))
    P.lexi_moe_stack_forward([dl], [k], x, y, P.alloc_workspace([dl], T, k), routing=[rout], chained=True)
    torch.cuda.synchronize()
    u = rout.moe_input.view(torch.int16).cpu().numpy().view("uint16")
    ref = O.moe_layer(hl, u, k, round_act=True)
    check_routing(rout, ref)
    assert rel_err(y.cpu().numpy() - x.float().cpu().numpy(), ref.out) <= TOL_BF16


@pytest.mark.parametrize("T,E", [(8, 64), (5, 17), (8, 5), (16, 40)])
def test_selection_inside_the_gate_up_launch_with_infinite_and_nan_logits(T, E):
    import numpy as np
    import oracle as O
    from helpers import to_numpy
    cfg = replace(S.mini(S.C2, L=1, d=256, F=64, F_shared=0), E=E)
    x = np.random.default_rng(T * E).standard_normal((T, cfg.d)).astype(np.float32)
    x[3, 5], x[3, 200] = np.inf, np.inf
    x[T - 1, 77] = np.nan
    dl, hl, xd, xh = _with_router(cfg, 1.0, x, "bf16")
    k = 1 if E < 8 else 2
    logits = O.moe_layer(hl, xh, k, routing_only=True).logits
    want = np.argsort(-np.where(np.isnan(logits), -np.inf, logits), axis=1, kind="stable")[:, :k]
    rout = _route(dl, xd, k, E)
    assert np.array_equal(to_numpy(rout.topk_idx), want)
    assert np.array_equal(np.sort(to_numpy(rout.perm)), np.arange(T * k))


@pytest.mark.parametrize("T,k,E,d,kind", [
    # all routing in one workgroup: one to 64 tokens (a wave's four partly there), one to three segments, one to 64 experts, on
    # both sides of the line to the three launches
    (1, 1, 1, 128, "c1"), (3, 60, 60, 128, "c1"), (64, 3, 8, 128, "c1"), (64, 3, 64, 128, "c2"), (63, 4, 64, 128, "c1"), (5, 2, 17, 384, "c1"),
    (21, 3, 5, 384, "c2"), (24, 5, 40, 256, "c1"), (33, 1, 64, 256, "c2"), (21, 4, 5, 384, "c1"), (50, 1, 8, 256, "c1"),
])
def test_routing_in_one_workgroup(T, k, E, d, kind):
    cfg = replace(S.mini(S.C1 if kind == "c1" else S.C2, L=1, d=d, F=64, F_shared=0), E=E)
    run_and_check_layer(cfg, 0, T, k)


@pytest.mark.parametrize("T,k,E,d,F,Fs,routed,shared", [
    # the two jobs of a GEMM launch, as (gate/up, down) of each: both stream; routed streams beside shared tiles; the other way round;
    # tiles of both, low, of 96 rows and tall; eight waves; more than 1024 tokens, together and one after the other
    (20, 2, 64, 256, 192, 320, ("stream x4", "stream x4"), ("stream x4", "stream x4")),
    (100, 1, 64, 256, 192, 320, ("stream x4", "stream x4"), ("128 rows x4", "64 rows x4")),
    (40, 4, 60, 384, 192, 704, ("64 rows x4", "stream x4"), ("stream x4", "stream x4")),
    (40, 8, 8, 1024, 448, 320, ("64 rows x4", "64 rows x4"), ("stream x4", "stream x4")),
    (200, 4, 60, 384, 192, 2048, ("64 rows x4", "64 rows x4"), ("64 rows x4", "64 rows x4 cut")),
    (65, 2, 2, 512, 576, 64, ("96 rows x4", "96 rows x4"), ("96 rows x4", "96 rows x4")),
    (800, 8, 16, 1152, 448, 320, ("160 rows x4", "160 rows x4"), ("160 rows x4", "160 rows x4")),
    (1000, 4, 4, 4096, 192, 192, ("64 rows x4", "160 rows x8"), ("64 rows x4", "128 rows x8")),
    (2401, 8, 8, 1664, 192, 192, ("160 rows x4", "160 rows x8"), ("160 rows x4", "96 rows x4")),
    (1100, 2, 16, 256, 192, 320, ("64 rows x4", "64 rows x4"), ("160 rows x4", "64 rows x4")),
    # the shared reduction cut in two in eight-wave workgroups; selection in the gate/up launch, of four and of eight waves
    (1000, 4, 4, 4096, 192, 2048, ("64 rows x4", "160 rows x8"), ("64 rows x4", "128 rows x8 cut")),
    (9, 3, 60, 384, 1408, 704, ("stream x4", "stream x4"), ("stream x4", "stream x4")),
    (12, 2, 64, 256, 192, 320, ("stream x4", "stream x4"), ("stream x4", "stream x4")),
    (16, 1, 16, 256, 64, 320, ("stream x8", "stream x8"), ("stream x8", "stream x8")),
])
@pytest.mark.parametrize("kind", [S.SHARED_UNGATED, S.SHARED_SIGMOID])
def test_shared_expert_as_second_job_of_the_routed_launches(T, k, E, d, F, Fs, routed, shared, kind):
    """Every combination of schedules the routed and the shared expert's GEMMs meet in, against the oracle."""
    import numpy as np
    import paper_2509_02753_amd as P
    from helpers import device_and_host_layer
    cfg = replace(S.mini(S.C2, L=1, d=d, F=F), E=E, F_shared=Fs, shared_kind=kind)
    dl, _ = device_and_host_layer(cfg, 0)
    for gemm, want, want_shared in zip(("gate_up", "down"), routed, shared):
        for sh, w in ((False, want), (True, want_shared)):
            p = P.lexi_moe_gemm_plan(dl, T, k, gemm, shared=sh)
            got = f"stream x{p['waves']}" if p["streams"] else f"{p['tile_rows']} rows x{p['waves']}" + (" cut" if p["ksplit"] > 1 else "")
            assert w is None or got == w, (gemm, sh, got)
    del dl
    tokens = None
    if T > 1000:
        tokens = np.unique(np.concatenate([[0, 1, T - 2, T - 1], np.random.default_rng(T).integers(0, T, 60)])).astype(np.int32)
    run_and_check_layer(cfg, 0, T, k, tokens=tokens)


def _random_layer(d, E, F, Fs, seed, zero=()):
    """An ungated layer of seeded weights (the same ones for the same seed and sizes), those named in `zero` all 0."""
    import torch
    import paper_2509_02753_amd as P
    t = {}
    shapes = dict(w_router=(d, E), w_gate=(E, F, d), w_up=(E, F, d), w_down=(E, d, F))
    if Fs:
        shapes.update(ws_gate=(Fs, d), ws_up=(Fs, d), ws_down=(d, Fs))
    for n, shape in shapes.items():
        gen = torch.Generator(device="cuda:0").manual_seed(seed + sum(map(ord, n)))
        w = torch.empty(shape, device="cuda:0").normal_(0.0, 0.05, generator=gen)
        t[n] = w if n == "w_router" else (w * (n not in zero)).to(torch.bfloat16)
    return P.Layer.from_tensors(t)


def _forward(dl, x, k):
    import torch
    import paper_2509_02753_amd as P
    y = torch.empty((x.shape[0], dl.d), dtype=torch.float32, device="cuda:0")
    P.lexi_moe_layer_forward(dl, x, y, k, P.alloc_workspace([dl], x.shape[0], k))
    torch.cuda.synchronize()
    return y


@pytest.mark.parametrize("T,d,Fs", [(9, 256, 320), (16, 2176, 2816), (20, 256, 64), (33, 384, 704), (64, 2048, 1408), (64, 128, 4160)])
def test_streamed_shared_expert_does_not_depend_on_the_routed_ones(T, d, Fs):
    """Rows of the shared expert, bit for bit, beside routed experts of any number and width: in launches of four and eight waves and
    beside tiles.  (Routed down weights of 0 leave the output to the shared expert.)"""
    import torch
    x = torch.empty((T, d), device="cuda:0").normal_(generator=torch.Generator(device="cuda:0").manual_seed(T)).to(torch.bfloat16)
    want = _forward(_random_layer(d, 64, 64, Fs, 3, zero=("w_down",)), x, 1)
    assert float(want.abs().max()) > 0.0
    # few units: eight waves; many: four; more than two rows per expert: tiles
    for E, F, k in ((16, 64, 1), (64, 1408, 1), (4, 192, 3), (8, 1408, 8)):
        assert torch.equal(_forward(_random_layer(d, E, F, Fs, 3, zero=("w_down",)), x, k), want), (E, F, k)


@pytest.mark.parametrize("T,k,E,d,F", [
    (9, 2, 16, 256, 64), (16, 2, 16, 1152, 128), (24, 2, 24, 128, 64), (40, 3, 3, 640, 2624), (64, 2, 2, 512, 576),
    (70, 1, 40, 128, 64), (120, 2, 2, 384, 448),     # beside shared tiles; the last of up to 120 rows per expert
])
def test_streamed_routed_experts_do_not_depend_on_the_shared_one(T, k, E, d, F):
    """The same for the routed experts beside shared ones of several widths, against the layer without one."""
    import torch
    import paper_2509_02753_amd as P
    x = torch.empty((T, d), device="cuda:0").normal_(generator=torch.Generator(device="cuda:0").manual_seed(T)).to(torch.bfloat16)
    alone = _random_layer(d, E, F, 0, 5)
    assert P.lexi_moe_gemm_plan(alone, T, k, "down")["streams"] == 1
    want = _forward(alone, x, k)
    for Fs in (64, 704, 5632):
        assert torch.equal(_forward(_random_layer(d, E, F, Fs, 5, zero=("ws_down",)), x, k), want), Fs


@pytest.mark.parametrize("T,k,E,d,F,Fs", [(1, 6, 64, 2048, 1408, 2816), (8, 6, 64, 2048, 1408, 2816), (4, 4, 60, 2048, 1408, 5632),
                                          (4, 4, 64, 1280, 896, 1792), (8, 2, 8, 4096, 14336, 0), (5, 2, 32, 2560, 4544, 1216)])
def test_down_and_combine_in_one_launch_sums_in_short_chains(T, k, E, d, F, Fs):
    """fp32 rounding of the fused launch alone: token t is the unit vector e_t and all gate weights are 64, so an intermediate is
    64 * w_up[:, t] exactly (a bf16 number).  A sum of n MFMA steps in c chains rounds about n / c * n / 2 partial sums, each at
    up to 2^-24 of its size, so its error grows with sqrt(n / c): in eight parts or more it is 0.9e-7 to 1.3e-7 at n = 88
    (seen here: 0.9e-7 to 1.1e-7), in the one or two chains of a wave's whole share 1.6e-7 to 5e-7."""
    import torch
    import paper_2509_02753_amd as P
    gen = torch.Generator(device="cuda:0").manual_seed(11)
    normal = lambda *s: torch.empty(s, device="cuda:0").normal_(0.0, 0.02, generator=gen)
    full = lambda *s: torch.full(s, 64.0, device="cuda:0").to(torch.bfloat16)
    t = dict(w_router=normal(d, E), w_gate=full(E, F, d), w_up=normal(E, F, d).to(torch.bfloat16), w_down=normal(E, d, F).to(torch.bfloat16))
    if Fs:
        t.update(ws_gate=full(Fs, d), ws_up=normal(Fs, d).to(torch.bfloat16), ws_down=normal(d, Fs).to(torch.bfloat16))
    dl = P.Layer.from_tensors(t)
    assert P.lexi_moe_gemm_plan(dl, T, k, "down")["fused"] == 1
    x = torch.eye(T, d, device="cuda:0").to(torch.bfloat16)
    y, rout = torch.empty((T, d), dtype=torch.float32, device="cuda:0"), P.RoutingOut(T, k, E)
    P.lexi_moe_layer_forward(dl, x, y, k, P.alloc_workspace([dl], T, k), routing=rout)
    torch.cuda.synchronize()
    want = torch.zeros((T, d), dtype=torch.float64, device="cuda:0")
    for i in range(T):
        for s in range(k):
            e = int(rout.topk_idx[i, s])
            want[i] += rout.gates[i, s].double() * (t["w_down"][e].double() @ (64.0 * t["w_up"][e, :, i].double()))
        if Fs:
            want[i] += t["ws_down"].double() @ (64.0 * t["ws_up"][:, i].double())
    assert float((y.double() - want).norm() / want.norm()) <= 1.4e-7


@pytest.mark.parametrize("T,Fs", [(3, 320), (8, 64), (3, 0), (12, 320), (40, 320), (200, 320)])
def test_stage_events_are_recorded_in_their_order(T, Fs):
    """"Shared expert done" lies behind the launch that holds its down projection, also where that launch holds the combine."""
    import torch
    import paper_2509_02753_amd as P
    dl = _random_layer(256, 64, 384, Fs, 1)
    x = torch.zeros((T, 256), dtype=torch.bfloat16, device="cuda:0").normal_()
    y = torch.empty((T, 256), dtype=torch.float32, device="cuda:0")
    ws, ev = P.alloc_workspace([dl], T, 2), P.StageEvents(1)
    assert P.lexi_moe_gemm_plan(dl, T, 2, "down")["fused"] == (T <= 8)
    for _ in range(3):
        P.lexi_moe_stack_forward([dl], [2], x, y, ws, stage_events=ev)
        torch.cuda.synchronize()
        at = [ev.events[0][0].elapsed_time(e) for e in ev.events[0]]
        assert at == sorted(at) and at[3] > at[2], at


def _gate_logits(x, w, strided):
    """x . w per token in fp32 as 256 threads add it up: thread j takes elements j, j + 256, ... (strided) or 8 j .. 8 j + 7 of every
    2048, the 64 threads of a wave are added as a binary tree, the four waves in order.  (Products of bf16 numbers and their
    sums with an fp32 number are exact in float64 at these exponents: one rounding per step, as a fused multiply-add.)"""
    import numpy as np
    T, d = x.shape
    acc = np.zeros((T, 256), dtype=np.float32)
    for e in range(d):
        j = e % 256 if strided else (e % 2048) // 8
        acc[:, j] = (acc[:, j].astype(np.float64) + x[:, e].astype(np.float64) * np.float64(w[e])).astype(np.float32)
    v = acc.reshape(T, 4, 64)
    while v.shape[2] > 1:
        v = v[:, :, 0::2] + v[:, :, 1::2]
    v = v[:, :, 0]
    return ((v[:, 0] + v[:, 1]) + v[:, 2]) + v[:, 3]


@pytest.mark.parametrize("d", [128, 384, 2048, 2176, 4096, 4224])
def test_order_of_the_shared_gate_dot_product(d):
    """The gate coefficient 1 / (1 + exp(-z)) at z around -20 is exp(z), whose logarithm gives z back: the exponent z * log2(e) (below
    2^5) is rounded by up to 2^-20, 6.6e-7 of z, exp2 and the divide by 3 ulp or 3.6e-7 more; together 1.02e-6, where one ulp of
    z is 1.9e-6.  The routed experts contribute 0."""
    import numpy as np
    import torch
    import paper_2509_02753_amd as P
    T, E, F, Fs = 70, 8, 64, 64
    rng = np.random.default_rng(d)
    bf = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda().to(torch.bfloat16)
    x = bf(rng.standard_normal((T, d)))
    w = bf(rng.standard_normal(d) * 2.0 / np.sqrt(d))
    xf = x.float().cpu().numpy()
    wf = w.float().cpu().numpy()
    # shift every token's x along w so that z lands near -20
    x = bf(xf - np.outer((xf @ wf + 20.0) / (wf @ wf), wf))
    xf = x.float().cpu().numpy()
    t = dict(w_router=torch.zeros((d, E), device="cuda:0"), w_gate=bf(rng.standard_normal((E, F, d)) * 0.02),
             w_up=bf(rng.standard_normal((E, F, d)) * 0.02), w_down=bf(np.zeros((E, d, F))), ws_gate=bf(rng.standard_normal((Fs, d)) * 0.1),
             ws_up=bf(rng.standard_normal((Fs, d)) * 0.1), ws_down=bf(rng.standard_normal((d, Fs))))
    plain = _forward(P.Layer.from_tensors(t), x, 2).double()             # coefficient 1
    gated = _forward(P.Layer.from_tensors(dict(t, w_shared_gate=w)), x, 2).double()
    c = ((gated * plain).sum(1) / (plain * plain).sum(1)).cpu().numpy()  # (least squares: the roundings of d outputs average out)
    z = np.log(c) - np.log1p(-c)
    want, other = (_gate_logits(xf, wf, s).astype(np.float64) for s in (True, False))
    assert np.abs(want + 20.0).max() < 4.0
    assert np.abs(z - want).max() <= 1.02e-6, (np.abs(z - want).max(), np.abs(z - other).max())
    if d != 128:
        assert (np.abs(want - other) > 2.0 ** -20).sum() > T // 8        # (another order would not pass)


@pytest.mark.parametrize("T,k,E,d,F,Fs", [(1, 1, 2, 128, 64, 0), (3, 16, 16, 128, 64, 64), (64, 2, 8, 128, 256, 0), (17, 5, 8, 384, 64, 192),
                                          (9, 18, 40, 128, 64, 0)])
def test_fp32_down_and_combine_in_one_launch(T, k, E, d, F, Fs):
    """Against the oracle, and bit for bit against the separate launches of a larger batch that starts with the same tokens; one wave to more
    slots than waves, the shared expert as the last slot."""
    import torch
    import paper_2509_02753_amd as P
    from helpers import device_and_host_layer
    cfg = replace(S.mini(S.C1, L=1, d=d, F=F, F_shared=0), E=E, F_shared=Fs, shared_kind=S.SHARED_UNGATED if Fs else S.SHARED_NONE)
    run_and_check_layer(cfg, 0, T, k)
    dl, _ = device_and_host_layer(cfg, 0)
    many = T
    while P.lexi_moe_gemm_plan(dl, many, k, "down")["fused"]:
        many *= 2
    assert P.lexi_moe_gemm_plan(dl, T, k, "down")["waves"] == min(k + (Fs > 0), 16) and many > T
    x = S.device_x(cfg, 0, many)
    y = torch.empty((many, d), dtype=torch.float32, device="cuda:0")
    for n in (many, T):
        out = y if n == many else torch.empty((n, d), dtype=torch.float32, device="cuda:0")
        P.lexi_moe_layer_forward(dl, x[:n].contiguous(), out, k, P.alloc_workspace([dl], n, k))
    torch.cuda.synchronize()
    assert torch.equal(out, y[:T])


@pytest.mark.parametrize("base", ["C1", "C2"])
@pytest.mark.parametrize("T,d", [(1, 128), (3, 1024), (2, 1152), (5, 4096), (2, 4224), (1, 8320)])
def test_start_of_a_chained_stack_at_its_edges(base, T, d):
    """Rows of a part of a piece to more than a thread keeps: the normalised input against its definition, and the block on it."""
    import numpy as np
    from test_chained_gpu import _check_blocks
    cfg = replace(S.mini(getattr(S, base), L=2, d=d, F=64, F_shared=0), E=4, k_base=2)
    _check_blocks(cfg, T, np.array([1, 2]))


@pytest.mark.parametrize("base,T,d", [("C1", 3, 128), ("C1", 2, 1152), ("C1", 1, 4224), ("C2", 3, 384), ("C2", 2, 2176), ("C2", 1, 4224)])
def test_chained_stack_in_the_place_of_its_input(base, T, d):
    """The normalised input in the place of x, and for fp32 layers the hidden state there, give the bits of separate buffers."""
    import torch
    import paper_2509_02753_amd as P
    from helpers import device_and_host_layer
    cfg = replace(S.mini(getattr(S, base), L=2, d=d, F=64, F_shared=0), E=4, k_base=2)
    layers = [device_and_host_layer(cfg, l)[0] for l in range(2)]
    x, ws = S.device_x(cfg, 0, T), P.alloc_workspace(layers, T, 2)

    def run(x, y, moe_input=None):
        routing = [P.RoutingOut(T, k, cfg.E, moe_input=moe_input) for k in (1, 2)] if moe_input is not None else None
        P.lexi_moe_stack_forward(layers, [1, 2], x, y, ws, routing=routing, chained=True)
        return y

    want = run(x, torch.empty((T, d), dtype=torch.float32, device="cuda:0"))
    in_x = x.clone()
    assert torch.equal(run(in_x, torch.empty_like(want), moe_input=in_x), want)
    if cfg.dtype == "f32":
        own = x.clone()
        assert torch.equal(run(own, own), want)


@pytest.mark.parametrize("T,k,E,d,F", [(20, 2, 64, 128, 64), (40, 2, 64, 384, 192), (100, 1, 64, 1152, 576), (128, 1, 64, 2176, 1088), (33, 3, 60, 1280, 320)])
@pytest.mark.parametrize("zipf", [0.0, 1.1])
def test_streamed_parts_shorter_and_longer_than_the_loads_in_flight(T, k, E, d, F, zipf):
    """Parts of no, one, three, eight, nine, ten and seventeen K blocks, where up to eight are in flight; one row to many per expert."""
    import paper_2509_02753_amd as P
    from helpers import device_and_host_layer
    cfg = replace(S.mini(S.C5 if zipf else S.C2, L=1, d=d, F=F, F_shared=0), E=E, F_shared=0, shared_kind=S.SHARED_NONE)
    assert P.lexi_moe_gemm_plan(device_and_host_layer(cfg, 0)[0], T, k, "gate_up")["streams"] == 1
    run_and_check_layer(cfg, 0, T, k)


@pytest.mark.parametrize("T", [9, 30, 60])
@pytest.mark.parametrize("d,F,Fs,E", [
    # down in eight parts of 1, 2, 3, 4, 4 to 5, 5 to 6, 7 to 8 and 8 to 9 blocks; up to 16, 32 and 64 rows of one expert or the shared one, both
    # jobs streaming (E 64) and the routed one on tiles in gate/up (E 2), whose reductions are as long
    (128, 256, 256, 2), (384, 512, 0, 2), (640, 768, 576, 2), (896, 1088, 1088, 64), (1152, 1408, 704, 64), (1920, 1920, 0, 2), (2176, 2176, 64, 64),
])
def test_streamed_parts_of_every_length_around_the_depth_of_the_ring(T, d, F, Fs, E):
    import paper_2509_02753_amd as P
    from helpers import device_and_host_layer
    cfg = replace(S.mini(S.C2, L=1, d=d, F=F, F_shared=0), E=E, F_shared=Fs, shared_kind=S.SHARED_UNGATED if Fs else S.SHARED_NONE)
    k = 1 if E == 64 else 2
    dl, _ = device_and_host_layer(cfg, 0)
    if Fs:
        assert all(P.lexi_moe_gemm_plan(dl, T, k, g, shared=True)["streams"] for g in ("gate_up", "down"))
    else:
        assert P.lexi_moe_gemm_plan(dl, T, k, "down")["streams"]
    run_and_check_layer(cfg, 0, T, k)


@pytest.mark.parametrize("kind", ["c1", "c2"])
@pytest.mark.parametrize("T,k,E,d", [
    # rows of 16 lanes: one to 16 experts, a wave's four tokens partly there, on both sides of the line to three launches and to whole waves
    (1, 1, 2, 128), (2, 16, 16, 128), (63, 15, 16, 128), (64, 8, 15, 128), (64, 4, 8, 256), (64, 5, 8, 256), (32, 8, 16, 384), (33, 8, 16, 384),
    (42, 1, 3, 384), (9, 9, 17, 128),
])
def test_routing_in_one_workgroup_of_few_experts(T, k, E, d, kind):
    cfg = replace(S.mini(S.C1 if kind == "c1" else S.C2, L=1, d=d, F=64, F_shared=0), E=E)
    run_and_check_layer(cfg, 0, T, k)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("T,E", [(64, 16), (37, 5)])
def test_routing_in_one_workgroup_of_few_experts_keeps_subnormals_infinities_and_nan(T, E, dtype):
    test_router_keeps_subnormal_products_and_sums(T, E, dtype)
    test_router_with_infinite_and_nan_activations(T, E, dtype)
