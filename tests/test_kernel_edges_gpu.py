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


@pytest.mark.parametrize("T,k,E,d,F,zipf", [
    (161, 1, 1, 128, 64, 0.0), (160, 1, 1, 640, 192, 0.0),      # one tile of 160 rows; a second one of 16-row blocks
    (320, 2, 2, 512, 128, 0.0), (321, 2, 2, 1152, 128, 0.0),    # every expert: whole tiles; one row more
    (1100, 2, 8, 1152, 320, 0.0),     # column blocks of 512 whose last holds 128 features; gate/up blocks half empty
    (1100, 3, 16, 256, 1024, 1.5),    # skewed: tall tiles for few experts, cuts of the item list by cost
    (700, 4, 64, 384, 2048, 2.0),     # most experts with a handful of rows, a few with many; reduction cut in two
    (130, 2, 3, 256, 4096, 0.0),      # 87 rows per expert, few items: cut in two where it streamed
    (40, 2, 8, 256, 448, 0.0),        # 10 rows per expert, reduction too short to cut: whole, on tiles
    (1030, 1, 8, 512, 128, 1.0),      # output rows stored directly from the wide form
])
def test_grouped_gemm_tiles(T, k, E, d, F, zipf):
    """Token tiles of up to 160 rows dealt out evenly, the eight-wave down GEMM, the cuts of the work list, and the sizes
    around the streaming schedule's limits, against the oracle (routing bit for bit, TOL_BF16 of RMS)."""
    cfg = replace(S.mini(S.C5 if zipf else S.C2, L=1, d=d, F=F, F_shared=0), E=E, F_shared=0, shared_kind=S.SHARED_NONE)
    if zipf:
        cfg = replace(cfg, zipf_s=zipf)
    run_and_check_layer(cfg, 0, T, k)


@pytest.mark.parametrize("T,k,E,d,F", [
    (4, 4, 64, 2048, 1408), (6, 1, 64, 2048, 1408),     # 14 and 6 experts expected in use: 156 items of gate/up (tiles), 63 (streams)
    (16, 4, 64, 256, 1408), (20, 4, 64, 2048, 128),     # gate/up on tiles with a streaming down GEMM, and the reverse
    (2, 6, 64, 1024, 2816), (16, 1, 8, 2304, 8192),     # 240 items: streams; 443: tiles
    (33, 2, 64, 2048, 1408),                            # both on tiles
])
def test_decode_schedules_around_their_limits(T, k, E, d, F):
    """Decode-sized calls on either side of the line between weight streaming and tiles, against the oracle."""
    cfg = replace(S.mini(S.C2, L=1, d=d, F=F, F_shared=0), E=E)
    run_and_check_layer(cfg, 0, T, k)
