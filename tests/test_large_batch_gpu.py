"""Routing of batches of ten thousand tokens and more (narrow layers: the permutation is what grows)."""
from dataclasses import replace

import numpy as np
import pytest

import lexi_synth as S
from helpers import run_and_check_layer

pytestmark = pytest.mark.gpu


# 512 router blocks of 16 tokens are the most whose histograms every workgroup of the permutation reads itself; from 65536
# tokens on a workgroup owns more than eight blocks
@pytest.mark.parametrize("T,E,k", [(8192, 8, 2), (8193, 8, 1), (8192 + 16 * 5 + 3, 60, 4), (65536, 17, 2), (65537, 5, 1), (140001, 5, 1)])
def test_permutation_of_many_tokens(T, E, k):
    cfg = replace(S.mini(S.C2, L=1, d=128, F=64, F_shared=0), E=E)
    tokens = np.unique(np.concatenate([[0, T - 1], np.random.default_rng(T).integers(0, T, 62)])).astype(np.int32)
    run_and_check_layer(cfg, 0, T, k, tokens=tokens)


def test_permutation_does_not_grow_faster_than_the_batch():
    """Eight times the tokens: eight times the routing time in the limit, 64 times where every workgroup reads every
    histogram.  Medians of the routing stage; the bound of 12 leaves room for either end's fixed costs."""
    import torch
    import paper_2509_02753_amd as P
    from helpers import device_and_host_layer
    cfg = replace(S.mini(S.C2, L=1, d=128, F=64, F_shared=0), E=8)
    dl, _ = device_and_host_layer(cfg, 0)
    ms = []
    for T in (131072, 1048576):
        x = torch.zeros((T, cfg.d), dtype=torch.bfloat16, device="cuda:0").normal_()
        y = torch.empty((T, cfg.d), dtype=torch.float32, device="cuda:0")
        ws = P.alloc_workspace([dl], T, 1)
        ev, seen = P.StageEvents(1), []
        for _ in range(5):
            P.lexi_moe_stack_forward([dl], [1], x, y, ws, stage_events=ev)
            torch.cuda.synchronize()
            seen.append(ev.stage_ms()[0][0])
        ms.append(float(np.median(seen)))
    assert ms[1] <= 12.0 * ms[0], ms


def test_combine_time_follows_the_bytes_of_a_ragged_width():
    """d = 1280 is one whole and a quarter piece of 1024 features per token: the combine reads 1.25 times the bytes of d =
    1024.  (Threads past the row once re-read its start: 1.6 times.)  The bound of 1.45 is halfway."""
    import torch
    import paper_2509_02753_amd as P
    from helpers import device_and_host_layer
    T, k, us = 4096, 8, []
    for d in (1024, 1280):
        cfg = replace(S.mini(S.C2, L=1, d=d, F=64, F_shared=0), E=16)
        dl, _ = device_and_host_layer(cfg, 0)
        x, y = S.device_x(cfg, 0, T), torch.empty((T, d), dtype=torch.float32, device="cuda:0")
        ws, ev, seen = P.alloc_workspace([dl], T, k), P.StageEvents(1), []
        for _ in range(15):
            P.lexi_moe_stack_forward([dl], [k], x, y, ws, stage_events=ev)
            torch.cuda.synchronize()
            seen.append(ev.stage_ms()[0][4])
        us.append(1e3 * float(np.median(seen)))
    assert us[1] <= 1.45 * us[0], us


def test_fp32_down_gemm_of_more_workgroups_than_one_grid_dimension_holds():
    """The most tokens of d = 4096 that an fp32 call takes, every expert selected (k = E = 17): 64 column blocks x 278544 tiles of 16
    rows are 2^32 threads and more (in one dimension the launch went through and most rows stayed unwritten).  Outputs of the
    first, the last and some other tokens against float64.  Bound: a chain of 4096 fp32 fused multiply-adds rounds by about 2^-24 *
    sqrt(4096) / 2 = 1.9e-6 of the result's RMS, the product of two by 2.7e-6, five times that at the largest of 3 * 10^5
    outputs: 1.4e-5 (seen: 1.1e-5)."""
    import torch
    import paper_2509_02753_amd as P
    T, d, E, F = 262143, 4096, 17, 64
    assert (d // 64) * (T * E // 16) * 256 >= 1 << 32
    gen = torch.Generator(device="cuda:0").manual_seed(2)
    normal = lambda sigma, *s: torch.empty(s, device="cuda:0").normal_(0.0, sigma, generator=gen)
    t = dict(w_router=normal(0.02, d, E), w_gate=normal(0.02, E, F, d), w_up=normal(0.02, E, F, d), w_down=normal(0.02, E, d, F))
    x = normal(1.0, T, d)
    dl = P.Layer.from_tensors(t)
    y = torch.full((T, d), float("nan"), device="cuda:0")
    P.lexi_moe_layer_forward(dl, x, y, E, P.alloc_workspace([dl], T, E))
    torch.cuda.synchronize()
    assert not torch.isnan(y[:, ::64]).any()
    at = torch.cat([torch.tensor([0, 1, T - 2, T - 1]), torch.randint(0, T, (60,), generator=torch.Generator().manual_seed(3))]).cuda()
    xs = x[at].double()
    gates = torch.softmax(xs @ t["w_router"].double(), dim=1)
    want = torch.zeros((len(at), d), dtype=torch.float64, device="cuda:0")
    for e in range(E):
        h = torch.nn.functional.silu(xs @ t["w_gate"][e].double().T) * (xs @ t["w_up"][e].double().T)
        want += gates[:, e:e + 1] * (h @ t["w_down"][e].double().T)
    assert float((y[at].double() - want).abs().max() / want.square().mean().sqrt()) <= 1.4e-5
    del x, y, dl
    torch.cuda.empty_cache()


def test_packing_of_more_runs_than_one_grid_dimension_holds():
    """2^32 + 2^19 runs of eight bf16 weights (64 GiB and 8 MiB more): the first, the last and the matrices around run 2^32."""
    import torch
    import paper_2509_02753_amd as P
    R, K, n = 1024, 4096, 8193
    runs = R * K // 8
    assert n * runs > 1 << 32 and (n - 1) * runs == 1 << 32
    torch.cuda.empty_cache()
    w = torch.empty((n, R, K), dtype=torch.int16, device="cuda:0")
    some = [0, 1, 4095, 8190, 8191, 8192]
    w.zero_()
    for m in some:
        w[m].random_(-(1 << 15), 1 << 15, generator=torch.Generator(device="cuda:0").manual_seed(m))
    packed = P.lexi_pack_weights(w.view(torch.bfloat16)).view(torch.int16)
    torch.cuda.synchronize()
    for m in some:
        # [row block][row][K block][octet][8] -> [row block][K block][octet][row][8]
        want = w[m].view(R // 16, 16, K // 32, 4, 8).permute(0, 2, 3, 1, 4).reshape(R, K)
        assert torch.equal(packed[m], want), m
    del w, packed
    torch.cuda.empty_cache()
