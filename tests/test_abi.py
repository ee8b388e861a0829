"""The C-ABI library: loads, exports every declared symbol, and rejects bad arguments before touching the GPU."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_functions():
    """Every function any header under include/ declares."""
    names = set()
    inc = os.path.join(ROOT, "include")
    for fn in sorted(os.listdir(inc)):
        if fn.endswith(".h"):
            text = re.sub(r"/\*.*?\*/", "", open(os.path.join(inc, fn)).read(), flags=re.S)
            names |= set(re.findall(r"\b(lexi_[a-z0-9_]+)\s*\(", text))
    return sorted(names)


def test_library_exports_every_declared_symbol():
    import paper_2509_02753_amd as P
    names = declared_functions()
    assert set(names) == set(P.EXPORTS)
    lib = ctypes.CDLL(P.LIB_PATH)
    for n in names:
        assert getattr(lib, n) is not None
    assert P.version().startswith("lexi-moe")
    assert P.strerror(0) == "ok" and "k" in P.strerror(-3)


def fake_layer(P, **over):
    """A lexi_layer_t with plausible shapes and fake (never dereferenced) aligned device addresses."""
    f = dict(d=256, E=8, F=128, F_shared=0, dtype=P.LEXI_BF16, shared_kind=0, w_router=0x10000, router_bias=None,
             w_gate=0x20000, w_up=0x30000, w_down=0x40000, ws_gate=None, ws_up=None, ws_down=None, w_shared_gate=None)
    f.update(over)
    from paper_2509_02753_amd.binding import lexi_layer_t
    return lexi_layer_t(*[f[n] for n, _ in lexi_layer_t._fields_])


def call_layer(P, ly, x=0x50000, y=0x60000, y_dtype=0, T=16, k=2, ws=0x70000, ws_bytes=1 << 40):
    from paper_2509_02753_amd.binding import _lib
    return _lib.lexi_moe_layer_forward(ctypes.byref(ly), x, y, y_dtype, T, k, ws, ws_bytes, None, None)


def test_argument_validation_returns_codes_without_launching():
    """Every case fails validation (or is T == 0), so no kernel is launched and no GPU is needed."""
    import paper_2509_02753_amd as P
    ok = fake_layer(P)
    assert call_layer(P, ok, T=0) == 0                                   # T = 0: nothing to do
    assert call_layer(P, ok, k=0) == -3 and call_layer(P, ok, k=9) == -3 and call_layer(P, ok, k=-1) == -3
    assert call_layer(P, ok, T=-1) == -2
    assert call_layer(P, ok, x=None) == -1 and call_layer(P, ok, y=None) == -1 and call_layer(P, ok, ws=None) == -1
    assert call_layer(P, ok, x=0x50004) == -6 and call_layer(P, ok, ws=0x70008) == -6
    assert call_layer(P, ok, y_dtype=7) == -4
    assert call_layer(P, ok, ws_bytes=1024) == -5
    assert call_layer(P, fake_layer(P, E=65)) == -2 and call_layer(P, fake_layer(P, E=0)) == -2
    assert call_layer(P, fake_layer(P, d=192)) == -2 and call_layer(P, fake_layer(P, F=100)) == -2
    assert call_layer(P, fake_layer(P, dtype=3)) == -4
    assert call_layer(P, fake_layer(P, w_gate=None)) == -1
    assert call_layer(P, fake_layer(P, w_up=0x30002)) == -6
    assert call_layer(P, fake_layer(P, F_shared=128, shared_kind=1)) == -1          # shared weights missing
    assert call_layer(P, fake_layer(P, F_shared=128, shared_kind=0)) == -2          # width without a kind
    assert call_layer(P, fake_layer(P, F_shared=128, shared_kind=2, ws_gate=0x80000, ws_up=0x90000,
                                    ws_down=0xA0000)) == -1                         # sigmoid gate vector missing
    assert call_layer(P, ok, T=1 << 23, k=2) == -2                                  # T*k >= 2^24
    assert call_layer(P, fake_layer(P, F=65536), T=16384, k=2) == -2                # intermediate of 4 GiB or more
    assert call_layer(P, fake_layer(P, d=65536), T=32768, k=1) == -2                # x of 4 GiB or more


def test_profile_entry_point_validates_before_launching():
    """lexi_moe_profile_layer applies the limits of the forward entry points up front (fake pointers: any launch
    would fail, so a validation code coming back shows nothing was enqueued)."""
    import paper_2509_02753_amd as P
    from paper_2509_02753_amd.binding import _lib

    def prof(ly, T=16, k_base=2, k_list=(1, 2), x=0x50000, delta=0x60000, ws=0x70000, ws_bytes=1 << 40):
        kl = (ctypes.c_int32 * len(k_list))(*k_list)
        return _lib.lexi_moe_profile_layer(ctypes.byref(ly), x, T, k_base, kl, len(k_list), delta, ws, ws_bytes, None)

    ok = fake_layer(P)
    assert prof(ok, T=0) == -2 and prof(ok, k_base=0) == -3 and prof(ok, k_base=9) == -3
    assert prof(ok, k_list=(3,)) == -3                                     # a listed k above k_base
    assert prof(ok, x=None) == -1 and prof(ok, delta=None) == -1 and prof(ok, ws=None) == -1
    assert prof(ok, ws_bytes=1024) == -5
    assert prof(ok, T=1 << 23) == -2                                       # T*k >= 2^24
    assert prof(fake_layer(P, F=65536), T=16384) == -2                     # intermediate of 4 GiB or more
    assert prof(fake_layer(P, d=65536), T=32768, k_base=1, k_list=(1,)) == -2   # x of 4 GiB or more


def test_static_scratch_entry_point_validates_before_launching():
    """lexi_moe_layer_forward_static: the same argument checks, and a call that needs more than the library's 64 MiB
    static scratch is refused with LEXI_ERR_WORKSPACE (fake pointers: nothing may be launched)."""
    import paper_2509_02753_amd as P
    from paper_2509_02753_amd.binding import _lib
    call = lambda ly, x=0x50000, y=0x60000, y_dtype=0, T=16, k=2: _lib.lexi_moe_layer_forward_static(
        ctypes.byref(ly), x, y, y_dtype, T, k, None, None)
    ok = fake_layer(P)
    assert call(ok, T=0) == 0
    assert call(ok, k=0) == -3 and call(ok, T=-1) == -2 and call(ok, x=None) == -1 and call(ok, y=0x60004) == -6
    assert call(ok, y_dtype=5) == -4
    assert call(fake_layer(P, d=2048, F=1024, E=64), T=4096, k=8) == -5       # 353 MB of workspace


def test_down_gemm_plan_is_host_logic():
    """lexi_moe_down_plan only reads the layer's sizes: the schedule of every case the GPU schedule test runs, and of
    the full-size workloads, checked here without a GPU (0 streaming, 1 tiles, 2 split reduction, 3 direct rows)."""
    import paper_2509_02753_amd as P
    from paper_2509_02753_amd.binding import _lib
    shared = dict(ws_gate=0x80000, ws_up=0x90000, ws_down=0xA0000, w_shared_gate=0xB0000)

    def plan(T, k, which=0, **kw):
        ly = fake_layer(P, dtype=1, **kw)
        return _lib.lexi_moe_down_plan(ctypes.byref(ly), T, k, which)

    assert plan(1300, 2, d=1024, E=64, F=2048) == 2
    assert plan(2600, 1, d=1024, E=64, F=2048) == 3
    assert plan(1300, 2, d=1024, E=64, F=1024) == 1
    assert plan(700, 3, d=1024, E=60, F=384, F_shared=2048, shared_kind=2, **shared) == 1
    assert plan(700, 3, 1, d=1024, E=60, F=384, F_shared=2048, shared_kind=2, **shared) == 2
    assert plan(3700, 2, d=1024, E=8, F=4096) == 2
    # full sizes: prefill runs plain tiles (several rounds of work items), decode streams the weights
    assert plan(4096, 2, d=4096, E=8, F=14336) == 1 and plan(32, 2, d=4096, E=8, F=14336) == 0
    # a handful of tokens (T <= 8, T*k <= 64, no sigmoid-gated shared expert): the combine rides in the down launch
    assert plan(1, 6, d=2048, E=64, F=1408, F_shared=2816, shared_kind=1, ws_gate=0x80000, ws_up=0x90000,
                ws_down=0xA0000) == 4
    assert plan(8, 2, d=4096, E=8, F=14336) == 4 and plan(9, 2, d=4096, E=8, F=14336) == 0
    assert plan(8, 8, d=2048, E=64, F=1024) == 4 and plan(8, 9, d=2048, E=64, F=1024) == 0
    assert plan(16, 16, d=2048, E=64, F=1024) == 1     # enough work items for the tile schedule: not fused
    assert plan(4, 4, d=2048, E=60, F=1408, F_shared=5632, shared_kind=2, **shared) == 0
    assert plan(4096, 8, d=2048, E=64, F=1024) == 1 and plan(4096, 1, d=2048, E=64, F=1024) == 3
    assert plan(8192, 4, 1, d=2048, E=60, F=1408, F_shared=5632, shared_kind=2, **shared) == 1
    assert plan(64, 4, 1, d=2048, E=60, F=1408, F_shared=5632, shared_kind=2, **shared) == 0
    # fp32 layers report by the size, however they are launched (lexi_moe_gemm_plan tells)
    f32 = lambda T, k, which=0, **kw: _lib.lexi_moe_down_plan(ctypes.byref(fake_layer(P, dtype=0, **kw)), T, k, which)
    assert f32(6343, 7, d=896, E=35, F=1088) == 1 and f32(64, 2, d=128, E=8, F=256) == 0 and f32(128, 1, d=896, E=64, F=64) == 0
    assert f32(94, 2, 1, d=1664, E=10, F=2944, F_shared=128, shared_kind=1, **shared) == 1
    assert f32(64, 2, 1, d=1664, E=10, F=2944, F_shared=128, shared_kind=1, **shared) == 0
    # a k = 1 layer with a shared expert still needs the combine
    assert plan(2600, 1, d=1024, E=60, F=2048, F_shared=2048, shared_kind=2, **shared) != 3
    assert plan(16, 1, 1, d=1024, E=8, F=2048) == -1 and plan(0, 1, d=1024, E=8, F=2048) == -1
    assert plan(16, 9, d=1024, E=8, F=2048) == -1


def gemm_plan(P, ly, T, k, which, chained=0):
    from paper_2509_02753_amd.binding import _lib, lexi_gemm_plan_t
    p = lexi_gemm_plan_t()
    st = _lib.lexi_moe_gemm_plan(ctypes.byref(ly), T, k, chained, which, ctypes.byref(p))
    return {n: getattr(p, n) for n, _ in p._fields_} if st == 0 else st


def test_gemm_plan_agrees_with_the_down_plan():
    import itertools

    import paper_2509_02753_amd as P
    from paper_2509_02753_amd.binding import _lib
    shared = dict(F_shared=2048, shared_kind=1, ws_gate=0x80000, ws_up=0x90000, ws_down=0xA0000)
    for T, k, E, F, sh in itertools.product((1, 8, 16, 64, 65, 300, 1025, 5000), (1, 2, 6), (1, 8, 60), (1024, 4096), ({}, shared)):
        ly = fake_layer(P, dtype=1, d=2048, E=E, F=F, **sh)
        if k > E:
            assert gemm_plan(P, ly, T, k, 1) == -3
            continue
        p, old = gemm_plan(P, ly, T, k, 1), _lib.lexi_moe_down_plan(ctypes.byref(ly), T, k, 0)
        assert old == (4 if p["fused"] else 0 if p["streams"] else 3 if p["direct"] else p["ksplit"])
        assert p["tile_rows"] % 16 == 0 and 16 <= p["tile_rows"] <= 160 and p["waves"] in (4, 8, 16)
        assert not (gemm_plan(P, ly, T, k, 1, chained=1)["fused"] or gemm_plan(P, ly, T, k, 1, chained=1)["direct"])
        if sh:
            p = gemm_plan(P, ly, T, k, 3)
            assert _lib.lexi_moe_down_plan(ctypes.byref(ly), T, k, 1) == (0 if p["streams"] else p["ksplit"])
        else:
            assert gemm_plan(P, ly, T, k, 3) == -2
    small, large = fake_layer(P, dtype=0, d=128, E=8, F=256), fake_layer(P, dtype=0, d=896, E=35, F=1088)
    assert gemm_plan(P, small, 64, 2, 1)["fused"] == 1 and gemm_plan(P, small, 64, 2, 1, chained=1)["fused"] == 0
    assert gemm_plan(P, large, 6343, 7, 1)["fused"] == 0
    assert gemm_plan(P, fake_layer(P), 0, 1, 0) == -2 and gemm_plan(P, fake_layer(P), 1, 1, 4) == -2


def test_decode_sized_calls_stream_whatever_the_router():
    """Up to two rows per expert both routed GEMMs take the weight-streaming schedule: how many experts really get rows is
    only known on the device (behind a biased router a third of what a uniform one would use), so no schedule -- and with
    it no summation order -- may depend on a guess of it."""
    import itertools

    import paper_2509_02753_amd as P
    for T, k, E, d, F, bias in itertools.product((1, 4, 12, 16, 20, 33, 64), (1, 2, 4, 6), (8, 32, 60, 64), (1024, 2048, 4096),
                                                 (896, 1408, 2496, 8192), (None, 0xC0000)):
        if k > E or T * k > 2 * E:
            continue
        ly = fake_layer(P, dtype=1, d=d, E=E, F=F, router_bias=bias)
        for which in (0, 1):
            assert gemm_plan(P, ly, T, k, which)["streams"] == 1, (T, k, E, d, F, which)


def test_plan_does_not_depend_on_the_presence_of_a_router_bias():
    """A bias may balance the load, skew it or be zero; its pointer says nothing about the rows an expert gets."""
    import itertools

    import paper_2509_02753_amd as P
    for T, k, (d, E, F), which, chained in itertools.product(
            (1, 16, 64, 256, 1500, 4096, 8192), (1, 2, 4, 8),
            ((2048, 64, 1024), (2048, 60, 1408), (4096, 8, 14336), (4096, 8, 7168), (1024, 32, 2048)), (0, 1), (0, 1)):
        shape = dict(dtype=1, d=d, E=E, F=F)
        assert gemm_plan(P, fake_layer(P, router_bias=0xC0000, **shape), T, k, which, chained) == \
            gemm_plan(P, fake_layer(P, **shape), T, k, which, chained)


@pytest.mark.parametrize("T,k,E,d,F,streams", [
    (13, 3, 3, 640, 2624, 1), (20, 2, 2, 640, 1984, 1), (15, 4, 6, 640, 4096, 1), (28, 1, 1, 512, 1408, 1),   # few units
    (35, 1, 4, 128, 896, 1), (86, 4, 24, 640, 2624, 1), (48, 3, 3, 512, 1408, 1), (64, 1, 1, 2048, 1408, 1),
    (65, 1, 1, 2048, 1408, 0), (45, 4, 8, 2560, 1408, 0), (58, 4, 6, 1024, 4096, 0),    # 65 rows; 2560 and 3072 units
    (64, 2, 8, 4096, 14336, 0), (512, 2, 8, 4096, 14336, 0),
    (89, 3, 4, 512, 192, 1), (128, 2, 2, 512, 384, 1), (129, 2, 2, 512, 384, 0), (100, 2, 2, 512, 576, 0),   # short reductions
    (128, 1, 1, 640, 384, 0),     # the tile schedule stores the output rows of a layer with one active expert itself
])
def test_down_gemm_of_few_units_streams(T, k, E, d, F, streams):
    """More than eight rows per expert in a launch of few units: one long chain of steps on a few CUs on tiles."""
    import paper_2509_02753_amd as P
    assert gemm_plan(P, fake_layer(P, dtype=1, d=d, E=E, F=F), T, k, 1)["streams"] == streams


@pytest.mark.parametrize("T,k,E,d,F,gate_up,down", [
    # launches of at most one item per CU: the height whose items fill more of them, never eight waves for 128 features
    (190, 4, 6, 2048, 896, (64, 4), (64, 4)), (300, 5, 5, 128, 64, (64, 4), (64, 4)), (1300, 1, 5, 128, 64, (64, 4), (64, 4)),
    # one item per CU at 128 rows, two on some at 64
    (3315, 1, 8, 2560, 896, (128, 4), None), (198, 4, 8, 3328, 2624, (128, 4), None), (1296, 1, 16, 3328, 1408, (128, 4), None),
    # eight waves from 250 rows per expert on
    (1464, 5, 60, 1792, 2240, None, (None, 4)), (2999, 5, 60, 1792, 2240, None, (None, 4)),
    (4096, 2, 8, 4096, 14336, (160, 4), (160, 8)), (4096, 8, 64, 2048, 1024, (160, 4), (160, 8)),
])
def test_tile_plans(T, k, E, d, F, gate_up, down):
    import paper_2509_02753_amd as P
    for which, want in ((0, gate_up), (1, down)):
        p = gemm_plan(P, fake_layer(P, dtype=1, d=d, E=E, F=F), T, k, which)
        assert p["streams"] == 0
        if want is not None:
            assert want[0] in (None, p["tile_rows"]) and p["waves"] == want[1], (which, p)


@pytest.mark.parametrize("T,k,E,d,F,Fs,which,waves", [
    # down projections and combine in one launch: as many waves as output features of a workgroup, 8 up to d = 2048
    (1, 1, 8, 128, 704, 320, 1, 8), (8, 6, 64, 2048, 1408, 2816, 1, 8), (8, 6, 64, 2048, 1408, 2816, 3, 8), (4, 2, 64, 2048, 1408, 0, 1, 8),
    (4, 2, 64, 2176, 1408, 0, 1, 16), (4, 2, 64, 4096, 1408, 320, 1, 16), (4, 2, 64, 4096, 1408, 320, 3, 16),
    # two streaming jobs: eight where both sums have eight parts, four where one has; beside tiles four
    (12, 1, 16, 256, 64, 320, 0, 8), (12, 1, 16, 256, 64, 320, 2, 8), (12, 2, 64, 256, 1408, 320, 0, 4), (12, 2, 64, 256, 1408, 320, 2, 4),
    (40, 8, 8, 1024, 448, 320, 3, 4),
])
def test_waves_of_streaming_launches(T, k, E, d, F, Fs, which, waves):
    import paper_2509_02753_amd as P
    shared = dict(F_shared=Fs, shared_kind=1, ws_gate=0x80000, ws_up=0x90000, ws_down=0xA0000) if Fs else {}
    p = gemm_plan(P, fake_layer(P, dtype=1, d=d, E=E, F=F, **shared), T, k, which)
    assert p["streams"] == 1 and p["waves"] == waves


@pytest.mark.parametrize("T,k,E,d,F,Fs", [(65, 1, 33, 128, 64, 64), (100, 1, 64, 4096, 1024, 1408), (128, 1, 64, 2048, 1408, 5632),
                                          (120, 2, 2, 384, 448, 1408), (200, 2, 16, 512, 448, 2816)])
def test_shared_tiles_beside_a_streaming_down_gemm_are_low(T, k, E, d, F, Fs):
    """Up to 64 rows the tile kernel has four workgroups per CU for the routed units of the launch, above two."""
    import paper_2509_02753_amd as P
    ly = fake_layer(P, dtype=1, d=d, E=E, F=F, F_shared=Fs, shared_kind=1, ws_gate=0x80000, ws_up=0x90000, ws_down=0xA0000)
    assert gemm_plan(P, ly, T, k, 1)["streams"] == 1
    p = gemm_plan(P, ly, T, k, 3)
    assert (p["streams"], p["waves"], p["tile_rows"]) == (0, 4, 64)


def test_workspace_of_small_calls_has_not_grown():
    """The workspace was once laid out as these arrays, each at a multiple of 256 bytes, with 32 bytes per token tile of 128
    rows and a tile count; a caller that keeps a buffer of that size may go on using it."""
    import itertools

    import paper_2509_02753_amd as P
    from paper_2509_02753_amd.binding import _lib
    for T, k, E, d, F, dt in itertools.product(list(range(1, 21)) + [64, 65, 130, 1024, 1025, 9000], (1, 2, 7, 8, 9, 64), (1, 8, 64),
                                               (128, 256, 384, 2048), (64, 128, 2048), (0, 1)):
        if k > E:
            continue
        A, es = T * k, (4, 2)[dt]
        planes = 2 if dt == 1 and F // 64 >= 32 and F // 64 % 2 == 0 else 1
        arrays = [T * d * es, d // 128 * T * 256, *[4 * A] * 6, (T + 7) // 8 * 256, 256, 272, 32 * (A // 128 + min(A, E)), 16,
                  A * F * es, A * d * 4 * planes]
        earlier = sum((n + 255) // 256 * 256 for n in arrays)
        size = _lib.lexi_moe_workspace_bytes(ctypes.byref(fake_layer(P, dtype=dt, d=d, E=E, F=F)), 1, T, k)
        assert size <= earlier, (T, k, E, d, F, dt, size, earlier)


def test_workspace_query_is_monotone_and_checked():
    import paper_2509_02753_amd as P
    from paper_2509_02753_amd.binding import _lib, lexi_layer_t
    arr = (lexi_layer_t * 2)(fake_layer(P), fake_layer(P, F=256, F_shared=128, shared_kind=1, ws_gate=0x80000,
                                                       ws_up=0x90000, ws_down=0xA0000))
    q = lambda T, k: int(_lib.lexi_moe_workspace_bytes(arr, 2, T, k))
    assert q(64, 2) > 0 and q(128, 2) > q(64, 2) and q(64, 4) > q(64, 2)
    assert q(64, 9) == q(64, 8) and q(-1, 2) == 0 and q(64, 0) == 0     # k is capped by the layer's E (8 here)
    assert int(_lib.lexi_moe_workspace_bytes(None, 1, 64, 2)) == 0
    # a stack call validates every layer before launching: bad k in the second layer is reported, nothing runs
    kv = (ctypes.c_int32 * 2)(2, 0)
    st = _lib.lexi_moe_stack_forward(arr, 2, kv, 0x50000, 0, 0x60000, 64 * 256, 0, 64, 0, 0x70000, 1 << 40, None, None)
    assert st == -3
    kv = (ctypes.c_int32 * 2)(2, 2)
    call = lambda y_dtype, x_stride, mode: _lib.lexi_moe_stack_forward(
        arr, 2, kv, 0x50000, x_stride, 0x60000, 64 * 256, y_dtype, 64, mode, 0x70000, 1 << 40, None, None)
    assert call(0, 0, 2) == -4                       # unknown mode
    assert call(1, 0, 1) == -4                       # chained mode keeps the hidden state in fp32
    assert call(0, 64 * 256, 1) == -4                # chained mode has one input
    assert _lib.lexi_moe_stack_forward(arr, 2, kv, 0x50000, 0, 0x60000, 10, 0, 64, 0, 0x70000, 1 << 40, None, None) == -2
    assert _lib.lexi_moe_stack_forward(arr, 2, None, 0x50000, 0, 0x60000, 64 * 256, 0, 64, 0, 0x70000, 1 << 40, None, None) == -1


def test_build_does_not_load_the_library_it_replaces():
    import subprocess
    import sys
    code = "import sys, __graft_entry__ as g; g._lib_build(); assert 'paper_2509_02753_amd' not in sys.modules"
    subprocess.run([sys.executable, "-c", code], cwd=ROOT, check=True, timeout=100)


def test_product_does_not_import_the_oracle():
    pkg = os.path.join(ROOT, "paper_2509_02753_amd")
    for dirpath, _, files in os.walk(pkg):
        for fn in files:
            if fn.endswith((".py", ".hip", ".hpp", ".h", ".cpp")):
                src = open(os.path.join(dirpath, fn)).read()
                assert "oracle" not in src.lower(), f"{fn} mentions the oracle"
    src = open(os.path.join(ROOT, "oracle", "__init__.py")).read() + open(os.path.join(ROOT, "oracle", "lexi_oracle.c")).read()
    assert "paper_2509_02753_amd" not in src and "lexi_moe.h" not in src
