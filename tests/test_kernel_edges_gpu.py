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
