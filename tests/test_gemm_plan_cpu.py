"""The plan of the products: the kernels that the GPU tests of the row tiles are there for are the
ones that the library picks, and malformed requests are refused."""

import dataclasses

import pytest

import paper_2512_04752_amd as sv
import workload as wl
from tests.test_gpu_row_tiles import RING_TILES, ROW_TILES, check_plan


@pytest.mark.parametrize("case", list(ROW_TILES.values()) + list(RING_TILES.values()),
                         ids=list(ROW_TILES) + [f"ring-{k}" for k in RING_TILES])
def test_cases_reach_their_kernels(case):
    check_plan(*case)


def test_every_epilogue_on_both_wide_tiles_with_one_live_row():
    """Over the cases whose last 256-row tile holds one row: each product kind on 256 x 256 and
    256 x 128 tiles, and the residual products both split over K and not."""
    got = {("resid" if k in ("gemm_o", "gemm_down") else k, tile[1], tile[2] > 1)
           for _, sizes, kernels in ROW_TILES.values() if sum(sizes) % 256 == 1
           for k, tile in kernels.items() if tile[0] == 256}
    for kind in ("gemm_qkv", "gemm_gate_up", "lm_head"):
        assert (kind, 256, False) in got and (kind, 128, False) in got
    for kind in ("gemm_qkv", "gemm_gate_up"):
        assert (kind, 128, True) in got
    assert {("resid", c, split) for c in (128, 256) for split in (False, True)} <= got


def test_few_rows_and_refusals():
    assert sv.spec_gemm_plan(wl.LLAMA_8B, "gemm_gate_up", 4) == (0, 16, 1)
    assert sv.spec_gemm_plan(wl.LLAMA_8B, "gemm_gate_up", 5)[0] == 64
    with pytest.raises(sv.SpecError):
        sv.spec_gemm_plan(wl.LLAMA_8B, "attention", 4)
    with pytest.raises(sv.SpecError):
        sv.spec_gemm_plan(wl.LLAMA_8B, "gemm_o", 0)
    with pytest.raises(sv.SpecError):
        sv.spec_gemm_plan(dataclasses.replace(wl.LLAMA_8B, hidden=100), "gemm_o", 4)
