"""GPU parity of the products' row tiles at their edges: one row past a tile,
remainders, every epilogue on 256 x 256 and 256 x 128 tiles, the blocked tile
order (more than 8 M tiles) and the shortest K loop.  Every case names the
kernels it is there for, and the library's plan has to agree."""

import dataclasses

import numpy as np
import pytest
import torch

import paper_2512_04752_amd as sv
import workload as wl
from tests.gpu_util import check_tree_kv, full_check, release, say

pytestmark = pytest.mark.gpu

# 64 query heads over 4 K/V heads: wide q/k/v and gate/up products over a short K (4 steps)
WIDE = dataclasses.replace(wl.TINY, n_layers=1, n_heads=64, n_kv_heads=4, head_dim=64, ffn=4096,
                           vocab=4096)
# residual products of 2048 columns (K = 2048 and 8192, split), head dim 128
LONG = dataclasses.replace(wl.TINY, n_layers=1, hidden=2048, n_heads=16, n_kv_heads=2, head_dim=128,
                           ffn=8192, vocab=2048)


# wide products over K = 256
FLAT = dataclasses.replace(wl.TINY, n_layers=1, n_heads=16, n_kv_heads=8, head_dim=128, ffn=8192,
                           vocab=8192)
# K = 128, two K steps: the shortest loop
SHORT = dataclasses.replace(wl.TINY, n_layers=1, hidden=128, n_heads=2, n_kv_heads=2, ffn=4096,
                            vocab=8192)
SHORT_NARROW = dataclasses.replace(SHORT, ffn=1024, vocab=2048)


def _shape(hidden, n_heads, n_kv_heads, head_dim, ffn):
    return dataclasses.replace(wl.TINY, n_layers=1, hidden=hidden, n_heads=n_heads,
                               n_kv_heads=n_kv_heads, head_dim=head_dim, ffn=ffn)


ROW_TILES = {   # configuration, tree sizes, {product: (tile rows, tile columns, K splits)}
    "257": (WIDE, [200, 57], dict(gemm_qkv=(64, 128, 1), gemm_o=(64, 64, 8))),
    # the same rows as a full tree and a root
    "256+1": (WIDE, [256, 1], dict(gemm_gate_up=(64, 128, 1), lm_head=(64, 128, 1))),
    "1100": (WIDE, [250, 250, 250, 250, 100],
             dict(gemm_qkv=(256, 128, 1), gemm_gate_up=(256, 256, 1), lm_head=(256, 128, 1))),
    # 9 M tiles: blocked order
    "2100": (WIDE, [234] * 8 + [228], dict(gemm_qkv=(256, 256, 1), lm_head=(256, 256, 1))),
    "601-long": (LONG, [200, 200, 201],
                 dict(gemm_o=(128, 128, 2), gemm_gate_up=(256, 256, 1), gemm_down=(256, 128, 4))),
    # one live row in the last 256-row tile
    "257-flat": (FLAT, [256, 1], dict(gemm_gate_up=(256, 128, 1))),
    "513-flat": (FLAT, [256, 256, 1], dict(gemm_gate_up=(256, 256, 1), lm_head=(256, 128, 1))),
    "1025-flat": (FLAT, [256] * 4 + [1], dict(gemm_qkv=(256, 128, 1), lm_head=(256, 256, 1))),
    "2049-flat": (FLAT, [256] * 8 + [1],
                  dict(gemm_qkv=(256, 256, 1), gemm_gate_up=(256, 256, 1), gemm_down=(256, 128, 8))),
    "257-split": (_shape(4096, 16, 8, 128, 2048), [256, 1],
                  dict(gemm_qkv=(256, 128, 4), gemm_gate_up=(256, 128, 4))),
    "769-o-split": (_shape(1280, 32, 4, 128, 128), [256] * 3 + [1], dict(gemm_o=(256, 128, 4))),
    "2049-o": (_shape(2048, 4, 2, 64, 128), [256] * 8 + [1], dict(gemm_o=(256, 128, 1))),
    "2049-o-wide": (_shape(4096, 4, 2, 64, 128), [256] * 8 + [1], dict(gemm_o=(256, 256, 1))),
    "1537-down-split": (_shape(1280, 4, 2, 64, 8192), [256] * 6 + [1], dict(gemm_down=(256, 256, 4))),
    "1537-short": (SHORT, [256] * 6 + [1], dict(gemm_gate_up=(256, 256, 1), lm_head=(256, 256, 1))),
    "3073-short": (SHORT_NARROW, [256] * 12 + [1], dict(gemm_gate_up=(256, 128, 1), lm_head=(256, 128, 1))),
}
RING_TILES = {
    # few rows on 64 x 64 tiles, q/k/v and gate/up unsplit
    "5": (WIDE, [5], dict(gemm_qkv=(64, 64, 1), gemm_o=(64, 64, 16), gemm_gate_up=(64, 64, 1))),
    "64": (WIDE, [64], dict(gemm_qkv=(64, 64, 1), gemm_down=(64, 64, 16))),
    "65": (WIDE, [40, 25], dict(gemm_qkv=(64, 64, 1), gemm_o=(64, 64, 16))),    # one row past a tile
    "129": (WIDE, [64, 65], dict(gemm_gate_up=(64, 128, 1), lm_head=(64, 64, 1))),
    # K = 2048 and 8192, split
    "5-long": (LONG, [3, 2], dict(gemm_qkv=(64, 64, 4), gemm_o=(64, 64, 8), gemm_down=(64, 64, 8))),
    "65-long": (LONG, [65], dict(gemm_qkv=(64, 128, 4), gemm_gate_up=(64, 128, 1), gemm_down=(64, 128, 8))),
    "128-long": (LONG, [128], dict(gemm_qkv=(64, 64, 2), gemm_o=(64, 64, 4))),
}


def check_plan(cfg, sizes, kernels):
    assert {k: sv.spec_gemm_plan(cfg, k, sum(sizes)) for k in kernels} == kernels


@pytest.mark.parametrize("name", ROW_TILES)
def test_row_tiles(name):
    run_case(*ROW_TILES[name])


@pytest.mark.parametrize("name", RING_TILES)
def test_ring_tiles(name):
    run_case(*RING_TILES[name])


def run_case(cfg, sizes, kernels):
    check_plan(cfg, sizes, kernels)
    say(f"row tiles: {sum(sizes)} rows, hidden {cfg.hidden}")
    W_cpu = wl.make_weights(cfg, 71, dtype=torch.bfloat16)
    W_dev = {"tok_embed": W_cpu["tok_embed"].cuda(), "final_norm": W_cpu["final_norm"].cuda(),
             "lm_head": W_cpu["lm_head"].cuda(),
             "layers": [{k: v.cuda() for k, v in lw.items()} for lw in W_cpu["layers"]]}
    rng = np.random.default_rng(sum(sizes))
    pars = [wl.recursive_tree(rng, n, min(n, 9), 4) for n in sizes]
    lens = [int(x) for x in rng.integers(0, 120, size=len(sizes))]
    ver = sv.Verifier(cfg, W_dev, [S + n for S, n in zip(lens, sizes)], max_batch=len(sizes),
                      max_tokens=sum(sizes))
    gen = torch.Generator(device="cuda").manual_seed(71)
    for b, S in enumerate(lens):
        k, v = ver.kv.sample_view(b)
        wl.fill_prefix_kv(k, v, S, wl.prefix_kv_std(cfg), gen)
    torch.cuda.synchronize()
    ids = list(range(len(sizes)))
    trees = [(wl.random_tokens(rng, len(p), cfg.vocab), p) for p in pars]
    out, r, exc = full_check(cfg, W_cpu, ver, ids, trees, lens, envelope=max(cfg.hidden, cfg.ffn) >= 8192 or cfg.hidden >= 2048)
    check_tree_kv(cfg, ver, ids, trees, lens, r, ids)
    release(ver, W_dev)

