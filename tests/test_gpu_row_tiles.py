"""GPU parity of the products' row tiles at their edges: one row past a 256-row
tile, remainders, every epilogue on 256 x 256 and 256 x 128 tiles, K split and
unsplit, and the blocked tile order (more than 8 M tiles)."""

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


@pytest.mark.parametrize("cfg,sizes", [
    (WIDE, [200, 57]),                  # 257 rows: 256 x 128 tiles, the last with one row
    (WIDE, [256, 1]),                   # the same rows as a full tree and a root
    (WIDE, [250, 250, 250, 250, 100]),  # 1100 rows: gate/up and the LM head on 256 x 256
    (WIDE, [234] * 8 + [228]),          # 2100 rows, 9 M tiles: q/k/v on 256 x 256, blocked order
    (LONG, [200, 200, 201]),            # 601 rows: residual products split over K
], ids=["257", "256+1", "1100", "2100", "601-long"])
def test_row_tiles(cfg, sizes):
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
    out, r, exc = full_check(cfg, W_cpu, ver, ids, trees, lens, envelope=cfg is LONG)
    check_tree_kv(cfg, ver, ids, trees, lens, r, ids)
    release(ver, W_dev)


@pytest.mark.parametrize("cfg,sizes", [
    (WIDE, [5]),              # few rows on 64 x 64 tiles, q/k/v and gate/up unsplit or split
    (WIDE, [64]),
    (WIDE, [40, 25]),         # one row past a 64-row tile
    (WIDE, [64, 65]),         # one row past 128
    (LONG, [3, 2]),           # residual products split over K at 5 rows, K = 2048 and 8192
    (LONG, [65]),
    (LONG, [128]),
], ids=["5", "64", "65", "129", "5-long", "65-long", "128-long"])
def test_ring_tiles(cfg, sizes):
    test_row_tiles(cfg, sizes)
