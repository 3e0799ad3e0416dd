"""The order of the tiles over the workgroups (runs of 1, 2, 8 or 16
neighbouring tiles on one XCD): three Nesterov rounds, bit for bit against the
oracle.  Every operation of a round rounds once in a fixed order, so any tile
done twice, left out or given to a wrong cluster shows as different bits.  Grids
end inside a cycle of eight runs, at one and one workgroup past one; cluster
grids also end with fewer tiles than a run, and hold fewer than one run."""
import sys

import numpy as np
import pytest
import torch

import oracle
import paper_2110_04175_amd as rs
import workloads as wl
from oracle.double import DoubleOracle
from parity import bit_mismatches

pytestmark = pytest.mark.gpu

T = 512   # coordinates of a tile

# path, tree, n, d.  Tile kernel: past half of the MALL (432*d bytes at 16
# workers), runs of 16 for d % 16 != 0 and pairs otherwise.  The cluster
# kernels and dtree_seq for d % 32 != 0: runs of 16, but below 3 workgroups per
# CU runs of 8 on single trees and launch order on double trees whose number of
# clusters is no multiple of 4; by 1 otherwise.  dtree: launch order, here on
# both sides of the cache-allocating accesses.
CASES = [
    ("tile", "chain", 16, 640 * T - 1),        # five cycles of 128 tiles exactly
    ("tile", "chain", 16, 640 * T + 1),        # one tile past them
    ("tile", "heap", 16, 671 * T + 16),        # pairs, 42 cycles of 16
    ("tile", "chain", 20, 639 * T + 5),        # two workers in some waves, inside a cycle
    # 124 KB of messages, one workgroup per CU: 512 workgroups in two dispatch
    # rounds of 256, the excess over 512 tiles as spill coordinates, whose
    # owners are in launch order beside tiles in runs of 16 and in pairs.
    ("tile", "chain", 32, 270_001),
    ("tile", "chain", 32, 270_000),
    ("cluster", "chain", 40, 36 * T + 3),      # runs of 8, inside a cycle of 8 * 8
    ("cluster", "chain", 64, 32 * T - 1),      # 32 tiles of 4 clusters: two cycles exactly
    ("cluster", "random", 100, 50 * T + 7),    # a last run of 3 tiles
    ("cluster", "chain", 64, 192 * T - 1),     # 3 workgroups per CU: runs of 16, six cycles of 8 * 16
    ("cluster", "chain", 64, 191 * T - 1),     # the longest in runs of 8
    ("cluster", "random", 100, 97 * T - 7),    # runs of 16, a last run of 1 tile
    ("cluster", "hubs", 90, 142 * T + 5),      # the same with hubs, a last run of 15 tiles
    ("cluster", "hubs", 90, 33 * T - 16),      # hubs, a last run of 1 tile
    ("cluster", "random", 40, 5 * T + 1),      # fewer tiles than a run
    ("cluster", "chain", 48, 40 * T),          # rows of whole lines: no runs
    ("dtree", "double", 16, 640 * T + 3),      # streaming: past half of the MALL
    ("dtree", "double", 20, 520 * T),          # the same, two workers in some waves
    ("dtree", "double", 16, 600 * T + 1),      # near the largest that stay in the caches
    ("dtree_seq", "double", 33, 128 * T - 1),  # one cycle of 128 tiles exactly
    ("dtree_seq", "double", 40, 129 * T + 17),
    ("cluster_dtree", "double", 70, 50 * T + 3),    # 3 clusters: launch order
    ("cluster_dtree", "double", 70, 256 * T + 1),   # 3 workgroups per CU: runs of 16, a last run of 1 tile
    ("cluster_dtree", "double", 100, 16 * T + 8),   # 4 clusters: runs of 16, a last run of 1 tile
]


@pytest.mark.parametrize("path,tree,n,d", CASES)
def test_every_tile_once(path, tree, n, d):
    sys.__stderr__.write(f"[gpu] tile order {path} {tree} n={n} d={d}\n")
    sys.__stderr__.flush()
    if tree == "double":
        edges, edges_b = wl.double_binary_tree_edges(n)
        ref = DoubleOracle(n, d, edges, edges_b)
    else:
        make = {"chain": wl.chain_edges, "heap": wl.heap_edges,
                "random": lambda k: wl.random_tree_edges(k, 0),
                "hubs": lambda k: wl.preferential_attachment_edges(k, 0)}[tree]
        edges, edges_b = make(n), None
        ref = oracle.Oracle(n, d, edges, np.float32)
    rng = np.random.default_rng(n + d)
    xo = rng.standard_normal((n, d), dtype=np.float32)
    mo = np.zeros_like(xo)
    x, mom = torch.from_numpy(xo.copy()).cuda(), torch.zeros(n, d, device="cuda")
    with rs.RelaySum(n, d, edges, edges_b=edges_b) as h:
        assert h.path == path
        for _ in range(3):
            g = rng.standard_normal((n, d), dtype=np.float32)
            h.step(x, torch.from_numpy(g).cuda(), mom, 0.1, 0.9)
            ref.round_ex(xo, g, mo, update="model", optimizer="sgd", lr=0.1, beta1=0.9)
        assert bit_mismatches(x.cpu().numpy(), xo) == 0
        assert bit_mismatches(mom.cpu().numpy(), mo) == 0
