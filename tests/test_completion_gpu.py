"""The completion of the boundary workers of clusters on its two widths: 16-byte
chunks (with and without a partial last one) once their blocks fill the
device, single floats below.  Three rounds, bit for bit against the oracle: the
completion adds in a fixed order, one rounding per operation."""
import sys

import numpy as np
import pytest
import torch

import oracle
import paper_2110_04175_amd as rs
import workloads as wl
from parity import bit_mismatches

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tree,n,d,offset,update", [
    # Chunks: a random tree of 1,000 workers has 134 boundary workers, 5 blocks
    # of 1,024 coordinates per CU from about 9,800 coordinates on; 600 workers
    # with hubs have 26, 8 blocks per CU from about 80,000.
    ("random", 1000, 30_720, 0, "model"),
    ("random", 1000, 30_721, 0, "model"),
    ("random", 1000, 30_722, 1, "robust"),
    ("random", 1000, 30_719, 3, "mean"),
    ("random", 1000, 10_243, 0, "model"),
    ("hubs", 600, 80_897, 0, "grad"),
    ("hubs", 600, 80_898, 2, "model"),
    # Single floats, on rows of whole chunks too.
    ("hubs", 600, 61_441, 0, "grad"),
    ("hubs", 600, 61_440, 2, "model"),
    ("random", 300, 1_024, 0, "model"),
    ("hubs", 100, 4_000, 0, "robust"),
    ("chain", 40, 3, 0, "model"),
    ("hubs", 200, 1_001, 1, "mean"),
])
def test_boundary_workers(tree, n, d, offset, update):
    sys.__stderr__.write(f"[gpu] completion {tree} n={n} d={d} offset={offset} {update}\n")
    sys.__stderr__.flush()
    edges = {"chain": wl.chain_edges, "random": lambda k: wl.random_tree_edges(k, 0),
             "hubs": lambda k: wl.preferential_attachment_edges(k, 0)}[tree](n)
    beta = 0.9 if update in ("model", "robust") else 0.0
    rng = np.random.default_rng(n + d)

    def device(a):
        t = torch.zeros(n * d + offset, device="cuda")[offset:].view(n, d)
        return t.copy_(torch.from_numpy(a))

    xo = rng.standard_normal((n, d), dtype=np.float32)
    so = np.zeros_like(xo)
    x, s = device(xo), device(so)
    state = update != "grad"
    ref = oracle.Oracle(n, d, edges, np.float32)
    with rs.RelaySum(n, d, edges) as h:
        assert h.path == "cluster"
        for _ in range(3):
            g = rng.standard_normal((n, d), dtype=np.float32)
            h.step_ex(x, device(g), s if state else None, update=update, lr=0.1, beta1=beta)
            ref.round_ex(xo, g, so if state else None, update=update, lr=0.1, beta1=beta)
        assert bit_mismatches(x.cpu().numpy(), xo) == 0
        assert bit_mismatches(s.cpu().numpy(), so) == 0
