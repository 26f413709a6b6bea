"""Rows at the edges of the sampler's lane groups: degrees around every bin boundary (16, 32, 64, ..., 1024,
4096), fanouts around the groups' limits, both id widths, with and without weights.  Bit-exact against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2511_07421_amd as a3
from helpers import blocks_equal

pytestmark = pytest.mark.gpu
Q = 65536
DEV = "cuda:0"


def _graph(dtype):
    """3 rows of each degree, neighbours distinct and ascending, among 6000 nodes; the others have none"""
    edges = [0, 1, 3, 4, 5, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 512, 513, 1023, 1024, 1025,
             4095, 4096, 4097]
    n, rng = 6000, np.random.default_rng(5)
    deg = np.zeros(n, dtype=np.int64)
    deg[rng.permutation(n)[:3 * len(edges)]] = np.repeat(edges, 3)
    indptr = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(deg, out=indptr[1:])
    indices = np.concatenate([np.sort(rng.choice(n, size=d, replace=False)) for d in deg if d]).astype(dtype)
    return indptr, indices, np.nonzero(deg)[0].astype(dtype)


@pytest.mark.parametrize("dtype", [np.int32, np.int64])
@pytest.mark.parametrize("flags", [0, a3.A3_TEST_FEW_DRAWS])
def test_rows_at_the_edges_of_the_lane_groups(dtype, flags):
    indptr, indices, seeds = _graph(dtype)
    d_ip, d_ix, d_seeds = (torch.from_numpy(t).to(DEV) for t in (indptr, indices, seeds))
    ctx = a3.Context(len(seeds), [64], flags=flags)
    rng = np.random.default_rng(6)
    for fan in (1, 4, 5, 15, 16, 17, 20, 31, 32, 33, 64):
        for cached, gamma in ((1.0, 1.0), (0.7, 4.0), (0.03, 1.5)):
            print(f"[case] {np.dtype(dtype).name} flags={flags} fanout={fan} cached={cached} gamma={gamma}", flush=True)
            cm = np.where(rng.random(len(indptr) - 1) < cached, 1, -1).astype(np.int32)  # only the sign counts here
            got = ctx.sample_blocks(d_ip, d_ix, d_seeds, [fan], torch.from_numpy(cm).to(DEV), int(gamma * Q), fan).to_host()
            blocks_equal(got, oracle.sample_blocks(indptr, indices, seeds, [fan], cm, int(gamma * Q), fan))
    ctx.close()
