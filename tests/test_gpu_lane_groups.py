"""Rows at the edges of the sampler's degree bins (16, 32, 64, ... 2048 neighbours, hubs above 4096 or 8192), fanouts
around the lane groups' limits (16 with weights, 32 without), both id widths, with and without weights.  A hop of up to
8 192 nodes leaves rows above 64 neighbours to a wavefront each, a larger one to groups of sixteen lanes: both sizes run.
Bit-exact against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2511_07421_amd as a3
from helpers import blocks_equal

pytestmark = pytest.mark.gpu
Q = 65536
DEV = "cuda:0"
FEW, MANY = 120, 8200


def _graph(dtype, n_seeds):
    """3 rows of each degree, neighbours distinct and ascending, among 20 000 nodes; in a batch of `n_seeds` the other seeds
    have one to three neighbours, the other nodes none"""
    edges = [0, 1, 3, 4, 5, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 512, 513, 1023, 1024, 1025,
             2047, 2048, 2049, 4095, 4096, 4097, 8191, 8192, 8193]
    n, rng = 20000, np.random.default_rng(5)
    seeds = np.sort(rng.permutation(n)[:n_seeds])
    deg = np.zeros(n, dtype=np.int64)
    deg[seeds] = rng.integers(1, 4, size=n_seeds)
    deg[rng.permutation(seeds)[:3 * len(edges)]] = np.repeat(edges, 3)
    indptr = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(deg, out=indptr[1:])
    indices = np.concatenate([np.sort(rng.choice(n, size=d, replace=False)) for d in deg if d]).astype(dtype)
    return indptr, indices, seeds.astype(dtype)


@pytest.mark.parametrize("n_seeds", [FEW, MANY])
@pytest.mark.parametrize("dtype", [np.int32, np.int64])
@pytest.mark.parametrize("flags", [0, a3.A3_TEST_FEW_DRAWS, a3.A3_TEST_SMALL_GRID])
def test_rows_at_the_edges_of_the_lane_groups(dtype, flags, n_seeds):
    indptr, indices, seeds = _graph(dtype, n_seeds)
    d_ip, d_ix, d_seeds = (torch.from_numpy(t).to(DEV) for t in (indptr, indices, seeds))
    ctx = a3.Context(len(seeds), [64], flags=flags)
    rng = np.random.default_rng(6)
    for fan in (1, 4, 5, 15, 16, 17, 20, 31, 32, 33, 64):
        for cached, gamma in ((1.0, 1.0), (0.7, 4.0), (0.03, 1.5)):
            print(f"[case] {np.dtype(dtype).name} flags={flags} seeds={n_seeds} fanout={fan} cached={cached} gamma={gamma}", flush=True)
            cm = np.where(rng.random(len(indptr) - 1) < cached, 1, -1).astype(np.int32)  # only the sign counts here
            got = ctx.sample_blocks(d_ip, d_ix, d_seeds, [fan], torch.from_numpy(cm).to(DEV), int(gamma * Q), fan).to_host()
            blocks_equal(got, oracle.sample_blocks(indptr, indices, seeds, [fan], cm, int(gamma * Q), fan))
            # a large hop leaves few of its nodes to the second launch, so none of its calls is a single full launch,
            # which has no groups for rows above 64
            assert n_seeds == FEW or ctx.sample_stats()["launch_plan"] == (1 if gamma > 1.0 else 0)
    ctx.close()
