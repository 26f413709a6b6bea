"""Weighted choices whose cut falls between keys that single precision cannot tell apart: the error that the
sampler allows for, over all draws, and neighbourhoods made so that the cut is that close.  Bit-exact
against the oracle."""
import ctypes as C

import numpy as np
import pytest
import torch

import oracle
import paper_2511_07421_amd as a3
from helpers import blocks_equal
from native import build as native

pytestmark = pytest.mark.gpu
Q = 65536
DEV = "cuda:0"


@pytest.mark.parametrize("gamma", [1.0, 1.25, 4.0, 1000.0, 65535.0])
def test_error_of_the_single_precision_keys(gamma):
    """Two keys are told apart from 4 (1 / w + key) kKeyError on: 2 for each of them.  Expected: 0.12 for the
    logarithm and 2^-23 / 2^-20 = 0.125 for the division by the weight (a rounded reciprocal and a product).
    At least eightfold room is left below the limit."""
    lib = C.CDLL(native.build(force=False))
    lib.key_error.argtypes = [C.c_uint32, C.c_uint32, C.c_void_p, C.c_void_p]
    blocks = 8192
    worst = torch.zeros(blocks * 256, dtype=torch.float64, device=DEV)
    print(f"[case] all draws, weight {gamma}", flush=True)
    assert lib.key_error(int(gamma * Q), blocks, worst.data_ptr(), torch.cuda.current_stream().cuda_stream) == 0
    got = float(worst.max())
    print(f"largest error: {got:.4f} kKeyError (1 / w + key)", flush=True)
    assert 0.0 < got <= (0.12 if gamma == 1.0 else 0.245)


DEGREES = (12, 30, 33, 60, 64, 65, 300, 1500)   # groups of 4, 8, 16 lanes; whole and partial lists


def _graph(dtype, n_seeds):
    """one row of each degree, no two rows with a common neighbour; the other seeds have none"""
    first = n_seeds
    n = n_seeds + sum(DEGREES)
    deg = np.zeros(n, dtype=np.int64)
    deg[:len(DEGREES)] = DEGREES
    indptr = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(deg, out=indptr[1:])
    return indptr, np.arange(first, n).astype(dtype), np.arange(n_seeds).astype(dtype)


@pytest.mark.parametrize("n_seeds", [64, 8200])   # up to 8 192 nodes, rows above 64 go to a wavefront each
@pytest.mark.parametrize("dtype", [np.int32, np.int64])
def test_cuts_between_a_cached_and_an_uncached_neighbour(dtype, n_seeds):
    """All neighbours cached but one of the best draws, whose key the bias rate moves next to the m-th best cached
    one: below it, above it, by a rounding of the rate (2^-16) to some millionths of it."""
    indptr, indices, seeds = _graph(dtype, n_seeds)
    d_ip, d_ix, d_seeds = (torch.from_numpy(t).to(DEV) for t in (indptr, indices, seeds))
    ctx = a3.Context(n_seeds, [5])
    n_cases = 0
    for v, deg in enumerate(DEGREES):
        for trial in range(6):
            seed = 1000 * v + trial
            log = np.array([oracle.key(oracle.draw(seed, 0, v, s), Q) for s in range(deg)], dtype=np.int64)
            order = np.argsort(log, kind="stable")
            for m, rank in ((5, 0), (5, 2), (3, 1)):
                u = order[rank]
                cut = log[np.delete(order, rank)[m - 1]]      # the m-th best cached key, times its weight
                rate = cut / log[u] if log[u] > 0 else np.inf
                if not 1.0 < rate < 60000.0:
                    continue
                cm = np.full(len(indptr) - 1, 1, dtype=np.int32)
                cm[indices[indptr[v] + u]] = -1
                d_cm = torch.from_numpy(cm).to(DEV)
                for off in (-3e-6, -4e-7, 0.0, 4e-7, 3e-6):
                    for up in (0, 1):
                        bias = max(int(rate * (1 + off) * Q) + up, Q + 1)
                        print(f"[case] {np.dtype(dtype).name} deg={deg} m={m} seed={seed} bias={bias}", flush=True)
                        got = ctx.sample_blocks(d_ip, d_ix, d_seeds, [m], d_cm, bias, seed).to_host()
                        blocks_equal(got, oracle.sample_blocks(indptr, indices, seeds, [m], cm, bias, seed))
                        n_cases += 1
    assert n_cases > 300
    ctx.close()


@pytest.mark.parametrize("gamma", [300.0, 5000.0, 65535.0])
@pytest.mark.parametrize("n_seeds", [64, 8200])
def test_high_bias_rates(gamma, n_seeds):
    """keys of cached neighbours that lie 1 / gamma as close, down to equal upper halves and equal keys"""
    indptr, indices, seeds = _graph(np.int32, n_seeds)
    d_ip, d_ix, d_seeds = (torch.from_numpy(t).to(DEV) for t in (indptr, indices, seeds))
    ctx = a3.Context(n_seeds, [16])
    rng = np.random.default_rng(int(gamma))
    for share in (0.05, 0.3, 0.9):
        cm = np.where(rng.random(len(indptr) - 1) < share, 1, -1).astype(np.int32)
        d_cm = torch.from_numpy(cm).to(DEV)
        for fan in (1, 5, 15, 16):
            for seed in range(20):
                print(f"[case] gamma={gamma} share={share} fanout={fan} seed={seed}", flush=True)
                got = ctx.sample_blocks(d_ip, d_ix, d_seeds, [fan], d_cm, int(gamma * Q), seed).to_host()
                blocks_equal(got, oracle.sample_blocks(indptr, indices, seeds, [fan], cm, int(gamma * Q), seed))
    ctx.close()
