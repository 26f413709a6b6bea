"""The sampler's single-precision keys against its exact ones, over all draws."""
import ctypes as C

import pytest
import torch

from native import build as native

pytestmark = pytest.mark.gpu
Q = 65536
DEV = "cuda:0"


@pytest.mark.parametrize("gamma", [1.0, 1.25, 4.0, 1000.0, 65535.0])
def test_error_of_the_single_precision_keys(gamma):
    """Two keys are told apart from 4 (1 / w + key) kKeyError on: 2 for each of them.  Expected: 0.12 for the
    logarithm and 2^-23 / 2^-20 = 0.125 for the division by the weight (a rounded reciprocal and a product).
    Sixteenfold room is left below the limit."""
    lib = C.CDLL(native.build(force=False))
    lib.key_error.argtypes = [C.c_uint32, C.c_uint32, C.c_void_p, C.c_void_p]
    blocks = 8192
    worst = torch.zeros(blocks * 256, dtype=torch.float64, device=DEV)
    print(f"[case] all draws, weight {gamma}", flush=True)
    assert lib.key_error(int(gamma * Q), blocks, worst.data_ptr(), torch.cuda.current_stream().cuda_stream) == 0
    got = float(worst.max())
    print(f"largest error: {got:.4f} kKeyError (1 / w + key)", flush=True)
    assert 0.0 < got <= (0.12 if gamma == 1.0 else 0.245)
