"""unstep_linear at the edges of each tile size its launch rule picks, against the float64 oracle.

Bound per element: one bf16 rounding of the result (2^-8 of its value covers it twice) plus K
float32 roundings of the running sum, each at most 2^-24 of sum |x| |w| + |b|.
"""
import numpy as np
import pytest
import torch

import synth
from oracle import numerics, svd
from tests.gpu_helpers import dev, host, log

pytestmark = pytest.mark.gpu

SHAPES = [
    # 128 x 256 tiles: ragged in both, a k tail of one chunk, and one k step in all
    (4681, 1544, 136), (4608, 1536, 40),
    # 128 x 128: ragged in both, k tails; whole tiles, fewer stages than the ring holds
    (1537, 1544, 72), (1536, 1536, 192),
    # 64 x 128: rows of 2064 bytes, ragged; whole tiles
    (1365, 1000, 1032), (1281, 1024, 320),
    # 64 x 64: one value more and less than a tile, the smallest call, deep k
    (65, 72, 8), (63, 64, 64), (1, 8, 8), (64, 136, 4104), (129, 3072, 200),
    # rows longer than the tiles' 32-bit offsets address: the register-staged kernel (the bound is wider
    # than the values there; test_gpu_linear_exact.py checks those)
    (2, 8, (1 << 22) + 8),
]


@pytest.mark.parametrize("M,N,K", SHAPES)
@pytest.mark.parametrize("bias", [True, False])
def test_linear_tiles(M, N, K, bias):
    import paper_2609_32518_amd as u

    log(f"linear tiles: M {M} N {N} K {K} bias {bias}")
    x = synth.normal_bf16((M, K), (M, N, K, 21))
    w = synth.normal_bf16((N, K), (M, N, K, 22), 1.0 / np.sqrt(K))
    b = synth.normal_bf16((N,), (M, N, K, 23)) if bias else None
    guard = 64                                       # y stays inside its buffer
    buf = torch.full((M * N + 2 * guard,), 7.0, dtype=torch.bfloat16, device="cuda")
    y = buf[guard:guard + M * N].view(M, N)
    u.unstep_linear(dev(x), dev(w), dev(b) if bias else None, out=y)
    torch.cuda.synchronize()
    want = svd.linear(x, w, b)
    mag = np.abs(numerics.bf16_to_f64(x)) @ np.abs(numerics.bf16_to_f64(w)).T
    if bias:
        mag = mag + np.abs(numerics.bf16_to_f64(b))
    err = np.abs(numerics.bf16_to_f64(host(y)) - want)
    assert np.all(err <= 2.0 ** -8 * np.abs(want) + K * 2.0 ** -24 * mag)
    assert bool((buf[:guard] == 7).all()) and bool((buf[guard + M * N:] == 7).all())
