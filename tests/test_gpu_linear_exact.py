"""unstep_linear on small whole numbers, where its float32 sums are exact in any order: y must equal the
one rounding to bf16 of the exact result, bit for bit, in every tile size of the launch rule, with rings
that wrap many times and k tails after a wrap, and in the register-staged kernel.

Sums of at most 2^22 products of magnitude at most 4 (of 1 in rows of 2^22 values and more) and a bias of at
most 8 stay below 2^24, so every partial sum is a whole number that float32 holds.
"""
import numpy as np
import pytest
import torch

from oracle import numerics, svd
from tests.gpu_helpers import dev, host, log

pytestmark = pytest.mark.gpu

# M, N, K and the tile (columns, rows of y) that the launch rule gives them; staged: the
# register-staged kernel.  tests/test_linear_plan_cpu.py checks the rule against this list.
SHAPES = [
    # one frame's projection (24 stages in a ring of 5), and ragged in both with a k tail after three wraps
    (1560, 1536, 1536, (128, 128, False)), (1537, 1544, 1032, (128, 128, False)),
    # fewer and as many stages as the ring holds
    (1537, 1544, 72, (128, 128, False)), (1536, 1536, 320, (128, 128, False)),
    # a chunk's projection (24 stages in a ring of 3), ragged with a k tail after wraps, one stage
    (4680, 1536, 1536, (128, 256, False)), (4681, 1544, 1032, (128, 256, False)), (4608, 1536, 40, (128, 256, False)),
    (1365, 1000, 1032, (64, 128, False)), (1281, 1024, 1536, (64, 128, False)),
    (64, 136, 4104, (64, 64, False)), (129, 3072, 200, (64, 64, False)), (1, 8, 8, (64, 64, False)),
    # rows longer than the tiles' 32-bit offsets address, and no whole number of k steps
    (9, 16, (1 << 22) + 8, (128, 128, True)), (130, 8, (1 << 22), (128, 128, True)),
]


def _whole(M, N, K):
    """x [M, K] and w [N, K] as float32.  Long rows: row 0 of x dense, the others zero but for some
    200 places, both ends and a step's edge among them, so that sums stay exact in bf16 too and one
    chunk left out shows."""
    rng = np.random.default_rng((M, N, K))
    if K < 1 << 20:
        return (rng.integers(-2, 3, s).astype(np.float32) for s in ((M, K), (N, K)))
    w = rng.integers(0, 2, (N, K)).astype(np.float32) * 2 - 1
    x = np.zeros((M, K), np.float32)
    x[0] = rng.integers(0, 2, K) * 2 - 1
    for r in range(1, M):
        at = np.concatenate([rng.integers(0, K, 200), [0, 7, 63, 64, K - 65, K - 8, K - 1], rng.integers(K - 72, K, 8)])
        x[r, at] = 1
    return x, w


def _bits(v):
    return (np.ascontiguousarray(v, np.float32).view(np.uint32) >> 16).astype(np.uint16)     # whole numbers: exact


@pytest.mark.parametrize("M,N,K,bias", [s[:3] + (b,) for s in SHAPES for b in (True, False) if b or s[2] < 1 << 20])
def test_exact(M, N, K, bias):
    import paper_2609_32518_amd as u

    log(f"linear exact: M {M} N {N} K {K} bias {bias}")
    x, w = _whole(M, N, K)
    b = np.random.default_rng(7).integers(-8, 9, N).astype(np.float32) if bias else None
    xb, wb, bb = _bits(x), _bits(w), _bits(b) if bias else None
    want = svd.linear(xb, wb, bb)
    # what the comparison has to notice: nothing computed, or a row's last 16-byte chunk left out
    cut = want - x[:, K - 8:].astype(np.float64) @ w[:, K - 8:].T.astype(np.float64)
    want_bits = numerics.f32_to_bf16_bits(want)
    assert M * N < 64 or (want_bits != numerics.f32_to_bf16_bits(cut)).any() and want_bits.any()
    guard = 64                                       # y stays inside its buffer
    buf = torch.full((M * N + 2 * guard,), 7.0, dtype=torch.bfloat16, device="cuda")
    y = buf[guard:guard + M * N].view(M, N)
    u.unstep_linear(dev(xb), dev(wb), dev(bb) if bias else None, out=y)
    torch.cuda.synchronize()
    got = host(y)
    assert np.array_equal(numerics.bf16_to_f64(got), numerics.bf16_to_f64(want_bits)), \
        f"{np.count_nonzero(got != want_bits)} of {got.size} values differ"
    assert bool((buf[:guard] == 7).all()) and bool((buf[guard + M * N:] == 7).all())
