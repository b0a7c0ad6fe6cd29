"""The exact-max re-walk in the one-segment kernel (ranges of at most 32 key tiles per work-group), whole
and in equal parts, against the float64 oracle.

A row's exponent offset is the maximum of the first key tile of its range; needle keys (raw keys drawn
N(0, 40^2)) placed after the first tile of the part that holds them push some rows more than 64 / (scale
log2 e) ~ 502 raw units past it, the row sum overflows its 2^64 guard and the work-group walks its range
again, for the exact maximum and then for the sums.  Only the parts with needles do.
"""
import math

import numpy as np
import pytest
import torch

import synth
from oracle import numerics
from tests.gpu_helpers import LSE_ABS, Mirror, check_attention, host, log

pytestmark = pytest.mark.gpu

ROWS = 2 * 256 * 130 * 4          # scratch bytes per work-group
SHORT = 32                        # most key tiles of a work-group in the one-segment kernel

# B, H, grid, C, S, W, R, f0, parts, runs of cache rows, needle tokens of the chunk
CASES = [
    # whole range, one run; the last waves of the only query tile have no query
    (1, 3, 10, 10, 2, 0, 2, 4, 6, 1, 1, (20, 90, 150)),
    # whole range, two runs: frames 11-14 of a 6-frame ring in slots 5 and 0-2
    (2, 2, 10, 10, 2, 0, 2, 6, 13, 1, 2, (20, 90, 150)),
    # equal parts merged in eight slices, needles in one part; one run
    (1, 2, 16, 16, 1, 0, 20, 21, 30, 21, 1, (70, 130, 200)),
    # equal parts, batch 2, sinks, ragged last query tile with idle waves, two runs (also whole)
    (2, 12, 15, 13, 2, 2, 5, 9, 14, 5, 2, (40, 200, 300)),
    # equal parts of 30 key tiles each
    (1, 12, 24, 40, 1, 0, 9, 10, 9, 5, 1, (200, 500, 900)),
]


@pytest.mark.parametrize("B,H,gh,gw,C,S,W,R,f0,parts,runs,needles,use_split",
                         [c + (True,) for c in CASES] + [CASES[3] + (False,)])      # the others are too long whole
def test_rewalk_short(B, H, gh, gw, C, S, W, R, f0, parts, runs, needles, use_split):
    import paper_2609_32518_amd as u

    log(f"rewalk short: B {B} H {H} grid {gh}x{gw} C {C} S {S} W {W} R {R} f0 {f0} parts {parts} split {use_split}")
    m = Mirror(u, B, H, gh, gw, S, R, guard_rows=64)
    for f in range(0, f0, C):
        m.append(f, min(C, f0 - f), (41, f))
    tiles = B * H * -(-C * m.T // 256)
    groups = m.lib.workspace_bytes(f0, C, W) // ROWS or tiles
    assert groups == parts * tiles
    key, n = (41, 100), C * m.T
    k = synth.normal_bf16((B, n, H, 128), key + (synth.K,))
    for j, t in enumerate(needles):
        k[0, t, 0] = synth.normal_bf16((128,), key + (50 + j,), scale=40.0)
    q_rot, out, lse, ref = m.step(f0, C, W, key, use_split=use_split, lse=True, k_bits=k)
    torch.cuda.synchronize()
    assert np.array_equal(host(q_rot), ref)
    m.check_cache("rewalk short")

    # the kernel walks the retained rows in ascending cache order; its parts start at tile i Tk / parts
    rows = m.orc.key_rows(f0, C, W)
    order = np.sort(rows)
    assert 1 + np.count_nonzero(np.diff(order) != 1) == runs
    p = parts if use_split else 1
    tk = -(-len(rows) // 64)
    assert -(-tk // p) <= SHORT
    starts = np.array([i * tk // p for i in range(p)])
    qh = numerics.bf16_to_f64(ref[0, :, 0])
    kc = numerics.bf16_to_f64(m.orc.k[0, 0])
    jump = np.full(n, -np.inf)
    for t in needles:
        row = rows[len(rows) - n + t]
        tile = int(np.searchsorted(order, row)) // 64
        first = starts[np.searchsorted(starts, tile, side="right") - 1]
        assert tile > first, (t, tile, first)            # not in the tile that sets the offset
        jump = np.maximum(jump, qh @ kc[row] - (qh @ kc[order[64 * first:64 * first + 64]].T).max(axis=1))
    past = int((jump > 64 / (128 ** -0.5 * math.log2(math.e))).sum())
    log(f"  rows past the guard: {past} of {n}")
    assert (jump > 530).sum() > n // 20
    want, want_lse = m.expected(ref, f0, C, W)
    log(f"  {check_attention(host(out), want, 'rewalk short')}")
    assert np.max(np.abs(lse.cpu().numpy() - want_lse)) <= LSE_ABS
