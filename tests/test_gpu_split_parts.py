"""Attention split into the kinds of parts the plan makes, against the float64 oracle: query tiles
whole and cut into 3, 4, 5, 9, 11 and 21 parts of four and more key tiles (the merge loads four partials at
a time, in one, two, four or eight slices), a ragged last query tile whose merge blocks past the chunk
return at once, and the contiguous split whose work-groups walk the ends of two query tiles."""
import numpy as np
import pytest
import torch

from tests.gpu_helpers import LSE_ABS, Mirror, check_attention, host, log

pytestmark = pytest.mark.gpu

ROWS = 2 * 256 * 130 * 4          # scratch bytes per work-group


# B, H, grid, chunk, sinks, window, expected work-groups per query tile (None: contiguous split)
CASES = [
    (1, 2, 5, 7, 2, 1, 4, 1),             # whole: the split would save less than the merge costs
    (1, 1, 6, 10, 1, 0, 11, 3),           # one slice, parts of four key tiles
    (2, 12, 15, 13, 2, 2, 5, 5),          # five partials: a batch of four and one more
    (1, 8, 10, 10, 3, 0, 9, 4),           # two slices
    (1, 12, 6, 54, 1, 1, 12, 9),          # two slices of five and four, ragged last query tile
    (1, 5, 16, 17, 1, 0, 11, 11),         # four slices
    (1, 2, 16, 16, 1, 0, 20, 21),         # eight slices
    (1, 130, 5, 7, 2, 0, 44, None),       # contiguous split (of 130 query tiles)
]


@pytest.mark.parametrize("B,H,gh,gw,C,S,W,parts", CASES)
def test_parts(B, H, gh, gw, C, S, W, parts):
    import paper_2609_32518_amd as u

    log(f"parts: B {B} H {H} grid {gh}x{gw} C {C} S {S} W {W} -> {parts}")
    R = W + C + 1
    m = Mirror(u, B, H, gh, gw, S, R, guard_rows=64)
    f0 = S + W + C                               # past the sinks; the ring has not wrapped ...
    for f in range(0, f0, C):
        m.append(f, min(C, f0 - f), (31, f))
    for i, f in enumerate((f0, f0 + C)):         # ... and has wrapped or is about to
        tiles = B * H * -(-C * gh * gw // 256)
        groups = m.lib.workspace_bytes(f, C, W) // ROWS or tiles
        assert (groups % tiles != 0) if parts is None else groups == parts * tiles, (groups, tiles)
        q_rot, out, lse, ref = m.step(f, C, W, (31, 100 + i), lse=True)
        torch.cuda.synchronize()
        assert np.array_equal(host(q_rot), ref)
        m.check_cache(f"parts {f}")
        want, want_lse = m.expected(ref, f, C, W)
        check_attention(host(out), want, f"parts {f}")
        assert np.max(np.abs(lse.cpu().numpy() - want_lse)) <= LSE_ABS


@pytest.mark.parametrize("groups,parts", [(216, 9), (215, 8), (72, 3), (71, 2), (47, 1), (1, 1)])
def test_scratch_for_some_of_the_parts(groups, parts):
    """A scratch of fewer work-groups than the plan's 9 parts of 24 query tiles: as many parts as it holds,
    and nothing written past it."""
    import paper_2609_32518_amd as u

    log(f"parts: scratch of {groups} work-groups -> {parts}")
    C, W = 1, 12
    m = Mirror(u, 1, 12, 6, 54, 1, W + C + 1, guard_rows=64)
    f0 = W + 2
    for f in range(f0):
        m.append(f, C, (33, f))
    ws = torch.full((groups * ROWS + 4096,), 0x5a, dtype=torch.uint8, device="cuda")
    q_rot, _, _, ref = m.step(f0, C, W, (33, 100))
    lse = torch.empty((1, 12, C * m.T), device="cuda")
    out = m.lib.unstep_window_attn(f0, C, W, q_rot, lse=lse, workspace=ws[:groups * ROWS])
    torch.cuda.synchronize()
    assert bool((ws[groups * ROWS:] == 0x5a).all())
    assert bool((ws == 0x5a).all()) == (parts == 1)
    # the last work-group's partial outputs: written by the last of parts * 24 work-groups, none after it
    o = ws[:parts * 24 * 2 * 256 * 128 * 4].view(-1, 2 * 256 * 128 * 4)[-1] if parts > 1 else ws[:0]
    assert parts == 1 or not bool((o == 0x5a).all())
    want, want_lse = m.expected(ref, f0, C, W)
    check_attention(host(out), want, f"scratch of {groups}")
    assert np.max(np.abs(lse.cpu().numpy() - want_lse)) <= LSE_ABS
