"""Sizes of the decode workspace, computed on the host: a workspace of the size reported for a
plan's largest context serves every shorter one, as decode calls with max_ctx below the capacity
expect.  Calls are made with NULL device pointers: whether the workspace is large enough is
checked before they are."""
import ctypes as C

import pytest

from paper_2606_08382_amd import starkv as S

R8 = [16, 48, 32, 32, 16, 48, 32, 32]
R128 = [128] * 8
CASES = [
    # batch, query heads, key ranks, value rank, qmode, theta
    (65, 32, R8, 256, S.Q_MIX8_4, 5e5),        # equal split grid, one or two head groups
    (70, 32, R8, 384, S.Q_MIX8_4, 5e5),
    (85, 32, R8, 256, S.Q_F16, 1e4),
    (100, 32, R8, 384, S.Q_MIX8_4, 1e4),
    (127, 32, R8, 384, S.Q_MIX8_4, 5e5),
    (128, 32, R8, 384, S.Q_MIX8_4, 5e5),
    (200, 32, R8, 384, S.Q_MIX8_4, 5e5),       # near the fixed scratch's size
    (255, 32, R8, 384, S.Q_MIX8_4, 5e5),
    (300, 32, R8, 384, S.Q_MIX8_4, 5e5),
    (66, 64, [48] * 16, 384, S.Q_MIX8_4, 5e5),
    (70, 8, [32], 64, S.Q_INT4, 5e5),          # general kernel
    (70, 64, R128, 384, S.Q_MIX8_4, 5e5),
    (1, 32, R8, 256, S.Q_F16, 1e4),            # work plan on the device
    (8, 32, R128, 384, S.Q_MIX8_4, 1e4),
    (64, 32, R8, 384, S.Q_MIX8_4, 5e5),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"b{c[0]}_h{c[1]}x{len(c[2])}_rv{c[3]}_q{c[4]}_th{c[5]:g}")
def test_largest_context_serves_all(case):
    batch, n_q, ranks, rv, qmode, theta = case
    cap = 20000
    plan = S.starkv_plan_create(S.make_config(batch, n_q, len(ranks), 128, cap, ranks, rv, qmode, theta))
    sizes = sorted({c for k in range(1, 157) for c in (128 * k - 1, 128 * k, 128 * k + 1) if c <= cap}
                   | {1, 300, 8192, 8193, 16385, cap})
    full = S.starkv_decode_workspace_bytes(plan, cap)
    last = 0
    fake = C.c_void_p(256)                     # aligned, never read

    def status(ctx, n_bytes):
        return S.lib().starkv_decode_attn(plan.handle, None, None, None, None, None, ctx, None, fake,
                                          n_bytes, None)

    for c in sizes:
        need = S.starkv_decode_workspace_bytes(plan, c)
        assert last <= need <= full, f"context {c}: {need} bytes, {last} for a shorter one, {full} for {cap}"
        last = need
        assert status(c, full) == 1, f"context {c}"          # INVALID_ARG: the NULL pointers
        assert status(c, need) == 1, f"context {c}"
        assert status(c, 1024) == 4                           # WORKSPACE


def test_items_follow_the_fixed_scratch():
    """255 sequences whose split grid by the polynomial kernel's single head group (510 items)
    would exceed the scratch array of the no-allocation entry point, by the general kernel's two
    (255 items) not: the call is not refused for its workspace."""
    ranks, rv, ctx = R8, 384, 8192
    plan = S.starkv_plan_create(S.make_config(255, 32, 8, 128, ctx, ranks, rv, S.Q_MIX8_4, 5e5))
    info = S.starkv_decode_describe(plan, ctx)
    assert info["items"] == 255 and info["head_groups"] == 1
    assert S.starkv_decode_workspace_bytes(plan, ctx) <= 32 << 20
    st = S.lib().starkv_decode_attn_noalloc(plan.handle, None, None, None, None, None, ctx, None, None)
    assert st in (1, 6)                        # NULL pointers, or no device
    smaller = S.starkv_plan_create(S.make_config(120, 32, 8, 128, ctx, ranks, rv, S.Q_MIX8_4, 5e5))
    assert S.starkv_decode_describe(smaller, ctx)["items"] == 360
