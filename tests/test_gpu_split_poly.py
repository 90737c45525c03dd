"""GPU parity of the polynomial-rotation split kernel at the edges of its dispatch: every
pair count of a key head (ranks 16 .. 128), one to four query heads per KV head, head groups
that leave waves without a head or give a head two waves, one and two fast RoPE blocks (rope
bases 5e5 and 1e4), both head dimensions, mixed precision tiles, paged rows, contexts that end
inside a lane's tokens, a 16-token block, a step and a split; and the general kernel where it
takes over (a rope base whose frequencies are all fast, eight query heads per KV head).  fp32
outputs at the bare 2e-3 + 1e-3 |o| bound."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2606_08382_amd import starkv as S
from paper_2606_08382_amd import synth

from _helpers import assert_close, oracle_cfg, say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

F16, INT4, MIX84, MIX43 = synth.Q_F16, synth.Q_INT4, synth.Q_MIX8_4, synth.Q_MIX4_3
ALL = [16, 32, 48, 64, 80, 96, 112, 128]
MID = [16, 64, 32, 48, 16, 48, 64, 32]
CASES = [
    # n_q, n_kv, d, ranks, rv, qmode, theta, ctx lengths, page tokens, fast blocks (0: general kernel)
    (32, 8, 128, ALL, 256, INT4, 5e5, (1, 127, 128, 129, 641), 0, 1),
    (32, 8, 128, ALL, 256, MIX84, 5e5, (2, 63, 255, 257, 1030), 128, 1),
    (32, 8, 128, ALL, 256, MIX43, 5e5, (3, 64, 65, 300, 777), 0, 1),
    (32, 8, 128, MID, 256, F16, 5e5, (1, 17, 33, 500, 640), 256, 1),
    (32, 8, 128, MID, 272, MIX84, 1e4, (5, 130, 700), 0, 2),        # two fast blocks, mixed value tile
    (16, 8, 128, MID, 144, MIX43, 1e4, (31, 32, 900), 0, 2),
    (8, 8, 128, MID, 64, INT4, 1e6, (16, 15, 400), 0, 1),           # one query head per KV head
    (32, 8, 128, MID, 256, INT4, 50.0, (100, 200), 0, 0),           # all frequencies fast: general kernel
    (12, 3, 128, [16, 128, 48], 384, MIX84, 5e5, (64, 66, 515), 128, 1),   # two waves a head, idle waves
    (16, 4, 128, [112, 16, 80, 32], 320, MIX43, 5e5, (1, 2, 66, 450), 0, 1),
    (16, 4, 128, [48, 64, 16, 32], 256, F16, 1e4, (65, 300), 0, 2),
    (20, 5, 128, [32, 16, 96, 48, 128], 128, INT4, 5e5, (7, 390), 0, 1),
    (64, 16, 128, MID * 2, 256, MIX43, 5e5, (129, 640), 0, 1),      # two groups of eight heads
    (32, 8, 128, [128] * 8, 384, MIX84, 5e5, (90, 300), 0, 1),      # groups by LDS size
    (32, 8, 64, [16, 64, 32, 48] * 2, 256, MIX84, 1e4, (77, 128, 400), 0, 1),
    (8, 4, 64, [16, 64, 32, 48], 96, MIX43, 5e5, (3, 333), 0, 1),
    (64, 8, 128, ALL, 384, MIX84, 5e5, (1, 64, 127, 700), 128, 0),  # eight query heads per KV head
    (64, 8, 128, ALL, 384, MIX43, 5e5, (2, 300), 0, 0),
    (32, 4, 128, [16, 128, 96, 48], 256, INT4, 5e5, (65, 1000), 0, 0),
    (24, 3, 128, [64, 16, 48], 256, F16, 5e5, (40, 260), 0, 0),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"h{c[0]}x{c[1]}_d{c[2]}_rv{c[4]}_q{c[5]}_th{c[6]:g}")
def test_split_forms(case):
    from paper_2606_08382_amd.device import Layer, to_dev
    n_q, n_kv, d, ranks, rv, qmode, theta, lens, page, fast_blocks = case
    ctx, batch = max(lens), len(lens)
    w = synth.Workload("poly", batch, n_q, n_kv, d, ctx, ranks, "fixed", rv, qmode, theta,
                       synth.DT_F16, synth.DT_F32, outlier_frac=0.01, seed=77)
    inp = synth.generate(w)
    inp.ctx_len[:] = lens
    kw = {}
    if page:
        per = -(-ctx // page)
        kw = dict(page_tokens=page, n_pages=batch * per + 2, page_rng=np.random.default_rng(3))
    layer = Layer(batch, n_q, n_kv, d, ctx, ranks, rv, qmode, theta, w.q_dtype, w.out_dtype, **kw)
    assert S.starkv_decode_fast_blocks(layer.plan, ctx) == fast_blocks
    if page:
        for b in range(batch):
            layer.pool.ensure(b, ctx)
        layer.pool.sync()
    layer.cache.fill_(0xFF)            # rows past a context hold NaN scales
    layer.append(to_dev(inp.latents), torch.zeros(batch, dtype=torch.int32, device="cuda"))
    args = [to_dev(x) for x in (inp.q, inp.Bk, inp.Bv, inp.ctx_len)]
    layer.decode(*args)
    first = layer.out.clone()
    layer.decode(*args)
    torch.cuda.synchronize()
    assert torch.equal(first, layer.out), "two calls differ"
    cfg = oracle_cfg(w, inp)
    cache = O.new_cache(cfg)
    O.append(cfg, cache, inp.latents, [0] * batch)
    ref, _ = O.decode_attn(cfg, cache, inp.q, False, inp.Bk, inp.Bv, inp.ctx_len)
    err, scale = assert_close(layer.out_float(), ref, "split", synth.DT_F32)
    say(f"max err {err:.3e}, max |o| {scale:.3e}")
