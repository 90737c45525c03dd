"""GPU parity of the polynomial split kernel's head groups: groups of up to eight KV heads (a
wave a head), which plans take whose max_ctx gives the compute units enough work, on the cases
whose short contexts take groups of four; and more than 64 sequences (the equal split grid) with
splits of 64 steps, the longest.  fp32 outputs at the bare 2e-3 + 1e-3 |o| bound."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2606_08382_amd import starkv as S
from paper_2606_08382_amd import synth

from _helpers import assert_close, oracle_cfg, say
from test_gpu_split_poly import ALL, F16, INT4, MID, MIX43, MIX84

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CASES = [
    # n_q, n_kv, d, ranks, rv, qmode, theta, ctx lengths, page tokens, head groups short and long
    (32, 8, 128, ALL, 128, INT4, 5e5, (1, 127, 128, 129, 641), 0, 2, 2),     # (too large for one)
    (32, 8, 128, [16, 96, 48, 64, 32, 96, 16, 64], 256, INT4, 5e5, (1, 127, 129, 641), 0, 2, 1),
    (32, 8, 128, [16, 96, 48, 64, 32, 96, 16, 64], 256, MIX84, 5e5, (2, 63, 257, 1030), 128, 2, 1),
    (32, 8, 128, [16, 96, 48, 64, 32, 80, 16, 64], 272, MIX43, 5e5, (3, 64, 65, 777), 0, 2, 1),
    (32, 8, 128, MID, 256, F16, 5e5, (1, 17, 33, 500, 640), 256, 2, 1),
    (32, 8, 128, MID, 272, MIX84, 1e4, (5, 130, 700), 0, 2, 1),
    (32, 8, 128, MID, 256, F16, 1e4, (5, 130, 700), 0, 2, 2),                # never eight
    (16, 8, 128, MID, 144, MIX43, 1e4, (31, 32, 900), 0, 2, 1),
    (8, 8, 128, MID, 384, INT4, 1e6, (16, 15, 400), 0, 2, 1),
    (20, 5, 128, [32, 16, 96, 48, 128], 128, INT4, 5e5, (7, 390), 0, 2, 1),
    (24, 6, 128, [32, 16, 48, 48, 64, 16], 384, MIX84, 5e5, (7, 390), 0, 2, 1),
    (64, 16, 128, MID * 2, 256, MIX43, 5e5, (129, 640), 0, 4, 2),
    (32, 8, 64, [16, 64, 32, 48] * 2, 256, MIX84, 1e4, (77, 128, 400), 0, 2, 1),
    (32, 8, 64, [16, 64, 32, 48] * 2, 128, F16, 1e4, (77, 128, 400), 0, 2, 1),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"h{c[0]}x{c[1]}_d{c[2]}_rv{c[4]}_q{c[5]}_th{c[6]:g}")
def test_group_forms(case):
    from paper_2606_08382_amd.device import Layer, to_dev
    n_q, n_kv, d, ranks, rv, qmode, theta, lens, page, g_short, g_long = case
    ctx, batch, cap = max(lens), len(lens), 40000
    w = synth.Workload("groups", batch, n_q, n_kv, d, ctx, ranks, "fixed", rv, qmode, theta,
                       synth.DT_F16, synth.DT_F32, outlier_frac=0.01, seed=79)
    inp = synth.generate(w)
    inp.ctx_len[:] = lens
    kw = {}
    if page:
        per = -(-ctx // page)
        kw = dict(page_tokens=page, n_pages=batch * per + 2, page_rng=np.random.default_rng(3))
    layer = Layer(batch, n_q, n_kv, d, cap, ranks, rv, qmode, theta, w.q_dtype, w.out_dtype, **kw)
    for max_ctx, groups in ((ctx, g_short), (cap, g_long)):
        info = S.starkv_decode_describe(layer.plan, max_ctx)
        assert info["fast_blocks"] > 0 and info["head_groups"] == groups
    if page:
        for b in range(batch):
            layer.pool.ensure(b, ctx)
        layer.pool.sync()
    layer.cache.fill_(0xFF)            # rows past a context hold NaN scales
    layer.append(to_dev(inp.latents), torch.zeros(batch, dtype=torch.int32, device="cuda"))
    args = [to_dev(x) for x in (inp.q, inp.Bk, inp.Bv, inp.ctx_len)]
    cfg = oracle_cfg(w, inp)
    cache = O.new_cache(cfg)
    O.append(cfg, cache, inp.latents, [0] * batch)
    ref, _ = O.decode_attn(cfg, cache, inp.q, False, inp.Bk, inp.Bv, inp.ctx_len)
    for max_ctx in (ctx, cap):
        layer.decode(*args, max_ctx=max_ctx)
        first = layer.out.clone()
        layer.decode(*args, max_ctx=max_ctx)
        torch.cuda.synchronize()
        assert torch.equal(first, layer.out), "two calls differ"
        err, scale = assert_close(layer.out_float(), ref, f"max_ctx {max_ctx}", synth.DT_F32)
        say(f"max_ctx {max_ctx}: max err {err:.3e}, max |o| {scale:.3e}")


@pytest.mark.parametrize("qmode,page,peaked", [(INT4, 128, 1), (MIX84, 0, 0), (MIX43, 128, 0), (F16, 256, 1)])
def test_many_sequences_long_splits(qmode, page, peaked):
    """260 sequences of up to 8192 tokens are one split each: 64 steps, as many pages of 128
    tokens as a wave has lanes.  Three of them against the oracle, two of full length."""
    from paper_2606_08382_amd.device import Layer, to_dev
    batch, n_q, ranks, rv, cap = 260, 8, [16, 32, 16, 48], 32, 8192
    w = synth.Workload("many", 3, n_q, 4, 128, cap, ranks, "fixed", rv, qmode, 5e5, synth.DT_BF16,
                       synth.DT_F32, seed=83)
    inp = synth.generate(w, peaked=peaked)
    at = [0, 131, 259]
    inp.ctx_len[:] = [cap, 8065, 8191]
    rng = np.random.default_rng(4)
    lens = rng.integers(0, 200, batch).astype(np.int32)
    lens[at] = inp.ctx_len
    q = rng.standard_normal((batch, n_q, 128))
    q = synth.to_bits(q, synth.DT_BF16)
    q[at] = inp.q
    kw = {}
    if page:
        kw = dict(page_tokens=page, n_pages=3 * (cap // page) + 2 * batch + 2, page_rng=np.random.default_rng(5))
    layer = Layer(batch, n_q, 4, 128, cap, ranks, rv, qmode, 5e5, w.q_dtype, w.out_dtype, **kw)
    info = S.starkv_decode_describe(layer.plan, cap)
    assert info["fast_blocks"] == 1 and info["device_plan"] == 0 and info["split_tokens"] == 8192
    if page:
        for b in range(batch):
            layer.pool.ensure(b, int(lens[b]))
        layer.pool.sync()
    for t0 in range(0, cap, 1024):
        lat = np.zeros((batch, 1024, inp.width), np.uint16)
        lat[:] = inp.latents[0, :1024]
        lat[at] = inp.latents[:, t0:t0 + 1024]
        layer.append(to_dev(lat), torch.full((batch,), t0, dtype=torch.int32, device="cuda"))
    layer.decode(*[to_dev(x) for x in (q, inp.Bk, inp.Bv, lens)])
    torch.cuda.synchronize()
    out = layer.out_float()
    assert np.isfinite(out).all() and not out[lens == 0].any()
    cfg = oracle_cfg(w, inp)
    cache = O.new_cache(cfg)
    O.append(cfg, cache, inp.latents, [0] * 3)
    ref, _ = O.decode_attn(cfg, cache, inp.q, True, inp.Bk, inp.Bv, inp.ctx_len)
    err, scale = assert_close(out[at], ref, "long splits", synth.DT_F32)
    say(f"max err {err:.3e}, max |o| {scale:.3e}")
