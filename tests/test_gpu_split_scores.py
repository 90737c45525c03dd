"""Scores of the polynomial-rotation split kernel: any scale of the key factors that keeps the
keys themselves in fp16, and errors no larger than the general split kernel's, which rounds
every rotated key to fp16 once."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2606_08382_amd import starkv as S
from paper_2606_08382_amd import synth

from _helpers import assert_close, oracle_cfg, say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

F16, INT4, MIX84, MIX43 = synth.Q_F16, synth.Q_INT4, synth.Q_MIX8_4, synth.Q_MIX4_3


def _decode(w, inp):
    from paper_2606_08382_amd.device import Layer, to_dev
    layer = Layer(w.batch, w.n_q_heads, w.n_kv_heads, w.head_dim, w.ctx, inp.key_rank, w.value_rank,
                  w.qmode, w.rope_theta, w.q_dtype, w.out_dtype)
    assert S.starkv_decode_fast_blocks(layer.plan, w.ctx) == (1 if w.rope_theta >= 5e5 else 2)
    layer.append(to_dev(inp.latents), torch.zeros(w.batch, dtype=torch.int32, device="cuda"))
    layer.decode(*[to_dev(x) for x in (inp.q, inp.Bk, inp.Bv, inp.ctx_len)])
    torch.cuda.synchronize()
    return layer


@pytest.mark.parametrize("q_dtype", [synth.DT_F16, synth.DT_BF16])
@pytest.mark.parametrize("qmode,theta,shift", [
    (F16, 5e5, 16), (F16, 5e5, -10), (F16, 1e4, 16), (F16, 1e4, -10), (INT4, 5e5, 16),
    (MIX84, 1e4, 16), (MIX43, 5e5, 16), (MIX84, 5e5, -10)])
def test_factor_scale(qmode, theta, shift, q_dtype):
    """B_k times 2^shift and the key latents times 2^-shift: the same keys (entries up to 6e4 at
    shift 16, with queries of standard deviation 4).  With an fp16 cache every product is the same up to powers of two and what the
    smallest operands lose as fp16 subnormals, 2^-4 of a rounding: the error is the same.  All
    against the oracle."""
    ranks, rv = [16, 48, 64, 32], 64
    w = synth.Workload("scale", 3, 16, 4, 128, 300, ranks, "fixed", rv, qmode, theta, q_dtype,
                       synth.DT_F32, ragged=(1, 300), seed=5)
    inp = synth.generate(w)
    ks = sum(ranks)
    if shift > 0:
        exponent = 10 if q_dtype == synth.DT_F16 else 7
        inp.q = (inp.q + (2 << exponent)).astype(np.uint16)            # times four
    Bk = inp.Bk.view(np.float16).astype(np.float64)
    Bk = np.clip(np.round(Bk * 2 ** 14) / 2 ** 14, -0.99, 0.99)        # exact at 2^-10 and 2^16
    lat = inp.latents.view(np.float16).astype(np.float64)
    lat[..., :ks] = np.round(lat[..., :ks] * 256) / 256                # exact at 2^-16 and 2^10

    def scaled(k):
        l2 = lat.copy()
        l2[..., :ks] *= 2.0 ** -k
        inp.Bk, inp.latents = synth.to_bits(Bk * 2.0 ** k, synth.DT_F16), synth.to_bits(l2, synth.DT_F16)
        return _decode(w, inp)

    base = scaled(0).out_float()
    layer = scaled(shift)
    cfg = oracle_cfg(w, inp)
    cache = O.new_cache(cfg)
    O.append(cfg, cache, inp.latents, [0] * w.batch)
    ref, _ = O.decode_attn(cfg, cache, inp.q, q_dtype == synth.DT_BF16, inp.Bk, inp.Bv, inp.ctx_len)
    out = layer.out_float()
    err, scale = assert_close(out, ref, "scaled factors", synth.DT_F32)
    rms = [float(np.sqrt(np.mean((o - ref) ** 2))) for o in (out, base)]
    say(f"max err {err:.3e}, max |o| {scale:.3e}, rms err {rms[0]:.3e}, unscaled {rms[1]:.3e}")
    if qmode == F16:
        assert rms[0] <= 1.1 * rms[1]      # (the rms of 6144 errors, known to a few percent)


def _score_errors(d, theta, ranks, heads, q, Bk, lat, exact):
    """Errors of the split pass's candidate scores for these KV heads: (errors, tokens)."""
    from paper_2606_08382_amd.device import Layer, to_dev
    batch, n = lat.shape[:2]
    off = np.concatenate([[0], np.cumsum(ranks)])
    cols = np.concatenate([np.arange(off[g], off[g + 1]) for g in heads])
    rv, G = 16, q.shape[1] // len(ranks)
    qh = [g * G + i for g in heads for i in range(G)]
    layer = Layer(batch, len(qh), len(heads), d, n, [ranks[g] for g in heads], rv, F16, theta,
                  synth.DT_F16, synth.DT_F32)
    assert (S.starkv_decode_fast_blocks(layer.plan, n) > 0) == (len(heads) > 2)
    z = np.concatenate([lat[..., cols], np.zeros((batch, n, rv))], axis=-1)
    layer.append(to_dev(synth.to_bits(z, synth.DT_F16)),
                 torch.zeros(batch, dtype=torch.int32, device="cuda"))
    layer.dec_ws.zero_()
    ctx = torch.full((batch,), n, dtype=torch.int32, device="cuda")
    S.starkv_decode_split(layer.plan, layer.cache, to_dev(synth.to_bits(q[:, qh], synth.DT_F16)),
                          to_dev(synth.to_bits(Bk[cols], synth.DT_F16)), ctx, n, layer.dec_ws)
    torch.cuda.synchronize()
    # partials [items][heads][rv + 8] fp32 (maximum, normalizer, flags of four candidate blocks at
    # rv .. rv + 2), then [items][heads][64] (score, token); here sequence b is item b
    items = S.starkv_decode_describe(layer.plan, n)["items"]
    n_part = items * len(qh) * (rv + 8) * 4
    ws = layer.dec_ws.cpu().numpy()
    part = ws[:n_part].view(np.float32).reshape(items, len(qh), rv + 8)[:batch]
    at = -(-n_part // 256) * 256
    cand = ws[at:at + items * len(qh) * 512].view(np.float32).reshape(items, len(qh), 64, 2)[:batch]
    flags = np.ascontiguousarray(part[..., rv + 2]).view(np.uint8).reshape(batch, len(qh), 4)
    ok = (np.repeat(flags, 16, axis=2) != 0) & np.isfinite(cand[..., 0])
    tok = np.ascontiguousarray(cand[..., 1]).view(np.int32)
    b, h, e = np.nonzero(ok)
    t = tok[b, h, e]
    return cand[b, h, e, 0] - exact[b, np.array(qh)[h], t], t


@pytest.mark.parametrize("d,theta", [(64, 700.0), (128, 700.0), (128, 4.74e5), (128, 5e5), (128, 1e4)])
def test_score_error(d, theta):
    """64 * theta^(-2j/d) of the first polynomial frequency is 2.4 at the first four: there the
    series has its largest terms.  Two KV heads a plan take the general kernel."""
    rng = np.random.default_rng(11)
    ranks, G, batch, n = [16, 48, 64, 32], 4, 64, 128
    h16 = lambda a: a.astype(np.float16).astype(np.float64)
    Bk = h16(np.concatenate([rng.standard_normal((r, d)) / np.sqrt(r) for r in ranks]))
    q = h16(rng.standard_normal((batch, 4 * G, d)))
    lat = h16(2.0 * rng.standard_normal((batch, n, sum(ranks)))
              / np.sqrt(np.concatenate([np.arange(1, r + 1) for r in ranks])))
    half = d // 2
    ang = np.arange(n)[:, None] * theta ** (-2.0 * np.arange(half) / d)
    exact = np.empty((batch, 4 * G, n))
    off = 0
    for g, r in enumerate(ranks):
        k = lat[..., off:off + r] @ Bk[off:off + r]
        lo, hi = k[..., :half], k[..., half:]
        k = np.concatenate([lo * np.cos(ang) - hi * np.sin(ang), hi * np.cos(ang) + lo * np.sin(ang)], -1)
        exact[:, g * G:(g + 1) * G] = q[:, g * G:(g + 1) * G] @ k.transpose(0, 2, 1)
        off += r
    exact *= 1.4426950408889634 / np.sqrt(d)
    new, t_new = _score_errors(d, theta, ranks, [0, 1, 2, 3], q, Bk, lat, exact)
    parts = [_score_errors(d, theta, ranks, hs, q, Bk, lat, exact) for hs in ([0, 1], [2, 3])]
    old, t_old = (np.concatenate(x) for x in zip(*parts))
    assert min(new.size, old.size) > batch * 4 * G * 32
    rms = lambda e: float(np.sqrt(np.mean(e ** 2)))
    ratio = [rms(new[t_new // 16 == c]) / rms(old[t_old // 16 == c]) for c in range(n // 16)]
    say(f"rms {rms(new):.3e} of {rms(old):.3e}; by 16 tokens {[round(x, 3) for x in ratio]}")
    assert rms(new) <= rms(old)
    # (a group's rms over some 8000 scores is known to about 1 %)
    assert max(ratio) <= 1.01
