"""Scores of the polynomial-rotation split kernel: any scale of the key factors that keeps the
keys themselves in fp16."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2606_08382_amd import synth

from _helpers import assert_close, oracle_cfg, say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

F16, INT4, MIX84, MIX43 = synth.Q_F16, synth.Q_INT4, synth.Q_MIX8_4, synth.Q_MIX4_3


def _decode(w, inp):
    from paper_2606_08382_amd.device import Layer, to_dev
    layer = Layer(w.batch, w.n_q_heads, w.n_kv_heads, w.head_dim, w.ctx, inp.key_rank, w.value_rank,
                  w.qmode, w.rope_theta, w.q_dtype, w.out_dtype)
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
