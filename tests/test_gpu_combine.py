"""GPU parity of the combine pass where its dispatch and its loops turn: sixteen waves (at
most one workgroup per compute unit) and four waves, both head dimensions, value ranks that
are no multiple of a 256-channel chunk or exceed one channel per thread, fewer candidates
than a wave holds, all tokens of a short context rescored, and more than 64 splits.  Peaked
inputs, so that the exact rescoring runs; fp32 outputs at the bare 2e-3 + 1e-3 |o| bound."""
import pytest

from oracle import oracle as O
from paper_2606_08382_amd import synth

from _helpers import assert_close, oracle_cfg, say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CASES = [
    # batch, n_q, n_kv, d, ranks, rv, qmode, ctx, ragged
    (1, 4, 1, 64, [16], 16, synth.Q_F16, 3, None),
    (1, 8, 2, 64, [16, 64], 128, synth.Q_INT4, 300, None),
    (9, 32, 8, 64, [16, 32, 48, 64] * 2, 272, synth.Q_MIX8_4, 70, (1, 70)),
    (9, 32, 8, 128, [16, 128, 48, 96] * 2, 272, synth.Q_MIX4_3, 200, (1, 200)),
    (2, 32, 8, 128, [32] * 8, 768, synth.Q_MIX8_4, 257, None),
    (1, 8, 2, 128, [48, 112], 208, synth.Q_MIX4_3, 8400, None),     # 66 splits
    (65, 8, 2, 128, [16, 80], 64, synth.Q_F16, 150, (0, 150)),      # equal split grid
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"b{c[0]}_h{c[1]}x{c[2]}_d{c[3]}_rv{c[5]}_q{c[6]}_ctx{c[7]}")
def test_combine_forms(case):
    from paper_2606_08382_amd.device import Layer, to_dev
    batch, n_q, n_kv, d, ranks, rv, qmode, ctx, ragged = case
    w = synth.Workload("combine", batch, n_q, n_kv, d, ctx, ranks, "fixed", rv, qmode, 5e5,
                       synth.DT_BF16, synth.DT_F32, ragged=ragged, seed=31)
    inp = synth.generate(w, peaked=1)
    layer = Layer(batch, n_q, n_kv, d, ctx, ranks, rv, qmode, w.rope_theta, w.q_dtype, w.out_dtype)
    layer.append(to_dev(inp.latents), torch.zeros(batch, dtype=torch.int32, device="cuda"))
    q, Bk, Bv, n = (to_dev(x) for x in (inp.q, inp.Bk, inp.Bv, inp.ctx_len))
    layer.decode(q, Bk, Bv, n)
    first = layer.out.clone()
    layer.decode(q, Bk, Bv, n)
    torch.cuda.synchronize()
    assert torch.equal(first, layer.out), "two calls differ"
    cfg = oracle_cfg(w, inp)
    cache = O.new_cache(cfg)
    O.append(cfg, cache, inp.latents, [0] * batch)
    ref, _ = O.decode_attn(cfg, cache, inp.q, True, inp.Bk, inp.Bv, inp.ctx_len)
    err, scale = assert_close(layer.out_float(), ref, "combine", synth.DT_F32)
    say(f"max err {err:.3e}, max |o| {scale:.3e}")
