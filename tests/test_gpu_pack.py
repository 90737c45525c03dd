"""Byte parity of the two packs at their edges.  Appends given as latents: rows that cover
64-row blocks, value words (eight tokens four apart) and key blocks in part, groups of 8, 16, 24
and 32 channels, every precision, ties and scales at fp16's edges (subnormal spans, spans of up
to 131008), single infinities and NaNs beside finite tokens, latents at an odd 2-byte address,
pages, rows outside the cache.  Appends of a few hidden states (a lane per channel): the same
values through a projection that copies them."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2606_08382_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

KINDS = ["normal", "ties", "subnormal", "huge", "mixed", "inf", "nan"]


def _latents(kind, shape, rng):
    if kind == "normal":
        x = rng.standard_normal(shape)
    elif kind == "ties":                    # small multiples of 1/8 and constant groups
        x = rng.integers(-40, 41, shape) / 8.0
        x[:, ::5] = 0.375
    elif kind == "subnormal":
        x = rng.integers(-90, 91, shape) * 2.0 ** -24
    elif kind == "huge":
        x = rng.choice([-65504.0, 65504.0, 2.0 ** -24, 1.0, -3.0], shape) * rng.choice([1.0, 0.5], shape)
    else:
        x = rng.standard_normal(shape) * 2.0 ** rng.integers(-24, 13, shape)
        if kind != "mixed":                 # a few single values, most tokens without one
            n = max(1, x.size // 500)
            at = rng.choice(x.size, n, replace=False)
            x.reshape(-1)[at] = rng.choice([np.inf, -np.inf], n) if kind == "inf" else np.nan
    # (no negative zeros: which sign a group's zero point takes among both is not defined)
    return np.ascontiguousarray(x.astype(np.float16) + np.float16(0)).view(np.uint16)


@pytest.mark.parametrize("qmode", [synth.Q_F16, synth.Q_INT4, synth.Q_MIX8_4, synth.Q_MIX4_3])
@pytest.mark.parametrize("page", [0, 128])
def test_append_bytes(qmode, page):
    from paper_2606_08382_amd.device import Layer, to_dev
    rng = np.random.default_rng(1000 + 10 * qmode + page)
    ranks, rv, batch, cap = [16, 48, 80, 128], 272, 3, 400
    if qmode == synth.Q_F16:
        ranks, rv = [16, 48, 64, 32], 144
    width = sum(ranks) + rv
    cfg = O.make_cfg(batch, 8, 4, 128, cap, ranks, rv, qmode, 1e4)
    for n_new, pos in [(5, [0, 30, 63]), (33, [1, 64, 97]), (64, [0, 17, 333]), (131, [3, 64, 200]),
                       (260, [7, 128, 390])]:
        for kind in KINDS:
            lat = _latents(kind, (batch, n_new, width), rng)
            kw = {}
            if page:
                kw = dict(page_tokens=page, n_pages=4 * batch)
            layer = Layer(batch, 8, 4, 128, cap, ranks, rv, qmode, 1e4, synth.DT_F16, synth.DT_F32, **kw)
            if page:
                for b in range(batch):      # in order: the pool is laid out like padded rows
                    layer.pool.ensure(b, cap)
                layer.pool.sync()
            layer.cache.fill_(0xA5)
            buf = torch.zeros(lat.size + 1, dtype=torch.int16, device="cuda")
            buf[1:] = to_dev(lat).flatten()
            layer.append(buf[1:].view(lat.shape), torch.tensor(pos, dtype=torch.int32, device="cuda"))
            torch.cuda.synchronize()
            cache = O.new_cache(cfg)
            cache[:] = 0xA5
            O.append(cfg, cache, lat, pos)  # (drops rows beyond the capacity, too)
            got = layer.cache.cpu().numpy()
            assert got.shape == cache.shape
            bad = np.nonzero(got != cache)[0]
            assert bad.size == 0, f"{kind} n_new {n_new}: {bad.size} bytes differ, first at {bad[0]}"


def _bf16(x):
    """Rounded to bf16 (and to fp16's range and grid, which keeps eight bits of the first)."""
    u = synth.f32_to_bf16_bits(np.clip(x, -65280, 65280).astype(np.float32))
    return (u.astype(np.uint32) << 16).view(np.float32)


@pytest.mark.parametrize("qmode", [synth.Q_F16, synth.Q_INT4, synth.Q_MIX8_4, synth.Q_MIX4_3])
@pytest.mark.parametrize("n_new,pos", [(1, [0, 31, 333]), (4, [3, 62, 127]), (5, [0, 30, 63])])
def test_projected_bytes(qmode, n_new, pos):
    """A_all with a single one per column: the latents are inputs, exactly."""
    from paper_2606_08382_amd.device import Layer, to_dev
    rng = np.random.default_rng(2000 + 10 * qmode + n_new)
    ranks, rv, batch, cap = [16, 48, 80, 128], 272, 3, 400
    if qmode == synth.Q_F16:
        ranks, rv = [16, 48, 64, 32], 144
    width = sum(ranks) + rv
    d_model = -(-width // 64) * 64
    A = np.zeros((d_model, width))
    A[np.arange(width), np.arange(width)] = 1.0
    cfg = O.make_cfg(batch, 8, 4, 128, cap, ranks, rv, qmode, 1e4)
    for kind in ("normal", "ties", "subnormal", "huge", "mixed"):
        x = np.zeros((batch, n_new, d_model), np.float32)
        # (2^-24 multiples of at most eight bits are exact in both types)
        x[..., :width] = _bf16(_latents(kind, (batch, n_new, width), rng).view(np.float16).astype(np.float32))
        x = x.astype(np.float16).astype(np.float32)
        x = _bf16(x)
        x += np.float32(0)                  # (no negative zeros)
        lat = np.ascontiguousarray(x[..., :width].astype(np.float16))
        assert np.array_equal(lat.astype(np.float32), x[..., :width])
        layer = Layer(batch, 8, 4, 128, cap, ranks, rv, qmode, 1e4, synth.DT_F16, synth.DT_F32, d_model=d_model)
        layer.cache.fill_(0xA5)
        layer.append(to_dev(synth.f32_to_bf16_bits(x)), torch.tensor(pos, dtype=torch.int32, device="cuda"),
                     to_dev(synth.to_bits(A, synth.DT_BF16)))
        torch.cuda.synchronize()
        cache = O.new_cache(cfg)
        cache[:] = 0xA5
        O.append(cfg, cache, lat.view(np.uint16), pos)
        got = layer.cache.cpu().numpy()
        bad = np.nonzero(got != cache)[0]
        assert bad.size == 0, f"{kind} n_new {n_new}: {bad.size} bytes differ, first at {bad[0]}"
