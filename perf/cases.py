"""Performance cases of the decode-attention library: what a serving program calls.

A case is one call (or one append + decode step) of a single attention layer, through
``paper_2606_08382_amd.device.Layer``.  ``prepare`` builds what a serving loop holds before the
call: a filled cache, factors, queries, workspaces.  ``run`` is the call.  ``exact`` is the same
result in float64 with plain torch.

Kinds of case:
  decode    one decode-attention step over the cache; output [B][H_q][d]
  step      append of one token per sequence from hidden states, then the decode step;
            output and the updated cache
  absorbed  decode step with the value up-projection absorbed into the output projection
  prefill   append of many tokens from hidden states; the latents and the cache
  fill      append of many tokens given as latents; the cache
"""
from __future__ import annotations

import math

import torch

from paper_2606_08382_amd import starkv as S
from paper_2606_08382_amd.device import Layer

QMODES = {"f16": S.Q_F16, "int4": S.Q_INT4, "mix8_4": S.Q_MIX8_4, "mix4_3": S.Q_MIX4_3}
DTYPES = {"f16": S.DT_F16, "bf16": S.DT_BF16, "f32": S.DT_F32}
TORCH_DT = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}
CHUNK = 8192                     # tokens per sequence of one filling append


def _case(name, kind, batch, n_q, n_kv, d, ranks, rv, qmode, lo, hi, theta=5e5, q="bf16",
          out="bf16", d_model=0, n_new=1, page=0, peaked=False, d_out=0):
    """lo..hi: context lengths (drawn per sequence when they differ); ranks: one key rank per
    KV head; n_new: tokens appended per sequence; page: tokens per cache page (0: contiguous)."""
    return {"name": name, "kind": kind, "batch": batch, "n_q": n_q, "n_kv": n_kv, "d": d,
            "ranks": ",".join(str(r) for r in ranks), "rv": rv, "qmode": qmode, "lo": lo,
            "hi": hi, "theta": theta, "q": q, "out": out, "d_model": d_model, "n_new": n_new,
            "page": page, "peaked": peaked, "d_out": d_out}


R_8B = [16, 48, 32, 32, 16, 48, 32, 32]           # learned ranks of an 8B layer, about 75 % cut
R_8B_HI = [16, 96, 48, 64, 32, 96, 16, 64]        # the same layer kept at higher ranks
R_70B = [80, 32, 128, 128, 48, 112, 64, 96]       # a 70B layer


def listed():
    return [
        # smallest call: one short sequence, uncompressed latents; launch latency counts
        _case("decode_1x1k_f16_d64", "decode", 1, 4, 1, 64, [16], 16, "f16", 1024, 1024, 1e4,
              "f16", "f16"),
        # a single user's chat turn: one token appended and attended, batch 1
        _case("step_1x8k_mix84", "step", 1, 32, 8, 128, R_8B, 256, "mix8_4", 8192, 8192,
              d_model=4096),
        # a few short conversations of odd lengths in the paper's 4/3-bit format
        _case("decode_6x_ragged_short_mix43", "decode", 6, 32, 8, 128, R_8B, 256, "mix4_3", 97,
              3001, out="f32"),
        # medium contexts at higher key ranks, all 4-bit
        _case("decode_4x32k_int4", "decode", 4, 32, 8, 128, R_8B_HI, 256, "int4", 32768, 32768),
        # the long-context benchmark: 4 x 128K, 8-bit outliers and 4-bit inliers
        _case("decode_4x128k_mix84", "decode", 4, 32, 8, 128, R_8B, 256, "mix8_4", 131072, 131072),
        # the same context in the paper's format, attention concentrated on a few tokens
        _case("decode_4x128k_mix43_peaked", "decode", 4, 32, 8, 128, R_8B, 256, "mix4_3", 131071,
              131071, peaked=True),
        # a 70B layer: eight query heads per KV head, large ranks
        _case("decode_2x64k_gqa8_mix84", "decode", 2, 64, 8, 128, R_70B, 384, "mix8_4", 65536,
              65536),
        # continuous batching: 32 ragged sequences in pages, one token appended to each
        _case("step_32x_ragged_paged_int4", "step", 32, 32, 8, 128, R_8B, 256, "int4", 2048, 16384,
              d_model=4096, page=256),
        # latents kept in fp16 (rank compression only)
        _case("decode_8x4k_f16", "decode", 8, 32, 8, 128, R_8B, 256, "f16", 4096, 4096),
        # the attention block's output with absorbed weights, moderate context
        _case("absorbed_4x8k_mix84", "absorbed", 4, 32, 8, 128, R_8B, 256, "mix8_4", 8192, 8192,
              d_out=4096),
        # prompt processing of a 70B layer: 2 x 4096 tokens from hidden states
        _case("prefill_2x4096_h8192_mix84", "prefill", 2, 64, 8, 128, R_70B, 384, "mix8_4", 4096,
              4096, d_model=8192, n_new=4096),
        # a prompt's latents moved into the cache, odd length
        _case("fill_3x1501_mix43", "fill", 3, 32, 8, 128, R_8B, 256, "mix4_3", 1501, 1501,
              n_new=1501),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges."""
    kind = rng.choice(["decode", "decode", "decode", "step", "step", "absorbed", "prefill", "fill"])
    d = 64 if rng.random() < 0.15 else 128
    n_kv = rng.choice([1, 2, 4, 8, 8, 8])
    G = rng.choice([1, 2, 4, 4, 4, 8])
    ranks = [16 * rng.randint(1, rng.choice([3, d // 16])) for _ in range(n_kv)]
    rv = 16 * rng.randint(max(1, n_kv), max(1, min(n_kv * d, 384) // 16))
    qmode = rng.choice(["f16", "int4", "mix8_4", "mix8_4", "mix4_3"])
    theta = rng.choice([1e4, 5e5, 5e5])
    batch = _log_int(rng, 1, 40)
    width = sum(ranks) + rv
    page = rng.choice([0, 0, 128, 256, 1024])
    kw = dict(theta=theta, q=rng.choice(["f16", "bf16", "bf16"]),
              out=rng.choice(["bf16", "f16", "f32"]), page=page)
    if kind in ("prefill", "fill"):
        if kind == "prefill":
            kw["d_model"] = 8 * _log_int(rng, 32, 1024)
        n_new = _log_int(rng, 2, max(2, 6000 // batch))
        c = _case("", kind, batch, n_kv * G, n_kv, d, ranks, rv, qmode, n_new, n_new, n_new=n_new,
                  **kw)
    else:
        # at most a quarter of the largest listed case's cache contents
        top = max(64, min(131072, (1 << 26) // (batch * width)))
        hi = _log_int(rng, 33, top)
        lo = hi if rng.random() < 0.4 else rng.randint(max(1, hi // 8), hi)
        if kind == "step":
            kw["d_model"] = rng.choice([1024, 2048, 4096, 5120])
        if kind == "absorbed":
            kw["d_out"] = rng.choice([1024, 2048, 4096])
        c = _case("", kind, batch, n_kv * G, n_kv, d, ranks, rv, qmode, lo, hi,
                  peaked=rng.random() < 0.3, **kw)
    del c["name"]
    return c


# ------------------------------------------------------------------------------- inputs

class _Inputs:
    """Everything drawn from the seed.  Latent channel i of a block ~ N(0, 1/i) with 1 % of the
    channels eight times larger, as the singular values order them; factors and queries normal.
    Peaked: queries four times larger and four tokens per sequence with keys eight times larger."""

    def __init__(self, c, seed):
        g = torch.Generator(device="cuda")
        g.manual_seed(1000003 * (seed % 4000037) + 17)
        self.c, self.g = c, g
        self.ranks = [int(r) for r in c["ranks"].split(",")]
        B, d, n_q, n_kv, rv = c["batch"], c["d"], c["n_q"], c["n_kv"], c["rv"]
        self.sum_r, self.width = sum(self.ranks), sum(self.ranks) + rv

        def normal(*shape):
            return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)

        self.normal = normal
        sc = torch.cat([torch.arange(1, r + 1, device="cuda", dtype=torch.float32) ** -0.5
                        for r in self.ranks + [rv]])
        n_out = max(1, self.width // 100)
        idx = torch.randperm(self.width, generator=g, device="cuda")[:n_out]
        sc[idx] *= 8.0
        self.scale = sc
        self.Bk = torch.cat([normal(r, d) / math.sqrt(r) for r in self.ranks]).half()
        self.Bv = (normal(rv, n_kv * d) / math.sqrt(rv)).half()
        q = normal(B, n_q, d)
        self.q = (4.0 * q if c["peaked"] else q).to(TORCH_DT[c["q"]])
        lens = torch.randint(c["lo"], c["hi"] + 1, (B,), generator=g, device="cuda")
        self.ctx = lens.to(torch.int32)
        self.x = self.A = self.W = self.needles = None
        if c["d_model"]:
            self.x = normal(B, c["n_new"], c["d_model"]).bfloat16()
            self.A = (normal(c["d_model"], self.width) * (sc / math.sqrt(c["d_model"]))).bfloat16()
        if c["d_out"]:
            k = n_q * rv
            self.W = (normal(c["d_out"], k) / math.sqrt(k)).half()
        if c["peaked"]:
            self.needles = (torch.rand((B, 4), generator=g, device="cuda", dtype=torch.float64)
                            * lens[:, None]).long()

    def latents(self):
        """(first token, fp16 latents [B][n][width]) chunk by chunk over the contexts."""
        c = self.c
        for t0 in range(0, c["hi"], CHUNK):
            n = min(CHUNK, c["hi"] - t0)
            z = self.normal(c["batch"], n, self.width)
            z *= self.scale
            if self.needles is not None:
                hit = torch.zeros((c["batch"], n), device="cuda", dtype=torch.bool)
                rel = self.needles - t0
                ok = (rel >= 0) & (rel < n)
                b = torch.arange(c["batch"], device="cuda")[:, None].expand_as(rel)
                hit[b[ok], rel[ok]] = True
                z[..., :self.sum_r] *= torch.where(hit, 8.0, 1.0)[..., None]
            yield t0, z.half()


def _bits(t):
    return t.view(torch.int16) if t.dtype in (torch.float16, torch.bfloat16) else t


def prepare(case, seed):
    c = case
    inp = _Inputs(c, seed)
    B, page = c["batch"], c["page"]
    cap = max(c["hi"], c["n_new"])
    kw = {}
    if page:
        kw = dict(page_tokens=page, n_pages=B * -(-cap // page) + 3)
    layer = Layer(B, c["n_q"], c["n_kv"], c["d"], cap, inp.ranks, c["rv"], QMODES[c["qmode"]],
                  c["theta"], DTYPES[c["q"]], DTYPES[c["out"]], d_model=c["d_model"], **kw)
    if page:
        lens = inp.ctx.tolist()
        # pages handed out as sequences grow side by side
        for j in range(0, cap, page):
            for b in range(B):
                if j < max(lens[b], c["n_new"]):
                    layer.pool.ensure(b, min(j + page, cap))
        layer.pool.sync()
    st = {"kind": c["kind"], "layer": layer, "ctx": inp.ctx, "out": TORCH_DT[c["out"]],
          "q": _bits(inp.q), "Bk": _bits(inp.Bk), "Bv": _bits(inp.Bv),
          "pos": torch.zeros(B, dtype=torch.int32, device="cuda")}
    if c["kind"] == "fill":
        st["lat"] = _bits(next(inp.latents())[1])
        return st
    if c["d_model"]:
        st["x"], st["A"] = _bits(inp.x), _bits(inp.A)
        st["shape"] = (B, c["n_new"], inp.width)
    if c["kind"] == "prefill":
        return st
    # the cached context: its latents through a plan that takes them directly
    fill = layer.plan
    if c["d_model"]:
        cfg = S.make_config(B, c["n_q"], c["n_kv"], c["d"], cap, inp.ranks, c["rv"],
                            QMODES[c["qmode"]], c["theta"], q_dtype=DTYPES[c["q"]],
                            out_dtype=DTYPES[c["out"]], page_tokens=page,
                            n_pages=kw.get("n_pages", 0),
                            block_table=layer.pool.table if page else None)
        fill = S.starkv_plan_create(cfg)
    for t0, lat in inp.latents():
        pos = torch.full((B,), t0, dtype=torch.int32, device="cuda")
        ws = torch.empty(max(S.starkv_append_workspace_bytes(fill, lat.shape[1]), 256),
                         dtype=torch.uint8, device="cuda")
        S.starkv_append(fill, layer.cache, _bits(lat), None, pos, lat.shape[1], ws)
    torch.cuda.synchronize()
    if c["kind"] == "step":
        st["pos"] = inp.ctx - 1
    if c["kind"] == "absorbed":
        st["W"] = _bits(inp.W)
        st["y"] = torch.empty((B, c["d_out"]), device="cuda",
                              dtype=torch.float32 if c["out"] == "f32" else torch.int16)
    return st


def run(state):
    st, layer, kind = state, state["layer"], state["kind"]
    if kind == "fill":
        layer.append(st["lat"], st["pos"])
        return layer.cache
    if kind == "prefill":
        layer.append(st["x"], st["pos"], st["A"])
        b, n, w = st["shape"]
        return layer.app_ws[:2 * b * n * w].view(torch.float16).view(b, n, w), layer.cache
    if kind == "step":
        layer.append(st["x"], st["pos"], st["A"])
    if kind == "absorbed":
        y = layer.decode_absorbed(st["q"], st["Bk"], st["W"], st["ctx"], out=st["y"])
        return y.view(st["out"])
    o = layer.decode(st["q"], st["Bk"], st["Bv"], st["ctx"]).view(st["out"])
    return (o, layer.cache) if kind == "step" else o


# ------------------------------------------------------------------------------- work

def _outlier(qmode, r):
    if qmode == "mix8_4":
        return 8 * -(-r // 32)
    if qmode == "mix4_3":
        return min(r, 8 * max(1, (r + 20) // 40))
    return 0


def _regions(qmode, r):
    """(first channel, channels, bits) of the precision regions of a block."""
    ro = _outlier(qmode, r)
    hi, lo = (8 if qmode == "mix8_4" else 4), (3 if qmode == "mix4_3" else 4)
    return [(a, n, b) for a, n, b in ((0, ro, hi), (ro, r - ro, lo)) if n]


def _token_bytes(qmode, r):
    if qmode == "f16":
        return 2 * r
    return sum(n * b / 8 + 4 * -(-n // 32) for _, n, b in _regions(qmode, r))


def work(case):
    c = case
    ranks = [int(r) for r in c["ranks"].split(",")]
    B, d, n_q, rv = c["batch"], c["d"], c["n_q"], c["rv"]
    width = sum(ranks) + rv
    tok = sum(_token_bytes(c["qmode"], r) for r in ranks + [rv])
    es = {"f16": 2, "bf16": 2, "f32": 4}[c["out"]]
    nbytes = flops = 0.0
    if c["kind"] in ("step", "prefill", "fill"):
        m = B * c["n_new"]
        nbytes += m * tok
        if c["d_model"]:
            nbytes += 2 * c["d_model"] * (m + width)
            flops += 2.0 * m * c["d_model"] * width
        else:
            nbytes += 2 * m * width
        if c["kind"] == "prefill":
            nbytes += 2 * m * width
    if c["kind"] in ("decode", "step", "absorbed"):
        tokens = B * (c["lo"] + c["hi"]) / 2
        nbytes += tokens * tok + 2 * B * n_q * d + 2 * sum(ranks) * d
        # keys rebuilt, scores, values weighted
        flops += tokens * (2.0 * sum(ranks) * d + 2.0 * n_q * d + 2.0 * n_q * rv)
        if c["kind"] == "absorbed":
            nbytes += 2 * c["d_out"] * n_q * rv + es * B * c["d_out"]
            flops += 2.0 * B * c["d_out"] * n_q * rv
        else:
            nbytes += 2 * rv * c["n_kv"] * d + es * B * n_q * d
            flops += 2.0 * B * n_q * rv * d
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """About four times the difference from ``exact``: output rounding in 16-bit results (bf16
    1.7e-3, fp16 2.1e-4), fp16 operands of the matrix products in 32-bit ones (2e-4 .. 3.5e-4).
    Cache bytes follow the latents' last bit where fp32 sums are taken in another order (8e-5 of
    the bytes of a prefill against float64 sums, none of a one-token append)."""
    if case["kind"] == "fill":
        return "exact"
    if case["kind"] == "prefill":
        return {"rel": 8e-4, "max": 4e-3, "differ": 4e-4}
    if case["out"] == "bf16":
        return {"rel": 7e-3, "max": 5e-2, "differ": 1e-5}
    return {"rel": 1.4e-3, "max": 2e-2, "differ": 1e-5}


# ------------------------------------------------------------------------------- exact

def _scale_up(v):
    """The smallest float16 at or above v (float64, non-negative), as float64."""
    h = v.to(torch.float16)
    for step in (1, -1):
        up = (h.view(torch.int16) + step).clamp(min=0).view(torch.float16)
        if step == 1:
            h = torch.where(h.double() < v, up, h)
        else:
            h = torch.where((up.double() >= v) & (h.double() > v), up, h)
    return h.double()


def _round_trip(c, ranks, lat):
    """Latents after the cache's quantization, float64 [..., width]."""
    x = lat.double()
    if c["qmode"] == "f16":
        return x
    off = 0
    for r in ranks + [c["rv"]]:
        for a, n, bits in _regions(c["qmode"], r):
            for g in range(a, a + n, 32):
                s = x[..., off + g:off + min(g + 32, a + n)]
                z, top = s.amin(-1, keepdim=True), s.amax(-1, keepdim=True)
                sc = _scale_up((top - z) / (2 ** bits - 1))
                code = ((s - z) / torch.where(sc > 0, sc, 1.0)).round().clamp(0, 2 ** bits - 1)
                s.copy_(z + code * sc)
        off += r
    return x


def exact(case, seed):
    c = case
    if c["kind"] == "fill":
        return None
    inp = _Inputs(c, seed)
    B, d, n_q, n_kv, rv, ranks = c["batch"], c["d"], c["n_q"], c["n_kv"], c["rv"], inp.ranks
    proj = None
    if c["d_model"]:
        proj = inp.x.double().view(-1, c["d_model"]) @ inp.A.double()
        proj = proj.view(B, c["n_new"], inp.width)
        if c["kind"] == "prefill":
            return proj, None
    chunks = [lat for _, lat in inp.latents()]
    lens = inp.ctx.tolist()
    half = d // 2
    om = torch.arange(half, device="cuda", dtype=torch.float64)
    om = torch.exp(-(2.0 * om / d) * math.log(c["theta"]))
    G = n_q // n_kv
    heads = torch.zeros((B, n_q, d), device="cuda", dtype=torch.float64)
    value = torch.zeros((B, n_q, rv), device="cuda", dtype=torch.float64)
    for b in range(B):
        L = lens[b]
        lat = torch.cat([ch[b] for ch in chunks])[:L]
        if c["kind"] == "step":
            lat[L - 1] = proj[b, 0].half()
        x = _round_trip(c, ranks, lat)
        ang = torch.arange(L, device="cuda", dtype=torch.float64)[:, None] * om
        cs, sn = torch.cos(ang), torch.sin(ang)
        off = 0
        for g, r in enumerate(ranks):
            k = x[:, off:off + r] @ inp.Bk[off:off + r].double()
            lo, hi = k[:, :half], k[:, half:]
            k = torch.cat([lo * cs - hi * sn, hi * cs + lo * sn], dim=1)
            p = torch.softmax(inp.q[b, g * G:(g + 1) * G].double() @ k.T / math.sqrt(d), dim=1)
            v = p @ x[:, inp.sum_r:]
            value[b, g * G:(g + 1) * G] = v
            heads[b, g * G:(g + 1) * G] = v @ inp.Bv[:, g * d:(g + 1) * d].double()
            off += r
    if c["kind"] == "absorbed":
        return value.view(B, -1) @ inp.W.double().T
    return (heads, None) if c["kind"] == "step" else heads
