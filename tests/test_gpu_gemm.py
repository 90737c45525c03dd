"""The prefill down-projection where its tile choice and its copy pipeline turn: 256 x 128,
256 x 144 and 256 x 192 tiles, one, two, three and more k steps, ragged row and column tiles, fewer columns
than a tile.  Latents against a float64 product."""
import pytest

from paper_2606_08382_amd import starkv as S

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CASES = [
    # rows, key ranks, value rank, d_model
    (24600, [16], 16, 64),                          # tiles of 128, 32 of them used, one k step
    (12301, [48, 32], 192, 128),                    # two tiles of 128 columns, 16 of a third
    (8192, [80, 32, 128, 128, 48, 112, 64, 96], 384, 192),   # 256 tiles of 144 columns
    (10000, [80, 32, 128, 128, 48, 112, 64, 96], 384, 64),   # 240 tiles of 192 columns, one k step
    (10001, [80, 32, 128, 128, 48, 112, 64, 96], 384, 320),
]


@pytest.mark.parametrize("m,ranks,rv,d_model", CASES)
def test_prefill_tiles(m, ranks, rv, d_model):
    from paper_2606_08382_amd.device import Layer
    print(f"prefill tiles {m} x {sum(ranks) + rv} x {d_model}", flush=True)
    width = sum(ranks) + rv
    g = torch.Generator(device="cuda").manual_seed(5)
    x = torch.randn((1, m, d_model), generator=g, device="cuda").bfloat16()
    A = (torch.randn((d_model, width), generator=g, device="cuda") / d_model ** 0.5).bfloat16()
    layer = Layer(1, 8 * len(ranks), len(ranks), 128, m, ranks, rv, S.Q_MIX8_4, 5e5, S.DT_BF16,
                  S.DT_BF16, d_model=d_model)
    pos = torch.zeros(1, dtype=torch.int32, device="cuda")
    layer.append(x.view(torch.int16), pos, A.view(torch.int16))
    torch.cuda.synchronize()
    got = layer.app_ws[:2 * m * width].view(torch.float16).view(m, width).double()
    ref = x[0].double() @ A.double()
    # fp32 sums of d_model products (|error| <= d_model 2^-24 sum |x A|), one fp16 rounding
    bound = d_model * 2.0 ** -24 * (x[0].double().abs() @ A.double().abs())
    half_ulp = torch.clamp(ref.abs() * 2.0 ** -11, min=2.0 ** -25)
    assert bool(((got - ref).abs() <= bound + half_ulp * (1 + 2.0 ** -10)).all())
