"""The quantizer near the ends of the fp32 range: a step below 1e-36 or above 1e36 takes a division
instead of the reciprocal estimate with one Newton step.  A power of two scales every step and offset exactly (but for
subnormal ones, by half the smallest), so the codes are those of the unscaled tile and the aux are its
scaled ones.  The two ends are chosen so that every step lies past its line, and at the low one is
subnormal, where the hardware's reciprocal estimate is of no use though 1 / step is finite."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [2, 4])
@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("end", ["high", "near high", "middle", "near low", "low"])
def test_quantize_scaled_tiles(bits, kind, end):
    from paper_2606_03458_amd import kvarn as K
    exponent = {"high": 122, "near high": 118, "middle": -60, "near low": -119, "low": -128 if bits == 2 else -126}[end]
    p = K.kvarn_params_init(bits, varn_iters=0)  # (the variances' clamp is not scale-free)
    x = torch.randn((3, 128, 128), generator=torch.Generator().manual_seed(bits + kind))
    # multiples of 2^-12: the rotated sums are exact at every scale (at the low end multiples of 2^-140), and
    # quotients that lie on a tie are rare
    x = (torch.round(x * 4096) / 4096).cuda()
    if end == "low" and bits == 4:
        x = 1.25 * x  # (exact; every step then lies in the two octaves asserted below)
    got = []
    for t in (x, x * 2.0**exponent):
        out = torch.zeros((3, K.kvarn_tile_bytes(p)), dtype=torch.uint8, device="cuda")
        K.kvarn_quantize_block(p, kind, t.contiguous(), K.KVARN_F32, 3, 1, 128 * 128, 0, 128, out, 1, 1)
        got.append((out[:, :bits * 2048], out[:, bits * 2048:].view(torch.float32).clone()))
    (codes, aux), (scaled_codes, scaled_aux) = got
    assert torch.isfinite(scaled_aux).all()
    step = aux[:, :128].double() * 2.0**exponent
    assert {"high": step.min() > 1.01e36, "near high": step.max() < 1e36, "near low": step.min() > 2.0**-126,
            "low": step.max() < 2.0**-126 and step.min() > 2.0**-128, "middle": True}[end]
    # A quotient is off by 15 x 2^-24 for a rounded reciprocal, and at the low end by the rounding of a subnormal value,
    # 2^-150 / 2^-128: within 2^-18 of a tie, which a share of 2^-17 of the codes and 2^-15 of the bytes is.
    assert (codes != scaled_codes).float().mean() <= 1e-4
    b = aux[:, :256].double() * 2.0**exponent
    # (a range of two rounded subnormal values, divided and rounded)
    assert ((scaled_aux[:, :256].double() - b).abs() <= 2.0**-23 * b.abs() + 2.0**-148).all()
    assert torch.equal(scaled_aux[:, 256:], aux[:, 256:])
