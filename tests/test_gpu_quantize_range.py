"""The quantizer near the ends of the fp32 range: a step below 1e-36 or above 1e36 takes a division
instead of the corrected reciprocal.  A power of two scales every step and offset exactly, so the codes
are those of the unscaled tile and the aux are its scaled ones."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [2, 4])
@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("exponent", [-119, 118, -60])
def test_quantize_scaled_tiles(bits, kind, exponent):
    from paper_2606_03458_amd import kvarn as K
    p = K.kvarn_params_init(bits, varn_iters=0)  # (the variances' clamp is not scale-free)
    x = torch.randn((3, 128, 128), generator=torch.Generator().manual_seed(bits + kind))
    # multiples of 2^-4: the rotated sums are exact at every scale, and no value is subnormal
    x = (torch.round(x * 16) / 16).cuda()
    got = []
    for t in (x, torch.ldexp(x, torch.tensor(float(exponent), device="cuda"))):
        out = torch.zeros((3, K.kvarn_tile_bytes(p)), dtype=torch.uint8, device="cuda")
        K.kvarn_quantize_block(p, kind, t.contiguous(), K.KVARN_F32, 3, 1, 128 * 128, 0, 128, out, 1, 1)
        got.append((out[:, :bits * 2048], out[:, bits * 2048:].view(torch.float32).clone()))
    (codes, aux), (scaled_codes, scaled_aux) = got
    assert torch.isfinite(scaled_aux).all()
    # the reciprocal is within an ulp of the division: a code may differ only at a tie
    assert (codes != scaled_codes).float().mean() <= 1e-4
    a, b = scaled_aux[:, :256].double(), torch.ldexp(aux[:, :256].double(), torch.tensor(float(exponent), device="cuda"))
    assert ((a - b).abs() <= 2.0**-23 * b.abs() + 2.0**-149).all()
    assert torch.equal(scaled_aux[:, 256:], aux[:, 256:])
