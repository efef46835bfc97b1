"""Packed tiles byte for byte.  A cache holds tiles for as long as its sequences live, so the same
tokens must give the same bytes from one build of the library to the next: the sums of the statistics
keep their order (a different one moves the last bit of a scale, and an 8-bit scale that lies on a tie
with it).  tests/golden/quantized_tiles.txt holds the SHA-256 of the tiles and kept iterations for fixed
inputs, each line for one data set, kind, bit width and aux format, over fp32 and bf16 input with and
without the rotation."""
import hashlib
import os

import numpy as np
import pytest
import torch

GOLDEN = os.path.join(os.path.dirname(__file__), "golden", "quantized_tiles.txt")
N = 24  # tiles


def _hash(n, salt):
    """n 64-bit values by splitmix64 (integer arithmetic: the same on every machine)."""
    with np.errstate(over="ignore"):
        z = np.arange(1, n + 1, dtype=np.uint64) * np.uint64(0x9E3779B97F4A7C15) + np.uint64(salt)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
    return z ^ (z >> np.uint64(31))


def _bell(n, salt):
    """Roughly normal values, exact multiples of 2^-15: sums of four 16-bit pieces."""
    h = _hash(n, salt)
    return sum(((h >> np.uint64(16 * i)) & np.uint64(0xFFFF)).astype(np.float64) for i in range(4)) / 32768.0 - 4.0


def _data(name):
    x = _bell(N * 128 * 128, 1).reshape(N, 128, 128)
    channel = 1 + (_hash(N * 128, 2) % np.uint64(64)).astype(np.float64).reshape(N, 1, 128) / 8
    token = 1 + (_hash(N * 128, 3) % np.uint64(64)).astype(np.float64).reshape(N, 128, 1) / 16
    if name == "spread":
        x = x * channel * token
    elif name == "zeros":  # zeros of both signs with a few values among them, and constant tiles
        x = x * channel * (_hash(x.size, 4) % np.uint64(50) == 0).reshape(x.shape)
        x[N // 2:] = np.linspace(-2.0, 2.0, N // 2).reshape(-1, 1, 1)
    elif name == "huge":  # group ranges beyond the largest fp32 number
        x = x * (3.3e38 / 4)
    elif name == "tiny":  # down to subnormal values and steps
        x = x * channel * 2.0 ** -(100 + 2 * np.arange(N)).reshape(N, 1, 1)
    elif name == "infinite":  # one to four infinities in a token, of one sign or both
        x = x * channel * token
        for t in range(N):
            for k in range(1 + t % 4):
                x[t, 5 * t, (37 * k + 11 * t) % 128] = -np.inf if (t // 4 >> k) & 1 else np.inf
    elif name in ("nan", "nan rows"):  # a NaN, infinities of both signs, and a token of many, in 8 tiles each
        x = x * channel * token
        i = np.arange(N)
        x[i[0::3], 5 * i[0::3], 3 * i[0::3] + 1] = np.nan
        x[i[1::3], 4 * i[1::3], 2] = np.inf
        x[i[1::3], 127 - i[1::3], 100] = -np.inf
        many = (_hash(N * 128, 6) % np.uint64(6)).reshape(N, 128)
        for t in i[2::3]:
            x[t, 3 * t] = np.select([many[t] == 0, many[t] == 1, many[t] == 2], [np.inf, -np.inf, np.nan], x[t, 3 * t])
            if name == "nan rows":
                x[t, 3 * t, 40:64] = np.nan
    else:
        raise ValueError(name)
    return x.astype(np.float32)


def digest(K, name, kind, bits, aux):
    h = hashlib.sha256()
    x32 = torch.from_numpy(_data(name)).cuda()
    for x in (x32, x32.to(torch.bfloat16)):
        for rotate in (0,) if name == "huge" else (1, 0):  # (rotated, the huge tokens overflow themselves)
            p = K.kvarn_params_init(bits, aux_format=aux, rotate=rotate, varn_iters=0 if name == "nan rows" else 8)
            out = torch.zeros((N, K.kvarn_tile_bytes(p)), dtype=torch.uint8, device="cuda")
            best = torch.zeros(N, dtype=torch.int32, device="cuda")
            K.kvarn_quantize_block(p, kind, x, K._dtype(x), N, 1, 128 * 128, 0, 128, out, 1, 1, best)
            if name in ("nan", "nan rows", "infinite") and aux == 0:  # (the sign of a NaN is not a value)
                scales = out[:, bits * 2048:].view(torch.float32)
                scales[scales.isnan()] = float("nan")
            h.update(out.cpu().numpy().tobytes())
            h.update(best.cpu().numpy().tobytes())
    return h.hexdigest()


def _golden():
    with open(GOLDEN) as fh:
        rows = [line.rsplit(maxsplit=4) for line in fh if line.strip() and not line.startswith("#")]
    return [(name, int(kind), int(bits), int(aux), want) for name, kind, bits, aux, want in rows]


@pytest.mark.gpu
@pytest.mark.parametrize("name,kind,bits,aux,want", _golden())
def test_tiles_keep_their_bytes(name, kind, bits, aux, want):
    from paper_2606_03458_amd import kvarn as K
    assert digest(K, name, kind, bits, aux) == want
