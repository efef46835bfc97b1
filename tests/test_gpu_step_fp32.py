"""kvarn_append_decode with fp32 tokens on a dense body: the append inside the decode launch rounds the
token and puts it in place of the residual's last row.  Bit-equal, in output and cache, to the two calls
for each decode kernel, where the token is the first row of a chunk, the last, or inside; and with
head chunks (two waves read the token, one stores it)."""
import pytest
import torch

from test_gpu_step import SCALE, _clone

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits,aux,n_q,n_kv,batch,n_sink,context", [
    (2, 0, 4, 1, 1, 0, 0),            # an empty cache
    (2, 1, 32, 8, 2, 0, 128 + 30),    # rows 30, 31 and 0 of the next chunk
    (2, 0, 10, 2, 3, 7, 7 + 62),      # the extra-head kernel
    (4, 0, 12, 2, 3, 0, 3 * 128 + 95),
    (4, 1, 32, 2, 2, 0, 128 + 63),    # two head chunks of eight
    (2, 0, 18, 2, 150, 0, 17 * 128),  # two head chunks of five and four, 600 waves' worth of streams
])
def test_fp32_step_equals_two_calls(bits, aux, n_q, n_kv, batch, n_sink, context):
    from paper_2606_03458_amd import kvarn as K
    from paper_2606_03458_amd import workloads
    built, _ = workloads.build("llama", bits=bits, aux=aux, n_q=n_q, n_kv=n_kv, batch=batch, n_sink=n_sink,
                               context=context, extra_blocks=1)
    p, a = built.params, built.cache
    a.k_resid.fill_(float("nan")) if context % 128 == n_sink % 128 else None  # rows that were never written
    b = _clone(K, p, a)
    gen = torch.Generator(device="cuda").manual_seed(bits + n_q)
    L = built.length
    n = max(K.kvarn_decode_workspace_bytes(p, a, n_q, L + s + 1) for s in range(4))
    ws = torch.empty(max(n, 16), dtype=torch.uint8, device="cuda")
    for s in range(4):
        kt = 2 * torch.randn(batch, n_kv, 128, generator=gen, device="cuda")
        vt = torch.randn(batch, n_kv, 128, generator=gen, device="cuda")
        q = torch.randn(batch, n_q, 128, generator=gen, device="cuda")
        got, ref = torch.full_like(q, float("nan")), torch.full_like(q, float("nan"))
        K.kvarn_append_decode(p, a, kt, vt, K.KVARN_F32, L + s, n_q, q, K.KVARN_F32, got, K.KVARN_F32, SCALE, ws, n)
        K.kvarn_append_token(p, b, kt, vt, K.KVARN_F32, L + s)
        K.kvarn_decode_attention(p, b, n_q, q, K.KVARN_F32, ref, K.KVARN_F32, SCALE, L + s + 1, ws, n)
        torch.cuda.synchronize()
        assert bool(torch.isfinite(ref).all()) and torch.equal(got, ref), s
        for f in ("k_resid", "v_resid"):  # (bits: unwritten rows may hold NaN)
            assert torch.equal(getattr(a, f).view(torch.int16), getattr(b, f).view(torch.int16)), (s, f)
        assert torch.equal(a.seq_len, b.seq_len) and int(a.err_word.item()) == 0
