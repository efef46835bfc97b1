"""Decode attention at the edges of the launch plan: every rule of workgroups per stream and waves
per workgroup, with units (body tiles, 32-token chunks) that do not divide by the waves, fewer units
than waves, and ragged lengths down to empty, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import check_output, host_cache, q_to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,n_q,n_kv,bits,aux,n_sink,tiles", [
    (1, 4, 1, 2, 0, 0, 0),       # residual only: 4 waves of one chunk each
    (2, 8, 2, 2, 0, 0, 1),       # 5 units, 5 waves
    (2, 10, 2, 4, 1, 40, 9),     # 15 units, 8 waves, the extra-head kernel
    (4, 32, 8, 2, 0, 0, 13),     # 17 units, the CU's 12 waves
    (4, 64, 8, 2, 1, 0, 13),     # 17 units, the CU's 8 waves (two head groups)
    (4, 32, 8, 2, 0, 0, 33),     # 10 workgroups of 4 waves, merged by four waves per head
    (1, 32, 8, 2, 1, 128, 65),   # 19 workgroups
    (16, 64, 8, 4, 0, 0, 61),    # 4 workgroups, merged by one wave per head
    (129, 8, 2, 2, 0, 0, 5),     # 258 streams: 4 waves
    (129, 8, 2, 2, 1, 0, 96),    # 258 long streams: 4 waves
    (180, 8, 2, 2, 1, 0, 70),    # 360 long streams: 12 waves
    (140, 16, 2, 2, 0, 0, 97),   # 280 long streams of two head groups: 8 waves
    (100, 12, 3, 2, 0, 0, 65),   # 300 long streams, the longest sequences first (a batch above a wave)
    (33, 80, 8, 2, 0, 20, 34),   # 528 streams (two head chunks): 4 waves, the longest first
    (400, 8, 2, 2, 0, 7, 3),     # 800 streams: 2 waves
    (400, 8, 2, 2, 0, 0, 33),    # 800 longer streams: 4 waves, too many sequences to rank
    (100, 32, 8, 2, 1, 0, 33),   # 800 of fewer sequences, the longest first
    (300, 8, 2, 2, 0, 0, 65),    # 600 long streams of more sequences than a wave ranks
    (22, 64, 8, 2, 0, 0, 72),    # 176 streams that may be ragged: 4 workgroups
    (576, 8, 2, 4, 0, 0, 16),    # 1152 streams at 4 bits: 4 waves
    (800, 8, 2, 2, 0, 3, 16),    # 1600 streams: 4 waves
    (1600, 4, 2, 2, 1, 0, 2),    # 3200 streams: 1 wave
])
def test_decode_plan_edges(batch, n_q, n_kv, bits, aux, n_sink, tiles):
    from paper_2606_03458_amd import kvarn as K
    from paper_2606_03458_amd import workloads
    built, _ = workloads.build("llama", bits=bits, n_q=n_q, n_kv=n_kv, batch=batch, aux=aux, n_sink=n_sink,
                               context=n_sink + tiles * 128 + 77)
    L = built.length
    cycle = [L, L - 77, n_sink + 1, L - 45, n_sink // 2, 0, n_sink + tiles // 2 * 128 + 32]
    lens = [max(0, cycle[i % len(cycle)]) for i in range(batch)]
    built.cache.seq_len.copy_(torch.tensor(lens, dtype=torch.int32))
    q = workloads.decode_queries(built, seed=31)
    out = torch.full(q.shape, float("nan"), dtype=torch.float32, device="cuda")
    n = K.kvarn_decode_workspace_bytes(built.params, built.cache, n_q, L)
    ws = torch.full((max(n // 4, 4),), float("nan"), device="cuda")
    K.kvarn_decode_attention(built.params, built.cache, n_q, q, K.KVARN_BF16, out, K.KVARN_F32, 128**-0.5, L, ws, n)
    torch.cuda.synchronize()
    check_output(out.cpu().numpy(), oracle.decode(host_cache(built.cache), q_to_host(q), np.float64(128**-0.5)),
                 bf16_out=False)
