"""Ragged sequences in the many-row GQA kernel when its workgroups outnumber the
slots of the GPU, where sequences are dispatched longest first: ascending,
equal and zero lengths, 2 and 64 sequences, and 65 (the order given), against
the fp64 oracle (max-abs 2e-2, mean-abs 2e-3, relative L2 1e-2)."""
import math

import numpy as np
import pytest
import torch

import oracle
from helpers import Guarded, check_attention_close, host_bits, log
from paper_2606_17107_amd import pkv, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nq,L,d", [(2, 40, 48, 64), (7, 33, 12, 128), (64, 9, 3, 64), (65, 9, 3, 64)])
def test_longest_first(n, nq, L, d):
    H, Hkv = 16, 4
    log("longest first: %d sequences, %d layers, d %d" % (n, L, d))
    kv = [60 + 23 * (i // 2) for i in range(n)]   # ascending, in pairs
    kv[0] = 0
    g = synth.Draws(90 + n, "cuda")
    base = np.concatenate([[0], np.cumsum(kv)]).astype(np.int64)
    q, k, v = g.normal((L, n * nq, H, d)), g.normal((L, Hkv, int(base[-1]), d)), g.normal((L, Hkv, int(base[-1]), d))
    q_pos = np.concatenate([np.arange(max(kv[s], nq) - nq, max(kv[s], nq)) for s in range(n)]).astype(np.int32)
    out = Guarded((L, n * nq, H, d), torch.bfloat16)
    cu = torch.arange(n + 1, dtype=torch.int32, device="cuda") * nq
    pkv.suffix_attention(q, k, v, out.t, torch.from_numpy(q_pos).cuda(), torch.tensor(kv, dtype=torch.int32, device="cuda"),
                         1 / math.sqrt(d), max(kv), n_seqs=n, cu_q=cu, kv_base=torch.from_numpy(base[:n]).cuda(), max_q=nq,
                         n_splits=1)
    torch.cuda.synchronize()
    out.check("attention output")
    got, qh, kh, vh = host_bits(out.t), host_bits(q), host_bits(k), host_bits(v)
    assert np.all(got[:, :nq] == 0)               # the sequence without slots
    for l in (0, L - 1):
        want = [np.zeros((nq, H, d))]
        for s in range(1, n):
            r, c = slice(s * nq, (s + 1) * nq), slice(base[s], base[s + 1])
            want.append(oracle.attention(np.ascontiguousarray(qh[l, r]), np.ascontiguousarray(kh[l][:, c]),
                                         np.ascontiguousarray(vh[l][:, c]), q_pos[r], kv[s], 1 / math.sqrt(d))[0])
        check_attention_close(got[l], np.concatenate(want))
