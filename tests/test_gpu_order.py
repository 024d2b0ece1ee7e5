"""Dispatch order of the many-row attention kernels.  Ragged sequences in the GQA kernel when its workgroups outnumber the
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


@pytest.mark.parametrize("n,nq,L,d", [(2, 40, 48, 64), (7, 33, 12, 128), (64, 9, 3, 64)])
def test_longest_first_long_caches(n, nq, L, d):
    """Caches long enough for the order to pay (2048 keys and more), in no order: equal lengths, lengths above the
    stated bound (cut to it) and a negative one, contiguous and paged, against the oracle on the first and last
    layer.  The order is by 1/64 of the bound, so equal classes occur as well."""
    H, Hkv, bound, page = 16, 4, 2100, 64
    kv = [min(bound + 5, 30 + (i * 977) % 2200) for i in range(n)]
    kv[n // 2] = kv[0]
    kv[1] = -3 if n > 2 else kv[1]
    own = [min(max(m, 0), bound) for m in kv]
    log("longest first, long caches: %d sequences, %d layers, d %d" % (n, L, d))
    g = synth.Draws(190 + n, "cuda")
    base = np.concatenate([[0], np.cumsum([-(-m // page) * page + page for m in own])]).astype(np.int64)
    q, k, v = g.normal((L, n * nq, H, d)), g.normal((L, Hkv, int(base[-1]), d)), g.normal((L, Hkv, int(base[-1]), d))
    q_pos = np.concatenate([np.arange(max(m, nq) - nq, max(m, nq)) for m in own]).astype(np.int32)
    i32 = lambda a: torch.tensor(a, dtype=torch.int32, device="cuda")
    args = dict(n_seqs=n, cu_q=i32([nq * i for i in range(n + 1)]), max_q=nq, n_splits=1)
    out, out_p = Guarded((L, n * nq, H, d), torch.bfloat16), Guarded((L, n * nq, H, d), torch.bfloat16)
    pkv.suffix_attention(q, k, v, out.t, i32(q_pos.tolist()), i32(kv), 1 / math.sqrt(d), bound,
                         kv_base=torch.from_numpy(base[:n]).cuda(), **args)
    # the same cache as pages: [layer][page][slot][head][channel]
    pool = lambda t: t.view(L, Hkv, -1, page, d).permute(0, 2, 3, 1, 4).contiguous()
    per = -(-bound // page)
    table = i32([[min(base[s] // page + e, base[-1] // page - 1) for e in range(per)] for s in range(n)])
    pkv.suffix_attention_paged(q, pool(k), pool(v), out_p.t, i32(q_pos.tolist()), i32(kv), table, 1 / math.sqrt(d), bound,
                               **args)
    torch.cuda.synchronize()
    out.check("attention output")
    out_p.check("paged attention output")
    assert torch.equal(out.t, out_p.t)
    got, qh, kh, vh = host_bits(out.t), host_bits(q), host_bits(k), host_bits(v)
    for l in (0, L - 1):
        want = []
        for s in range(n):
            r, c = slice(s * nq, (s + 1) * nq), slice(base[s], base[s] + own[s])
            want.append(oracle.attention(np.ascontiguousarray(qh[l, r]), np.ascontiguousarray(kh[l][:, c]),
                                         np.ascontiguousarray(vh[l][:, c]), q_pos[r], own[s], 1 / math.sqrt(d))[0]
                        if own[s] else np.zeros((nq, H, d)))
        # one bf16 ulp of outputs of size 4 (few visible keys) is 2^-6
        check_attention_close(got[l], np.concatenate(want), max_abs=2e-2 if np.abs(want).max() < 2.5 else 2 ** -5)


@pytest.mark.parametrize("variant,H,Hkv,d,nq,splits", [
    ("gqa", 8, 1, 64, 150, 1),      # 1 group, 10 row blocks: shared by 8 XCDs
    ("gqa", 8, 2, 128, 97, 3),      # 6 groups, 4 row blocks
    ("gqa", 12, 3, 128, 33, 1),     # 3 groups, 2 row blocks: more XCDs than row blocks
    ("gqa", 20, 5, 64, 300, 1),     # 5 groups, 10 row blocks
    ("mla", 16, 1, 576, 70, 3),     # 3 groups, 9 row blocks
    ("f32", 6, 3, 64, 130, 1),      # 3 groups, 5 row blocks of 64
])
def test_row_blocks_shared_by_xcds(variant, H, Hkv, d, nq, splits):
    """Group counts that do not divide over the XCDs: every row block is dealt to exactly one workgroup."""
    log("shared groups:", variant, H, Hkv, nq, splits)
    mla, dt = variant == "mla", torch.float32 if variant == "f32" else torch.bfloat16
    kv, dv = 700, 512 if mla else d
    scale = 1 / math.sqrt(192 if mla else d)
    g = synth.Draws(300 + H + nq, "cuda")
    q, k = g.normal((1, nq, H, d), dt), g.normal((1, Hkv, kv, d), dt)
    v = k[..., :512] if mla else g.normal((1, Hkv, kv, d), dt)
    out = Guarded((1, nq, H, dv), dt)
    q_pos = np.arange(kv - nq, kv, dtype=np.int32)
    pkv.suffix_attention(q, k, v, out.t, torch.from_numpy(q_pos).cuda(), torch.tensor([kv], dtype=torch.int32, device="cuda"),
                         scale, kv, n_splits=splits, variant=pkv.PKV_ATTN_MLA if mla else pkv.PKV_ATTN_GQA)
    torch.cuda.synchronize()
    out.check("attention output")
    got = host_bits(out.t)
    want, _ = oracle.attention(host_bits(q)[0], host_bits(k)[0], host_bits(v.contiguous())[0], q_pos, kv, scale)
    check_attention_close(got[0], want)
