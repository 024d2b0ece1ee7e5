"""fp32 attention at the edges of its two kernels (up to one workgroup of 32
rows per CU the four waves split the keys; above that they split the rows),
against the fp64 oracle at fp32 tolerance (relative L2 1e-5, max-abs 1e-5 as
in the other fp32 tests)."""
import math

import numpy as np
import pytest
import torch

import oracle
from helpers import Guarded, host_bits, log
from paper_2606_17107_amd import pkv, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,Hkv,d,nq,kv,splits,window", [
    (4, 2, 64, 1, 1, 1, 0),          # one key
    (4, 2, 64, 16, 31, 1, 0),        # less than a tile
    (4, 2, 64, 16, 129, 1, 0),       # one key in the first wave's second tile
    (8, 2, 128, 8, 100, 1, 0),       # 32 rows exactly, three tiles for four waves
    (8, 2, 128, 9, 300, 2, 0),       # 36 rows: a second row block of four rows
    (6, 2, 64, 11, 500, 5, 70),      # 33 rows, groups of 3, a window
    (8, 8, 64, 1024, 1100, 1, 0),    # 256 workgroups of 32 rows: the last that split the keys
    (8, 8, 64, 1025, 1100, 1, 0),    # the first that split the rows
])
def test_f32_keys(H, Hkv, d, nq, kv, splits, window):
    log("fp32 keys:", H, Hkv, d, nq, kv, splits, window)
    g = synth.Draws(500 + nq + kv, "cuda")
    f = torch.float32
    q, k, v = g.normal((1, nq, H, d), f), g.normal((1, Hkv, kv, d), f), g.normal((1, Hkv, kv, d), f)
    out, lse = Guarded((1, nq, H, d), f), torch.zeros(1, nq, H, device="cuda")
    q_pos = np.arange(kv - nq, kv, dtype=np.int32)       # negative positions see nothing
    pkv.suffix_attention(q, k, v, out.t, torch.from_numpy(q_pos).cuda(), torch.tensor([kv], dtype=torch.int32, device="cuda"),
                         1 / math.sqrt(d), kv, n_splits=splits, window=window, lse_out=lse)
    torch.cuda.synchronize()
    out.check("fp32 attention output")
    rows = np.unique(np.linspace(0, nq - 1, 60).astype(int))
    got = out.t.cpu().numpy()[0][rows]
    want, want_lse = oracle.attention(np.ascontiguousarray(q.cpu().numpy()[0][rows]), k.cpu().numpy()[0], v.cpu().numpy()[0],
                                      q_pos[rows], kv, 1 / math.sqrt(d), window=window)
    assert np.linalg.norm(got - want) / np.linalg.norm(want) <= 1e-5
    assert np.abs(got - want).max() <= 1e-5
    np.testing.assert_allclose(lse.cpu().numpy()[0][rows], want_lse, rtol=1e-5, atol=1e-5)
