"""NaN and infinities through every attention kernel and both merges of partials,
against a float64 softmax: a row that sees a NaN score or one of +inf is NaN in
the output and in the log-sum-exp, a NaN in one value channel stays in that
channel, keys whose score is -inf weigh nothing, and the other KV head's rows are
as close as elsewhere (max-abs 2e-2; 1e-5 in fp32).  "few": the library's choice
of splits, for calls of few rows; "many": the same work with splits given, which
runs the many-row kernels."""
import math

import numpy as np
import pytest
import torch

from helpers import log
from paper_2606_17107_amd import pkv, synth

pytestmark = pytest.mark.gpu

ROUTES = {   # variant, query heads, KV heads, head size, queries, cache lengths, splits
    "few, pieces": ("gqa", 8, 2, 128, 1, [3000, 900], 0),
    "few, many pieces": ("gqa", 4, 2, 64, 2, [9000, 40], 0),
    "few, one sequence": ("gqa", 8, 2, 128, 1, [5000], 0),
    "few, whole items": ("gqa", 8, 2, 128, 1, [700], 0),
    "few, MLA": ("mla", 16, 1, 576, 1, [2500, 333], 0),
    "many, one split": ("gqa", 8, 2, 128, 40, [700], 1),
    "many, 3 splits": ("gqa", 8, 2, 64, 40, [700, 500], 3),
    "many, 20 splits": ("gqa", 8, 2, 128, 2, [3000], 20),
    "many, MLA, one split": ("mla", 16, 1, 576, 3, [600], 1),
    "many, MLA, 4 splits": ("mla", 16, 1, 576, 3, [900, 700], 4),
    "fp32, keys": ("f32", 4, 2, 64, 16, [600], 1),
    "fp32, keys, 5 splits": ("f32", 4, 2, 64, 16, [600], 5),
    "fp32, rows": ("f32", 8, 8, 64, 1100, [1200], 1),
    "fp32, rows, 3 splits": ("f32", 8, 8, 64, 1100, [1200], 3),
}
# what is planted: first and last key (of the first sequence, KV head 0), channel, value
PLANTS = {"NaN key": (100, 101, 0, math.nan), "NaN keys": (0, None, 0, math.nan), "+inf score": (100, 101, 0, math.inf),
          "-inf scores": (0, 64, 0, -math.inf), "-inf scores, half": (0, 0.5, 0, -math.inf),
          "NaN value": (100, 101, None, math.nan)}


@pytest.mark.parametrize("plant", PLANTS)
@pytest.mark.parametrize("route", ROUTES)
def test_nonfinite(route, plant):
    variant, H, Hkv, d, nq, kv, splits = ROUTES[route]
    lo, hi, channel, value = PLANTS[plant]
    hi = kv[0] - nq if hi is None else min(int(kv[0] * hi), kv[0] - nq) if isinstance(hi, float) else hi
    mla, dt = variant == "mla", torch.float32 if variant == "f32" else torch.bfloat16
    n, dv, G = len(kv), 512 if mla else d, H // Hkv
    scale = 1 / math.sqrt(192 if mla else d)
    log("non-finite:", route, "/", plant)
    g = synth.Draws(900, "cuda")
    base = np.concatenate([[0], np.cumsum(kv)])
    q, k = g.normal((1, n * nq, H, d), dt), g.normal((1, Hkv, int(base[-1]), d), dt)
    v = k[..., :512] if mla else g.normal((1, Hkv, int(base[-1]), dv), dt)
    if channel is None:
        if mla:
            pytest.skip("MLA values are part of the keys")
        v[0, 0, lo:hi, 5] = value
    else:
        # positive queries in that channel: scores of +-inf, not NaN.  (The MLA channel is a k_pe one, so that the
        # values, which are the first 512 channels, stay finite.)
        channel = 575 if mla else channel
        q[..., channel] = q[..., channel].abs() + 1
        k[0, 0, lo:hi, channel] = value
    out = torch.zeros(1, n * nq, H, dv, dtype=dt, device="cuda")
    lse = torch.zeros(1, n * nq, H, device="cuda")
    q_pos = np.concatenate([np.arange(m - nq, m) for m in kv])
    pkv.suffix_attention(q, k, v, out, torch.tensor(q_pos, dtype=torch.int32, device="cuda"),
                         torch.tensor(kv, dtype=torch.int32, device="cuda"), scale, max(kv), n_seqs=n,
                         cu_q=torch.arange(n + 1, dtype=torch.int32, device="cuda") * nq,
                         kv_base=torch.from_numpy(base[:n]).cuda(), max_q=nq, n_splits=splits, lse_out=lse,
                         variant=pkv.PKV_ATTN_MLA if mla else pkv.PKV_ATTN_GQA)
    torch.cuda.synchronize()
    f64 = lambda t: t.double().cpu().numpy()
    got, got_lse, q, k, v = f64(out)[0], f64(lse)[0], f64(q)[0], f64(k)[0], f64(v)[0]
    want, want_lse = np.zeros_like(got), np.zeros_like(got_lse)
    with np.errstate(invalid="ignore"):
        for s in range(n):
            rows, keys = slice(s * nq, (s + 1) * nq), slice(base[s], base[s + 1])
            hidden = np.arange(kv[s])[None, :] > q_pos[rows][:, None]
            for h in range(H):
                sc = (q[rows, h] @ k[h // G, keys].T) * scale
                sc[hidden] = -np.inf
                top = sc.max(1, keepdims=True)
                p = np.exp(sc - top)
                total = p.sum(1, keepdims=True)
                want_lse[rows, h] = (top + np.log(total))[:, 0]
                want[rows, h] = (p / total) @ v[h // G, keys]
    bad = np.isnan(want)
    assert bad.any() == (not plant.startswith("-inf"))
    np.testing.assert_array_equal(np.isnan(got), bad)
    np.testing.assert_array_equal(np.isnan(got_lse), np.isnan(want_lse))
    tol = 1e-5 if variant == "f32" else 2e-2
    assert np.abs(got - want)[~bad].max(initial=0) <= tol
    np.testing.assert_allclose(got_lse, want_lse, atol=max(tol, 1e-4))   # NaN where NaN
