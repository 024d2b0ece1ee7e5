"""Batched splice at the edges of its partition (a block copies a run of three
token tiles, 16 tokens each at 8 + 8 lanes a token; above 88 runs, and for other
tiles above 1024 tokens or 64 tiles, 32 blocks loop over a segment): segment
lengths around one tile, one run and the longest of either form, a bound far above
the longest segment or below it, row counts that do and do not divide over the
XCDs, more blocks than a launch dimension holds, against the fp64 oracle (values
bit-exact, keys within one bf16 ulp)."""
import numpy as np
import pytest
import torch

import oracle
from helpers import check_rotated_keys, dev, host_bits, log
from paper_2606_17107_amd import pkv, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,H,lens,bound", [
    (2, 4, [1, 15, 16, 17, 47, 48, 49, 96, 97], None),    # 8 rows: 1-D grid
    (1, 3, [1, 48, 49, 0, 200], None),                    # 3 rows: 3-D grid
    (2, 4, [48 * 128, 48 * 128 + 1, 5], None),            # looping blocks, several rounds
    (2, 4, [48 * 128, 5], None),
    (2, 4, [48 * 88, 5], None),                           # 88 runs, one per block
    (2, 4, [48 * 88 + 1, 5], None),                       # one token more: looping blocks
    (1, 1, [100, 33], 1 << 20),                           # a loose bound
    (2, 4, [100, 33, 5000, 49], 20),                      # segments beyond the bound are copied whole
    (1, 3, [3000, 1, 97], 48),
])
def test_run_edges(L, H, lens, bound):
    splice_and_check(L, H, 128, lens, bound)


@pytest.mark.parametrize("d,lens", [
    (64, [1024, 5, 33]), (64, [1025, 5, 33]),      # 32 tokens a tile: by the 1024 tokens
    (256, [512, 5, 9]), (256, [513, 5, 9]),        # 8 tokens a tile: by the 64 tiles
])
@pytest.mark.parametrize("L,H", [(2, 4), (1, 3)])
def test_form_edges(L, H, d, lens):
    splice_and_check(L, H, d, lens, None)


def splice_and_check(L, H, d, lens, bound):
    theta = 5e5
    log("segments:", L, H, d, lens, bound)
    g = synth.Draws(7 + len(lens) + H, "cpu")
    S, gap = sum(lens), 7
    src_k, src_v = host_bits(g.normal((L, H, S, d))), host_bits(g.normal((L, H, S, d)))
    cap = S + gap * (len(lens) + 1)
    dst_k, dst_v = host_bits(g.normal((L, H, cap, d))), host_bits(g.normal((L, H, cap, d)))
    segs, slot, at = [], 0, gap
    for i, n in enumerate(lens):
        segs.append(dict(src_slot0=slot, dst_seq_base=0, n_tokens=n, src_pos0=1000 * i, dst_pos0=at, dst_seq_len=cap))
        slot, at = slot + n, at + n + gap
    gk, gv, err = dev(dst_k), dev(dst_v), torch.zeros(1, dtype=torch.int32, device="cuda")
    pkv.reposition_splice_batched(dev(src_k), dev(src_v), gk, gv, pkv.make_segments(segs, "cuda"), len(segs),
                                  bound or max(lens), theta, d, err_flag=err)
    torch.cuda.synchronize()
    assert int(err.item()) == 0
    for sg in segs:
        n, s = sg["n_tokens"], slice(sg["src_slot0"], sg["src_slot0"] + sg["n_tokens"])
        if n:
            oracle.reposition_splice(np.ascontiguousarray(src_k[:, :, s]), np.ascontiguousarray(src_v[:, :, s]), dst_k,
                                     dst_v, np.arange(sg["src_pos0"], sg["src_pos0"] + n, dtype=np.int32),
                                     np.arange(sg["dst_pos0"], sg["dst_pos0"] + n, dtype=np.int32), theta, d)
    np.testing.assert_array_equal(host_bits(gv), dst_v)   # every slot no segment owns included
    check_rotated_keys(host_bits(gk), dst_k, 0, d, synth.HALF)


@pytest.mark.parametrize("n,L,H,d,bound", [
    (2979, 8, 8, 256, 88 * 48),     # one token each under a loose bound: in runs, 16.8e6 blocks
    (65535, 4, 4, 16, 1 << 20),     # the most segments: the looping blocks exceed it as well
])
def test_blocks_above_a_launch_dimension(n, L, H, d, bound):
    """A launch dimension holds 2^32 - 1 threads, 2^24 - 1 blocks of 256."""
    theta = 1e4
    log("segments:", n, L, H, bound)
    g = synth.Draws(11, "cpu")
    src_k, dst_k = host_bits(g.normal((L, H, n, d))), host_bits(g.normal((L, H, n + 5, d)))
    src_pos, dst_pos = np.arange(n, dtype=np.int32) % 1000, np.random.default_rng(5).permutation(n).astype(np.int32)
    segs = [dict(src_slot0=i, dst_seq_base=0, n_tokens=1, src_pos0=int(src_pos[i]), dst_pos0=int(dst_pos[i]),
                 dst_seq_len=n + 5) for i in range(n)]
    gk, err = dev(dst_k), torch.zeros(1, dtype=torch.int32, device="cuda")
    pkv.reposition_splice_batched(dev(src_k), None, gk, None, pkv.make_segments(segs, "cuda"), n, bound, theta, d,
                                  err_flag=err)
    torch.cuda.synchronize()
    assert int(err.item()) == 0
    oracle.reposition_splice(src_k, None, dst_k, None, src_pos, dst_pos, theta, d)
    check_rotated_keys(host_bits(gk), dst_k, 0, d, synth.HALF)
