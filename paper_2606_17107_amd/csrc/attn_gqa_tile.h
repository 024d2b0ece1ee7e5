// LDS layout of the 32-key bf16 K and V tiles of the GQA attention kernels: the
// chunk swizzles and the MFMA operand reads.
#pragma once

#include "attn_common.h"

namespace pkv {

// XOR swizzles of a row's 16-byte chunk index by its key.  LDS has 64 banks
// of 4 bytes (256 bytes per cycle); the rows one read touches must spread
// over the 16 bank groups of 16 bytes.
//   D = 128 (16 chunks per row, every row starting at bank 0):
//     K tiles: an operand read takes one logical chunk from 16 consecutive
//     keys, so the swizzle is a bijection of key & 15.
//     V tiles: a transposed read takes a 4-chunk window from 4 consecutive
//     keys, so bits 2..3 follow key & 3; depending on key & 7 only, it is the
//     same for keys 8 apart, which keeps their reads one immediate apart.
//     (Measured: K reads conflict free; V reads at the transposed-read rate.)
//   D = 64 (8 chunks per row, rows alternating between bank halves): keys of
//     one parity share a half, 3 bits suffice for both.
template <int D>
__device__ inline int swz_k(int key) {
    if constexpr (D == 128) return ((key & 3) << 2) | ((key >> 2) & 3);
    else return ((key & 3) << 1) | ((key >> 2) & 1);
}
template <int D>
__device__ inline int swz_v(int key) {
    if constexpr (D == 128) return (key & 3) << 2;
    else return ((key & 3) << 1) | ((key >> 2) & 1);
}

// Per-lane LDS element offsets of the 32x32x16 MFMA operands within a tile.
// The K swizzle depends only on key & 15 and the V swizzle on key & 7, the same
// for a lane's V reads of every 8 keys, so those strides are immediates:
//   K (A of S^T = K Q^T), k-step ks: kofs[ks]
//   V^T (A of O^T = V^T P^T), 16-key step st, half b, channel block db:
//       vofs[db] + (st * 16 + b * 8) * D
template <int D>
__device__ inline void gqa_operand_offsets(int lane, int (&kofs)[D / 16], int (&vofs)[D / 32]) {
    const int j = lane & 31, hl = lane >> 5;
    const int sk = swz_k<D>(j);
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) kofs[ks] = j * D + (((ks * 2 + hl) ^ sk) << 3);
    const int g = lane >> 4, sl = lane & 15;
    const int vkey = (g >> 1) * 4 + (sl >> 2);   // key within its group of 8
    const int sv = swz_v<D>(vkey);
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
        vofs[db] = vkey * D + (((db * 4 + (g & 1) * 2 + ((sl & 3) >> 1)) ^ sv) << 3) + (sl & 1) * 4;
}

// V^T operand of one 16-key step: two transposed reads, 8 keys apart (base
// holds vofs and the step).
template <int D>
__device__ inline bf16x8 gqa_v_operand(const uint16_t* base) {
    const s16x4 p0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(PKV_LDS(s16x4, base));
    const s16x4 p1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(PKV_LDS(s16x4, base + 8 * D));
    return __builtin_bit_cast(bf16x8, (short __attribute__((ext_vector_type(8)))){p0[0], p0[1], p0[2], p0[3],
                                                                                  p1[0], p1[1], p1[2], p1[3]});
}

}  // namespace pkv
