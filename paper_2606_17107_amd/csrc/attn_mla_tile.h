// LDS layout of the 32-key bf16 latent tiles of the MLA attention kernels.
#pragma once

#include "attn_common.h"

namespace pkv {

constexpr int MBN = 32;        // keys per tile
constexpr int DQK = 576;       // score channels
constexpr int DV = 512;        // value (latent) channels
constexpr int MCH = DQK / 8;   // 16-byte chunks per row: 72

// XOR swizzle of the low three bits of a row's 16-byte chunk index by its key.
// A row is 72 chunks, so consecutive keys start in alternate halves of the 16
// bank groups (16 bytes each).  K operand reads take one chunk from each of 16
// consecutive keys: for either key parity the swizzle is a bijection of
// (key >> 1) & 7, so the 16 reads hit 16 groups.  Transposed V reads take a
// 4-chunk aligned window from each of 4 consecutive keys: keys 4q and 4q+2
// (and 4q+1, 4q+3) differ in bit 2 of the swizzle, which moves the window to
// the other half of its 8-chunk group.
__device__ inline int mswz(int key) { return (((key >> 1) & 1) << 2) | ((key >> 2) & 3); }

}  // namespace pkv
