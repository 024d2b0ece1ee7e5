// bf16 MLA suffix attention (absorbed form) for few query rows: token-by-token
// generation with up to 16 (query, head) rows a sequence (paper Sec. 8, MLA
// adapter; Sec. 5 "Linear-time TTFT").
//
// 16 rows are all heads of one query of a 16-head model.  The call is bound by the
// stream of latent rows from HBM, so, as in the GQA few-row kernel, the workgroup
// splits the KEYS over its waves:
//   * MFMA 16x16x32 bf16 (N = 16 rows, no idle columns).  Every wave holds the
//     16 rows' Q^T over 576 channels (72 VGPRs) and their O^T over 512 channels
//     (128 VGPRs) and takes every fourth 32-key tile of the workgroup's run.
//   * S^T = K Q^T: a lane holds keys 4g + r and 16 + 4g + r (g = lane / 16) of one
//     row, which is the operand layout of O^T = V^T P^T with the keys in that
//     order; V^T comes from the same LDS tile by transposed reads.
//   * Each wave stages its own tiles (36 KB, one stage) by LDS-DMA: no barrier in
//     the loop; while one wave computes, the others' tiles are in flight.
//   * The four waves' (O, max, sum) are merged in LDS at the end of an item.
// Workgroups take equal runs of the tile axis (attn_columns.h), short caches whole
// items.  One query for
// each of 16 caches of 4096..32768 keys (351 MB): 85 us a call against 119 us in
// the many-row kernel, where 112 of a workgroup's 128 rows are idle and every
// sequence has 16 splits, long or short; one sequence of 32768 keys: 52 us against
// 67 us, of 512 keys: 21 us against 33 us.
#include <type_traits>

#include "attn_columns.h"
#include "attn_mla_tile.h"

namespace pkv {
namespace {

constexpr int kMlaRowWaves = 4;

template <bool PAGED>
__global__ __launch_bounds__(kMlaRowWaves * 64, 1) void attn_mla_rows_kernel(AttnArgs a, ColPlan p) {
    constexpr int NW = kMlaRowWaves;
    constexpr int BN = kColTile;            // keys per tile
    constexpr int KS = DQK / 32;            // MFMA k-steps over the score channels: 18
    constexpr int CB = DV / 16;             // 16-channel output blocks: 32
    constexpr int TE = BN * DQK;            // elements per tile
    constexpr int NBLK = BN * MCH / 64;     // LDS-DMA loads per tile: 36
    constexpr int HBLK = NBLK / 2;          // ... per 16 keys, after which the swizzle repeats: 18
    constexpr int ROWS = 16;                // rows per workgroup
    static_assert(HBLK * 64 == 16 * MCH, "16 keys are a whole number of loads");
    static_assert(ROWS * DV * 4 <= TE * 2, "a wave's O^T fits its own stage");

    __shared__ __attribute__((aligned(16))) uint16_t stage_lds[NW * TE];
    __shared__ float row_max_lds[NW][ROWS], row_sum_lds[NW][ROWS];

    const uint32_t column = col_decode(p);
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int j = lane & 15;     // row of the block (N axis), key or channel of an operand (M axis)
    const int g = lane >> 4;
    uint16_t* const st = stage_lds + wave * TE;

    // Source byte offsets of the first 16 keys' loads (the other 16 repeat them
    // 16 keys on): lane l of load b fills chunk slot 64 b + l of the tile.
    const int64_t kss = a.k_stride[2];
    uint32_t src_off[HBLK];
#pragma unroll
    for (int b = 0; b < HBLK; ++b) {
        const int slot = b * 64 + lane, key = slot / MCH;
        src_off[b] = (uint32_t)(key * kss * 2) + (uint32_t)((slot % MCH) ^ mswz(key)) * 16u;
    }
    // LDS element offsets of the MFMA operands:
    //   K, k-step ks, 16-key block b: chunk 4 ks + g of key 16 b + j, at
    //     kofs[ks & 1] + (ks >> 1) * 64 + b * 16 * 576;
    //   V^T, channel block cb, half b: lane group g reads channels 16 cb .. +15 of
    //     keys 16 b + 4 g + 0..3, at vofs[cb & 3] + (cb >> 2) * 64 + b * 16 * 576.
    int kofs[2], vofs[4];
#pragma unroll
    for (int q = 0; q < 2; ++q) kofs[q] = j * DQK + ((q * 4 + g) ^ mswz(j)) * 8;
    {
        const int key = g * 4 + (j >> 2);
#pragma unroll
        for (int q = 0; q < 4; ++q) vofs[q] = key * DQK + ((q * 2 + ((j & 3) >> 1)) ^ mswz(key)) * 8 + (j & 1) * 4;
    }
    const float sc2 = a.scale * kLog2e;

    ColSeqs cs{};
    uint32_t x = 0, x1 = 1;
    if (p.columns) {
        cs = col_seqs(a, p);
        const uint64_t lo = (uint64_t)column * cs.col, axis = (uint64_t)cs.total * p.streams;
        if (lo >= axis) return;   // uniform
        x = (uint32_t)lo;
        x1 = (uint32_t)min(lo + cs.col, axis);
    } else if (column >= (uint32_t)p.streams * (uint32_t)a.n_seqs) {
        return;
    }

    while (x < x1) {
        ColSegment sg;
        if (p.columns) {
            sg = col_segment(cs, p, x, x1, column);
            x += sg.length;
            if (sg.first == sg.last) continue;   // uniform
        } else {
            sg.seq = (int)(column / (uint32_t)p.streams);   // by sequence: neighbours take about equally long
            sg.stream = (int)(column - (uint32_t)sg.seq * (uint32_t)p.streams);
            sg.first = 0;
            sg.last = sg.tiles = 1;
            sg.piece = 0;
            sg.pieces = 1;
            x = x1;
        }
        const int layer = sg.stream;   // one KV head
        const SeqInfo si = p.columns ? col_seq_info(cs, sg.seq) : seq_info(a, sg.seq);
        const int H = a.n_heads;
        const int M = si.nq * H;
        if (M <= 0) continue;

        // The lane's row and its Q^T operands (the same in every wave).
        const bool row_ok = j < M;
        const int qi = row_ok ? j / H : 0;
        const int pos = a.q_pos[si.q0 + qi], qpos = row_ok ? pos : -1;
        bf16x8 qf[KS];
        {
            const int head = row_ok ? j - qi * H : 0;   // rows past M repeat the first (never written)
            const uint16_t* qrow = (const uint16_t*)a.q + (int64_t)layer * a.q_stride[0] +
                                   (int64_t)(si.q0 + qi) * a.q_stride[1] + (int64_t)head * a.q_stride[2];
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
                qf[ks] = __builtin_bit_cast(bf16x8, *(const u32x4*)(qrow + ks * 32 + g * 8));
        }
        int row_start, row_end;
        visible_range(qpos, si.kvl, a.window, row_start, row_end);   // (0, 0) for rows past M
        const int e_min = wave_min_u(row_ok ? row_end : 0x7fffffff);
        const int e_max = wave_max_u(row_end);
        const int s_min = wave_min_u(row_ok ? row_start : 0x7fffffff);
        const int s_max = wave_max_u(row_start);
        const int lo = s_min == 0x7fffffff ? 0 : s_min / BN * BN;
        const int hi = min(si.kvl, e_max);
        const int real = hi > lo ? (hi - lo + BN - 1) / BN : 0;
        const int t_begin = __builtin_amdgcn_readfirstlane(col_real_tile(sg.first, sg.tiles, real)) + wave;
        const int t_end = __builtin_amdgcn_readfirstlane(col_real_tile(sg.last, sg.tiles, real));
        const int n_tiles = t_end > t_begin ? (t_end - t_begin + NW - 1) / NW : 0;   // t_begin, + NW, ...
        auto key_of = [&](int i) __attribute__((always_inline)) { return lo + (t_begin + i * NW) * BN; };

        const char* const kbase =
            (const char*)((const uint16_t*)a.k + (int64_t)layer * a.k_stride[0] + si.base * kss);
        PageWindow pw;
        if constexpr (PAGED) pw.init(a.block_table, a, sg.seq, key_of(0) >> a.page_shift);
        // A tile that runs past the last visible key re-reads that key for the
        // missing rows (masked later).
        auto issue = [&](int t0) __attribute__((always_inline)) {
            const char* tile;
            if constexpr (PAGED) tile = kbase + pw.offset(a, t0, a.k_page_stride * 2, kss * 2);
            else tile = kbase + (int64_t)t0 * kss * 2;
            const uint32_t lds0 = lds_addr_of(st);
            if (t0 + BN <= hi) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    uint64_t at = uniform_u64((uint64_t)(uintptr_t)(tile + h * 16 * kss * 2));
                    asm volatile("" : "+s"(at));
#pragma unroll
                    for (int b = 0; b < HBLK; ++b)
                        lds_dma16(lds0 + (h * HBLK + b) * 1024, (const void*)at, src_off[b]);
                }
            } else {
                const int last = hi - 1 - t0;
                int slot0 = lane;
                asm volatile("" : "+v"(slot0));   // once per item at most: keep its addresses out of the set-up
#pragma unroll
                for (int b = 0; b < NBLK; ++b) {
                    const int slot = b * 64 + slot0, key = slot / MCH;
                    lds_dma16(lds0 + b * 1024, tile,
                              (uint32_t)(min(key, last) * kss * 2) + (uint32_t)((slot % MCH) ^ mswz(key)) * 16u);
                }
            }
        };
        if (n_tiles > 0) issue(key_of(0));

        f32x4 o[CB];
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) o[cb] = f32x4{0.f, 0.f, 0.f, 0.f};
        float m_run = -INFINITY, l_run = 0.f;
        constexpr float kLazy = 8.0f;   // the reference maximum moves only past this many log2 units

#pragma unroll 1
        for (int i = 0; i < n_tiles; ++i) {
            const int t0 = key_of(i);
            wait_vmcnt<0>();
            asm volatile("" ::: "memory");
            // S^T = K Q^T of two 16-key blocks, two accumulation chains
            f32x4 s[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    s[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        __builtin_bit_cast(bf16x8, *(const u32x4*)(st + kofs[ks & 1] + (ks >> 1) * 64 + b * 16 * DQK)),
                        qf[ks], s[b], 0, 0, 0);
            auto hidden = [&](int b, int r) __attribute__((always_inline)) {
                const int key = t0 + b * 16 + g * 4 + r;
                return key >= row_end || key < row_start;
            };
            const bool mask = t0 + BN > e_min || t0 < s_max;   // uniform
            if (mask) {
#pragma unroll
                for (int b = 0; b < 2; ++b)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (hidden(b, r)) s[b][r] = sc2 >= 0.f ? -INFINITY : INFINITY;
            }
            // Largest scaled score of the row: over the lane's 8 keys, then the
            // four lane groups.
            float mx = s[0][0] * sc2;
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int r = 0; r < 4; ++r) mx = fmaxf(mx, s[b][r] * sc2);
            const auto s32 = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
            mx = fmaxf(__uint_as_float(s32[0]), __uint_as_float(s32[1]));
            const auto s16 = __builtin_amdgcn_permlane16_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
            mx = fmaxf(__uint_as_float(s16[0]), __uint_as_float(s16[1]));
            const bool up = mx > m_run + kLazy;
            if (__builtin_amdgcn_ballot_w64(up) != 0) {
                const float m_new = up ? mx : m_run;
                const float alpha = m_run == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_run - m_new);
                l_run *= alpha;
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) o[cb] *= alpha;
                m_run = m_new;
            }
            const float neg_m = m_run == -INFINITY ? 0.f : -m_run;
            f32x8 e8;
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float e = __builtin_amdgcn_exp2f(fmaf(s[b][r], sc2, neg_m));
                    if (mask && hidden(b, r)) e = 0.f;
                    e8[b * 4 + r] = e;
                    l_run += e;
                }
            const bf16x8 pb = __builtin_convertvector(e8, bf16x8);
            // O^T += V^T P^T
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) {
                const uint16_t* base = st + vofs[cb & 3] + (cb >> 2) * 64;
                const s16x4 p0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(PKV_LDS(s16x4, base));
                const s16x4 p1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(PKV_LDS(s16x4, base + 16 * DQK));
                const bf16x8 vf = __builtin_bit_cast(
                    bf16x8, (short __attribute__((ext_vector_type(8)))){p0[0], p0[1], p0[2], p0[3], p1[0], p1[1],
                                                                        p1[2], p1[3]});
                o[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pb, o[cb], 0, 0, 0);
            }
            // The tile's reads are done before its stage is filled again.
            __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (0 << 8) | (3 << 14));
            asm volatile("" ::: "memory");
            if (i + 1 < n_tiles) issue(key_of(i + 1));
        }

        // Merge the four waves: O^T to this wave's stage (row-major fp32, 16-byte
        // chunks XOR-swizzled by row), maxima and sums beside.
        constexpr int OC = DV / 4;   // 16-byte fp32 chunks per row
        {
            float* const my_o = (float*)st;
            float l_tot = l_run + __shfl_xor(l_run, 32);
            l_tot += __shfl_xor(l_tot, 16);
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) *(f32x4*)(my_o + j * DV + ((cb * 4 + g) ^ j) * 4) = o[cb];
            if (g == 0) {
                row_max_lds[wave][j] = m_run;
                row_sum_lds[wave][j] = l_tot;
            }
        }
        __syncthreads();
        col_merge_rows<NW, ROWS, DV>(a, p, sg, si, layer, 0, H, M, (const float*)stage_lds, TE / 2,
                                     &row_max_lds[0][0], &row_sum_lds[0][0]);
        __syncthreads();   // the stages are free for the next item
    }
}

}  // namespace

hipError_t launch_attn_mla_rows(const AttnArgs& a, const ColPlan& p, dim3 grid, hipStream_t stream) {
    if (a.block_table)
        hipLaunchKernelGGL((attn_mla_rows_kernel<true>), grid, dim3(kMlaRowWaves * 64), 0, stream, a, p);
    else
        hipLaunchKernelGGL((attn_mla_rows_kernel<false>), grid, dim3(kMlaRowWaves * 64), 0, stream, a, p);
    return hipGetLastError();
}

}  // namespace pkv
