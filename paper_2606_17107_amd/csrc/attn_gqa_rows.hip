// bf16 GQA suffix attention for few query rows: token-by-token generation and
// short suffixes (paper Sec. 5 "Linear-time TTFT"; Sec. 4 erratum).
//
// With few (query, head-in-group) rows per KV head the call is bound by the
// K/V stream from HBM and by fixed costs, not by the matrix cores, so the
// workgroup splits the KEYS over its waves instead of the rows:
//   * every wave holds all rows (at most 32: Q^T operands and O^T
//     accumulators in registers) and takes every fourth 32-key tile of the
//     workgroup's run;
//   * each wave stages its own tiles in its own LDS stages (2 x 16 KB at head
//     size 128) by LDS-DMA: no barrier in the loop, only the wave's own vmcnt
//     waits, so the waves drift apart and keep the memory system busy;
//   * the four waves' (O, max, sum) are merged in LDS at the end of an item.
// Workgroups take equal runs of the tile axis (attn_columns.h), short caches whole
// items.  One query for each of 16 paged caches of 8448..12544 keys, one layer of
// the 8B shape: 131 us a call with the merge (every key read once: 683 MB by the
// counters, 681 MB at least), against 142 us in the many-row kernel with 4 splits a
// sequence; five sequences of 20000 and 4 x 300 keys: 33 us against 47 us; one of
// 512 keys: 10 us against 16, of 8192 keys: 16 us against 22.
#include <type_traits>

#include "attn_columns.h"
#include "attn_gqa_tile.h"

namespace pkv {
namespace {

constexpr int kRowWaves = 4;

__device__ inline int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

template <int D, bool PAGED>
__global__ __launch_bounds__(kRowWaves * 64, 2) void attn_gqa_rows_kernel(AttnArgs a, ColPlan p) {
    constexpr int NW = kRowWaves;
    constexpr int BN = kColTile;           // keys per tile
    constexpr int CH = D / 8;              // 16-byte chunks per row
    constexpr int KBLK = BN * CH / 64;     // LDS-DMA loads per K (or V) tile
    constexpr int KPB = 64 / CH;           // keys per LDS-DMA load
    constexpr int KP = D == 128 ? 4 : 1;   // LDS-DMA loads after which the K swizzle repeats
    constexpr int KS = D / 16;             // MFMA k-steps over channels
    constexpr int DB = D / 32;             // 32-channel output blocks
    constexpr int TE = BN * D;             // elements of one K or V tile
    constexpr int ROWS = 32;               // rows per workgroup
    static_assert(6 * KBLK < 64, "loads in flight within the vmcnt range");
    static_assert(ROWS * D * 4 <= 4 * TE * 2, "a wave's O^T fits its own stages");

    // Per wave: K stages 0 and 1, V stages 0 and 1; after the loop, its O^T.
    __shared__ __attribute__((aligned(16))) uint16_t stage_lds[NW * 4 * TE];
    __shared__ float row_max_lds[NW][ROWS], row_sum_lds[NW][ROWS];

    const uint32_t column = col_decode(p);
    const int tid = threadIdx.x;
    const int wave = uniform(tid >> 6);
    const int lane = tid & 63;
    const int j = lane & 31;
    const int hl = lane >> 5;
    const int lkey = lane / CH, phys = lane % CH;
    uint16_t* const my_lds = stage_lds + wave * 4 * TE;
    auto kst = [&](int st) __attribute__((always_inline)) -> uint16_t* { return my_lds + st * TE; };
    auto vst = [&](int st) __attribute__((always_inline)) -> uint16_t* { return my_lds + (2 + st) * TE; };

    // Per-lane LDS element offsets of the MFMA operands within a stage, as in
    // the many-row kernel.
    int kofs[KS], vofs[DB];
    gqa_operand_offsets<D>(lane, kofs, vofs);
    const float sc2 = a.scale * kLog2e;

    // Touch the tensors that the sequence bounds lead to, so that their address
    // translations are fetched while the bounds are.
    const uint32_t touch = (uint32_t)a.q_pos[0] ^ *(const uint32_t*)a.q ^ (PAGED ? (uint32_t)a.block_table[0] : 0u);
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

    asm volatile("" ::"v"(touch));

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
        const int layer = sg.stream / a.n_kv_heads;
        const int kvh = sg.stream - layer * a.n_kv_heads;
        const SeqInfo si = p.columns ? col_seq_info(cs, sg.seq) : seq_info(a, sg.seq);
        const int M = si.nq * p.G;
        if (M <= 0) continue;

        // The lane's row and its Q^T operands (the same in every wave).
        const bool row_ok = j < M;
        const int qi = row_ok ? j / p.G : 0;
        const int pos = a.q_pos[si.q0 + qi], qpos = row_ok ? pos : -1;
        bf16x8 qf[KS];
        {
            // rows past M repeat the first (never written)
            const int head = kvh * p.G + (row_ok ? j - qi * p.G : 0);
            const uint16_t* qrow = (const uint16_t*)a.q + (int64_t)layer * a.q_stride[0] +
                                   (int64_t)(si.q0 + qi) * a.q_stride[1] + (int64_t)head * a.q_stride[2];
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
                qf[ks] = __builtin_bit_cast(bf16x8, *(const u32x4*)(qrow + ks * 16 + hl * 8));
        }
        int row_start, row_end;
        visible_range(qpos, si.kvl, a.window, row_start, row_end);   // (0, 0) for rows past M
        // Every wave holds every row, so these are the workgroup's bounds.
        const int e_min = wave_min_u(row_ok ? row_end : 0x7fffffff);
        const int e_max = wave_max_u(row_end);
        const int s_min = wave_min_u(row_ok ? row_start : 0x7fffffff);
        const int s_max = wave_max_u(row_start);
        const int lo = s_min == 0x7fffffff ? 0 : s_min / BN * BN;
        const int hi = min(si.kvl, e_max);
        const int real = hi > lo ? (hi - lo + BN - 1) / BN : 0;
        const int t_begin = uniform(col_real_tile(sg.first, sg.tiles, real)) + wave;   // this wave: t_begin, + NW, ...
        const int t_end = uniform(col_real_tile(sg.last, sg.tiles, real));
        const int n_tiles = t_end > t_begin ? (t_end - t_begin + NW - 1) / NW : 0;
        auto key_of = [&](int i) __attribute__((always_inline)) { return lo + (t_begin + i * NW) * BN; };

        const char* const kbase = (const char*)((const uint16_t*)a.k + (int64_t)layer * a.k_stride[0] +
                                                (int64_t)kvh * a.k_stride[1] + si.base * a.k_stride[2]);
        const char* const vbase = (const char*)((const uint16_t*)a.v + (int64_t)layer * a.v_stride[0] +
                                                (int64_t)kvh * a.v_stride[1] + si.base * a.v_stride[2]);
        const int64_t krow = a.k_stride[2] * 2, vrow = a.v_stride[2] * 2;   // bytes between keys
        PageWindow kw, vw;
        if constexpr (PAGED) {
            kw.init(a.block_table, a, sg.seq, key_of(0) >> a.page_shift);
            if (a.v_block_table) vw.init(a.v_block_table, a, sg.seq, key_of(0) >> a.page_shift);
        }
        // LDS-DMA of one tile of one tensor.  Lane l of load b fills LDS chunk
        // slot 64 b + l: key KPB b + l / CH, physical chunk l % CH, holding logical
        // chunk phys ^ swizzle(key).  The K swizzle repeats every KP loads, the
        // V swizzle every load.  A tile that runs past the last visible key
        // re-reads that key for the missing rows (masked later).
        uint32_t kchunk[KP];
#pragma unroll
        for (int b = 0; b < KP; ++b) kchunk[b] = (uint32_t)(phys ^ swz_k<D>(b * KPB + lkey)) * 16u;
        const uint32_t vchunk = (uint32_t)(phys ^ swz_v<D>(lkey)) * 16u;
        auto issue = [&](const char* tile, int64_t row_bytes, int t0, uint16_t* dst, auto v_tag) __attribute__((always_inline)) {
            constexpr bool V = decltype(v_tag)::value;
            const uint32_t lds0 = lds_addr_of(dst);
            if (t0 + BN <= hi) {
                const uint32_t lane_off = (uint32_t)(lkey * row_bytes);
                uint64_t at = uniform_u64((uint64_t)(uintptr_t)tile);
#pragma unroll
                for (int b = 0; b < KBLK; ++b) {
                    lds_dma16(lds0 + b * 1024, (const void*)at, lane_off + (V ? vchunk : kchunk[b % KP]));
                    at += (uint64_t)(KPB * row_bytes);
                    asm volatile("" : "+s"(at));   // step by step: KBLK hoisted offsets would spill scalar registers
                }
            } else {
                int key0 = lkey;
                asm volatile("" : "+v"(key0));   // once per item at most: keep its addresses out of the set-up
#pragma unroll
                for (int b = 0; b < KBLK; ++b)
                    lds_dma16(lds0 + b * 1024, tile, (uint32_t)(min(b * KPB + key0, hi - 1 - t0) * row_bytes) +
                                                        (V ? vchunk : kchunk[b % KP]));
            }
        };
        auto issue_k = [&](int i) __attribute__((always_inline)) {
            const int t0 = key_of(i);
            const char* tile;
            if constexpr (PAGED) tile = kbase + kw.offset(a, t0, a.k_page_stride * 2, krow);
            else tile = kbase + (int64_t)t0 * krow;
            issue(tile, krow, t0, kst(i & 1), std::false_type{});
        };
        auto issue_v = [&](int i) __attribute__((always_inline)) {
            const int t0 = key_of(i);
            const char* tile;
            if constexpr (PAGED) {
                const int64_t off = a.v_block_table ? vw.offset(a, t0, a.v_page_stride * 2, vrow)
                                                    : kw.offset(a, t0, a.v_page_stride * 2, vrow);
                tile = vbase + off;
            } else {
                tile = vbase + (int64_t)t0 * vrow;
            }
            issue(tile, vrow, t0, vst(i & 1), std::true_type{});
        };
        if (n_tiles > 0) {
            issue_k(0);
            issue_v(0);
        }
        if (n_tiles > 1) {
            issue_k(1);
            issue_v(1);
        }

        f32x16 o[DB];
#pragma unroll
        for (int db = 0; db < DB; ++db) o[db] = f32x16{};
        float m_run = -INFINITY, l_run = 0.f;
        auto lds_reads_done = []() __attribute__((always_inline)) {
            __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (0 << 8) | (3 << 14));
            asm volatile("" ::: "memory");
        };

        // One tile: S^T = K Q^T, online softmax with a lazily moved reference
        // maximum (probabilities stay below 2^kLazy), O^T += V^T P^T.
        constexpr float kLazy = 8.0f;
        auto scores = [&](const uint16_t* ks_src) __attribute__((always_inline)) {
            f32x16 s = f32x16{};
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const bf16x8 kf = __builtin_bit_cast(bf16x8, *(const u32x4*)(ks_src + kofs[ks]));
                s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[ks], s, 0, 0, 0);
            }
            return s;
        };
        auto softmax = [&](int t0, f32x16& s, bf16x8 (&pb)[2], auto mask_tag) __attribute__((always_inline)) {
            constexpr bool MASK = decltype(mask_tag)::value;
            auto hidden = [&](int r) __attribute__((always_inline)) {   // register -> key of the tile
                const int key = t0 + (r >> 2) * 8 + hl * 4 + (r & 3);
                return key >= row_end || key < row_start;
            };
            if (MASK) {
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (hidden(r)) s[r] = sc2 >= 0.f ? -INFINITY : INFINITY;
            }
            // largest scaled score: the largest raw score, or the smallest when the scale is negative
            float mx = s[0];
            if (sc2 >= 0.f) {
#pragma unroll
                for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
            } else {
#pragma unroll
                for (int r = 1; r < 16; ++r) mx = fminf(mx, s[r]);
            }
            const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
            const float msc = fmaxf(__uint_as_float(sw[0]) * sc2, __uint_as_float(sw[1]) * sc2);
            const bool up = msc > m_run + kLazy;
            if (__builtin_amdgcn_ballot_w64(up) != 0) {
                const float m_new = up ? msc : m_run;
                const float alpha = m_run == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_run - m_new);
                l_run *= alpha;
#pragma unroll
                for (int db = 0; db < DB; ++db) o[db] *= alpha;
                m_run = m_new;
            }
            const float neg_m = m_run == -INFINITY ? 0.f : -m_run;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                float e = __builtin_amdgcn_exp2f(fmaf(s[r], sc2, neg_m));
                if (MASK && hidden(r)) e = 0.f;
                s[r] = e;
            }
#pragma unroll
            for (int st = 0; st < 2; ++st) {
                f32x8 pv;
#pragma unroll
                for (int e = 0; e < 8; ++e) pv[e] = s[st * 8 + e];
                pb[st] = __builtin_convertvector(pv, bf16x8);
            }
            // The row sum takes the probabilities as they enter PV, rounded to bf16, as in
            // the many-row kernel: the rounding of a key that dominates its row cancels.
            const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
            float lsum = 0.f;
#pragma unroll
            for (int e = 0; e < 16; e += 2)
                lsum = __builtin_amdgcn_fdot2_f32_bf16((bf16x2){pb[e >> 3][e & 7], pb[e >> 3][(e & 7) + 1]}, ones, lsum, false);
            l_run += lsum;
        };
        auto add_values = [&](const uint16_t* vs_src, const bf16x8 (&pb)[2]) __attribute__((always_inline)) {
#pragma unroll
            for (int st = 0; st < 2; ++st)
#pragma unroll
                for (int db = 0; db < DB; ++db)
                    o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(gqa_v_operand<D>(vs_src + vofs[db] + st * 16 * D),
                                                                    pb[st], o[db], 0, 0, 0);
        };
        // Loads retire in order: K(i), V(i), K(i+1), V(i+1), then K(i+2) once
        // the scores of tile i have been read, V(i+2) once its values have.
        auto tile = [&](int i, int st) __attribute__((always_inline)) {
            const int t0 = key_of(i);
            const bool more = i + 1 < n_tiles, more2 = i + 2 < n_tiles;
            if (more) wait_vmcnt<3 * KBLK>();
            else wait_vmcnt<KBLK>();
            asm volatile("" ::: "memory");
            f32x16 s = scores(kst(st));
            lds_reads_done();
            if (more2) issue_k(i + 2);
            bf16x8 pb[2];
            if (t0 + BN > e_min || t0 < s_max) softmax(t0, s, pb, std::true_type{});
            else softmax(t0, s, pb, std::false_type{});
            if (more2) wait_vmcnt<3 * KBLK>();
            else if (more) wait_vmcnt<2 * KBLK>();
            else wait_vmcnt<0>();
            asm volatile("" ::: "memory");
            add_values(vst(st), pb);
            lds_reads_done();
            if (more2) issue_v(i + 2);
        };
#pragma unroll 1
        for (int i = 0; i < n_tiles; ++i) tile(i, i & 1);

        // Merge the four waves: O^T to this wave's stages (row-major fp32,
        // 16-byte chunks XOR-swizzled by row), maxima and sums beside.
        constexpr int OC = D / 4;   // 16-byte fp32 chunks per row
        float* const my_o = (float*)my_lds;
        const float l_tot = l_run + __shfl_xor(l_run, 32);
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int b = 0; b < 4; ++b)
                *(f32x4*)(my_o + j * D + ((db * 8 + b * 2 + hl) ^ (j & (OC - 1))) * 4) =
                    f32x4{o[db][4 * b], o[db][4 * b + 1], o[db][4 * b + 2], o[db][4 * b + 3]};
        if (hl == 0) {
            row_max_lds[wave][j] = m_run;
            row_sum_lds[wave][j] = l_tot;
        }
        __syncthreads();
        col_merge_rows<NW, ROWS, D>(a, p, sg, si, layer, kvh * p.G, p.G, M, (const float*)stage_lds, 2 * TE,
                                    &row_max_lds[0][0], &row_sum_lds[0][0]);
        __syncthreads();   // the stages are free for the next item
    }
}

template <int D>
hipError_t launch_d(const AttnArgs& a, const ColPlan& p, dim3 grid, hipStream_t stream) {
    if (a.block_table)
        hipLaunchKernelGGL((attn_gqa_rows_kernel<D, true>), grid, dim3(kRowWaves * 64), 0, stream, a, p);
    else
        hipLaunchKernelGGL((attn_gqa_rows_kernel<D, false>), grid, dim3(kRowWaves * 64), 0, stream, a, p);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_attn_gqa_rows(const AttnArgs& a, const ColPlan& p, dim3 grid, hipStream_t stream) {
    return a.head_dim == 64 ? launch_d<64>(a, p, grid, stream) : launch_d<128>(a, p, grid, stream);
}

}  // namespace pkv
