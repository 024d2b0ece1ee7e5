// Even partition of a few-row attention call over the workgroups, formed on
// the device because the cache lengths live there.
//
// The key tiles of every (layer, KV head) stream and sequence are laid end to
// end on one axis (stream-major, then sequence), and the axis is cut into
// columns of equal length, one workgroup each, so all workgroups get the same
// number of tiles however ragged the cache lengths are.  A column's run of tiles
// covers the end of one item (stream, sequence), any number of whole items, and
// the beginning of another: an item inside one column is finished there, an item
// cut by column borders leaves one partial per column for the combine pass.  The
// borders follow all lengths of the call, so where one sequence is cut, and with
// it the rounding of its result, depends on the others.  Short caches are not cut:
// a workgroup takes a whole item, and sequences do not affect each other.
#pragma once

#include "attn_common.h"

namespace pkv {

constexpr int kColTile = 32;      // keys per unit of the axis
constexpr int kColMaxSeqs = 64;   // one lane of a wave per sequence

// Wave reductions and prefix sum by DPP (a register move within the wave: no
// trip through LDS, whose six dependent round trips cost about 0.4 us a
// reduction).  Rotations within the 16-lane rows leave every row's result in all
// its lanes; the four rows are combined in scalar registers, so the result is
// uniform.
template <int CTRL, int ROWS = 0xf>
__device__ inline int dpp(int old, int v) {
    return __builtin_amdgcn_update_dpp(old, v, CTRL, ROWS, 0xf, false);
}
constexpr int kDppRor = 0x120;      // row_ror:n = kDppRor + n
constexpr int kDppShr = 0x110;      // row_shr:n = kDppShr + n
constexpr int kDppBcast15 = 0x142;  // lane 15 of a row to the next row
constexpr int kDppBcast31 = 0x143;  // lane 31 to rows 2 and 3
template <typename F>
__device__ inline int wave_reduce_i(int v, F f) {
    v = f(v, dpp<kDppRor + 8>(v, v));
    v = f(v, dpp<kDppRor + 4>(v, v));
    v = f(v, dpp<kDppRor + 2>(v, v));
    v = f(v, dpp<kDppRor + 1>(v, v));
    return f(f(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
             f(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}
__device__ inline int wave_max_u(int v) {
    return wave_reduce_i(v, [](int x, int y) { return max(x, y); });
}
__device__ inline int wave_min_u(int v) {
    return wave_reduce_i(v, [](int x, int y) { return min(x, y); });
}
// Inclusive prefix sum over the 64 lanes.
__device__ inline int wave_prefix_sum_i(int v) {
    v += dpp<kDppShr + 1>(0, v);
    v += dpp<kDppShr + 2>(0, v);
    v += dpp<kDppShr + 4>(0, v);
    v += dpp<kDppShr + 8>(0, v);
    v += dpp<kDppBcast15, 0xa>(0, v);
    v += dpp<kDppBcast31, 0xc>(0, v);
    return v;
}

// The sequences as one wave sees them: lane s holds sequence s.
struct ColSeqs {
    int q0, nq, kvl;      // as seq_info
    int64_t base;
    uint32_t tiles;       // this lane's sequence: tiles of its axis share (0: no rows)
    uint32_t end;         // inclusive prefix sum of tiles
    uint32_t total;       // tiles of one stream
    uint32_t col;         // tiles of one column
};

__device__ inline SeqInfo col_seq_info(const ColSeqs& c, int s) {
    SeqInfo si;
    si.q0 = __builtin_amdgcn_readlane(c.q0, s);
    si.nq = __builtin_amdgcn_readlane(c.nq, s);
    si.kvl = __builtin_amdgcn_readlane(c.kvl, s);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)c.base, s);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)c.base >> 32), s);
    si.base = (int64_t)(((uint64_t)hi << 32) | lo);
    return si;
}

// Sequence s's share of the axis: the tiles up to its length, or with a sliding
// window the most that a row block sees (the window and the span of the
// queries), after p.item_cost tiles that stand for the cost of starting an
// item.  At least one tile, so that every row is visited and written.  The
// bounds are those of seq_info.
__device__ inline ColSeqs col_seqs(const AttnArgs& a, const ColPlan& p) {
    ColSeqs c;
    const int s = (int)__lane_id();
    // All loads first (lanes past the last sequence repeat it), so that they
    // share one round trip.
    const int i = min(s, a.n_seqs - 1);
    const int64_t len = a.kv_len[i];
    int64_t base = 0;
    int lo = 0, hi = a.total_q;
    if (a.kv_base) base = a.kv_base[i];
    if (a.cu_q) {
        lo = a.cu_q[i];
        hi = a.cu_q[i + 1];
    }
    c.q0 = lo;
    c.nq = hi - lo;
    if (lo < 0 || c.nq < 0 || (int64_t)lo + c.nq > a.total_q || s >= a.n_seqs) c.nq = 0;
    c.base = base;
    const int64_t kvl = min(min(len, (int64_t)a.max_kv_len), a.cache_slots - base);
    c.kvl = base < 0 ? 0 : (int)max(kvl, (int64_t)0);
    int64_t seen = c.kvl;
    if (a.window > 0) seen = min(seen, (int64_t)a.window + a.max_q);
    c.tiles = c.nq > 0 ? p.item_cost + max(1u, (uint32_t)((seen + kColTile - 1) / kColTile)) : 0u;
    const uint32_t top = (uint32_t)wave_max_u((int)c.tiles);
    c.end = (uint32_t)wave_prefix_sum_i((int)c.tiles);
    c.total = (uint32_t)__builtin_amdgcn_readlane((int)c.end, 63);
    // Equal columns, long enough that no item is cut into more pieces than
    // the workspace has records for, and never shorter than p.min_tiles.
    const uint32_t axis = c.total * (uint32_t)p.streams;
    c.col = (axis + p.columns - 1) / p.columns;
    if (p.pieces > 1) c.col = max(c.col, (top + p.pieces - 2) / (p.pieces - 1));
    c.col = max(c.col, (uint32_t)p.min_tiles);
    c.col = (uint32_t)__builtin_amdgcn_readfirstlane((int)c.col);
    return c;
}

// One item's run of tiles inside a column.
struct ColSegment {
    int stream, seq;
    uint32_t length;               // on the axis
    uint32_t first, last, tiles;   // tiles [first, last) of the item's `tiles`
    int piece, pieces;             // which of the item's pieces this is
};

// Tile t of an item's axis share as a tile of the `real` ones its row block
// really sees (positions may hide keys): proportional, exact at both ends, and
// the same at a border for the two columns that meet there.
__device__ inline int col_real_tile(uint32_t t, uint32_t tiles, int real) {
    return t == 0 ? 0 : t == tiles ? real : (int)((double)t * (double)real / (double)tiles);
}

// Workgroup id -> column (or item).  Ids are dealt to the XCDs round-robin;
// consecutive columns read consecutive keys and stay on one XCD.
__device__ inline uint32_t col_decode(const ColPlan& p) {
    const uint32_t xcd = blockIdx.x % kXcds, slot = blockIdx.x / kXcds;
    return p.columns ? xcd * (p.columns / kXcds) + slot : blockIdx.x;
}

// The segment that starts at axis position x of a column that ends at x1.
__device__ inline ColSegment col_segment(const ColSeqs& c, const ColPlan& p, uint32_t x, uint32_t x1,
                                        uint32_t column) {
    ColSegment g;
    const uint32_t stream = (uint32_t)__builtin_amdgcn_readfirstlane((int)(x / c.total));
    const uint32_t rem = x - stream * c.total;
    const int s = __builtin_popcountll(__builtin_amdgcn_ballot_w64(c.end <= rem));
    const uint32_t share = (uint32_t)__builtin_amdgcn_readlane((int)c.tiles, s);
    const uint32_t start = (uint32_t)__builtin_amdgcn_readlane((int)c.end, s) - share;
    const uint32_t cost = (uint32_t)p.item_cost;
    const uint32_t first = rem - start, last = min(share, first + (x1 - x));
    g.stream = (int)stream;
    g.seq = s;
    g.length = last - first;
    g.tiles = share - cost;
    g.first = max(first, cost) - cost;
    g.last = max(last, cost) - cost;   // == first: the column ends before the item's first tile
    const uint32_t item = stream * c.total + start;   // axis position of the item
    const uint32_t c0 = (item + cost) / c.col, c1 = (item + share - 1) / c.col;
    g.piece = __builtin_amdgcn_readfirstlane((int)(column - c0));
    g.pieces = __builtin_amdgcn_readfirstlane((int)(c1 - c0)) + 1;
    return g;
}

// End of an item: the NW waves' O (row-major fp32 in LDS, wave w's at
// o_lds + w * wave_stride, 16-byte chunk c of row r at chunk c ^ (r mod chunks)),
// maxima and sums are merged over all threads of the workgroup and written: as
// the output row when the item lies in this column, else as piece sg.piece of
// the workspace (normalised, with its log2-sum-exp).  Row r < M is (query r / G,
// head head0 + r % G) of the item.
template <int NW, int ROWS, int DV>
__device__ __forceinline__ void col_merge_rows(const AttnArgs& a, const ColPlan& p, const ColSegment& sg,
                                               const SeqInfo& si, int layer, int head0, int G, int M,
                                               const float* o_lds, int wave_stride, const float* max_lds,
                                               const float* sum_lds) {
    constexpr int OC = DV / 4;
    const int64_t items = (int64_t)a.n_layers * a.total_q * a.n_heads;
    constexpr int PASS = NW * 64 / OC;   // rows per pass
    static_assert(NW * 64 % OC == 0 && ROWS % PASS == 0, "whole rows per pass");
    const int c = (int)threadIdx.x % OC, r0 = (int)threadIdx.x / OC;
#pragma unroll 4
    for (int r = r0; r < ROWS; r += PASS) {
        if (r >= M) break;
        float mw[NW], mx = -INFINITY, sum = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            mw[w] = max_lds[w * ROWS + r];
            mx = fmaxf(mx, mw[w]);
        }
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float wt = mw[w] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mw[w] - mx);
            acc += wt * *(const f32x4*)(o_lds + w * wave_stride + r * DV + (c ^ (r & (OC - 1))) * 4);
            sum += wt * sum_lds[w * ROWS + r];
        }
        const float inv = row_inverse(sum);
        const float lse2 = row_lse2(mx, sum);
        const int q = r / G;
        const int head = head0 + r - q * G;
        const int64_t row = si.q0 + q;
        const int64_t item = ((int64_t)layer * a.total_q + row) * a.n_heads + head;
        acc *= inv;
        if (sg.pieces == 1) {
            u32x2 w;
            w[0] = bf_rne(acc[0]) | (bf_rne(acc[1]) << 16);
            w[1] = bf_rne(acc[2]) | (bf_rne(acc[3]) << 16);
            *(u32x2*)((uint16_t*)a.out + (int64_t)layer * a.o_stride[0] + row * a.o_stride[1] +
                      (int64_t)head * a.o_stride[2] + c * 4) = w;
            if (c == 0) {
                if (a.lse_out) a.lse_out[item] = lse2 * kLn2;
                if (a.ws_lse) a.ws_lse[item] = INFINITY;   // the combine pass leaves this row alone
            }
        } else {
            *(f32x4*)(a.ws_o + (sg.piece * items + item) * DV + c * 4) = acc;
            if (c == 0) {
                a.ws_lse[sg.piece * items + item] = lse2;
                if (sg.piece == sg.pieces - 1)   // records beyond the item's pieces weigh nothing
                    for (int k = sg.pieces; k < p.pieces; ++k) a.ws_lse[k * items + item] = -INFINITY;
            }
        }
    }
}

}  // namespace pkv
