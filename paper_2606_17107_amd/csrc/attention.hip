// Suffix attention: plan, fp32 kernel, split-KV combine and dispatch.
// (Paper Sec. 5 "Linear-time TTFT": the transplant costs a re-rotation pass
// plus the causal attention of the suffix over the spliced cache.)
// The bf16 GQA kernel lives in attn_gqa_bf16.hip.
#include <algorithm>

#include "attn_columns.h"

namespace pkv {

hipError_t launch_attn_gqa_bf16(const AttnArgs& a, const Plan& p, dim3 grid, hipStream_t stream);
hipError_t launch_attn_mla_bf16(const AttnArgs& a, const Plan& p, dim3 grid, hipStream_t stream);
hipError_t launch_attn_gqa_rows(const AttnArgs& a, const ColPlan& p, dim3 grid, hipStream_t stream);
hipError_t launch_attn_mla_rows(const AttnArgs& a, const ColPlan& p, dim3 grid, hipStream_t stream);

namespace {

constexpr int kCUs = 256;   // compute units of an MI355X

// fp32 GQA kernel on fp32 matrix cores (v_mfma_f32_32x32x2_f32).  Each of the
// two waves owns 32 rows (query, head-in-group) of one KV head.  As in the
// bf16 kernel the scores are formed transposed, S^T = K Q^T, so a lane holds 16
// keys of one row and its probabilities are already the B operand of
// O^T = V^T P^T: a 2-key step pairs key 8jj + rr (held by lanes 0-31) with key
// 8jj + 4 + rr (lanes 32-63), both in accumulator register 4jj + rr.  K/V tiles
// of 32 keys move through registers into LDS (the next tile's loads are in
// flight while one is consumed): K transposed ([channel][key], a half-wave's 32
// reads of one score step are 32 consecutive words), V row-major ([key][channel],
// likewise for the PV operand).  fp32 online softmax with an exact rescale per
// tile, in log2 units.
template <int D>
__global__ __launch_bounds__(128) void attn_gqa_f32(AttnArgs a, Plan p) {
    constexpr int BN = 32;                 // keys per tile
    constexpr int NW = 2;                  // waves, 32 rows each
    constexpr int KSF = D / 2;             // score steps (2 channels each)
    constexpr int DB = D / 32;             // 32-channel output blocks
    constexpr int NL = BN * D / 4 / (NW * 64);   // 16-byte loads per thread per tensor and tile
    __shared__ __attribute__((aligned(16))) float kt_lds[D * BN];   // [channel][key]
    __shared__ __attribute__((aligned(16))) float v_lds[BN * D];    // [key][channel]
    __shared__ int red[NW], red_min[NW], red_start[NW], red_smax[NW];

    int group, rb;
    if (!decode(p, group, rb)) return;
    const int split = group % p.splits;
    int rest = group / p.splits;
    const int kvh = rest % a.n_kv_heads;
    rest /= a.n_kv_heads;
    const int layer = rest % a.n_layers;
    const int seq = rest / a.n_layers;
    const SeqInfo si = seq_info(a, seq);
    const int M = si.nq * p.G;
    const int m0 = rb * (NW * 32);
    if (m0 >= M) return;

    const int tid = threadIdx.x;
    const int wave = tid >> 6;
    const int lane = tid & 63;
    const int j = lane & 31;
    const int hl = lane >> 5;
    const int m = m0 + wave * 32 + j;
    const bool row_ok = m < M;
    const int qi = row_ok ? m / p.G : 0;
    const int head = kvh * p.G + (row_ok ? m - qi * p.G : 0);

    // Q^T B operand: channel 2s + hl of the lane's row for step s, scaled.
    float qf[KSF];
    {
        const float* qrow = (const float*)a.q + (int64_t)layer * a.q_stride[0] +
                            (int64_t)(si.q0 + qi) * a.q_stride[1] + (int64_t)head * a.q_stride[2];
#pragma unroll
        for (int s = 0; s < KSF; ++s) qf[s] = row_ok ? qrow[2 * s + hl] * a.scale : 0.f;
    }
    const int qpos = row_ok ? a.q_pos[si.q0 + qi] : -1;
    int row_start, row_end;
    visible_range(qpos, si.kvl, a.window, row_start, row_end);   // (0, 0) for rows past M
    const int wmin = wave_min_i(row_ok ? row_end : 0x7fffffff);
    const int wmax = wave_max_i(row_end);
    const int wsmin = wave_min_i(row_ok ? row_start : 0x7fffffff);
    const int wsmax = wave_max_i(row_start);
    if (lane == 0) {
        red[wave] = wmax;
        red_min[wave] = wmin;
        red_start[wave] = wsmin;
        red_smax[wave] = wsmax;
    }
    __syncthreads();
    const int e_max = max(red[0], red[1]);
    const int s_min = min(red_start[0], red_start[1]);
    // Keys [lo, hi) hold every key a row of the workgroup sees (whole tiles
    // from the first window start); the splits share them in equal runs of
    // whole tiles.
    const int lo = s_min == 0x7fffffff ? 0 : s_min / BN * BN;
    const int hi = min(si.kvl, e_max);
    const int run = hi > lo ? ((hi - lo + p.splits - 1) / p.splits + BN - 1) / BN * BN : 0;
    const int k_begin = lo + split * run;
    const int k_end = min(hi, k_begin + run);

    const float* kbase = (const float*)a.k + (int64_t)layer * a.k_stride[0] + (int64_t)kvh * a.k_stride[1] +
                         si.base * a.k_stride[2];
    const float* vbase = (const float*)a.v + (int64_t)layer * a.v_stride[0] + (int64_t)kvh * a.v_stride[1] +
                         si.base * a.v_stride[2];
    // Thread tid moves 16-byte pieces tid + 128 i of each tensor's tile.  K:
    // key (tid + 128 i) % 32, channels 4 ((tid + 128 i) / 32) .. +3 (consecutive
    // threads write consecutive words of the transposed tile); V: key
    // (tid + 128 i) / (D/4), channels 4 ((tid + 128 i) % (D/4)) .. +3.  Keys
    // past k_end load zeros (their scores are masked, and 0 * 0 adds nothing).
    f32x4 pk[NL], pv[NL];
    auto load_tile = [&](int t0) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int id = tid + i * (NW * 64);
            const int kk = id % BN, kc = id / BN, vk = id / (D / 4), vc = id % (D / 4);
            pk[i] = t0 + kk < k_end ? *(const f32x4*)(kbase + (int64_t)(t0 + kk) * a.k_stride[2] + kc * 4)
                                    : f32x4{0.f, 0.f, 0.f, 0.f};
            pv[i] = t0 + vk < k_end ? *(const f32x4*)(vbase + (int64_t)(t0 + vk) * a.v_stride[2] + vc * 4)
                                    : f32x4{0.f, 0.f, 0.f, 0.f};
        }
    };

    f32x16 o[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) o[db] = f32x16{};
    float m_run = -INFINITY, l_run = 0.f;   // running maximum (log2 units) and sum
    if (k_begin < k_end) load_tile(k_begin);
    for (int t0 = k_begin; t0 < k_end; t0 += BN) {
        __syncthreads();   // every wave is done with the previous tile
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int id = tid + i * (NW * 64);
            const int kk = id % BN, kc = id / BN, vk = id / (D / 4), vc = id % (D / 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) kt_lds[(kc * 4 + e) * BN + kk] = pk[i][e];
            *(f32x4*)(v_lds + vk * D + vc * 4) = pv[i];
        }
        __syncthreads();
        if (t0 + BN < k_end) load_tile(t0 + BN);

        // S^T = K Q^T: step s takes channels 2s (lanes 0-31) and 2s + 1 (lanes 32-63).
        f32x16 sc = f32x16{};
#pragma unroll
        for (int s = 0; s < KSF; ++s)
            sc = __builtin_amdgcn_mfma_f32_32x32x2f32(kt_lds[(2 * s + hl) * BN + j], qf[s], sc, 0, 0, 0);
        // Element r of the lane holds key t0 + 8 (r / 4) + 4 hl + r % 4 of row j.
        float mx = -INFINITY;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int key = t0 + (r >> 2) * 8 + hl * 4 + (r & 3);
            const float v = key < row_end && key >= row_start && key < k_end ? sc[r] * kLog2e : -INFINITY;
            sc[r] = v;
            mx = fmaxf(mx, v);
        }
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        // Branch-free (the MFMAs below run for the whole wave): a row that has
        // seen no visible key keeps o = 0 and l = 0 (alpha 0, probabilities 0).
        const float m_new = fmaxf(m_run, mx);
        const float alpha = m_run == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_run - m_new);
        float lsum = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float e = sc[r] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(sc[r] - m_new);
            sc[r] = e;
            lsum += e;
        }
        l_run = l_run * alpha + lsum;
        m_run = m_new;
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            o[db] *= alpha;
#pragma unroll
            for (int jj = 0; jj < 4; ++jj)
#pragma unroll
                for (int rr = 0; rr < 4; ++rr)
                    o[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(v_lds[(8 * jj + 4 * hl + rr) * D + db * 32 + j],
                                                                 sc[4 * jj + rr], o[db], 0, 0, 0);
        }
    }

    // The two halves of a row hold disjoint keys.
    const float l_tot = l_run + __shfl_xor(l_run, 32);
    if (!row_ok) return;
    const float inv = row_inverse(l_tot);
    const float lse2 = row_lse2(m_run, l_tot);
    const int64_t row = si.q0 + qi;
    // Element 4 jj + rr of block db holds channel 32 db + 8 jj + 4 hl + rr of the row.
    float* dst;
    if (p.splits == 1) {
        dst = (float*)a.out + (int64_t)layer * a.o_stride[0] + row * a.o_stride[1] + (int64_t)head * a.o_stride[2];
        if (a.lse_out && hl == 0)
            a.lse_out[((int64_t)layer * a.total_q + row) * a.n_heads + head] = lse2 * kLn2;
    } else {
        // split partial: normalised output and its log2-sum-exp (the combine's domain)
        const int64_t item = (((int64_t)split * a.n_layers + layer) * a.total_q + row) * a.n_heads + head;
        dst = a.ws_o + item * D;
        if (hl == 0) a.ws_lse[item] = lse2;
    }
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int jj = 0; jj < 4; ++jj)
            *(f32x4*)(dst + db * 32 + jj * 8 + hl * 4) =
                f32x4{o[db][4 * jj] * inv, o[db][4 * jj + 1] * inv, o[db][4 * jj + 2] * inv, o[db][4 * jj + 3] * inv};
}

// fp32 kernel for calls that do not fill the GPU: a workgroup covers 32 rows, its
// four waves hold the same rows and split the keys (wave w takes every fourth
// 32-key tile of the workgroup's run through its own LDS stages: no barrier in
// the loop) and are merged in LDS at the end.  Such a call is a chain of memory
// round trips and of one tile's 64 MFMAs after another, so the chain is what is
// cut: 16 queries over 528 keys, 2 KV heads: 16.8 us with two row waves of which
// one is idle and three tiles one after another, 10.2 us here.  Layout as above,
// except that a score step takes channel s from one half-wave and s + D/2 from
// the other, so a lane's query channels are contiguous; LDS rows are padded so
// that the two halves' reads fall into different banks.
template <int D>
__global__ __launch_bounds__(256) void attn_gqa_f32_keys(AttnArgs a, Plan p) {
    constexpr int BN = 32, NW = 4;
    constexpr int KSF = D / 2;              // score steps (2 channels each)
    constexpr int DB = D / 32;              // 32-channel output blocks
    constexpr int NL = BN * D / 4 / 64;     // 16-byte loads per lane per tensor and tile
    constexpr int KT = D * BN + 32;         // transposed K tile: [channel][key], the upper half 32 words on
    constexpr int VS = D + 8;               // V row stride
    constexpr int WAVE = KT + BN * VS;      // floats per wave
    constexpr int OC = D / 4;               // 16-byte chunks per output row
    static_assert(32 * D <= WAVE && KT % 4 == 0 && WAVE % 4 == 0, "a wave's O^T fits its stages");
    __shared__ __attribute__((aligned(16))) float lds[NW * WAVE];
    __shared__ float max_lds[NW][32], sum_lds[NW][32];

    int group, rb;
    if (!decode(p, group, rb)) return;
    const int split = group % p.splits;
    int rest = group / p.splits;
    const int kvh = rest % a.n_kv_heads;
    rest /= a.n_kv_heads;
    const int layer = rest % a.n_layers;
    const int seq = rest / a.n_layers;
    const SeqInfo si = seq_info(a, seq);
    const int M = si.nq * p.G;
    const int m0 = rb * 32;
    if (m0 >= M) return;

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int j = lane & 31;
    const int hl = lane >> 5;
    const int m = m0 + j;
    const bool row_ok = m < M;
    const int qi = row_ok ? m / p.G : 0;                       // rows past M repeat row 0 (never written)
    const int head = kvh * p.G + (row_ok ? m - qi * p.G : 0);
    const int pos = a.q_pos[si.q0 + qi];
    f32x4 q4[KSF / 4];   // channels hl D/2 .. of the lane's row
    {
        const float* qrow = (const float*)a.q + (int64_t)layer * a.q_stride[0] +
                            (int64_t)(si.q0 + qi) * a.q_stride[1] + (int64_t)head * a.q_stride[2] + hl * KSF;
#pragma unroll
        for (int i = 0; i < KSF / 4; ++i) q4[i] = *(const f32x4*)(qrow + i * 4);
    }
    int row_start, row_end;
    visible_range(row_ok ? pos : -1, si.kvl, a.window, row_start, row_end);   // (0, 0) for rows past M
    const int e_max = wave_max_u(row_end);
    const int s_min = wave_min_u(row_ok ? row_start : 0x7fffffff);
    const int lo = s_min == 0x7fffffff ? 0 : s_min / BN * BN;
    const int hi = min(si.kvl, e_max);
    const int run = hi > lo ? ((hi - lo + p.splits - 1) / p.splits + BN - 1) / BN * BN : 0;
    const int k_begin = lo + split * run;
    const int k_end = min(hi, k_begin + run);

    const float* kbase = (const float*)a.k + (int64_t)layer * a.k_stride[0] + (int64_t)kvh * a.k_stride[1] +
                         si.base * a.k_stride[2];
    const float* vbase = (const float*)a.v + (int64_t)layer * a.v_stride[0] + (int64_t)kvh * a.v_stride[1] +
                         si.base * a.v_stride[2];
    float* const kt = lds + wave * WAVE;
    float* const vt = kt + KT;
    // Piece id = lane + 64 i of a tile: K key id % 32, channels 4 (id / 32) .. +3;
    // V key id / (D/4), channels 4 (id % (D/4)) .. +3.  Keys past k_end load zeros.
    f32x4 pk[NL], pv[NL];
    auto load_tile = [&](int t0) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int id = lane + i * 64;
            const int kk = id % BN, kc = id / BN, vk = id / (D / 4), vc = id % (D / 4);
            pk[i] = t0 + kk < k_end ? *(const f32x4*)(kbase + (int64_t)(t0 + kk) * a.k_stride[2] + kc * 4)
                                    : f32x4{0.f, 0.f, 0.f, 0.f};
            pv[i] = t0 + vk < k_end ? *(const f32x4*)(vbase + (int64_t)(t0 + vk) * a.v_stride[2] + vc * 4)
                                    : f32x4{0.f, 0.f, 0.f, 0.f};
        }
    };

    // A wave executes its LDS accesses in order; the compiler, which sees one
    // lane at a time, must not move one lane's reads over another's writes.
    auto wave_fence = []() __attribute__((always_inline)) {
        __builtin_amdgcn_wave_barrier();
        asm volatile("" ::: "memory");
    };

    f32x16 o[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) o[db] = f32x16{};
    float m_run = -INFINITY, l_run = 0.f;   // running maximum (log2 units) and sum
    const int first = k_begin + wave * BN;
    if (first < k_end) load_tile(first);
#pragma unroll 1
    for (int t0 = first; t0 < k_end; t0 += NW * BN) {
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int id = lane + i * 64;
            const int kk = id % BN, kc = id / BN, vk = id / (D / 4), vc = id % (D / 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) kt[(kc * 4 + e) * BN + (kc * 4 >= KSF ? 32 : 0) + kk] = pk[i][e];
            *(f32x4*)(vt + vk * VS + vc * 4) = pv[i];
        }
        wave_fence();
        if (t0 + NW * BN < k_end) load_tile(t0 + NW * BN);
        f32x16 sc = f32x16{};
#pragma unroll
        for (int s = 0; s < KSF; ++s)
            sc = __builtin_amdgcn_mfma_f32_32x32x2f32(kt[(s + hl * KSF) * BN + hl * 32 + j], q4[s / 4][s % 4] * a.scale,
                                                      sc, 0, 0, 0);
        // Element r of the lane holds key t0 + 8 (r / 4) + 4 hl + r % 4 of row j.
        float mx = -INFINITY;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int key = t0 + (r >> 2) * 8 + hl * 4 + (r & 3);
            if (!(key < row_end && key >= row_start && key < k_end)) sc[r] = -INFINITY;
            mx = fmaxf(mx, sc[r]);
        }
        const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
        mx = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1])) * kLog2e;
        // Branch-free: a row that has seen no visible key keeps o = 0 and l = 0.
        const float m_new = fmaxf(m_run, mx);
        const float alpha = m_run == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_run - m_new);
        float lsum = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            // (one rounding of the exponent: the product is not rounded by itself)
            const float e = sc[r] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(fmaf(sc[r], kLog2e, -m_new));
            sc[r] = e;
            lsum += e;
        }
        l_run = l_run * alpha + lsum;
        m_run = m_new;
#pragma unroll
        for (int db = 0; db < DB; ++db) o[db] *= alpha;
#pragma unroll
        for (int jj = 0; jj < 4; ++jj)
#pragma unroll
            for (int rr = 0; rr < 4; ++rr)
#pragma unroll
                for (int db = 0; db < DB; ++db)
                    o[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(vt[(8 * jj + 4 * hl + rr) * VS + db * 32 + j],
                                                                 sc[4 * jj + rr], o[db], 0, 0, 0);
        wave_fence();
    }

    // Merge the waves: O row-major in each wave's own stages, 16-byte chunks
    // XOR-swizzled by row.  Element 4 jj + rr of block db is channel 32 db + 8 jj + 4 hl + rr.
    const float l_tot = l_run + __shfl_xor(l_run, 32);
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int jj = 0; jj < 4; ++jj)
            *(f32x4*)(kt + j * D + ((db * 8 + jj * 2 + hl) ^ (j & (OC - 1))) * 4) =
                f32x4{o[db][4 * jj], o[db][4 * jj + 1], o[db][4 * jj + 2], o[db][4 * jj + 3]};
    if (hl == 0) {
        max_lds[wave][j] = m_run;
        sum_lds[wave][j] = l_tot;
    }
    __syncthreads();
    const int c = tid % OC;
#pragma unroll
    for (int r = tid / OC; r < 32; r += 256 / OC) {
        if (m0 + r >= M) break;
        float mw[NW], top = -INFINITY, sum = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            mw[w] = max_lds[w][r];
            top = fmaxf(top, mw[w]);
        }
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float wt = mw[w] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mw[w] - top);
            acc += wt * *(const f32x4*)(lds + w * WAVE + r * D + (c ^ (r & (OC - 1))) * 4);
            sum += wt * sum_lds[w][r];
        }
        const float inv = row_inverse(sum);
        const float lse2 = row_lse2(top, sum);
        const int q = (m0 + r) / p.G;
        const int hd = kvh * p.G + m0 + r - q * p.G;
        const int64_t row = si.q0 + q;
        if (p.splits == 1) {
            *(f32x4*)((float*)a.out + (int64_t)layer * a.o_stride[0] + row * a.o_stride[1] +
                      (int64_t)hd * a.o_stride[2] + c * 4) = acc * inv;
            if (a.lse_out && c == 0)
                a.lse_out[((int64_t)layer * a.total_q + row) * a.n_heads + hd] = lse2 * kLn2;
        } else {
            const int64_t item = (((int64_t)split * a.n_layers + layer) * a.total_q + row) * a.n_heads + hd;
            *(f32x4*)(a.ws_o + item * D + c * 4) = acc * inv;
            if (c == 0) a.ws_lse[item] = lse2;
        }
    }
}

// Merge split-KV partials: out = sum_s w_s O_s / sum_s w_s with
// w_s = 2^(lse_s - max lse).  Grid (row tiles, sequences from seq0, layers).
// With few rows the pass is latency-bound: the split partials of one row are
// dealt to SG groups of threads, one 16-byte chunk of the row per thread, so that
// a thread loads few records and the whole GPU takes part; the groups are merged
// in LDS.  With many rows (SG 1) it is bound by the stream of partials and a
// thread takes two chunks.  Rows that no sequence owns (outside every cu_q range) are
// left untouched, as the one-pass kernels leave them.  COLUMNS: the partials of
// the few-row kernels, which write a varying number of records per row (the
// rest have log-sum-exp -inf and are not read) and mark rows that need no merge.
template <int SG, bool COLUMNS>
__global__ __launch_bounds__(256) void attn_combine(AttnArgs a, int seq0) {
    constexpr int CB = SG == 1 ? 8 : 4;   // records loaded in one batch
    constexpr int CV = SG == 1 ? 2 : 1;   // 16-byte chunks per thread
    __shared__ f32x4 acc_lds[SG > 1 ? 256 : 1];
    __shared__ float max_lds[SG > 1 ? 256 : 1], sum_lds[SG > 1 ? 256 : 1];
    const int dv = a.head_dim_v;
    const int64_t items = (int64_t)a.n_layers * a.total_q * a.n_heads;   // partial records per split
    const uint32_t chunks = (uint32_t)dv / (4 * CV);                    // threads per (query, head) and group
    const uint32_t per_block = 256u / (chunks * SG);                    // rows per block
    const uint32_t t = threadIdx.x;
    const uint32_t rl = t / (chunks * SG);
    const uint32_t rest = t - rl * (chunks * SG);
    const uint32_t sg = rest / chunks;
    const int c0 = (int)(rest - sg * chunks) * CV;
    const uint32_t rh = blockIdx.x * per_block + rl;
    const uint32_t qi = rh / (uint32_t)a.n_heads;
    const int head = (int)(rh - qi * (uint32_t)a.n_heads);
    const int seq = seq0 + (int)blockIdx.y;
    const int layer = (int)blockIdx.z;
    int q0 = 0, nq = a.total_q;
    if (a.cu_q) {
        q0 = a.cu_q[seq];
        nq = a.cu_q[seq + 1] - q0;
    }
    if (q0 < 0 || nq < 0 || (int64_t)q0 + nq > a.total_q) nq = 0;   // as seq_info
    const bool mine = rl < per_block && qi < (uint32_t)a.max_q && (int)qi < nq;
    const int64_t row = q0 + (int)qi;
    const int64_t item = mine ? ((int64_t)layer * a.total_q + row) * a.n_heads + head : 0;
    // Records sg, sg + SG, ..: CB at a time, loaded in one batch (one memory
    // round trip), weighted by w_s = 2^(lse_s - max) and summed in order; a
    // later batch rescales the sums to its larger maximum.
    const int ns = a.n_splits;
    float mx = -INFINITY, wsum = 0.f;
    f32x4 acc[CV];
#pragma unroll
    for (int k = 0; k < CV; ++k) acc[k] = f32x4{0.f, 0.f, 0.f, 0.f};
    const float first_lse = COLUMNS && mine ? a.ws_lse[item] : 0.f;
    if (mine) {
        for (int s0 = (int)sg; s0 < ns; s0 += SG * CB) {
            float l[CB];
            f32x4 v[CB][CV];
            auto load_part = [&](int j, bool in) __attribute__((always_inline)) {
                const float* src = a.ws_o + ((int64_t)(s0 + j * SG) * items + item) * dv + c0 * 4;
#pragma unroll
                for (int k = 0; k < CV; ++k) v[j][k] = in ? *(const f32x4*)(src + k * 4) : f32x4{0.f, 0.f, 0.f, 0.f};
            };
#pragma unroll
            for (int j = 0; j < CB; ++j) {
                const bool in = s0 + j * SG < ns;
                l[j] = in ? a.ws_lse[(int64_t)(s0 + j * SG) * items + item] : -INFINITY;
                if (!COLUMNS) load_part(j, in);
            }
            if (COLUMNS && first_lse == INFINITY) break;   // the few-row kernel wrote the row itself
            if (COLUMNS) {
#pragma unroll
                for (int j = 0; j < CB; ++j) load_part(j, l[j] != -INFINITY);
            }
            // (fmaxf passes over a NaN: a batch whose only records are NaN has bm -inf)
            float bm = l[0];
            bool any = l[0] != -INFINITY;
#pragma unroll
            for (int j = 1; j < CB; ++j) {
                bm = fmaxf(bm, l[j]);
                any |= l[j] != -INFINITY;
            }
            if (!any) continue;
            if (bm > mx) {
                if (mx != -INFINITY) {
                    const float r = __builtin_amdgcn_exp2f(mx - bm);
#pragma unroll
                    for (int k = 0; k < CV; ++k) acc[k] *= r;
                    wsum *= r;
                }
                mx = bm;
            }
#pragma unroll
            for (int j = 0; j < CB; ++j) {
                if (l[j] == -INFINITY) continue;
                const float w = __builtin_amdgcn_exp2f(l[j] - mx);
#pragma unroll
                for (int k = 0; k < CV; ++k) acc[k] += w * v[j][k];
                wsum += w;
            }
        }
    }
    if constexpr (SG > 1) {
        acc_lds[t] = acc[0];
        max_lds[t] = mx;
        sum_lds[t] = wsum;
        __syncthreads();
        if (sg != 0) return;
        for (int k = 1; k < SG; ++k) {
            const float m2 = max_lds[t + k * chunks], sum2 = sum_lds[t + k * chunks];
            if (sum2 == 0.f) continue;   // no record (NaN records have a NaN sum and a maximum of -inf)
            const float m_new = fmaxf(mx, m2);
            const float r1 = mx == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mx - m_new);
            const float r2 = __builtin_amdgcn_exp2f(m2 - m_new);
            acc[0] = acc[0] * r1 + acc_lds[t + k * chunks] * r2;
            wsum = wsum * r1 + sum2 * r2;
            mx = m_new;
        }
    }
    if (!mine || (COLUMNS && first_lse == INFINITY)) return;
    const float inv = row_inverse(wsum);
    const int64_t oofs = (int64_t)layer * a.o_stride[0] + row * a.o_stride[1] + (int64_t)head * a.o_stride[2] + c0 * 4;
#pragma unroll
    for (int k = 0; k < CV; ++k) {
        if (a.dtype == 1) {
            *(f32x4*)((float*)a.out + oofs + k * 4) =
                f32x4{acc[k][0] * inv, acc[k][1] * inv, acc[k][2] * inv, acc[k][3] * inv};
        } else {
            u32x2 w;
            w[0] = bf_rne(acc[k][0] * inv) | (bf_rne(acc[k][1] * inv) << 16);
            w[1] = bf_rne(acc[k][2] * inv) | (bf_rne(acc[k][3] * inv) << 16);
            *(u32x2*)((uint16_t*)a.out + oofs + k * 4) = w;
        }
    }
    if (a.lse_out && c0 == 0)
        a.lse_out[item] = row_lse2(mx, wsum) * kLn2;
}

// rows: rows per workgroup, 0 for the dtype's usual count.
Plan make_plan(const AttnArgs& a, int splits, int rows = 0) {
    Plan p;
    p.G = a.n_heads / a.n_kv_heads;
    const int64_t m_rows = (int64_t)a.max_q * p.G;
    if (a.variant == 1) {
        // MLA: four waves of 32 whole rows; 32-key tiles in 2 LDS stages.
        p.qb = 1;
        p.nw = 4;
        p.ns = 2;
    } else {
        // bf16 GQA: 4 waves x 32 rows, two workgroups per CU, pipelined over
        // 32-key tiles in 4 LDS stages.  (The fp32 kernel also uses 32-key
        // tiles.)
        p.qb = 1;
        p.nw = 4;
        p.ns = 4;
    }
    p.BM = rows ? rows : a.dtype == 1 ? 64 : p.nw * 32 * p.qb;
    p.rbs = (int)((m_rows + p.BM - 1) / p.BM);
    if (p.rbs < 1) p.rbs = 1;
    p.splits = splits;
    p.n_groups = a.n_layers * a.n_kv_heads * a.n_seqs * splits;
    p.longest_first = 0;
    // Row blocks on the fullest XCD when a group is shared by 1, 2, 4 or 8 XCDs;
    // one XCD (every K/V byte through one L2) unless sharing fills them better:
    // 4 groups of 64 row blocks on four XCDs 1543 us, shared by two each 790 us.
    int64_t best = INT64_MAX / 20;
    for (int sh = 1; sh <= kXcds; sh *= 2) {
        const int rbs = (p.rbs + sh - 1) / sh;
        const int64_t load = ((int64_t)p.n_groups * sh + kXcds - 1) / kXcds * rbs;
        if (load * 20 < best * 19) {
            best = load;
            p.shares = sh;
            p.share_rbs = rbs;
        }
    }
    return p;
}

// Workgroups that fit on one CU at once (LDS and register bound).
int wgs_per_cu(const AttnArgs& a, const Plan& p) {
    if (a.variant == 1) return 1;                     // MLA: two 36 KB stages, one wave per SIMD
    const int tile = 32;                              // keys per K/V tile
    const int lds = p.ns * 2 * tile * a.head_dim * 2;
    const int n = (160 * 1024) / lds;
    return n < 1 ? 1 : (n > 2 ? 2 : n);               // two waves per SIMD at most (registers)
}

// Keys one workgroup's rows see at most: with a sliding window, about the window
// plus the span of the queries (contiguous suffix positions).
int64_t seen_keys(const AttnArgs& a) {
    return a.window > 0 && (int64_t)a.window + a.max_q < a.max_kv_len ? (int64_t)a.window + a.max_q : a.max_kv_len;
}

// Dispatching the longest sequences first costs every workgroup a dependent load
// and a selection, about 1 us: worth it where a workgroup runs much longer.
bool order_pays(const AttnArgs& a) { return a.n_seqs > 1 && a.n_seqs <= 64 && seen_keys(a) >= 2048; }

// ---- few query rows (attn_columns.h) -----------------------------------------

// Rows (queries x heads per KV head) of one sequence up to which the few-row
// kernels run: one row block.  Above it the many-row kernels are faster, since
// they stage a tile once for 128 rows (GQA, 64 queries x 4 heads over 8256 keys:
// 44 us with 32-row blocks, 27.5 us with 128-row ones; MLA, 16 sequences of 32
// rows over 16384 keys: 95 us with two 16-row blocks, 74 us).
constexpr int kRowsGqa = 32;
constexpr int kRowsMla = 16;

int64_t col_items(const AttnArgs& a) { return (int64_t)a.n_layers * a.n_kv_heads * a.n_seqs; }

// Whole items, one workgroup each: many items (the last round is a small part of
// the call), or short ones, where one launch without a merge is faster (4 sequences;
// whole / cut / many-row kernel: GQA, 8 KV heads of 128, 768 keys 13.1 / 13.3 / 21.5
// us, 1024 keys 15.7 / 13.3 / 18.9; of 64, 768 keys 10.2 / 12.0 / 17.7, 1024 keys
// 11.7 / 12.1 / 16.4; MLA, 16 heads, 512 keys 21.8 / 23.6 / 33.8, 768 keys 27.3 /
// 24.4 / 46.0; 64 MLA sequences of which one has 512 keys, the others 32: 21.6 / 18.8,
// so several are cut a little earlier than one).  Head size 64 has two workgroups a
// CU, but columns use one: whole items up to twice the length when they outnumber
// the slots.
bool col_whole(const AttnArgs& a) {
    const int64_t items = col_items(a);
    const int64_t cut = a.variant == 1       ? (a.n_seqs == 1 ? 640 : 512)
                        : a.head_dim == 128  ? 832
                        : items > 2 * kCUs   ? 2048
                                             : 1024;
    return items >= 8 * kCUs || seen_keys(a) < cut;
}

// Starting an item costs the few-row kernels more than the many-row ones, the more
// so the more rows it merges, and outside head size 64 their tiles leave one
// workgroup a CU, where the many-row GQA kernel has two.  So short caches stay with
// the many-row kernels: two tiles of keys for more than 8 rows (64 keys, 32 rows, 8
// KV heads of 128: 7.7 us against 8.7; 4 rows: 7.1 against 7.0), and, with more items
// than CUs (head size 64: than two a CU), until the stream of keys outweighs the
// rounds (64 sequences, 8 KV heads of 128: all of 512 keys 28.9 us against 31.3, all
// of 1024 keys 49.5 against 50.4, up to 1024 keys 39.5 against 35.9).
bool col_long_enough(const AttnArgs& a, int64_t rows) {
    const int64_t kv = seen_keys(a), items = col_items(a);
    if (a.head_dim != 64 && rows > 8 && kv <= 2 * kColTile) return false;
    if (a.variant == 1 || items <= kCUs) return true;
    if (a.head_dim == 64) return items <= 2 * kCUs || kv >= 512;
    return kv >= (items >= 8 * kCUs ? 2048 : 1024);
}

bool col_route(const AttnArgs& a) {
    if (!a.auto_splits || a.dtype != 0 || a.n_seqs > kColMaxSeqs) return false;
    const int64_t rows = (int64_t)a.max_q * (a.n_heads / a.n_kv_heads);
    if (rows < 1 || rows > (a.variant == 1 ? kRowsMla : kRowsGqa) || !col_long_enough(a, rows))
        return false;
    // axis positions and workgroup ids are 32-bit
    return col_items(a) * ((int64_t)a.max_kv_len / kColTile + 16) < 0x7fffffff;
}

}  // namespace

int attention_splits(const AttnArgs& a) {
    if (a.n_splits == 0 && col_route(a)) {
        // Columns have records for twice the pieces that sequences of one length
        // would be cut into (a sequence longer than that makes the columns longer).
        if (col_whole(a)) return 1;
        const int64_t items = col_items(a);
        return (int)std::min<int64_t>(32, 2 * ((kCUs + items - 1) / items) + 2);
    }
    if (a.n_splits > 0) {
        int s = a.n_splits;
        const int max_s = (a.max_kv_len + 63) / 64;
        if (s > max_s) s = max_s < 1 ? 1 : max_s;
        return s;
    }
    // Pick the split count that minimises the estimated time: the workgroup
    // rounds over the CUs times the duration of one workgroup (a fixed cost
    // for its start-up, first loads and partial write, plus 1/s of the keys),
    // plus, for s > 1, the split partials written and read back by the
    // combine pass.  Nominal rates (measured on MI355X): the bf16 kernels
    // sustain about 1.0 PFLOP/s (GQA) and 1.1 PFLOP/s (MLA), a workgroup's
    // fixed cost is about 20 us, the combine streams at about 5 TB/s.  At
    // least 512 keys per split, at most 32 splits.
    const Plan p = make_plan(a, 1);
    const int64_t wgs = (int64_t)p.n_groups * p.rbs;   // workgroups per split
    const int64_t kv = seen_keys(a);
    if (a.dtype == 1) {
        // fp32 path (small problems): one workgroup per CU, at least 64 keys
        // per split, at most 32 splits.
        int64_t s = (kCUs + wgs - 1) / wgs;
        const int64_t max_s = kv / 64;
        if (s > max_s) s = max_s;
        if (s > 32) s = 32;
        return s < 1 ? 1 : (int)s;
    }
    const int64_t slots = kCUs * (int64_t)wgs_per_cu(a, p);
    const double rate = a.variant == 1 ? 1.1e15 : 1.0e15;
    const double slot_rate = rate / (double)slots;
    const double wg_flops = (double)p.BM * kv * (a.head_dim + a.head_dim_v) * 2.0;
    const double comb_bytes = (double)a.n_layers * a.total_q * a.n_heads * (a.head_dim_v + 1) * 4.0 * 2.0;
    int best = 1;
    double best_t = 1e30;
    for (int s = 1; s <= 32; ++s) {
        if (s > 1 && kv / s < 512) break;
        const double rounds = (double)((wgs * s + slots - 1) / slots);
        const double t = rounds * (20e-6 + (wg_flops / s) / slot_rate) + (s > 1 ? s * comb_bytes / 5e12 + 5e-6 : 0.0);
        if (t < best_t * (1.0 - 1e-9)) {
            best_t = t;
            best = s;
        }
    }
    return best;
}

size_t attention_workspace_bytes(const AttnArgs& a, int n_splits) {
    if (n_splits <= 1) return 0;
    const size_t rows = (size_t)n_splits * a.n_layers * a.total_q * a.n_heads;
    return rows * a.head_dim_v * sizeof(float) + rows * sizeof(float);
}

namespace {

template <int SG, bool COLUMNS>
hipError_t launch_combine_groups(const AttnArgs& a, hipStream_t stream) {
    const int per_block = 256 / (a.head_dim_v / (SG == 1 ? 8 : 4) * SG);
    const int64_t blocks = ((int64_t)a.max_q * a.n_heads + per_block - 1) / per_block;
    if (blocks > 0x7fffffff || a.n_layers > 65535) return hipErrorInvalidValue;
    // One (row tiles, sequences, layers) grid per 65535 sequences.
    for (int seq0 = 0; seq0 < a.n_seqs; seq0 += 65535) {
        const int nseq = a.n_seqs - seq0 < 65535 ? a.n_seqs - seq0 : 65535;
        hipLaunchKernelGGL((attn_combine<SG, COLUMNS>), dim3((unsigned)blocks, (unsigned)nseq, (unsigned)a.n_layers),
                           dim3(256), 0, stream, a, seq0);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Split groups per row: one while the rows alone give four blocks a CU (the MLA
// layer: 2048 rows of 512 channels, 16 splits, 13 us), more below that (one 8B
// layer: 2048 rows of 128 channels, 16 splits, 6.2 us with one group, 5.7 us
// with four), within a block of 256 threads.
hipError_t launch_combine(const AttnArgs& a, bool columns, hipStream_t stream) {
    if (a.max_q == 0 || a.n_layers == 0 || a.n_seqs == 0) return hipSuccess;
    const int chunks = a.head_dim_v / 4;
    if (a.head_dim_v % 4 || chunks > 256 || 256 % chunks) return hipErrorInvalidValue;
    const int64_t threads = (int64_t)a.max_q * a.n_heads * a.n_layers * a.n_seqs * chunks;
    int sg = 1;
    while (sg < 4 && threads * sg < 4 * 256 * (int64_t)kCUs && sg * 4 < a.n_splits && sg * 2 * chunks <= 256) sg *= 2;
    if (columns)
        return sg == 1   ? launch_combine_groups<1, true>(a, stream)
               : sg == 2 ? launch_combine_groups<2, true>(a, stream)
                         : launch_combine_groups<4, true>(a, stream);
    return sg == 1   ? launch_combine_groups<1, false>(a, stream)
           : sg == 2 ? launch_combine_groups<2, false>(a, stream)
                     : launch_combine_groups<4, false>(a, stream);
}

hipError_t launch_columns(const AttnArgs& a, hipStream_t stream) {
    ColPlan p;
    p.G = a.n_heads / a.n_kv_heads;
    p.streams = a.n_layers * a.n_kv_heads;
    p.pieces = a.n_splits;
    // One workgroup per CU: its tiles fill the LDS, except at head size 64, where a
    // second one would fit.
    p.columns = p.pieces > 1 ? kCUs : 0;
    // Measured costs of a column's shortest useful run and of starting an item
    // (set-up, first loads and merge: about 7 us), in tiles of one workgroup at head
    // size 128; the tiles of head size 64 take half as long, with the same counts.
    p.min_tiles = a.variant == 1 ? 4 : 8;
    p.item_cost = a.variant == 1 ? 4 : 12;
    const int64_t cols = p.columns ? p.columns : (col_items(a) + kXcds - 1) / kXcds * kXcds;
    if (cols > 0x7fffffff) return hipErrorInvalidValue;
    const dim3 grid((unsigned)cols);
    const hipError_t e = a.variant == 1 ? launch_attn_mla_rows(a, p, grid, stream)
                                        : launch_attn_gqa_rows(a, p, grid, stream);
    if (e != hipSuccess || p.columns == 0) return e;
    return launch_combine(a, true, stream);
}

}  // namespace

hipError_t launch_attention(const AttnArgs& a, hipStream_t stream) {
    if (col_route(a)) return launch_columns(a, stream);
    Plan p = make_plan(a, a.n_splits < 1 ? 1 : a.n_splits);
    // fp32 calls of at most one workgroup of 32 rows per CU split the keys over
    // its waves.
    const bool keys = a.dtype == 1 && (int64_t)p.n_groups * (((int64_t)a.max_q * p.G + 31) / 32) <= kCUs;
    if (keys) p = make_plan(a, p.splits, 32);
    const int64_t n_wg = ((int64_t)p.n_groups * p.shares + kXcds - 1) / kXcds * kXcds * p.share_rbs;
    if (n_wg <= 0) return hipSuccess;
    if (n_wg > 0x7fffffff) return hipErrorInvalidValue;
    // More workgroups than the CUs hold at once (bf16 GQA): the order matters.
    p.longest_first = a.dtype == 0 && a.variant == 0 && n_wg > kCUs * (int64_t)wgs_per_cu(a, p) && order_pays(a);
    dim3 grid((unsigned)n_wg);
    hipError_t e;
    if (keys) {
        if (a.head_dim == 64)
            hipLaunchKernelGGL((attn_gqa_f32_keys<64>), grid, dim3(256), 0, stream, a, p);
        else
            hipLaunchKernelGGL((attn_gqa_f32_keys<128>), grid, dim3(256), 0, stream, a, p);
        e = hipGetLastError();
    } else if (a.dtype == 1) {
        if (a.head_dim == 64)
            hipLaunchKernelGGL((attn_gqa_f32<64>), grid, dim3(128), 0, stream, a, p);
        else
            hipLaunchKernelGGL((attn_gqa_f32<128>), grid, dim3(128), 0, stream, a, p);
        e = hipGetLastError();
    } else {
        e = a.variant == 1 ? launch_attn_mla_bf16(a, p, grid, stream) : launch_attn_gqa_bf16(a, p, grid, stream);
    }
    if (e != hipSuccess || p.splits == 1) return e;
    return launch_combine(a, false, stream);
}

}  // namespace pkv
