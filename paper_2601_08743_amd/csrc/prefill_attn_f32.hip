// Suffix prefill attention, fp32 storage and fp32 arithmetic (no reduced-precision operands).
// App. E.4 of the paper: the suffix rows attend to all stitched schema keys, and causally to
// the suffix itself.
//
// Bound: the fp32 matrix rate (v_mfma_f32_32x32x2_f32, 64 cycles for 4096 operations: 157 TFLOP/s on
// the chip, twice what v_fma_f32 reaches).  A work-group is 32 rows (row = token * G + head in the
// group) of one (query, KV head) against a key range; its four waves split the KEYS: wave w takes the
// 32-key units w, w + 4, ... of the range, streams each straight into its own LDS area (nobody else
// reads it, so the loop has no barrier), and keeps its own running maximum, sum and output; the four
// are combined through LDS at the end.  Splitting keys rather than rows keeps the row tile small - a
// suffix of a few tokens fills it, and ragged lengths waste little - and costs only L2 reads, of which
// this rate needs 16 bytes a cycle and CU.
//
// Operand layouts.  S^T = K . Q^T: the order of the depth index is free as long as both operands agree,
// so lane half hh holds elements hh * D/2 .. of its row, and four instructions' worth of K is one
// 16-byte LDS read.  A lane then holds 16 scores of ONE row, and score e is directly the B operand of
// O^T += V^T . P^T for the key pair that its two lane halves stand for; V is read from its token rows
// D/32 neighbouring columns at a time.
//
// A query in several ranges: the last of a row tile's ranges to end combines their partials (arrive.h), or a launch of its own does
// where one CU would take longer: heads of 128, whose partials are twice as large, and more than eight ranges (two round
// trips).  Us a layer, in one launch and in two: one query of 1.6 k + 64 tokens, 8 / 2 heads of 64, 4 ranges 18.4 and 19.5, 8 13.9
// and 13.9, 16 13.7 and 12.6; of 128, 4 32.1 and 31.9, 8 23.8 and 22.2, 16 22.7 and 19.1.
//
// Measured (8 queries, 23 k prefix and 1.4 k suffix tokens, 8 query / 2 KV heads of 64: 8.3 GFLOP): 109 us a layer with
// the ranges combined (110 with a launch of its own for that: 102 + 4.5 us and the gap between them); one wave per row
// with v_fma_f32, keys from LDS one float at a time, values straight from the pool, took 1049 us.  A batch long enough
// to drown its edges runs at 112 TFLOP/s (a 4096^3 library product: 140).  A whole pass over one query of 731 + 64 tokens:
// 30.5 us with two launches, 29.1 with one.
#include "arrive.h"
#include "kv_append.h"
#include "lds_dma.h"
#include "tc_internal.h"

namespace tc {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kF32Unit = 32;                                       // keys per unit

template <int D>
struct F32Lds {
    static constexpr int kPart = kF32Unit * D * 4;                 // K (or V) of one unit
    static constexpr int kWave = 2 * kPart;
    static constexpr int kBid = 4 * kWave;                         // block ids behind the four waves' areas
    static constexpr int kBytes = kBid + kF32MaxTiles * (kF32Keys / kBlockTokens) * 4 + 256;   // + alignment slack
    static constexpr int kRow = D + 4;                             // padded row of the final exchange (floats)
};

// kLong: some range of the batch has more key tiles than the table in LDS has block ids for; the planner makes such
// ranges only for a workspace that has no room for the partials of shorter ones.
// kFold: the last work-group of a row tile combines its ranges' partials; else they are left to a merge launch.
template <int D, bool kLong, bool kFold>
__global__ __launch_bounds__(256, D == 64 ? 2 : 1) void attn_f32_kernel(Geom g, BatchDev b, AttnArgs a)
{
    typedef F32Lds<D> L;
    constexpr int kPieces = L::kPart / 1024;     // load instructions per operand and unit
    constexpr int kChunks = D / 4;               // 16-byte chunks of a row
    constexpr int kRowsPer = 64 / kChunks;       // rows per load instruction
    constexpr int kCols = D / 32;                // neighbouring output columns per lane
    extern __shared__ __attribute__((aligned(16))) char lds_raw[];
    if ((int)blockIdx.x >= a.n_items) {          // extra work-groups: append the suffix to the pool
        append_unit<false, kF32AppendTokens>(g, b, a.layer, (const char *)a.k_new, (const char *)a.v_new, blockIdx.x - a.n_items, threadIdx.x);
        return;
    }
    const AttnItem it = load_item(a, blockIdx.x);
    if (it.q < 0) return;                        // padding item (uniform for the work-group)
    // the XOR addressing of the K rows needs them 256-byte aligned
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds_raw;
    const uint32_t slack = (256u - (lds_base & 255u)) & 255u;
    char *lds = lds_raw + slack;
    const uint32_t lds0 = lds_base + slack;
    int32_t *s_bid = (int32_t *)(lds + L::kBid);

    const int tid = threadIdx.x, lane = tid & 63, r32 = lane & 31, hh = lane >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int P = it.P, S = it.S, G = g.G;
    const int n_rows = S * G;
    const int m = min(it.m0 + r32, n_rows - 1);  // rows behind the last one repeat it and are dropped
    const int s_tok = m / G;
    const int64_t row = (int64_t)(it.cu + s_tok) * g.Hq + it.kvh * G + (m - s_tok * G);
    const int limit = P + s_tok;                 // last key this row sees
    const int u_begin = it.tile_begin * (kF32Keys / kF32Unit);
    // units behind the last key that any row of the tile sees are left out
    const int last_key = P + (min(it.m0 + kF32Rows, n_rows) - 1) / G;
    const int u_end = min(it.tile_end * (kF32Keys / kF32Unit), last_key / kF32Unit + 1);

    // block ids of the range's prefix part, as many as the table in LDS holds
    constexpr int kIds = kF32MaxTiles * (kF32Keys / kBlockTokens);
    const int blk0 = it.tile_begin * (kF32Keys / kBlockTokens);
    const int32_t *bt = b.block_table + (int64_t)it.q * b.max_blocks + blk0;
    {
        const int n_pblk = (P + kBlockTokens - 1) >> 4;
        const int n_range = min(it.tile_end * (kF32Keys / kBlockTokens), n_pblk) - blk0, n = kLong ? min(n_range, kIds) : n_range;
        for (int idx = tid; idx < n; idx += 256) s_bid[idx] = bt[idx];
    }
    // block `idx` of the range, the same for the whole wave (by a scalar load where LDS does not have it: a vector
    // load would have to wait for the tile loads in flight)
    typedef const __attribute__((address_space(4))) int32_t *const_ints;
    auto block_id = [&](int idx) {
        return !kLong || idx < kIds ? __builtin_amdgcn_readfirstlane(s_bid[idx]) : ((const_ints)(uintptr_t)bt)[idx];
    };
    // Q^T fragments (B operand): lane (row r32, half hh) holds q[row][hh * D/2 ..]
    float qf[D / 2];
    {
        const f32x4 *qp = (const f32x4 *)((const float *)a.q + row * D + hh * (D / 2));
#pragma unroll
        for (int j = 0; j < D / 8; ++j) {
            const f32x4 v = qp[j];
#pragma unroll
            for (int e = 0; e < 4; ++e) qf[4 * j + e] = v[e];
        }
    }
    // (used once here, so that the compiler's wait for these loads stands in front of the loop, not in it,
    // where it would drain the loads of the next unit as well)
#pragma unroll
    for (int j = 0; j < D / 2; ++j) asm volatile("" : "+v"(qf[j]));
    __syncthreads();                             // block ids visible

    const char *pool_l = g.pool + (int64_t)a.layer * g.layer_stride + (int64_t)it.kvh * kBlockTokens * D * 4;
    const int64_t v_half = g.block_bytes >> 1;
    const char *new_k = (const char *)a.k_new + ((int64_t)it.cu * g.Hkv + it.kvh) * D * 4;
    const char *new_v = (const char *)a.v_new + ((int64_t)it.cu * g.Hkv + it.kvh) * D * 4;
    const uint32_t lds_w = lds0 + w * L::kWave;
    const int l_row = lane / kChunks, l_chunk = lane % kChunks;

    // One operand of one unit -> LDS rows of D floats; of K, chunk c of row r lands at position
    // c ^ (r & 15), so that 16 lanes reading one chunk of 16 rows touch all banks.
    auto issue = [&](int u, bool is_v) {
        const uint32_t dst = lds_w + (is_v ? L::kPart : 0);
        const int key0 = u * kF32Unit;
        if (key0 + kF32Unit <= P) {              // two whole blocks of the pool
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const char *src = pool_l + (int64_t)block_id(2 * u + j - blk0) * g.block_bytes + (is_v ? v_half : 0);
#pragma unroll
                for (int i = 0; i < kPieces / 2; ++i) {
                    const int r = i * kRowsPer + l_row;
                    load_to_lds(dst + (j * (kPieces / 2) + i) * 1024, src, (r * kChunks + (is_v ? l_chunk : l_chunk ^ (r & 15))) * 16);
                }
            }
        } else {                                 // the end of the prefix and / or suffix tokens
            const int id0 = key0 < P ? block_id(2 * u - blk0) : 0, id1 = key0 + kBlockTokens < P ? block_id(2 * u + 1 - blk0) : 0;
#pragma unroll
            for (int i = 0; i < kPieces; ++i) {
                const int r = i * kRowsPer + l_row;
                const int key = key0 + r;
                const int st = min(max(key - P, 0), S - 1);
                const char *src = (is_v ? new_v : new_k) + (int64_t)st * g.row_bytes;
                if (key < P) src = pool_l + (int64_t)(r < kBlockTokens ? id0 : id1) * g.block_bytes + (is_v ? v_half : 0) + (key & 15) * (D * 4);
                load_to_lds_each(dst + i * 1024, src + (is_v ? l_chunk : l_chunk ^ (r & 15)) * 16);
            }
        }
    };

    f32x16 o[kCols];
#pragma unroll
    for (int j = 0; j < kCols; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) o[j][e] = 0.f;
    float m_run = -INFINITY, l_lane = 0.f;
    typedef const __attribute__((address_space(3))) f32x4 *lds_f4;
    typedef float vcols __attribute__((ext_vector_type(kCols)));
    typedef const __attribute__((address_space(3))) vcols *lds_cols;
    const uint32_t k_row = lds_w + r32 * (D * 4);
    const uint32_t v_at = lds_w + L::kPart + hh * 4 * (D * 4) + r32 * (kCols * 4);

    // The loads run one operand ahead: K of the wave's next unit is requested as soon as this unit's
    // scores are done, V likewise; loads complete in the order issued, so a wait that leaves the
    // kPieces youngest outstanding has everything older in LDS.
    int u = u_begin + w;
    if (u < u_end) {
        issue(u, false);
        issue(u, true);
    }
    for (; u < u_end; u += 4) {
        const bool more = u + 4 < u_end;
        wait_loads<kPieces>();                   // K(u) has landed; V(u) may still be on its way
        f32x16 s;
#pragma unroll
        for (int e = 0; e < 16; ++e) s[e] = 0.f;
#pragma unroll
        for (int j = 0; j < D / 8; ++j) {
            const f32x4 kf = *(lds_f4)(uintptr_t)(k_row + (((hh * (D / 8) + j) ^ (r32 & 15)) << 4));
#pragma unroll
            for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[e], qf[4 * j + e], s, 0, 0, 0);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // K area read out: free for the next unit
        if (more) issue(u + 4, false);
        // score e of the lane belongs to key 8 * (e >> 2) + 4 * hh + (e & 3) of the unit
        const int key0 = u * kF32Unit;
        if (key0 + kF32Unit - 1 > P) {           // some row may not see all of the unit
#pragma unroll
            for (int e = 0; e < 16; ++e) s[e] = key0 + 8 * (e >> 2) + 4 * hh + (e & 3) <= limit ? s[e] : -INFINITY;
        }
        float mx = s[0];
#pragma unroll
        for (int e = 1; e < 16; ++e) mx = fmaxf(mx, s[e]);
        mx = fmaxf(mx, __shfl_xor(mx, 32)) * a.scale_log2;       // (the scale is positive)
        if (__any(mx > m_run)) {
            const float m_new = fmaxf(m_run, mx);
            const float alpha = (m_run == -INFINITY) ? 0.f : exp2f(m_run - m_new);
            l_lane *= alpha;
#pragma unroll
            for (int j = 0; j < kCols; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) o[j][e] *= alpha;
            m_run = m_new;
        }
        const float ref = (m_run == -INFINITY) ? 0.f : m_run;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            s[e] = exp2f(s[e] * a.scale_log2 - ref);
            l_lane += s[e];
        }
        if (more) wait_loads<kPieces>();         // V(u) has landed, K(u + 4) may be outstanding
        else wait_loads<0>();
        // A matrix instruction multiplies a key that a row must not see by zero, which an infinity or a NaN in
        // its value would not survive.  Units that hold such keys are looked through first, and values that are
        // not finite are added to the rows that see them here and then taken as zero.
        if (key0 + kF32Unit - 1 > P) {
            float zero = 0.f;                    // stays so unless something is not finite
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const vcols vf = *(lds_cols)(uintptr_t)(v_at + (8 * (e >> 2) + (e & 3)) * (D * 4));
#pragma unroll
                for (int j = 0; j < kCols; ++j) zero = fmaf(vf[j], 0.f, zero);
            }
            if (__any(!(zero == 0.f))) {
#pragma unroll 1
                for (int kr = 0; kr < kF32Unit; ++kr) {
                    float p = s[0];
#pragma unroll
                    for (int e = 1; e < 16; ++e) p = e == 4 * (kr >> 3) + (kr & 3) ? s[e] : p;
                    p = __shfl(p, r32 + 32 * ((kr >> 2) & 1));
                    const bool seen = key0 + kr <= limit;
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        const vcols vf = *(lds_cols)(uintptr_t)(lds_w + L::kPart + (kr * D + kCols * (8 * (e >> 2) + 4 * hh + (e & 3))) * 4);
#pragma unroll
                        for (int j = 0; j < kCols; ++j) o[j][e] += seen && !__builtin_isfinite(vf[j]) ? p * vf[j] : 0.f;
                    }
                }
                asm volatile("" ::: "memory");
                typedef __attribute__((address_space(3))) float *lds_float;
#pragma unroll 1
                for (int i = lane; i < kF32Unit * D; i += 64) {
                    const lds_float at = (lds_float)(uintptr_t)(lds_w + L::kPart + i * 4);
                    if (!__builtin_isfinite(*at)) *at = 0.f;
                }
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            }
        }
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const vcols vf = *(lds_cols)(uintptr_t)(v_at + (8 * (e >> 2) + (e & 3)) * (D * 4));
#pragma unroll
            for (int j = 0; j < kCols; ++j) o[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(vf[j], s[e], o[j], 0, 0, 0);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // V area read out
        if (more) issue(u + 4, true);
    }

    // ---- combine the four waves: each writes O as padded rows and (max, sum) per row into its own area
    // (dead now), then the work-group folds the four and writes the rows (unsplit) or their partials
    {
        float *wo = (float *)(lds + w * L::kWave);
        const float l_row_sum = l_lane + __shfl_xor(l_lane, 32);
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            vcols v;
#pragma unroll
            for (int j = 0; j < kCols; ++j) v[j] = o[j][e];
            *(vcols *)(wo + r32 * L::kRow + kCols * (8 * (e >> 2) + 4 * hh + (e & 3))) = v;
        }
        if (hh == 0) { wo[32 * L::kRow + 2 * r32] = m_run; wo[32 * L::kRow + 2 * r32 + 1] = l_row_sum; }
    }
    __syncthreads();
    constexpr int kPass = 256 / kChunks, kPasses = kF32Rows / kPass;      // rows at a time
    const int r0 = tid / kChunks, d4 = tid % kChunks;
    auto fold_waves = [&](int r, float &M, float &sum) {                // four columns of a row of this range
        M = -INFINITY;
        sum = 0.f;
#pragma unroll
        for (int k = 0; k < 4; ++k) M = fmaxf(M, ((const float *)(lds + k * L::kWave))[32 * L::kRow + 2 * r]);
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float *wk = (const float *)(lds + k * L::kWave);
            const float mk = wk[32 * L::kRow + 2 * r];
            const float wgt = (mk == -INFINITY) ? 0.f : exp2f(mk - M);
            sum += wgt * wk[32 * L::kRow + 2 * r + 1];
            const f32x4 v = *(const f32x4 *)(wk + r * L::kRow + 4 * d4);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e] = fmaf(wgt, v[e], acc[e]);
        }
        return acc;
    };
    auto write = [&](int mr, f32x4 acc, float sum) {
        const float inv = 1.f / sum;
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] *= inv;
        const int tok = mr / G;
        *(f32x4 *)((float *)a.out + ((int64_t)(it.cu + tok) * g.Hq + it.kvh * G + (mr - tok * G)) * D + 4 * d4) = acc;
    };
    if (!kFold || it.n_splits == 1) {
#pragma unroll 2
        for (int r = r0; r < kF32Rows; r += kPass) {
            const int mr = it.m0 + r;
            if (mr >= n_rows) continue;
            float M, sum;
            const f32x4 acc = fold_waves(r, M, sum);
            if (kFold || it.n_splits == 1) {
                write(mr, acc, sum);
            } else {
                const int tok = mr / G;
                const int64_t prow = (int64_t)(it.part0 + tok * it.part_stride + it.split) * g.Hq + it.kvh * G + (mr - tok * G);
                *(f32x4 *)(a.part_o + prow * D + 4 * d4) = acc;
                if (d4 == 0) *(float2 *)(a.part_ml + prow * 2) = make_float2(M, sum);
            }
        }
        return;
    }

    // ---- a range of several: its partial, and by the last work-group of the row tile to end the rows from all of them (arrive.h):
    // with reference maxima m_s (log2 units), sums l_s and unnormalised outputs O_s, sum_s 2^(m_s - M) O_s / sum_s 2^(m_s - M) l_s.
    // All of a thread's rows at a time, four partials a round trip, eight at most.
    const int tok0 = it.m0 / G, m_last = min(it.m0 + kF32Rows, n_rows) - 1, ns = it.n_splits;
    const int64_t first_slot = ((int64_t)it.part0 + (int64_t)tok0 * it.part_stride) * g.Hq + it.kvh * G;
    const uint32_t n_slots = (uint32_t)min((int64_t)(m_last / G - tok0 + 1) * it.part_stride * g.Hq, (int64_t)(0x7fffffff / (D * 4)));
    const SharedPart part_o(a.part_o + first_slot * D, n_slots * (D * 4)), part_ml(a.part_ml + first_slot * 2, n_slots * 8);
    uint32_t slot[kPasses];
#pragma unroll
    for (int j = 0; j < kPasses; ++j) {
        const int r = r0 + j * kPass, mr = min(it.m0 + r, m_last), tok = mr / G;
        slot[j] = (uint32_t)((tok - tok0) * it.part_stride * g.Hq + mr - tok * G);
        if (it.m0 + r > m_last) continue;
        float M, sum;
        const f32x4 acc = fold_waves(r, M, sum);
        const uint32_t at = slot[j] + it.split * g.Hq;
        part_o.put4(at * (D * 4) + d4 * 16, acc);
        if (d4 == 0) part_ml.put2(at * 8, M, sum);
    }
    if (!last_to_arrive(arrival_counter(a, it), ns, s_bid)) return;
    constexpr int kBatch = 4;
    float M[kPasses], den[kPasses];
    f32x4 acc[kPasses];
#pragma unroll
    for (int j = 0; j < kPasses; ++j) { M[j] = -INFINITY; den[j] = 0.f; acc[j] = f32x4{0.f, 0.f, 0.f, 0.f}; }
    for (int s0 = 0; s0 < ns; s0 += kBatch) {
        float2 ml[kPasses][kBatch];
        f32x4 po[kPasses][kBatch];
#pragma unroll
        for (int k = 0; k < kBatch; ++k)
#pragma unroll
            for (int j = 0; j < kPasses; ++j) {
                const uint32_t at = slot[j] + (s0 + k) * g.Hq;
                ml[j][k] = part_ml.get2(s0 + k < ns ? at * 8 : kNowhere);
                po[j][k] = part_o.get4(s0 + k < ns ? at * (D * 4) + d4 * 16 : kNowhere);
            }
#pragma unroll
        for (int j = 0; j < kPasses; ++j) {
            float Mc = M[j];
#pragma unroll
            for (int k = 0; k < kBatch; ++k) Mc = s0 + k < ns ? fmaxf(Mc, ml[j][k].x) : Mc;
            const float r = M[j] == -INFINITY ? 0.f : exp2f(M[j] - Mc);
            den[j] *= r;
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[j][e] *= r;
            M[j] = Mc;
#pragma unroll
            for (int k = 0; k < kBatch; ++k) {
                if (s0 + k >= ns) continue;
                // a partition without a maximum saw no key of this row (sum and output are 0) or only scores that are NaN
                // (so are they, and so is the row)
                const float wgt = ml[j][k].x == -INFINITY ? 1.f : exp2f(ml[j][k].x - Mc);
                den[j] = fmaf(wgt, ml[j][k].y, den[j]);
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[j][e] = fmaf(wgt, po[j][k][e], acc[j][e]);
            }
        }
    }
#pragma unroll
    for (int j = 0; j < kPasses; ++j)
        if (it.m0 + r0 + j * kPass <= m_last) write(it.m0 + r0 + j * kPass, acc[j], den[j]);
}

template <int D, bool kLong, bool kFold>
static hipError_t launch_attn(const Geom &g, const BatchDev &b, const AttnArgs &a, const Launch &L)
{
    static PerDeviceOnce configured;
    const hipError_t e = configured.run([] {
        return hipFuncSetAttribute((const void *)attn_f32_kernel<D, kLong, kFold>, hipFuncAttributeMaxDynamicSharedMemorySize, F32Lds<D>::kBytes);
    });
    if (e != hipSuccess) return e;
    TC_LAUNCH((attn_f32_kernel<D, kLong, kFold>), a.n_items + a.n_append, F32Lds<D>::kBytes, L, g, b, a);
    return hipGetLastError();
}

hipError_t launch_attn_f32(const Geom &g, const BatchDev &b, const AttnArgs &a, const Launch &L)
{
    if (a.n_items + a.n_append == 0) return hipSuccess;
    const bool fold = a.part_o && a.arrivals;
    if (fold && (g.D != 64 || a.long_ranges)) return hipErrorInvalidValue;        // (the planner's rule)
    if (g.D == 64 && fold) return launch_attn<64, false, true>(g, b, a, L);
    if (g.D == 64) return a.long_ranges ? launch_attn<64, true, false>(g, b, a, L) : launch_attn<64, false, false>(g, b, a, L);
    if (g.D == 128) return a.long_ranges ? launch_attn<128, true, false>(g, b, a, L) : launch_attn<128, false, false>(g, b, a, L);
    return hipErrorInvalidValue;
}

// ------------------------------------------------------------------------------------ merge
// Combine split-KV partials of one output row: with reference maxima m_s (log2 units), sums l_s
// and unnormalised partial outputs O_s:  out = sum_s 2^(m_s - M) O_s / sum_s 2^(m_s - M) l_s.
// D/4 threads per (suffix token, head) row, four columns each.  Bound: the latency of the loads of a
// short launch, so those of eight partitions are issued before the first use, and (kEven) before it is known how
// many there are (slots beyond a token's last partition are loaded and ignored).
// Measured (2 queries, 9 k keys, 2 + 59 tokens, 20 partitions): 5.3 us; one partition after the other 18.4 us.
template <int D, bool kEven>
__global__ __launch_bounds__(256) void merge_f32_kernel(Geom g, BatchDev b, AttnArgs a)
{
    constexpr int kThreads = D / 4;
    constexpr int kBatch = 8;
    const int64_t row = (int64_t)blockIdx.x * (256 / kThreads) + threadIdx.x / kThreads;
    const int d = 4 * (threadIdx.x % kThreads);
    const int64_t n_rows = (int64_t)b.total_S * g.Hq;
    if (row >= n_rows) return;
    const int n = (int)(row / g.Hq), head = (int)(row - (int64_t)n * g.Hq);
    const PartSlots slots = part_slots<kEven>(b, n);
    if (!kEven && slots.count <= 1) return;      // written directly by the attention kernel
    float2 ml[kBatch];
    f32x4 po[kBatch];
    auto fetch = [&](int s0) {
#pragma unroll
        for (int j = 0; j < kBatch; ++j) {
            const int64_t slot = (int64_t)min(slots.first + s0 + j, slots.last) * g.Hq + head;
            ml[j] = *(const float2 *)(a.part_ml + slot * 2);
            po[j] = *(const f32x4 *)(a.part_o + slot * D + d);
        }
    };
    fetch(0);
    const int ns = slots.count;
    if (kEven && ns <= 1) return;
    float M = -INFINITY, den = 0.f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0; s0 < ns; s0 += kBatch) {
        if (s0 > 0) fetch(s0);
        float Mc = M;
#pragma unroll
        for (int j = 0; j < kBatch; ++j) Mc = s0 + j < ns ? fmaxf(Mc, ml[j].x) : Mc;
        const float r = M == -INFINITY ? 0.f : exp2f(M - Mc);
        den *= r;
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] *= r;
        M = Mc;
#pragma unroll
        for (int j = 0; j < kBatch; ++j) {
            if (s0 + j >= ns) continue;
            // a partition without a maximum saw no key of this row (sum and output are 0) or only scores that are NaN
            // (so are they, and so is the row)
            const float wgt = ml[j].x == -INFINITY ? 1.f : exp2f(ml[j].x - M);
            den = fmaf(wgt, ml[j].y, den);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e] = fmaf(wgt, po[j][e], acc[e]);
        }
    }
    const float inv = 1.f / den;
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] *= inv;
    *(f32x4 *)((float *)a.out + row * D + d) = acc;
}

hipError_t launch_merge_f32(const Geom &g, const BatchDev &b, const AttnArgs &a, const Launch &L)
{
    const int64_t n_rows = (int64_t)b.total_S * g.Hq;
    if (n_rows == 0) return hipSuccess;
    if (!b.part_tab) return hipErrorInvalidValue;
    const int per = 256 / (g.D / 4);
    const int grid = (int)((n_rows + per - 1) / per);
    const bool even = b.part_stride > 0;
    if (g.D == 64 && even) TC_LAUNCH((merge_f32_kernel<64, true>), grid, 0, L, g, b, a);
    else if (g.D == 64) TC_LAUNCH((merge_f32_kernel<64, false>), grid, 0, L, g, b, a);
    else if (g.D == 128 && even) TC_LAUNCH((merge_f32_kernel<128, true>), grid, 0, L, g, b, a);
    else if (g.D == 128) TC_LAUNCH((merge_f32_kernel<128, false>), grid, 0, L, g, b, a);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace tc
