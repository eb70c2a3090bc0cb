// Prefill attention for batches of few suffix tokens over short prefixes: launches that the other
// prefill kernels spend on getting started (a follow-up question of a few tokens against a few tables).
//
// Bound: latency.  The other kernels give a work-group 128 rows and all of its waves the same keys, tile
// after tile behind barriers, and fill the chip by cutting the keys into partitions that a second launch
// merges.  Here a work-group is 32 rows (row = token * G + head in the group) of one (query, KV head)
// and its EIGHT waves split the keys: wave w takes the 32-key units w, w + 8, ... of the range, streams
// each straight into its own LDS area and keeps its own running maximum, sum and output, so there is no
// barrier before the waves are combined at the end.  A prefix of a thousand tokens is four or five units
// per wave, needs no cut, and two waves on a SIMD cover each other's round trips.  What it
// costs is that 32 rows, not 128, share a key tile on its way from the L2, which is why it is only
// chosen where a launch is one or two rounds of work-groups.
//
// Masked keys get a weight of zero, and their values are multiplied by it: as in the other bf16 kernels those
// have to be finite.  (So are the zeros and the suffix values that the tail of the prefix's last block holds before
// and after the append of the same launch, which may run beside a tile's loads.)
//
// Where a query is cut all the same, the last of a row tile's ranges to end combines their partials (16 KB each) in the same
// launch (arrive.h), or, with more than eight ranges, a launch of its own does.  The same batches in the same ranges either way, us
// a layer: one query of 1.4 k + 17 tokens, 28 / 4 heads, in 7 ranges 10.1 against 10.6 in two launches, in 10 11.4 against 10.3;
// of 2.4 k + 8 in 8 ranges 10.5 either way, in 10 11.5 against 10.5, in 20 12.7 against 10.2; four of 2.4 k + 12, 32 / 8 heads, in 4 13.9
// against 14.4, in 12 30.4 against 25.0.  28 layers of a short question 362 us in two launches, 340 in one.
//
// Measured per layer, against the pipelined or general kernel, partials combined by a launch of its own: 28 / 4
// heads, one query of 1.1 k prefix and 17 new tokens 10.3 us (14.9); thirteen of 4 k and 3 .. 6 tokens 27.1
// (35.4); 40 / 8 heads, eight of 350 and 40 tokens 17.7 (28.3), sixteen of 1 k and 2 tokens 16.2 (36.0), four of
// 1 k and 40 tokens 14.4 (24.0).
#include "arrive.h"
#include "kv_append.h"
#include "lds_dma.h"
#include "tc_internal.h"

namespace tc {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kShWaves = 8;
constexpr int kShUnit = 32;                          // keys per unit: two pool blocks
constexpr int kShHeadBlk = 4096;                     // one head's K (or V) in one block: 16 * 128 * 2
constexpr int kShPart = 2 * kShHeadBlk;              // K of a unit: 32 rows of 256 B, 16-byte chunks XOR-swizzled; V: as in two blocks
constexpr int kShWave = 2 * kShPart;
constexpr int kShQ = kShWaves * kShWave;             // query rows (32 of 256 B), the same bytes written by every wave
constexpr int kShIds = kShQ + kShortRows * 256;      // block ids of the range, likewise
constexpr int kShMl = kShIds + kAttnMaxTiles * (kAttnKeys / kBlockTokens) * 4;     // (maximum, sum) per wave and row
constexpr int kShLds = kShMl + kShWaves * kShortRows * 8 + 256;                    // + alignment slack
constexpr float kShRescale = 8.f;

// Four columns of an output row.
__device__ __forceinline__ void write_part(const AttnArgs &a, int64_t row, int ch, f32x4 acc, float l)
{
    const float inv = 1.f / l;
    unsigned short r[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const __bf16 x = (__bf16)(acc[e] * inv);
        r[e] = *(const unsigned short *)&x;
    }
    *(uint2 *)((unsigned short *)a.out + row * 128 + 4 * ch) = make_uint2(r[0] | ((uint32_t)r[1] << 16), r[2] | ((uint32_t)r[3] << 16));
}

// Is some query of the batch in several ranges, and who combines them.  (With their end compiled in, batches without any paid
// 0.1 us for it.)
enum ShortCut { kUncut, kFolded, kMerged };
template <ShortCut kCut>
__global__ __launch_bounds__(64 * kShWaves, 2) void attn_bf16_short_kernel(Geom g, BatchDev b, AttnArgs a)
{
    extern __shared__ __attribute__((aligned(16))) char lds_raw[];
    const AttnItem it = load_item(a, blockIdx.x);
    if (it.q < 0) return;                            // padding item (uniform for the work-group)
    // the XOR addressing of the K rows needs them 256-byte aligned
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds_raw;
    const uint32_t slack = (256u - (lds_base & 255u)) & 255u;
    char *lds = lds_raw + slack;
    const uint32_t lds0 = lds_base + slack;

    const int tid = threadIdx.x, lane = tid & 63, r32 = lane & 31, hh = lane >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int G = g.G, P = it.P, S = it.S;
    const int n_rows = S * G, m_last = min(it.m0 + kShortRows, n_rows) - 1;
    // the range's units: first those of the prefix (from the pool), then those of the suffix (from k_new /
    // v_new) up to the last one that a row of the tile sees.  Key tiles are two units, and the suffix
    // starts a tile of its own.
    const int n_ptiles = (P + kAttnKeys - 1) / kAttnKeys, n_punits = (P + kShUnit - 1) / kShUnit;
    const int p_begin = min(2 * it.tile_begin, n_punits), n_p = min(2 * it.tile_end, n_punits) - p_begin;
    const int s_begin = max(2 * (it.tile_begin - n_ptiles), 0);
    const int n_s = max(min(2 * (it.tile_end - n_ptiles), m_last / G / kShUnit + 1) - s_begin, 0);
    const int n_units = n_p + n_s;

    const char *pool_l = g.pool + (int64_t)a.layer * g.layer_stride + (int64_t)it.kvh * kShHeadBlk;
    const int64_t bb = g.block_bytes;
    const uint32_t v_half = (uint32_t)(g.block_bytes >> 1);
    const char *new_k = (const char *)a.k_new + ((int64_t)it.cu * g.Hkv + it.kvh) * 256;
    const char *new_v = (const char *)a.v_new + ((int64_t)it.cu * g.Hkv + it.kvh) * 256;
    const uint32_t lds_w = lds0 + w * kShWave;
    const int32_t *ids = (const int32_t *)(lds + kShIds);
    const int last_id = ((P + kBlockTokens - 1) >> 4) - 1 - 2 * p_begin;     // the prefix's last block, counted from the range's first
    const float c = a.scale_log2;
    typedef const __attribute__((address_space(3))) bf16x8 *lds_frag;

    // K of a unit: rows of 256 bytes in pieces of four, chunk c of row r at chunk position c ^ (r & 15); 8
    // load instructions per operand and unit
    const int k_off0 = (lane >> 4) * 256;
    auto issue_k = [&](int k, int2 e) {
        if (k < n_p) {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const char *src = pool_l + (int64_t)entry_bid(j ? e.y : e.x) * bb;
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    load_to_lds(lds_w + j * 4096 + i * 1024, src, k_off0 + i * 1024 + (((lane & 15) ^ (4 * i + (lane >> 4))) * 16));
            }
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int r = 4 * i + (lane >> 4);
                const int tok = min((s_begin + k - n_p) * kShUnit + r, S - 1);
                load_to_lds_each(lds_w + i * 1024, new_k + (int64_t)tok * g.row_bytes + (((lane & 15) ^ (r & 15)) * 16));
            }
        }
    };
    auto issue_v = [&](int2 e) {                      // of a prefix unit: verbatim
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const char *src = pool_l + (int64_t)entry_bid(j ? e.y : e.x) * bb + v_half;
#pragma unroll
            for (int i = 0; i < 4; ++i) load_to_lds(lds_w + kShPart + j * 4096 + i * 1024, src + i * 1024, lane * 16);
        }
    };

    // The first key range also appends: a row tile takes the K and V of this head for the tokens whose first row
    // it holds, the last tile the zeros behind the sequence's end as well (extra work-groups for it would each
    // wait for a CU's LDS, and for a round of their own where the items fill the chip).  A thread's first 16
    // bytes of either are requested here, ahead of the counted loads; the stores come at the very end (a
    // store counts as an outstanding memory operation).
    const int a_begin = (it.m0 + G - 1) / G;
    const int a_end = m_last < n_rows - 1 ? (m_last + G) / G : S + ((-(P + S)) & (kBlockTokens - 1));
    const int n_append = it.split == 0 ? (a_end - a_begin) * 16 : 0;
    const int32_t *bt_q = b.block_table + (int64_t)it.q * b.max_blocks;
    struct Put { uint4 k, v; int phys; };
    auto fetch_new = [&](int idx) {
        const int t = a_begin + (idx >> 4);
        Put x{make_uint4(0, 0, 0, 0), make_uint4(0, 0, 0, 0), 0};
        x.phys = bt_q[(P + t) >> 4];
        if (t < S) {
            x.k = *(const uint4 *)(new_k + (int64_t)t * g.row_bytes + (idx & 15) * 16);
            x.v = *(const uint4 *)(new_v + (int64_t)t * g.row_bytes + (idx & 15) * 16);
        }
        return x;
    };
    Put put{make_uint4(0, 0, 0, 0), make_uint4(0, 0, 0, 0), 0};
    if (tid < n_append) put = fetch_new(tid);

    f32x16 o[4];
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int e = 0; e < 16; ++e) o[db][e] = 0.f;
    float m_run = -INFINITY, l_lane = 0.f;

    if (w < n_units) {
        int2 e_now = load_bids(a, blockIdx.x, 2 * w);  // a wave's first unit: its block ids come with the work item
        if (n_p > kShWaves) {                           // the others: the range's ids, 256 per load (rows of the table are padded to 16 bytes)
            const int32_t *bt = b.block_table + (int64_t)it.q * b.max_blocks + 2 * p_begin;
            const int last_chunk = ((b.max_blocks - 2 * p_begin) >> 2) - 1;
            for (int i = 0; i < 2 * n_p; i += 256)
                load_to_lds(lds0 + kShIds + i * 4, (const char *)bt, min((i >> 2) + lane, last_chunk) * 16);
        }
        issue_k(w, e_now);
        {                                               // the tile's query rows, chunk c of row r at c ^ (r & 15)
            const int tok0 = it.m0 / G;
            const char *qp = (const char *)a.q + ((int64_t)(it.cu + tok0) * g.Hq + it.kvh * G) * 256;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int r = 4 * i + (lane >> 4), m = min(it.m0 + r, n_rows - 1), tok = m / G;
                load_to_lds(lds0 + kShQ + i * 1024, qp, ((tok - tok0) * g.Hq + m - tok * G) * 256 + (((lane & 15) ^ (r & 15)) * 16));
            }
        }
        if (w < n_p) {
            issue_v(e_now);
            wait_loads<8>();
        } else {
            wait_loads<0>();
        }
        // Q^T fragments (B operand): lane (row r32, half hh) holds q[row][16*ks + 8*hh .. +8]
        bf16x8 qf[8];
        {
            const uint32_t qb = lds0 + kShQ + r32 * 256 + ((hh ^ (r32 & 15)) << 4);
#pragma unroll
            for (int ks = 0; ks < 8; ++ks) qf[ks] = *(lds_frag)(uintptr_t)(qb ^ (ks << 5));
        }
        const int s_tok = min(it.m0 + r32, n_rows - 1) / G;
        const uint32_t kb = lds_w + r32 * 256 + ((hh ^ (r32 & 15)) << 4);
        const uint32_t vb = lds_w + kShPart + r32 * 32 + hh * 16;

        // The loads run one operand ahead: K of the wave's next unit is requested as soon as this unit's
        // K fragments are in registers, V likewise; loads complete in the order issued, so a wait that
        // leaves the 8 youngest outstanding has everything older in LDS.
        for (int k = w; k < n_units; k += kShWaves) {
            const bool pre = k < n_p, more = k + kShWaves < n_units, more_pre = k + kShWaves < n_p;
            int2 e_next = make_int2(0, 0);
            if (more_pre) {
                const int i = 2 * (k + kShWaves);
                const int x = ids[i], y = ids[min(i + 1, last_id)];
                e_next = make_int2(__builtin_amdgcn_readfirstlane(x), __builtin_amdgcn_readfirstlane(y));
            }
            // values of a suffix unit come as token rows and are transposed on their way into LDS: a lane takes
            // 16 bytes of two neighbouring tokens
            uint4 vrow[8];
            const int pair = lane & 15;
            if (!pre) {
                const int tok = (s_begin + k - n_p) * kShUnit + 2 * pair;
                const char *r0 = new_v + (int64_t)min(tok, S - 1) * g.row_bytes, *r1 = new_v + (int64_t)min(tok + 1, S - 1) * g.row_bytes;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    vrow[2 * i] = *(const uint4 *)(r0 + (4 * i + (lane >> 4)) * 16);
                    vrow[2 * i + 1] = *(const uint4 *)(r1 + (4 * i + (lane >> 4)) * 16);
                }
                wait_loads<0>();
            } else {
                wait_loads<8>();
            }
            bf16x8 kf[8];
#pragma unroll
            for (int ks = 0; ks < 8; ++ks) kf[ks] = *(lds_frag)(uintptr_t)(kb ^ (ks << 5));
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // K area read out
            if (more) issue_k(k + kShWaves, e_next);
            f32x16 s;
#pragma unroll
            for (int e = 0; e < 16; ++e) s[e] = 0.f;
#pragma unroll
            for (int ks = 0; ks < 8; ++ks) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], qf[ks], s, 0, 0, 0);
            if (!pre) {
                char *vd = lds + w * kShWave + kShPart + (pair >> 3) * kShHeadBlk + vperm((2 * pair) & 15) * 2;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t x[4] = {vrow[2 * i].x, vrow[2 * i].y, vrow[2 * i].z, vrow[2 * i].w};
                    const uint32_t y[4] = {vrow[2 * i + 1].x, vrow[2 * i + 1].y, vrow[2 * i + 1].z, vrow[2 * i + 1].w};
#pragma unroll
                    for (int j = 0; j < 8; ++j)              // (tokens 2 pair and 2 pair + 1 are neighbours in the block, too)
                        *(uint32_t *)(vd + (8 * (4 * i + (lane >> 4)) + j) * 32) =
                            ((x[j >> 1] >> (16 * (j & 1))) & 0xffffu) | ((y[j >> 1] >> (16 * (j & 1))) << 16);
                }
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            } else if (more) {
                wait_loads<8>();
            } else {
                wait_loads<0>();
            }
            bf16x8 vf[8];                              // V^T fragments: in registers before the softmax starts
#pragma unroll
            for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                for (int db = 0; db < 4; ++db) vf[4 * kk + db] = *(lds_frag)(uintptr_t)(vb + kk * kShHeadBlk + db * 1024);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // V area read out
            if (more_pre) issue_v(e_next);
            if (pre) {
                // positions that hold no key: beyond the end of the prefix, and the unused tail of a table
                // block read in place (its count rides in the block-table entry)
                const int key0 = (p_begin + k) * kShUnit;
                const int pad0 = entry_pad(e_now.x), pad1 = entry_pad(e_now.y);
                if ((pad0 | pad1) != 0 || key0 + kShUnit > P) {
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        const int in_blk = 8 * ((e >> 2) & 1) + 4 * hh + (e & 3);
                        const int key = key0 + 8 * (e >> 2) + 4 * hh + (e & 3);
                        s[e] = (key >= P || in_blk >= kBlockTokens - (e < 8 ? pad0 : pad1)) ? -INFINITY : s[e];
                    }
                }
            } else {                                   // causal
                const int t0 = (s_begin + k - n_p) * kShUnit;
#pragma unroll
                for (int e = 0; e < 16; ++e) s[e] = t0 + 8 * (e >> 2) + 4 * hh + (e & 3) <= s_tok ? s[e] : -INFINITY;
            }
            float mx = s[0];
#pragma unroll
            for (int e = 1; e < 16; ++e) mx = fmaxf(mx, s[e]);
            mx = fmaxf(mx, __shfl_xor(mx, 32));
            const float mxs = mx * c;
            if (__any(mxs > m_run + kShRescale)) {     // also taken while m_run is still -inf
                const float m_new = fmaxf(m_run, mxs);
                const float alpha = (m_run == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m_run - m_new);
                l_lane *= alpha;
#pragma unroll
                for (int db = 0; db < 4; ++db)
#pragma unroll
                    for (int e = 0; e < 16; ++e) o[db][e] *= alpha;
                m_run = m_new;
            }
            const float neg_m = (m_run == -INFINITY) ? 0.f : -m_run;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                s[e] = __builtin_amdgcn_exp2f(fmaf(s[e], c, neg_m));
                l_lane += s[e];
            }
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) {
                bf16x8 pf;
#pragma unroll
                for (int e = 0; e < 8; ++e) pf[e] = (__bf16)s[8 * kk + e];
#pragma unroll
                for (int db = 0; db < 4; ++db) o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[4 * kk + db], pf, o[db], 0, 0, 0);
            }
            e_now = e_next;
        }
    }

    // ---- combine the waves: each writes O as 32 rows of 128 floats (16-byte chunk c of row r at c ^ r) into its own
    // area (dead now) and (maximum, sum) per row, then every thread folds the eight for a few (row, 4 columns)
    {
        char *wo = lds + w * kShWave + r32 * 512;
        const float l_row = l_lane + __shfl_xor(l_lane, 32);
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                f32x4 v;
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = o[db][4 * q + e];
                *(f32x4 *)(wo + (((8 * db + 2 * q + hh) ^ r32) << 4)) = v;
            }
        if (hh == 0) *(float2 *)(lds + kShMl + (w * kShortRows + r32) * 8) = make_float2(m_run, l_row);
    }
    __syncthreads();
    const int tok0 = it.m0 / G;
    auto fold_waves = [&](int row, int ch) {           // four columns of a row of this range
        float2 ml[kShWaves];
        RowSum x{-INFINITY, 0.f, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int k = 0; k < kShWaves; ++k) {
            ml[k] = *(const float2 *)(lds + kShMl + (k * kShortRows + row) * 8);
            x.M = fmaxf(x.M, ml[k].x);
        }
#pragma unroll
        for (int k = 0; k < kShWaves; ++k) {
            const float wgt = (ml[k].x == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(ml[k].x - x.M);
            x.L += wgt * ml[k].y;
            const f32x4 v = *(const f32x4 *)(lds + k * kShWave + row * 512 + ((ch ^ row) << 4));
#pragma unroll
            for (int e = 0; e < 4; ++e) x.acc[e] += wgt * v[e];
        }
        return x;
    };
    const int ch = tid & 31;
    if (kCut != kFolded || it.n_splits == 1) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int row = (tid >> 5) + 16 * j, m = it.m0 + row;
            if (m > m_last) continue;
            const RowSum x = fold_waves(row, ch);
            const int tok = m / G, head = it.kvh * G + (m - tok * G);
            if (kCut == kMerged && it.n_splits > 1) {
                const int64_t slot = (int64_t)(it.part0 + tok * it.part_stride + it.split) * g.Hq + head;
                *(f32x4 *)(a.part_o + slot * 128 + 4 * ch) = x.acc;
                if (ch == 0) *(float2 *)(a.part_ml + slot * 2) = make_float2(x.M, x.L);
            } else {
                write_part(a, (int64_t)(it.cu + tok) * g.Hq + head, ch, x.acc, x.L);
            }
        }
    } else {
        // A range of several: the last work-group of the row tile to end combines them (arrive.h), up to eight in one round of
        // loads.  32 threads take two rows at a time, four columns each; lanes 0 .. 15 and 16 .. 31 bring their weights.
        const int64_t first_slot = ((int64_t)it.part0 + (int64_t)tok0 * it.part_stride) * g.Hq + it.kvh * G;
        const uint32_t n_slots = (uint32_t)min((int64_t)(m_last / G - tok0 + 1) * it.part_stride * g.Hq, (int64_t)0x3fffff);
        const SharedPart part_o(a.part_o + first_slot * 128, n_slots * 512), part_ml(a.part_ml + first_slot * 2, n_slots * 8);
        const int ns = it.n_splits;
        const uint32_t step = (uint32_t)g.Hq * 512;
        uint32_t slot[2];
        int64_t orow[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int row = (tid >> 5) + 16 * j, m = min(it.m0 + row, m_last), tok = m / G;
            slot[j] = (uint32_t)((tok - tok0) * it.part_stride * g.Hq + m - tok * G);
            orow[j] = (int64_t)(it.cu + tok) * g.Hq + it.kvh * G + (m - tok * G);
            if (it.m0 + row > m_last) continue;
            const RowSum x = fold_waves(row, ch);
            part_o.put4(slot[j] * 512 + it.split * step + ch * 16, x.acc);
            if (ch == 0) part_ml.put2(slot[j] * 8 + it.split * (step >> 6), x.M, x.L);
        }
        const uint32_t ml_at = (ch < 16 ? slot[0] : slot[1]) * 8 + (ch & 15) * (step >> 6);
        float *s_w = (float *)(lds + kShMl) + (tid >> 5) * 32;
        if (last_to_arrive(arrival_counter(a, it), ns, (int32_t *)(lds + kShIds))) {
            const bool there = (ch & 15) < ns;
            const float2 ml = part_ml.get2(there ? ml_at : kNowhere);
            f32x4 o[kShortFold][2];
#pragma unroll
            for (int k = 0; k < kShortFold; ++k)
#pragma unroll
                for (int j = 0; j < 2; ++j) o[k][j] = part_o.get4(k < ns ? slot[j] * 512 + ch * 16 + k * step : kNowhere);
            const float m = there ? ml.x : -INFINITY, M = max16(m);
            const float w = m == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m - M);     // (no maximum: its sums are 0, or NaN and so is the row)
            s_w[ch] = w;
            f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                f32x4 wj[kShortFold / 4];
#pragma unroll
                for (int k = 0; k < kShortFold / 4; ++k) wj[k] = *(const f32x4 *)(s_w + 16 * j + 4 * k);
#pragma unroll
                for (int k = 0; k < kShortFold; ++k)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[j][e] += wj[k >> 2][k & 3] * o[k][j][e];
            }
            s_w[ch] = sum16(w * ml.y);
#pragma unroll
            for (int j = 0; j < 2; ++j)
                if (it.m0 + (tid >> 5) + 16 * j <= m_last) write_part(a, orow[j], ch, acc[j], s_w[16 * j]);
        }
    }

    for (int idx = tid; idx < n_append; idx += 64 * kShWaves) {
        if (idx != tid) put = fetch_new(idx);
        const int t = (P + a_begin + (idx >> 4)) & 15, ch = idx & 15;
        char *kd = const_cast<char *>(pool_l) + (int64_t)entry_bid(put.phys) * bb;
        *(uint4 *)(kd + t * 256 + ch * 16) = put.k;
        unsigned short *v16 = (unsigned short *)(kd + v_half) + 8 * ch * kBlockTokens + vperm(t);
        const uint32_t u[4] = {put.v.x, put.v.y, put.v.z, put.v.w};
#pragma unroll
        for (int e = 0; e < 8; ++e) v16[e * kBlockTokens] = (unsigned short)(u[e >> 1] >> (16 * (e & 1)));
    }
}

hipError_t launch_attn_short_bf16(const Geom &g, const BatchDev &b, const AttnArgs &a, const Launch &L)
{
    if (a.n_items == 0) return hipSuccess;
    if (g.D != 128 || g.esize != 2) return hipErrorInvalidValue;
    static PerDeviceOnce configured;
    const hipError_t e = configured.run([] {
        for (const void *k : {(const void *)attn_bf16_short_kernel<kUncut>, (const void *)attn_bf16_short_kernel<kFolded>, (const void *)attn_bf16_short_kernel<kMerged>}) {
            const hipError_t ek = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kShLds);
            if (ek != hipSuccess) return ek;
        }
        return hipSuccess;
    });
    if (e != hipSuccess) return e;
    auto launch = [&](auto *kernel) { hipExtLaunchKernelGGL(kernel, dim3(a.n_items), dim3(64 * kShWaves), kShLds, L.stream, L.start, L.stop, 0, g, b, a); };
    if (!a.part_o) launch(attn_bf16_short_kernel<kUncut>);
    else if (a.arrivals) launch(attn_bf16_short_kernel<kFolded>);
    else launch(attn_bf16_short_kernel<kMerged>);
    return hipGetLastError();
}

}  // namespace tc
