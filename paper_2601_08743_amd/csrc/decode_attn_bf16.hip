// Decode-step attention: one new token per query attends to everything its sequence already holds
// in the pool (the tables' tokens, the prompt's own suffix, the tokens generated so far) and to
// itself.  With one token, a KV head has only G rows (its group's query heads), so the work is
// reading K and V once: HBM-bound, and for short sequences bound by the chain of round trips from
// the launch to the first keys.
//
// A work-group is one (query, KV head, key range); its four waves split the KEYS: wave w takes the
// 32-key units w, w + 4, ... of the range, streams each straight into its own LDS ring of two units
// (32 KB), computes S^T = K . Q^T and O^T += V^T . P^T with the matrix cores exactly as the prefill
// kernels do (columns beyond G repeat row G-1 and are dropped) and keeps its own running maximum and
// sum.  No wave waits for another before the end: the range's block ids, the query rows and the keys
// all arrive by LDS-direct loads that the wave counts itself, the ids of a wave's first two units come
// with the work item, and so the first keys are requested one scalar fetch after the kernel starts.
// Units of 32 keys rather than 64 halve both the shortest useful range (a sequence of 4 k tokens
// makes 132 work-groups instead of 44) and what a wave loses when a range does not divide by four.  A
// wave works on two units at a time where it has them: over tables that many sequences read in place the keys come
// from the L2 and what counts is the wave's own work, of which one maximum, one vote and two waits for each
// unit were 6 % (47 sequences of 9.1 k tokens, 32 / 8 heads: 159 us in single units, 151 with the 64-key tiles, 134 so).
//
// At the end the four waves' (max, sum, O) are combined through LDS.  A work-group that has all the keys of its (query, KV
// head) adds the new token itself (its key and value come from k_new / v_new: one dot product and one scaled row per
// head) and writes the output; one of several stores one partial per row, and the last of them to end combines them
// (arrive.h): up to 36, one round of loads, of up to eight heads, a row for every 32 threads, 72 of up to four.  More are combined by a
// launch of its own: a second round on one CU takes longer than that (one sequence of 4.7 k tokens in 37 ranges, 32 / 1
// heads, 18.0 us in one launch, 10.0 in two; 24 / 2 heads 11.7 against 9.4; 28 / 4 heads in 33 8.7 against 9.5, in 72 13.9 against 12.8).  The new token's K/V are appended to the pool by the first key range of each (query, KV head): extra
// work-groups for it, as in prefill, would each wait for a CU's LDS.
//
// Measured, a layer of a token step (28 / 4 heads unless said; in parentheses with a second launch that combined the
// partials): one sequence of 200 tokens 5.3 us (7.5), of 4.2 k in 33 ranges 8.9 (10.0), of 14.4 k 12.5 (14.3); eight of 2.4 k 12.7
// (14.3); 32 sequences, 142 MB: 32.4 (33.7); four of 25 k, 32 / 8 heads, 412 MB: 65.0 (67.1) = 6.3 TB/s.  Where the 8.9 us
// go: 1.3 between two launches, 0.45 to the work item, 1.0 to the first keys, 1.5 for the unit, 0.5 to combine the waves, 0.3
// to store, 0.8 to count in, 2 to fold 33 partials (118 KB) on one CU and 0.1 to write.
#include "arrive.h"
#include "kv_append.h"
#include "lds_dma.h"
#include "tc_internal.h"

#include <type_traits>

namespace tc {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kDecUnit = 32;                         // keys per unit: two pool blocks
constexpr int kDecHeadBlk = 4096;                    // one head's K (or V) in one block: 16 * 128 * 2
constexpr int kDecPart = 2 * kDecHeadBlk;            // K of a unit: 32 rows of 256 B, 16-byte chunks XOR-swizzled; V: two blocks verbatim
constexpr int kDecSlot = 2 * kDecPart;
constexpr int kDecWave = 2 * kDecSlot;               // two units in flight per wave
constexpr int kDecQ = 4 * kDecWave;                  // query rows (32 of 256 B), the same bytes written by every wave
constexpr int kDecIds = kDecQ + 32 * 256;            // block ids of the range, likewise
constexpr int kDecLds = kDecIds + kAttnMaxTiles * (kAttnKeys / kBlockTokens) * 4 + 256;    // + alignment slack
constexpr int kDecRow = 132;                         // padded row of the final exchange (floats)
constexpr float kDecRescale = 8.f;

// Four columns of the new token's key and value and of one head's query row.
struct SelfRaw { uint2 q, k, v; };
__device__ __forceinline__ SelfRaw load_self(const Geom &g, const AttnArgs &a, int token, int kvh, int head, int d)
{
    const int64_t kv = ((int64_t)token * g.Hkv + kvh) * 128 + d;
    return SelfRaw{*(const uint2 *)((const unsigned short *)a.q + ((int64_t)token * g.Hq + head) * 128 + d),
                *(const uint2 *)((const unsigned short *)a.k_new + kv), *(const uint2 *)((const unsigned short *)a.v_new + kv)};
}

// The new token's score against itself and its value (32 neighbouring threads, four columns each).
struct Self { float score; f32x4 v; };
__device__ __forceinline__ Self score_self(const SelfRaw &s, float scale_log2)
{
    auto lo = [](uint32_t u) { return __uint_as_float(u << 16); };
    auto hi = [](uint32_t u) { return __uint_as_float(u & 0xffff0000u); };
    const float prod = sum32(lo(s.q.x) * lo(s.k.x) + hi(s.q.x) * hi(s.k.x) + lo(s.q.y) * lo(s.k.y) + hi(s.q.y) * hi(s.k.y));
    return Self{prod * scale_log2, {lo(s.v.x), hi(s.v.x), lo(s.v.y), hi(s.v.y)}};
}

// Four columns of an output row.
__device__ __forceinline__ void write_row(unsigned short *out, const RowSum &x)
{
    const float inv = 1.f / x.L;
    unsigned short r[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const __bf16 y = (__bf16)(x.acc[e] * inv);
        r[e] = *(const unsigned short *)&y;
    }
    *(uint2 *)out = make_uint2(r[0] | ((uint32_t)r[1] << 16), r[2] | ((uint32_t)r[3] << 16));
}

// The new token joins the row's keys.  (One key: a score of -infinity is no weight, not the mark of a partial without keys.)
__device__ __forceinline__ void add_self(RowSum &x, const Self &s)
{
    if (s.score != -INFINITY) x.add(s.score, 1.f, s.v);
}

// The new token joins, and the row is written.
__device__ __forceinline__ void finish_row(const Geom &g, const AttnArgs &a, const AttnItem &it, int row, int d, const Self &s, RowSum x)
{
    add_self(x, s);
    write_row((unsigned short *)a.out + ((int64_t)it.cu * g.Hq + it.kvh * g.G + row) * 128 + d, x);
}

// kFold: the last work-group of a (query, KV head) combines its ranges' partials; else they are left to a merge launch.
template <bool kFold>
__global__ __launch_bounds__(256, 1) void decode_attn_bf16_kernel(Geom g, BatchDev b, AttnArgs a)
{
    extern __shared__ __attribute__((aligned(16))) char lds_raw[];
    const AttnItem it = load_item(a, blockIdx.x);
    if (it.q < 0) return;
    // the XOR addressing of the K rows needs them 256-byte aligned
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds_raw;
    const uint32_t slack = (256u - (lds_base & 255u)) & 255u;
    char *lds = lds_raw + slack;
    const uint32_t lds0 = lds_base + slack;

    const int tid = threadIdx.x, lane = tid & 63, r32 = lane & 31, hh = lane >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int G = g.G, P = it.P;
    const int u_begin = it.tile_begin * (kAttnKeys / kDecUnit);
    const int n_units = min(it.tile_end * (kAttnKeys / kDecUnit), (P + kDecUnit - 1) / kDecUnit) - u_begin;
    const int n_mine = n_units > w ? (n_units - w + 3) >> 2 : 0;        // this wave's units: u_begin + w + 4 k

    const char *pool_l = g.pool + (int64_t)a.layer * g.layer_stride + (int64_t)it.kvh * kDecHeadBlk;
    const int64_t bb = g.block_bytes;
    const uint32_t v_half = (uint32_t)(g.block_bytes >> 1);
    const uint32_t lds_w = lds0 + w * kDecWave;
    const int32_t *ids = (const int32_t *)(lds + kDecIds);
    const int last_id = ((P + kBlockTokens - 1) >> 4) - 1 - 2 * u_begin;     // the prefix's last block, counted from the range's first
    const float c = a.scale_log2;
    typedef const __attribute__((address_space(3))) bf16x8 *lds_frag;

    // a unit's two block-table entries: the first two units' come with the item
    const int2 e_first = load_bids(a, blockIdx.x, 2 * w), e_second = load_bids(a, blockIdx.x, 2 * w + 8);
    auto read_entries = [&](int k) {                    // of a later unit, from LDS (the same for the whole wave)
        const int i = 2 * (w + 4 * k);
        return make_int2(ids[i], ids[min(i + 1, last_id)]);
    };
    // K of a unit: two blocks as four 1 KB pieces of four rows each (chunk c of row r at chunk
    // position c ^ r); V verbatim; 8 load instructions per operand
    uint32_t k_off[4], v_off[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        k_off[i] = (lane >> 4) * 256 + (((lane & 15) ^ (4 * i + (lane >> 4))) * 16);
        v_off[i] = lane * 16;
    }
    auto issue_k = [&](int k, int2 e) {
        const uint32_t dst = lds_w + (k & 1) * kDecSlot;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const char *src = pool_l + (int64_t)entry_bid(j ? e.y : e.x) * bb;
            load4_to_lds(dst + j * 4096, src, k_off);
        }
    };
    auto issue_v = [&](int k, int2 e) {
        const uint32_t dst = lds_w + (k & 1) * kDecSlot + kDecPart;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const char *src = pool_l + (int64_t)entry_bid(j ? e.y : e.x) * bb + v_half;
            load4_to_lds(dst + j * 4096, src, v_off);
        }
    };

    // The first range of a (query, KV head) also appends the new token's K and V of that head: the
    // loads are issued here, ahead of the counted ones, the stores come at the very end (a store counts
    // as an outstanding memory operation).  Behind the token the block is zero, as after every append.
    // K: thread -> 16 bytes of one token row.  V^T: thread d -> the 16 tokens of row d, merged.
    // (The new token's own key and value, and the query row that meets them, are needed last of all: requested here, too,
    // where most work-groups or the last of each (query, KV head) will need them.)
    const bool appends = it.split == 0;
    const int slot8 = tid >> 5, d4 = 4 * (tid & 31);   // at the end: eight groups of 32 threads, four columns each
    SelfRaw self_raw{};
    if (kFold) self_raw = load_self(g, a, it.cu, it.kvh, it.kvh * G + min(slot8, G - 1), d4);
    const int t_new = P & 15;
    char *k_dst = nullptr, *v_dst = nullptr;
    uint4 k_put = make_uint4(0, 0, 0, 0), v_old0 = k_put, v_old1 = k_put;
    uint32_t v_put = 0;
    if (appends) {
        const int phys = it.append_bid;
        k_dst = const_cast<char *>(pool_l) + (int64_t)phys * bb + tid * 16;
        v_dst = k_dst + v_half + tid * 16;             // (32 bytes per row d = tid)
        const char *k_src = (const char *)a.k_new + ((int64_t)it.cu * g.Hkv + it.kvh) * 256;
        if ((tid >> 4) == t_new) k_put = *(const uint4 *)(k_src + (tid & 15) * 16);
        if (tid < 128) {
            v_put = *((const uint16_t *)((const char *)a.v_new + ((int64_t)it.cu * g.Hkv + it.kvh) * 256) + tid);
            v_old0 = *(const uint4 *)v_dst;
            v_old1 = *(const uint4 *)(v_dst + 16);
        }
    }

    f32x16 o[4];
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int e = 0; e < 16; ++e) o[db][e] = 0.f;
    float m_run = -INFINITY, l_lane = 0.f;

    if (n_mine > 0) {
        if (n_mine > 2) {                               // the range's block ids, 256 per load (rows of the table are padded to 16 bytes)
            const int32_t *bt = b.block_table + (int64_t)it.q * b.max_blocks + 2 * u_begin;
            const int last_chunk = ((b.max_blocks - 2 * u_begin) >> 2) - 1;
            for (int i = 0; i < 2 * n_units; i += 256)
                load_to_lds(lds0 + kDecIds + i * 4, (const char *)bt, min((i >> 2) + lane, last_chunk) * 16);
        }
        {                                               // the group's query rows, four per load, chunk c of row r at c ^ r
            const char *qp = (const char *)a.q + ((int64_t)it.cu * g.Hq + it.kvh * G) * 256;
            for (int i = 0; i < (G + 3) >> 2; ++i) {
                const int r = 4 * i + (lane >> 4);
                load_to_lds(lds0 + kDecQ + i * 1024, qp, min(r, G - 1) * 256 + (((lane & 15) ^ (r & 15)) * 16));
            }
        }
        issue_k(0, e_first);
        issue_v(0, e_first);
        if (n_mine > 1) {
            issue_k(1, e_second);
            issue_v(1, e_second);
            wait_loads<32>();
        } else {
            wait_loads<16>();
        }
        // Q^T fragments (B operand): lane (row r32, half hh) holds q[row][16*ks + 8*hh .. +8]
        bf16x8 qf[8];
        {
            const int r = min(r32, G - 1);
            const uint32_t qb = lds0 + kDecQ + r * 256 + ((hh ^ (r & 15)) << 4);
#pragma unroll
            for (int ks = 0; ks < 8; ++ks) qf[ks] = *(lds_frag)(uintptr_t)(qb ^ (ks << 5));
        }
        const uint32_t kb = lds_w + r32 * 256 + ((hh ^ (r32 & 15)) << 4);
        const uint32_t vb = lds_w + kDecPart + r32 * 32 + hh * 16;

        // Two units at a time (64 keys: one maximum, one vote on the rescale, two waits), a last odd one by itself.
        // The ring holds both; K of the next two is requested as soon as these two's K fragments are in registers,
        // V likewise.  Loads complete in the order issued, so a wait that leaves N younger ones outstanding has
        // everything older in LDS.
        int2 e0 = e_first, e1 = e_second;              // block-table entries of the units at work
        auto step = [&](auto pair_c, int k) {
            constexpr int N = decltype(pair_c)::value; // units: k .. k + N - 1, k even: unit k + u stands in slot u
            const int left = n_mine - k - N;           // and how many follow
            // (for the first pair K and V were requested unit by unit: only V of the second may be outstanding)
            if (N == 2 && k > 0) wait_loads<16>();
            else wait_loads<8>();
            int2 n0 = make_int2(0, 0), n1 = n0;
            if (left >= 1) n0 = read_entries(k + N);
            if (left >= 2) n1 = read_entries(k + N + 1);
            bf16x8 kf[8 * N];
#pragma unroll
            for (int ks = 0; ks < 8; ++ks)
#pragma unroll
                for (int u = 0; u < N; ++u) kf[N * ks + u] = *(lds_frag)(uintptr_t)((kb + u * kDecSlot) ^ (ks << 5));
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // K area read out
            n0 = make_int2(__builtin_amdgcn_readfirstlane(n0.x), __builtin_amdgcn_readfirstlane(n0.y));
            n1 = make_int2(__builtin_amdgcn_readfirstlane(n1.x), __builtin_amdgcn_readfirstlane(n1.y));
            if (left >= 1) issue_k(k + N, n0);
            if (left >= 2) issue_k(k + N + 1, n1);
            f32x16 s[N];
#pragma unroll
            for (int u = 0; u < N; ++u)
#pragma unroll
                for (int e = 0; e < 16; ++e) s[u][e] = 0.f;
#pragma unroll
            for (int ks = 0; ks < 8; ++ks)
#pragma unroll
                for (int u = 0; u < N; ++u) s[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[N * ks + u], qf[ks], s[u], 0, 0, 0);
            if (left >= 2) wait_loads<16>();
            else if (left == 1) wait_loads<8>();
            else wait_loads<0>();
            bf16x8 vf[8 * N];                          // V^T fragments: in registers before the softmax starts
#pragma unroll
            for (int u = 0; u < N; ++u)
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    vf[8 * u + j] = *(lds_frag)(uintptr_t)(vb + u * kDecSlot + (j >> 2) * kDecHeadBlk + (j & 3) * 1024);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // V area read out
            if (left >= 1) issue_v(k + N, n0);
            if (left >= 2) issue_v(k + N + 1, n1);
            // positions that hold no key: beyond the end of the sequence, and the unused tail of a
            // table block read in place (its count rides in the block-table entry)
#pragma unroll
            for (int u = 0; u < N; ++u) {
                const int key0 = (u_begin + w + 4 * (k + u)) * kDecUnit;
                const int2 e_u = u ? e1 : e0;
                const int pad0 = entry_pad(e_u.x), pad1 = entry_pad(e_u.y);
                if ((pad0 | pad1) != 0 || key0 + kDecUnit > P) {
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        const int in_blk = 8 * ((e >> 2) & 1) + 4 * hh + (e & 3);
                        const int key = key0 + 8 * (e >> 2) + 4 * hh + (e & 3);
                        s[u][e] = (key >= P || in_blk >= kBlockTokens - (e < 8 ? pad0 : pad1)) ? -INFINITY : s[u][e];
                    }
                }
            }
            float mx = s[0][0];
#pragma unroll
            for (int u = 0; u < N; ++u)
#pragma unroll
                for (int e = 0; e < 16; ++e) mx = fmaxf(mx, s[u][e]);
            mx = fmaxf(mx, __shfl_xor(mx, 32));
            const float mxs = mx * c;
            if (__any(mxs > m_run + kDecRescale)) {    // also taken while m_run is still -inf
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
            for (int u = 0; u < N; ++u)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    s[u][e] = __builtin_amdgcn_exp2f(fmaf(s[u][e], c, neg_m));
                    l_lane += s[u][e];
                }
#pragma unroll
            for (int u = 0; u < N; ++u)
#pragma unroll
                for (int kk = 0; kk < 2; ++kk) {
                    bf16x8 pf;
#pragma unroll
                    for (int e = 0; e < 8; ++e) pf[e] = (__bf16)s[u][8 * kk + e];
#pragma unroll
                    for (int db = 0; db < 4; ++db)
                        o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[8 * u + 4 * kk + db], pf, o[db], 0, 0, 0);
                }
            e0 = n0;
            e1 = n1;
        };
        int k = 0;
        for (; k + 1 < n_mine; k += 2) step(std::integral_constant<int, 2>{}, k);
        if (k < n_mine) step(std::integral_constant<int, 1>{}, k);
    }

    // ---- combine the four waves: each writes (max, sum) per row and O as padded rows of floats into
    // its own ring (dead now), then every thread folds the four for a few (row, 4 columns)
    {
        float *wo = (float *)(lds + w * kDecWave);
        const float l_row = l_lane + __shfl_xor(l_lane, 32);
        if (r32 < G) {
#pragma unroll
            for (int db = 0; db < 4; ++db)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    f32x4 v;
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = o[db][4 * q + e];
                    *(f32x4 *)(wo + r32 * kDecRow + 32 * db + 8 * q + 4 * hh) = v;
                }
            if (hh == 0) { wo[32 * kDecRow + 2 * r32] = m_run; wo[32 * kDecRow + 2 * r32 + 1] = l_row; }
        }
    }
    __syncthreads();
    Self self{};
    if (kFold) self = score_self(self_raw, c);
    const int64_t first_slot = (int64_t)it.part0 * g.Hq + (int64_t)it.kvh * G * it.n_splits;
    const uint32_t n_slots = (uint32_t)(it.n_splits * G);
    const SharedPart part_o(a.part_o + first_slot * 128, n_slots * 512), part_ml(a.part_ml + first_slot * 2, n_slots * 8);
    auto fold_waves = [&](int row) {
        RowSum x{-INFINITY, 0.f, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int k = 0; k < 4; ++k) x.M = fmaxf(x.M, ((const float *)(lds + k * kDecWave))[32 * kDecRow + 2 * row]);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float *wk = (const float *)(lds + k * kDecWave);
            const float mk = wk[32 * kDecRow + 2 * row];
            const float wgt = (mk == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(mk - x.M);
            x.L += wgt * wk[32 * kDecRow + 2 * row + 1];
            const f32x4 v = *(const f32x4 *)(wk + row * kDecRow + d4);
#pragma unroll
            for (int e = 0; e < 4; ++e) x.acc[e] += wgt * v[e];
        }
        return x;
    };
    if (!kFold && it.n_splits > 1) {
        for (int row = slot8; row < G; row += 8) {
            const RowSum x = fold_waves(row);
            const int64_t slot = (int64_t)(it.part0 + it.split) * g.Hq + it.kvh * G + row;
            *(f32x4 *)(a.part_o + slot * 128 + d4) = x.acc;
            if (d4 == 0) *(float2 *)(a.part_ml + slot * 2) = make_float2(x.M, x.L);
        }
    } else {
        for (int row = slot8; row < G; row += 8) {
            const RowSum x = fold_waves(row);
            if (it.n_splits == 1) {
                finish_row(g, a, it, row, d4, kFold && row == slot8 ? self : score_self(load_self(g, a, it.cu, it.kvh, it.kvh * G + row, d4), c), x);
            } else {
                const uint32_t off = (uint32_t)(it.split * G + row);
                part_o.put4(off * 512 + d4 * 4, x.acc);
                if (d4 == 0) part_ml.put2(off * 8, x.M, x.L);
            }
        }
    }
    if (kFold && it.n_splits > 1 && last_to_arrive(arrival_counter(a, it), it.n_splits, (int32_t *)(lds + kDecIds))) {
        // a row to 32 threads; of up to four rows two such groups take every other partition each
        const bool two = G <= 4;
        float *s_w = (float *)lds + 8 * kDecRow + slot8 * kFoldBatch;
        const int row = two ? slot8 & 3 : slot8, half = two ? slot8 >> 2 : 0;
        RowSum x{-INFINITY, 0.f, {0.f, 0.f, 0.f, 0.f}};
        if (row < G) x = fold_partials(part_o, part_ml, row, G, it.n_splits, half, two ? 2 : 1, tid & 31, s_w);
        if (two) {
            float *sx = (float *)lds + slot8 * kDecRow;
            *(f32x4 *)(sx + d4) = x.acc;
            if (d4 == 0) { sx[128] = x.M; sx[129] = x.L; }
            __syncthreads();
            const float *other = (const float *)lds + (slot8 | 4) * kDecRow;
            if (half == 0) x.add(other[128], other[129], *(const f32x4 *)(other + d4));
        }
        if (row < G && half == 0) finish_row(g, a, it, row, d4, self, x);
    }
    if (appends) {
        if ((tid >> 4) >= t_new) *(uint4 *)k_dst = k_put;
        if (tid < 128) {
            const uint32_t old[8] = {v_old0.x, v_old0.y, v_old0.z, v_old0.w, v_old1.x, v_old1.y, v_old1.z, v_old1.w};
            uint32_t out[8];
#pragma unroll
            for (int p = 0; p < 8; ++p) {              // positions 2p and 2p + 1 hold tokens vperm(2p), vperm(2p + 1)
                const int ta = vperm(2 * p), tb = vperm(2 * p + 1);
                const uint32_t ea = ta < t_new ? old[p] & 0xffffu : ta == t_new ? v_put : 0u;
                const uint32_t eb = tb < t_new ? old[p] >> 16 : tb == t_new ? v_put : 0u;
                out[p] = ea | (eb << 16);
            }
            *(uint4 *)v_dst = make_uint4(out[0], out[1], out[2], out[3]);
            *(uint4 *)(v_dst + 16) = make_uint4(out[4], out[5], out[6], out[7]);
        }
    }
}

hipError_t launch_decode_bf16(const Geom &g, const BatchDev &b, const AttnArgs &a, const Launch &L)
{
    if (a.n_items == 0) return hipSuccess;
    if (g.D != 128 || g.esize != 2 || g.G > 32) return hipErrorInvalidValue;
    static PerDeviceOnce configured;
    const hipError_t e = configured.run([] {
        const hipError_t e0 = hipFuncSetAttribute((const void *)decode_attn_bf16_kernel<false>, hipFuncAttributeMaxDynamicSharedMemorySize, kDecLds);
        return e0 != hipSuccess ? e0 : hipFuncSetAttribute((const void *)decode_attn_bf16_kernel<true>, hipFuncAttributeMaxDynamicSharedMemorySize, kDecLds);
    });
    if (e != hipSuccess) return e;
    if (a.part_o && !a.arrivals) TC_LAUNCH(decode_attn_bf16_kernel<false>, a.n_items, kDecLds, L, g, b, a);
    else TC_LAUNCH(decode_attn_bf16_kernel<true>, a.n_items, kDecLds, L, g, b, a);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------ merge
// Partials by row combined by a launch of its own, where one CU would take longer over a row tile's than that: 32 threads, four
// columns each, per (suffix token, query head) row and group of partitions; a row's kGroups groups take every kGroups-th
// partition and are combined through LDS.  Bound: the latency of the loads of a short launch, so those of four partitions are issued
// before the first use, and (kEven) before it is known how many there are.  kSelf: a decode step, the new token joins.
template <int kGroups, bool kSelf, bool kEven>
__global__ __launch_bounds__(256) void merge_rows_bf16_kernel(Geom g, BatchDev b, AttnArgs a, int max_splits)
{
    constexpr int kBatch = 4, kRows = 8 / kGroups;
    __shared__ float s_acc[8][132], s_ml[8][2];
    const int tid = threadIdx.x, slot8 = tid >> 5, grp = slot8 % kGroups, d = 4 * (tid & 31);
    const int64_t n_rows = (int64_t)b.total_S * g.Hq;
    const int64_t want = (int64_t)blockIdx.x * kRows + slot8 / kGroups;
    const int row = (int)min(want, n_rows - 1);        // (the last work-group may have rows to spare: they repeat the last one)
    const int n = row / g.Hq, head = row - n * g.Hq;      // n: the token (queries may bring none)
    const PartSlots slots = part_slots<kEven>(b, n);
    float2 ml[kBatch];
    f32x4 po[kBatch];
    auto fetch = [&](int s0) {
#pragma unroll
        for (int j = 0; j < kBatch; ++j) {
            if (kGroups * j >= max_splits) break;
            const int64_t slot = (int64_t)min(slots.first + s0 + kGroups * j, slots.last) * g.Hq + head;
            ml[j] = *(const float2 *)(a.part_ml + slot * 2);
            po[j] = *(const f32x4 *)(a.part_o + slot * 128 + d);
        }
    };
    SelfRaw self;
    if (kSelf) self = load_self(g, a, n, head / g.G, head, d);
    if (kEven || slots.count > 0) fetch(grp);
    const int ns = slots.count;
    RowSum x{-INFINITY, 0.f, {0.f, 0.f, 0.f, 0.f}};
    for (int s0 = grp; s0 < ns; s0 += kGroups * kBatch) {
        if (s0 > grp) fetch(s0);
#pragma unroll
        for (int j = 0; j < kBatch; ++j)
            if (s0 + kGroups * j < ns) x.add(ml[j].x, ml[j].y, po[j]);
    }
    if (kGroups > 1) {
        *(f32x4 *)&s_acc[slot8][d] = x.acc;
        if (d == 0) { s_ml[slot8][0] = x.M; s_ml[slot8][1] = x.L; }
        __syncthreads();
    }
    if (grp > 0 || want >= n_rows || ns <= 1) return;          // (a row in one range was written by the attention kernel)
    if (kSelf) add_self(x, score_self(self, a.scale_log2));
#pragma unroll
    for (int k = 1; k < kGroups; ++k) x.add(s_ml[slot8 + k][0], s_ml[slot8 + k][1], *(const f32x4 *)&s_acc[slot8 + k][d]);
    write_row((unsigned short *)a.out + (int64_t)row * 128 + d, x);
}

template <bool kSelf, bool kEven>
static hipError_t launch_merge_rows(const Geom &g, const BatchDev &b, const AttnArgs &a, int max_splits, const Launch &L)
{
    const int n_rows = b.total_S * g.Hq;
    if (n_rows == 0) return hipSuccess;
    if (max_splits < 1 || !b.part_tab) return hipErrorInvalidValue;
    if (max_splits <= 4) TC_LAUNCH((merge_rows_bf16_kernel<1, kSelf, kEven>), (n_rows + 7) / 8, 0, L, g, b, a, max_splits);
    else if (max_splits <= 8) TC_LAUNCH((merge_rows_bf16_kernel<2, kSelf, kEven>), (n_rows + 3) / 4, 0, L, g, b, a, max_splits);
    else if (max_splits <= 16) TC_LAUNCH((merge_rows_bf16_kernel<4, kSelf, kEven>), (n_rows + 1) / 2, 0, L, g, b, a, max_splits);
    else TC_LAUNCH((merge_rows_bf16_kernel<8, kSelf, kEven>), n_rows, 0, L, g, b, a, max_splits);
    return hipGetLastError();
}

hipError_t launch_merge_rows_bf16(const Geom &g, const BatchDev &b, const AttnArgs &a, int max_splits, bool decode, const Launch &L)
{
    if (decode) return b.part_stride > 0 ? launch_merge_rows<true, true>(g, b, a, max_splits, L) : launch_merge_rows<true, false>(g, b, a, max_splits, L);
    return b.part_stride > 0 ? launch_merge_rows<false, true>(g, b, a, max_splits, L) : launch_merge_rows<false, false>(g, b, a, max_splits, L);
}

}  // namespace tc
