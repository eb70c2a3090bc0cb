// Combining the partials of a split range inside the launch that makes them: every work-group of a group stores its own, counts
// itself in, and the last one to do so reads them all and writes the result.  Nobody waits for anybody.
//
// The alternative is a launch of its own behind this one.  On this chip that is 1.3 us between the two and 2.5 us or more for a
// kernel that starts, fetches its indices, then the partials, and ends; counting in is 0.8 us and the fold as much or a little
// more, on one CU.  So it pays while the partials of a group are small (tens of KB: the row-wise kernels), and where they
// are large a launch that reads them with the whole chip stays the better one.
//
// What makes it correct across the eight L2s.  Partials, counter and nothing else are shared between work-groups of a launch,
// and all of them are accessed at device scope: stores and loads with sc1, for which the memory system, not the L2
// that happens to be nearer, is the point of coherence (the same instructions that relaxed atomic loads and stores at agent
// scope become; the builtins are used for their 16 bytes).  Order: a wave waits until its stores are complete (vmcnt, in which
// stores count), the barrier collects all waves, then one thread counts the work-group in; the reader's loads are issued
// behind the barrier behind that thread's answer.  An agent-scope release and acquire in their place would write back and
// invalidate whole L2s: 32 sequences' decode step 37.6 us a layer instead of 32.5.
//
// A row tile's counter has 128 bytes of its own behind the plan's device copy (132 arrivals at four neighbouring counters took
// 8 us), zeroed with the plan's upload without crossing the host link, and the last work-group sets it back to zero, so that every
// launch of the plan - replays of a graph, too - finds it so.  Where the workspace of fixed size has no room for them, the counter
// is a field of one of the tile's work items, which are 128 bytes as well and uploaded with the field at zero.  (Nobody else writes
// the items, and a work-group's scalar load of its own item ignores the field.)  An item that was counted in comes from memory and
// not from the L2s in the next launch: one decode step of 854 tokens, 32 / 8 heads, 9 ranges 7.45 us a layer instead of 7.05; two
// queries of 0.2 k + 30 tokens in fp32, two ranges 13.0 instead of 12.6.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "tc_types.h"

namespace tc {

typedef float part_f32x4 __attribute__((ext_vector_type(4)));

constexpr int kDeviceScope = 16;                     // sc1, in the buffer instructions' cache policy

// Memory that work-groups of one launch share: `bytes` (at most 2 GiB) from `base` on.  Reads beyond them give zero: the whole
// offset is in the vector register, for the hardware does not check the scalar one.
struct SharedPart {
    __amdgpu_buffer_rsrc_t r;
    __device__ __forceinline__ SharedPart(float *base, uint32_t bytes) : r(__builtin_amdgcn_make_buffer_rsrc(base, 0, bytes, 0x00020000)) {}
    __device__ __forceinline__ void put4(uint32_t off, part_f32x4 v) const
    {
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), r, off, 0, kDeviceScope);
    }
    __device__ __forceinline__ void put2(uint32_t off, float x, float y) const
    {
        typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
        const u32x2 v = {__float_as_uint(x), __float_as_uint(y)};
        __builtin_amdgcn_raw_buffer_store_b64(v, r, off, 0, kDeviceScope);
    }
    __device__ __forceinline__ part_f32x4 get4(uint32_t off) const
    {
        return __builtin_bit_cast(part_f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, kDeviceScope));
    }
    __device__ __forceinline__ float2 get2(uint32_t off) const
    {
        const auto v = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, kDeviceScope);
        return make_float2(__uint_as_float(v[0]), __uint_as_float(v[1]));
    }
};

__device__ __forceinline__ int32_t *arrival_counter(const AttnArgs &a, const AttnItem &it)
{
    return a.arrivals + (int64_t)it.arrival * (sizeof(AttnItem) / sizeof(int32_t));
}

// Counts the work-group in as one of `n` behind its stores to shared memory; true, in all of its threads, for the last one.
// `s_flag`: a word of LDS that nothing else uses by now.
__device__ __forceinline__ bool last_to_arrive(int32_t *counter, int n, int32_t *s_flag)
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
        const int before = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (before == n - 1) __hip_atomic_store(counter, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *s_flag = before == n - 1;
    }
    __syncthreads();
    return *s_flag != 0;
}

// (maximum, sum, output) of a row's keys so far, in one thread's four columns.
struct RowSum {
    float M, L;
    part_f32x4 acc;
    __device__ __forceinline__ void add(float m, float l, part_f32x4 o)
    {
        const float Mn = fmaxf(M, m);
        const float r = M == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(M - Mn);
        // (no maximum: no key for this row - l and o are 0 - or only scores that are NaN - so are they, and so is the row)
        const float wgt = m == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m - Mn);
        L = L * r + l * wgt;
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] = acc[e] * r + o[e] * wgt;
        M = Mn;
    }
};

constexpr uint32_t kNowhere = 0x80000000u;            // an offset beyond any SharedPart: reads as zero

// Over 16 neighbouring lanes, every lane's value exchanged with DPP; over 32, the two rows of 16 as well.
template <typename F>
__device__ __forceinline__ float reduce16(float x, F op)
{
    auto dpp = [](float v, auto ctrl) { return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), decltype(ctrl)::value, 0xf, 0xf, false)); };
    x = op(x, dpp(x, std::integral_constant<int, 0xb1>{}));      // lane ^ 1
    x = op(x, dpp(x, std::integral_constant<int, 0x4e>{}));      // lane ^ 2
    x = op(x, dpp(x, std::integral_constant<int, 0x141>{}));     // mirrored in each eight
    return op(x, dpp(x, std::integral_constant<int, 0x140>{}));  // mirrored in the sixteen
}
template <typename F>
__device__ __forceinline__ float reduce32(float x, F op)
{
    const unsigned u = __float_as_uint(reduce16(x, op));
    const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    return op(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float max16(float x) { return reduce16(x, [](float a, float b) { return fmaxf(a, b); }); }
__device__ __forceinline__ float sum16(float x) { return reduce16(x, [](float a, float b) { return a + b; }); }
__device__ __forceinline__ float max32(float x) { return reduce32(x, [](float a, float b) { return fmaxf(a, b); }); }
__device__ __forceinline__ float sum32(float x) { return reduce32(x, [](float a, float b) { return a + b; }); }

// Partials `first`, first + step, .. of the `n` of a row, folded by 32 neighbouring threads of a wave (lane: 0 .. 31), four
// columns each; row r's partial s stands in slot s * rows + r.  What this takes is the latency of its own instructions - a wave
// alone on its SIMD - and one round trip, so: up to 36 partials are requested at once, and slots
// beyond the group's last read as zeros; their weights come from one lane each and go around through LDS, where
// one shuffle and one branch a partial took three times as long (17 partials: 3.4 -> 1.3 us).
constexpr int kFoldBatch = kDecodeFold, kFoldGroup = 12;
__device__ __forceinline__ RowSum fold_partials(const SharedPart &po, const SharedPart &pml, int row, int rows, int n, int first, int step, int lane, float *s_w)
{
    RowSum x{-INFINITY, 0.f, {0.f, 0.f, 0.f, 0.f}};
    float l_lane = 0.f;
    const uint32_t o_step = (uint32_t)(rows * step) * 512, ml_step = (uint32_t)(rows * step) * 8;
    uint32_t o_at = (uint32_t)(first * rows + row) * 512 + lane * 16, ml_at = (uint32_t)(first * rows + row) * 8 + lane * ml_step;
    for (int m = (n - first + step - 1) / step; m > 0; m -= kFoldBatch, o_at += kFoldBatch * o_step, ml_at += kFoldBatch * ml_step) {
        float2 ml[2] = {pml.get2(ml_at), make_float2(0.f, 0.f)};
        if (m > 32) ml[1] = pml.get2(ml_at + 32 * ml_step);
        part_f32x4 o[kFoldBatch];
        auto fetch = [&](int j0) {
#pragma unroll
            for (int j = j0; j < j0 + kFoldGroup; ++j) o[j] = po.get4(o_at + j * o_step);
        };
        auto use = [&](int j0) {
            part_f32x4 w[kFoldGroup / 4];
#pragma unroll
            for (int k = 0; k < kFoldGroup / 4; ++k) w[k] = *(const part_f32x4 *)(s_w + j0 + 4 * k);
#pragma unroll
            for (int j = 0; j < kFoldGroup; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) x.acc[e] += w[j >> 2][j & 3] * o[j0 + j][e];
        };
        fetch(0);
        if (m > kFoldGroup) fetch(kFoldGroup);
        if (m > 2 * kFoldGroup) fetch(2 * kFoldGroup);
        const float m0 = lane < m ? ml[0].x : -INFINITY, m1 = lane + 32 < min(m, kFoldBatch) ? ml[1].x : -INFINITY;
        const float Mn = fmaxf(x.M, max32(fmaxf(m0, m1))), r = x.M == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(x.M - Mn);
        const float w0 = m0 == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m0 - Mn), w1 = m1 == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m1 - Mn);
        l_lane = l_lane * r + w0 * ml[0].y + (lane + 32 < kFoldBatch ? w1 * ml[1].y : 0.f);
        x.M = Mn;
#pragma unroll
        for (int e = 0; e < 4; ++e) x.acc[e] *= r;
        s_w[lane] = w0;
        if (lane < kFoldBatch - 32) s_w[32 + lane] = w1;
        use(0);
        if (m > kFoldGroup) use(kFoldGroup);
        if (m > 2 * kFoldGroup) use(2 * kFoldGroup);
    }
    x.L = sum32(l_lane);
    return x;
}

}  // namespace tc
