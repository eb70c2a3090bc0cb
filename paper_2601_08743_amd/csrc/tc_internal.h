// Internal declarations shared by the host side of libtablecache and its kernel files.
// Nothing here is part of the public ABI (see include/tablecache.h).
#pragma once
#include <hip/hip_runtime.h>
#include <atomic>
#include <hip/hip_ext.h>
#include <stdint.h>

#include "tc_types.h"

namespace tc {

// Where a kernel goes: the stream, and optionally two events that receive the dispatch's own begin
// and end timestamps (per-kernel timing without bracketing packets on the stream).
struct Launch {
    hipStream_t stream;
    hipEvent_t start, stop;
};
#define TC_LAUNCH(kernel, grid, lds_bytes, L, ...) \
    hipExtLaunchKernelGGL(kernel, dim3(grid), dim3(256), (lds_bytes), (L).stream, (L).start, (L).stop, 0, __VA_ARGS__)

// Work item `k` through scalar loads: the plan was uploaded before the launch and nothing writes it, which
// the compiler cannot see for itself in kernels that also store to memory.
__device__ __forceinline__ AttnItem load_item(const AttnArgs &a, unsigned k)
{
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    typedef const __attribute__((address_space(4))) u32x4 *const_words;
    const const_words src = (const_words)(uintptr_t)(a.items + k);
    union { u32x4 w[sizeof(AttnItem) / 16]; AttnItem item; } u;
#pragma unroll
    for (unsigned j = 0; j < sizeof(AttnItem) / 16; ++j) u.w[j] = src[j];
    return u.item;
}

// Two neighbouring block-table entries of item `k`, from bid[j] (j even, the same for the whole wave) on.
__device__ __forceinline__ int2 load_bids(const AttnArgs &a, unsigned k, int j)
{
    typedef int32_t i32x2 __attribute__((ext_vector_type(2)));
    typedef const __attribute__((address_space(4))) i32x2 *const_pair;
    const i32x2 v = *(const_pair)(uintptr_t)(&a.items[k].bid[j]);
    return make_int2(v.x, v.y);
}

// Where suffix token n's partials stand (kernels that keep them by row): its first slot, how many there are, and the
// last slot that may be read in their place.  Evenly spaced slots are known before the table answers, so their
// loads need not wait for it.
struct PartSlots { int first, count, last; };
template <bool kEven>
__device__ __forceinline__ PartSlots part_slots(const BatchDev &b, int n)
{
    if (kEven) return PartSlots{n * b.part_stride, b.part_tab[n], (n + 1) * b.part_stride - 1};
    const int first = b.part_tab[n], end = b.part_tab[n + 1];
    return PartSlots{first, end - first, end - 1};
}

// A kernel's dynamic-LDS limit (hipFuncSetAttribute) is a property of the kernel on one device: each
// launcher keeps one of these per kernel and raises the limit the first time it launches on a device.
// (Two threads that race on a device's first launch both set the same value.)
struct PerDeviceOnce {
    static constexpr int kDevices = 64;
    std::atomic<unsigned char> done[kDevices];
    template <typename F>
    hipError_t run(F &&set_attributes)
    {
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        if (dev < 0 || dev >= kDevices) return hipErrorInvalidDevice;
        if (done[dev].load(std::memory_order_acquire)) return hipSuccess;
        e = set_attributes();
        if (e == hipSuccess) done[dev].store(1, std::memory_order_release);
        return e;
    }
};

// kv_stitch.hip
hipError_t launch_upload(int32_t *dst, const int32_t *pinned_src, size_t ints, size_t zeros_at, size_t zeros, const Launch &L);
hipError_t launch_stitch(const Geom &g, const BatchDev &b, int l0, int l1, bool rope, const Launch &L);
hipError_t launch_format(const Geom &g, const void *raw, int64_t v_part, int n_tokens, int first_block, int l0,
                         int l1, const Launch &L);
hipError_t launch_readback(const Geom &g, int layer, const int32_t *blocks_dev, int n_tokens,
                           void *k_out_dev, void *v_out_dev, hipStream_t s);
// prefill_attn_bf16.hip / prefill_attn_f32.hip
hipError_t launch_attn_bf16(const Geom &g, const BatchDev &b, const AttnArgs &a, int row_blocks, bool pipelined,
                            const Launch &L);
// decode_attn_bf16.hip
hipError_t launch_attn_pp_bf16(const Geom &g, const BatchDev &b, const AttnArgs &a, const Launch &L);
hipError_t launch_decode_bf16(const Geom &g, const BatchDev &b, const AttnArgs &a, const Launch &L);
hipError_t launch_merge_rows_bf16(const Geom &g, const BatchDev &b, const AttnArgs &a, int max_splits, bool decode, const Launch &L);
hipError_t launch_attn_short_bf16(const Geom &g, const BatchDev &b, const AttnArgs &a, const Launch &L);
hipError_t launch_attn_f32(const Geom &g, const BatchDev &b, const AttnArgs &a, const Launch &L);
hipError_t launch_merge_f32(const Geom &g, const BatchDev &b, const AttnArgs &a, const Launch &L);
hipError_t launch_merge_bf16(const Geom &g, const AttnArgs &a, const MergeGroup *groups, int n_groups,
                             int row_blocks, int max_splits, const Launch &L);

}  // namespace tc
