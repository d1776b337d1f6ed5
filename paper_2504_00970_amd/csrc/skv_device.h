// Device helpers shared by the kernels of libsentencekv (gfx950, wave64): DPP adds and scans, the block scan
// of the 1024-thread kernels, the order-preserving image of a score.
#pragma once

#include "skv_internal.h"

namespace skv {

constexpr int kBlockWaves = kBlockThreads / kWave;

// x + (x moved by a DPP pattern): quad_perm [1,0,3,2] = 0xB1, [2,3,0,1] = 0x4E, row_ror:n = 0x120 + n
template <int CTRL>
__device__ __forceinline__ float dpp_add(float x) {
    const int moved = __builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, false);
    return x + __int_as_float(moved);
}

// sum over the lanes l and l ^ 32, in both
__device__ __forceinline__ float sum_halves(float x) {
    const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(a[0]) + __uint_as_float(a[1]);
}

// sum over the lanes l and l ^ 16, in both
__device__ __forceinline__ float sum_rows16(float x) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(a[0]) + __uint_as_float(a[1]);
}

// Block `id` of n in the order in which an XCD takes neighbours: the hardware deals consecutive blocks to the eight XCDs in turn, and of 8 * kXcdRun of them each
// XCD takes kXcdRun in a row here (blocks past the last whole group as they come).
constexpr uint32_t kXcdRun = 32;               // a power of two
__device__ __forceinline__ uint32_t xcd_run(uint32_t id, uint32_t n) {
    const uint32_t group = id / (8 * kXcdRun) * (8 * kXcdRun);
    return group + 8 * kXcdRun <= n ? group + (id & 7) * kXcdRun + ((id >> 3) & (kXcdRun - 1)) : id;
}

// 16 bytes that this launch reads or writes once (K/V rows, mean keys): the non-temporal forms.  Measured on one-shot reads of
// a 2.15 GB key pool (a wave requests 4 KB and ends): 6.45 TB/s with plain loads, 7.15 TB/s with these.
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 ld_stream(const void* p) {
    const u32x4_t t = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(p));
    return make_uint4(t[0], t[1], t[2], t[3]);
}
__device__ __forceinline__ void st_stream(void* p, const uint4& v) {
    const u32x4_t t = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(t, reinterpret_cast<u32x4_t*>(p));
}

// 16 bytes per lane from global memory at base + off straight to LDS at `lds` + 16 * lane (base and lds wave-uniform), non-temporal: one-shot
// reads of the same pool run at 7.1 TB/s with these, 6.2 with plain loads.  Asynchronous: counted by vmcnt, and only the
// kernel's own waits (wait_loads) order it against reads of the destination.  Written out because the compiler, where it
// knows that LDS is written, waits for everything outstanding before the next LDS read.  m0 (the LDS address) is declared as
// written: the compiler merges its own writes of m0 between uses, which it must not do across this.  (It warns that m0 is reserved, that
// is, not saved around the statement: nothing here expects it to be.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void load_lds_stream_at(const char* base, uint32_t off, uint32_t at /* address in LDS */) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(__builtin_amdgcn_readfirstlane((int)at)), "v"(off),
                 "s"(base)
                 : "memory", "m0");
}
__device__ __forceinline__ void load_lds_stream(const char* base, uint32_t off, char* lds) {
    load_lds_stream_at(base, off, (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds);
}
#pragma clang diagnostic pop
// waits until at most N of the wave's vector memory instructions are outstanding
template <int N>
__device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

// Stores that other blocks of the same launch read (possibly on another XCD, each with its own L2): device-scope
// relaxed atomic accesses go through to the level all XCDs share, so no L2 write-back / invalidate is needed around
// the arrival counters that publish them.
__device__ __forceinline__ void st_agent(float* p, float v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_agent(int32_t* p, int32_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_agent(unsigned int* p, unsigned int v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float ld_agent(const float* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int32_t ld_agent(const int32_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned int ld_agent(const unsigned int* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long ld_agent64(const float* p) {       // two consecutive floats
    return __hip_atomic_load(reinterpret_cast<const unsigned long long*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_agent64(float2* p, float x, float y) {                 // two floats in one store
    __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), ((unsigned long long)__float_as_uint(y) << 32) | __float_as_uint(x),
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Barrier behind which another thread of the block publishes what this block has stored (an arrival counter).  The
// workgroup barrier by itself does not wait for a wave's outstanding global stores (the waves of a block share their CU's
// cache, so the compiler leaves the store counter alone at workgroup scope): each wave waits for its own first.
// ASSUMPTION (of the kernels that publish with a counter: skv_attend, the two- and three-launch forms of
// skv_decode_step): a device-scope relaxed atomic store that has left the store counter (vmcnt == 0) has reached the
// level all XCDs share, so a device-scope relaxed load issued by any block after it observed the later counter
// increment returns the stored value.  The language's memory model does not promise this for relaxed accesses to
// different locations; it is how write-through stores and the store counter behave on this chip, and it is guarded by
// test_repeated_launches_reproduce_their_results.  The segmentation that reports its count relies on the same at system
// scope: its relaxed system-scope stores, once they have left the store counter, are in the memory that the host, copies and
// kernels of other streams read, so that whoever sees the count in host memory (stored relaxed, behind an arrival counter at
// device scope) finds them; guarded by test_segment_returns_behind_earlier_work.  The single-launch step does not rely on it: there every word
// carries its own validity tag (st_tagged).
__device__ __forceinline__ void block_sync_after_stores() {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
}
__device__ __forceinline__ float lo_f(unsigned long long v) { return __uint_as_float((uint32_t)v); }
__device__ __forceinline__ float hi_f(unsigned long long v) { return __uint_as_float((uint32_t)(v >> 32)); }

// A float and the tag of the launch that produced it, in one 64-bit word written and read with single relaxed
// device-scope atomic accesses.  A reader that finds the tag it expects holds the value that belongs to it: nothing has
// to be ordered against any other location (per-location coherence of atomics is all that is used), so there is no
// arrival counter, no wait for store acknowledgements and no cache maintenance between producer and consumer.
__device__ __forceinline__ void st_tagged(unsigned long long* p, float v, uint32_t tag) {
    __hip_atomic_store(p, ((unsigned long long)tag << 32) | (unsigned long long)__float_as_uint(v), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long ld_tagged(const unsigned long long* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t tag_of(unsigned long long w) { return (uint32_t)(w >> 32); }
__device__ __forceinline__ float val_of(unsigned long long w) { return __uint_as_float((uint32_t)w); }

// Order-preserving 32-bit image of a float: larger score <=> larger key.
__device__ __forceinline__ uint32_t score_key(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return 0u;          // NaN ranks below everything
    if (u == 0x80000000u) u = 0u;                             // -0 == +0
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// v + (v moved by a DPP pattern; lanes without a source, or rows masked out, add 0)
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t dpp_add_u32(uint32_t v) {
    return v + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROW_MASK, 0xf, true);
}
// inclusive prefix sum over the 64 lanes of a wave: row_shr 1,2,4,8 then row_bcast 15 and 31
__device__ __forceinline__ uint32_t wave_scan_u32(uint32_t v) {
    v = dpp_add_u32<0x111, 0xf>(v);
    v = dpp_add_u32<0x112, 0xf>(v);
    v = dpp_add_u32<0x114, 0xf>(v);
    v = dpp_add_u32<0x118, 0xf>(v);
    v = dpp_add_u32<0x142, 0xa>(v);
    v = dpp_add_u32<0x143, 0xc>(v);
    return v;
}
// v and (v moved by a DPP pattern), the larger of the two; lanes without a source, or rows masked out, keep v
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t dpp_max_u32(uint32_t v) {
    return max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROW_MASK, 0xf, true));
}
// inclusive running maximum over the 64 lanes of a wave (same DPP steps as the prefix sum)
__device__ __forceinline__ uint32_t wave_scan_max_u32(uint32_t v) {
    v = dpp_max_u32<0x111, 0xf>(v);
    v = dpp_max_u32<0x112, 0xf>(v);
    v = dpp_max_u32<0x114, 0xf>(v);
    v = dpp_max_u32<0x118, 0xf>(v);
    v = dpp_max_u32<0x142, 0xa>(v);
    v = dpp_max_u32<0x143, 0xc>(v);
    return v;
}
// Inclusive scan over the block's threads (thread order); one barrier.  A `slot` is used once per call
// of the selection.
__device__ __forceinline__ uint32_t block_scan_u32(uint32_t val, uint32_t* slot, uint32_t* total) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint32_t x = wave_scan_u32(val);
    if (lane == 63) slot[w] = x;
    __syncthreads();
    // prefix over the 16 wave totals: one more wave scan instead of 16 reads per thread
    const uint32_t t = slot[lane & (kBlockWaves - 1)];
    const uint32_t ti = wave_scan_u32(lane < kBlockWaves ? t : 0u);
    *total = (uint32_t)__builtin_amdgcn_readlane((int)ti, kBlockWaves - 1);
    const uint32_t pre = (uint32_t)__builtin_amdgcn_readlane((int)(ti - t), w);     // lane w < 16 holds slot[w]
    return x + pre;
}

}  // namespace skv
