// Prefill kernels: sentence segmentation (Sec. 4.1, Alg. 1 prefilling phase) and per-bucket mean key
// vectors (Eq. 1).  gfx950, wave64.
#include "skv_internal.h"
#include "skv_device.h"

#include <type_traits>

namespace skv {

// ------------------------------------------------------------------------------------------------
// Segmentation.  A token closes a bucket iff it is a terminator; seg_id is the exclusive prefix sum
// of the terminator flags.  Two launches over blocks of kSegTokPerBlock tokens:
//   seg_count : per block (number of terminators, 1 + position of the last terminator or 0)
//   seg_scan  : block prefix from the preceding blocks' partials, wave-level scan inside the block,
//               then each thread walks its 4 tokens and emits seg_id and, at every bucket end,
//               the bucket's start and length.
// The scan operator on (count, last_end) pairs is (a.count + b.count, max(a.last_end, b.last_end)).
// ------------------------------------------------------------------------------------------------

__device__ __forceinline__ bool is_terminator(const uint32_t* __restrict__ bitmap, int32_t vocab, int32_t id) {
    if (id < 0 || id >= vocab) return false;
    return (bitmap[id >> 5] >> (id & 31)) & 1u;
}

struct SegLocal {
    int flags;   // bit k set: token i0 + k is a terminator
    int cnt;
    int last;    // 1 + position of the thread's last terminator, 0 if none
};

__device__ __forceinline__ SegLocal seg_load(const int32_t* __restrict__ tok, int32_t T,
                                             const uint32_t* __restrict__ bitmap, int32_t vocab, int32_t i0) {
    int32_t t[kSegTokPerThread];
    if (i0 + kSegTokPerThread <= T) {
        const int4 v = *reinterpret_cast<const int4*>(tok + i0);
        t[0] = v.x; t[1] = v.y; t[2] = v.z; t[3] = v.w;
    } else {
#pragma unroll
        for (int k = 0; k < kSegTokPerThread; ++k) t[k] = (i0 + k < T) ? tok[i0 + k] : -1;
    }
    SegLocal r{0, 0, 0};
#pragma unroll
    for (int k = 0; k < kSegTokPerThread; ++k) {
        if (i0 + k < T && is_terminator(bitmap, vocab, t[k])) {
            r.flags |= 1 << k;
            r.cnt += 1;
            r.last = i0 + k + 1;
        }
    }
    return r;
}

__device__ __forceinline__ void wave_reduce_sum_max(int& s, int& m) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        s += __shfl_xor(s, off);
        m = max(m, __shfl_xor(m, off));
    }
}

// Block-wide (sum, max) over kSegThreads threads; result valid in every thread.
__device__ __forceinline__ void block_reduce_sum_max(int& s, int& m, int* sh /*[2 * waves]*/) {
    constexpr int kWaves = kSegThreads / kWave;
    wave_reduce_sum_max(s, m);
    const int w = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) { sh[w] = s; sh[kWaves + w] = m; }
    __syncthreads();
    s = 0; m = 0;
#pragma unroll
    for (int i = 0; i < kWaves; ++i) { s += sh[i]; m = max(m, sh[kWaves + i]); }
}

__global__ __launch_bounds__(kSegThreads) void seg_count_kernel(const int32_t* __restrict__ tok, int32_t T,
                                                                const uint32_t* __restrict__ bitmap, int32_t vocab,
                                                                unsigned long long* __restrict__ part) {
    __shared__ int sh[2 * (kSegThreads / kWave)];
    const int32_t i0 = (blockIdx.x * kSegThreads + threadIdx.x) * kSegTokPerThread;
    SegLocal loc = seg_load(tok, T, bitmap, vocab, i0);
    int s = loc.cnt, m = loc.last;
    block_reduce_sum_max(s, m, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = ((unsigned long long)(unsigned)s << 32) | (unsigned)m;
}

__global__ __launch_bounds__(kSegThreads) void seg_scan_kernel(const int32_t* __restrict__ tok, int32_t T,
                                                               const uint32_t* __restrict__ bitmap, int32_t vocab,
                                                               const unsigned long long* __restrict__ part,
                                                               int32_t* __restrict__ seg_id, int32_t* __restrict__ sent_off,
                                                               int32_t* __restrict__ sent_len, int32_t cap_sent,
                                                               int32_t* __restrict__ n_sent) {
    constexpr int kWaves = kSegThreads / kWave;
    __shared__ int sh[2 * kWaves];
    __shared__ int sh_scan[2 * kWaves];
    if (T == 0) {                       // launched with one block
        if (threadIdx.x == 0) { *n_sent = 0; sent_off[0] = 0; }
        return;
    }
    // prefix of the blocks before this one
    int base_cnt = 0, base_last = 0;
    for (int j = threadIdx.x; j < (int)blockIdx.x; j += kSegThreads) {
        const unsigned long long p = part[j];
        base_cnt += (int)(p >> 32);
        base_last = max(base_last, (int)(p & 0xffffffffu));
    }
    block_reduce_sum_max(base_cnt, base_last, sh);

    const int32_t i0 = (blockIdx.x * kSegThreads + threadIdx.x) * kSegTokPerThread;
    const SegLocal loc = seg_load(tok, T, bitmap, vocab, i0);

    // inclusive wave scan of (cnt, last)
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int c = loc.cnt, l = loc.last;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int tc = __shfl_up(c, off), tl = __shfl_up(l, off);
        if (lane >= off) { c += tc; l = max(l, tl); }
    }
    if (lane == 63) { sh_scan[w] = c; sh_scan[kWaves + w] = l; }
    __syncthreads();
    int ec = __shfl_up(c, 1), el = __shfl_up(l, 1);       // exclusive within the wave
    if (lane == 0) { ec = 0; el = 0; }
    for (int i = 0; i < w; ++i) { ec += sh_scan[i]; el = max(el, sh_scan[kWaves + i]); }

    int seg = base_cnt + ec;
    int start = max(base_last, el);
#pragma unroll
    for (int k = 0; k < kSegTokPerThread; ++k) {
        const int32_t i = i0 + k;
        if (i >= T) break;
        seg_id[i] = seg;
        const bool term = (loc.flags >> k) & 1;
        const bool closes = term || i == T - 1;
        if (closes) {
            if (seg < cap_sent) { sent_off[seg] = start; sent_len[seg] = i + 1 - start; }
            if (i == T - 1) {
                *n_sent = seg + 1;
                if (seg + 1 <= cap_sent) sent_off[seg + 1] = T;
            }
            start = i + 1;
            seg += 1;
        }
    }
}

// The same in ONE launch, for prompts of up to kSegOneMaxTok tokens: a block of 1024 threads owns 4096 tokens, keeps the
// terminator bitmap in LDS and counts the terminators of all tokens before its own by itself, which is cheaper than a second
// launch (4 tokens per thread and preceding block, from L2).  Bound by latency: two dependent memory round trips and a block
// scan.  REPORT: the block that finishes last also stores S to pinned host memory, when the results of every block are where the
// host and all XCDs see them, so that the host can poll the word instead of copying it and waiting for the stream.  They are written
// there store by store; a release at system scope goes through an XCD's whole L2.  Us a call as the host sees it, with ordinary stores, a release by a wave of every
// block, and words and blocks read one after the other / now, both in turn in one program (medians): 1531 tokens 16.4 / 16.7, 8192 16.9 / 16.8, 32768 19.3 / 18.9, 131072
// 27.2 / 24.2; behind a kernel that writes 64 MB 19.1 / 18.8, 20.4 / 19.8, 24.2 / 23.0, 38.6 / 32.5.
template <bool REPORT>
__global__ __launch_bounds__(kBlockThreads) void seg_one_kernel(const int32_t* __restrict__ tok, int32_t T,
                                                                const uint32_t* __restrict__ bitmap, int32_t vocab,
                                                                int32_t* __restrict__ seg_id, int32_t* __restrict__ sent_off,
                                                                int32_t* __restrict__ sent_len, int32_t cap_sent,
                                                                int32_t* __restrict__ n_sent, unsigned long long* arrive,
                                                                unsigned int* host_word) {
    extern __shared__ uint32_t sm_bits[];                       // [words]
    __shared__ uint32_t sm_cnt[kBlockWaves], sm_last[kBlockWaves], sm_pre[2][kBlockWaves];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int words = (vocab + 31) >> 5;
    const int32_t block0 = blockIdx.x * kSegOneBlockTok, i0 = block0 + 4 * tid;
    int32_t t[4];
    if (i0 + 4 <= T) {
        const int4 v = *reinterpret_cast<const int4*>(tok + i0);
        t[0] = v.x; t[1] = v.y; t[2] = v.z; t[3] = v.w;
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) t[k] = i0 + k < T ? tok[i0 + k] : -1;
    }
    for (int i = tid; i < words; i += 4 * kBlockThreads) {      // four at a time: 16 KB of bitmap in one round trip
        uint32_t v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = bitmap[min(i + u * kBlockThreads, words - 1)];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (i + u * kBlockThreads < words) sm_bits[i + u * kBlockThreads] = v[u];
    }
    __syncthreads();
    // REPORT: results are written through to memory (every store on its own, system scope), so that a wave that has waited for its stores has nothing left in the L2.
    auto put = [](int32_t* p, int32_t v) {
        if (REPORT) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        else *p = v;
    };
    auto is_term = [&](int32_t id) -> bool {
        return (uint32_t)id < (uint32_t)vocab && ((sm_bits[(uint32_t)id >> 5] >> (id & 31)) & 1u);
    };
    // Terminators before the block: number, and 1 + position of the last one (0: none).  Four preceding blocks at a time, what is left over one by one.  Us of kernel, one
    // by one / four at a time with the last four made up / this: 8192 tokens 4.4 / 4.7 / 4.4, 32768 7.2 / 7.05 / 6.95, 131072 18.2 / 16.8 / 15.5.  (The rest together, a form for
    // each number: 1531 tokens 3.5 -> 3.65, by the size of the code.)
    uint32_t pre_cnt = 0, pre_last = 0;
    auto count_before = [&](int32_t first, auto blocks) {
        constexpr int N = decltype(blocks)::value;
        int4 v[N];
#pragma unroll
        for (int u = 0; u < N; ++u) v[u] = *reinterpret_cast<const int4*>(tok + (first + u) * kSegOneBlockTok + 4 * tid);
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const int32_t p[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (is_term(p[k])) { pre_cnt += 1; pre_last = (uint32_t)((first + u) * kSegOneBlockTok + 4 * tid + k + 1); }
        }
    };
    int32_t first = 0;
    for (; first + 4 <= (int32_t)blockIdx.x; first += 4) count_before(first, std::integral_constant<int, 4>{});
#pragma unroll 1
    for (; first < (int32_t)blockIdx.x; ++first) count_before(first, std::integral_constant<int, 1>{});
    uint32_t cnt = 0, last = 0, flags = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if (is_term(t[k])) { flags |= 1u << k; cnt += 1; last = (uint32_t)(i0 + k + 1); }
    const uint32_t inc = wave_scan_u32(cnt), inl = wave_scan_max_u32(last);
    const uint32_t pc = wave_scan_u32(pre_cnt), pl = wave_scan_max_u32(pre_last);
    if (lane == 63) { sm_cnt[w] = inc; sm_last[w] = inl; sm_pre[0][w] = pc; sm_pre[1][w] = pl; }
    __syncthreads();
    uint32_t seg = 0, start = 0;
#pragma unroll
    for (int i = 0; i < kBlockWaves; ++i) {
        seg += sm_pre[0][i] + (i < w ? sm_cnt[i] : 0u);
        start = max(start, max(sm_pre[1][i], i < w ? sm_last[i] : 0u));
    }
    seg += inc - cnt;
    const uint32_t before = (uint32_t)__shfl_up((int)inl, 1);
    if (lane > 0) start = max(start, before);
    int32_t id[4];
    uint32_t total = 0;                                          // S, in the thread that closes the prompt
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int32_t i = i0 + k;
        id[k] = (int32_t)seg;
        if (i < T && (((flags >> k) & 1u) || i == T - 1)) {
            if ((int32_t)seg < cap_sent) { put(sent_off + seg, (int32_t)start); put(sent_len + seg, i + 1 - (int32_t)start); }
            if (i == T - 1) {
                total = seg + 1;
                put(n_sent, (int32_t)total);
                if ((int32_t)total <= cap_sent) put(sent_off + total, T);
            }
            start = (uint32_t)(i + 1);
            seg += 1;
        }
    }
    if (i0 + 4 <= T) {
        if (REPORT) {
#pragma unroll
            for (int k = 0; k < 4; k += 2)
                __hip_atomic_store(reinterpret_cast<unsigned long long*>(seg_id + i0 + k), ((unsigned long long)(uint32_t)id[k + 1] << 32) | (uint32_t)id[k],
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        } else {
            *reinterpret_cast<int4*>(seg_id + i0) = make_int4(id[0], id[1], id[2], id[3]);
        }
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (i0 + k < T) put(seg_id + i0 + k, id[k]);
    }
    if (REPORT) {
        __shared__ uint32_t sm_total;
        if (tid == 0) sm_total = 0u;
        __syncthreads();
        if (total != 0u) sm_total = total;
        block_sync_after_stores();                              // every wave's results are in memory
        if (tid == 0) {
            const unsigned long long mine = (1ull << 32) | (unsigned long long)sm_total;
            unsigned long long all = mine;
            if (gridDim.x > 1) {
                all += __hip_atomic_fetch_add(arrive, mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if ((uint32_t)(all >> 32) != gridDim.x) return;
                __hip_atomic_store(arrive, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);     // for the next call, which the word below may start
                wait_loads<0>();
            }
            __hip_atomic_store(host_word, (uint32_t)all, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
}

// One launch while the prompt and the bitmap fit it (an empty prompt takes the two-launch form's early exit).
static bool segment_in_one(int32_t T, int32_t vocab) { return T > 0 && T <= kSegOneMaxTok && (vocab - 1) / 32 < kSegOneMaxWords; }

bool segment_reports(const Ctx* c, int32_t T, int32_t vocab) { return c->n_sent_host && segment_in_one(T, vocab); }

hipError_t launch_segment(Ctx* c, const int32_t* tok, int32_t T, const uint32_t* bitmap, int32_t vocab,
                          int32_t* seg_id, int32_t* sent_off, int32_t* sent_len, int32_t* n_sent_dev, bool report) {
    if (segment_in_one(T, vocab)) {
        const dim3 grid((T + kSegOneBlockTok - 1) / kSegOneBlockTok), block(kBlockThreads);
        const size_t lds = (size_t)((vocab - 1) / 32 + 1) * sizeof(uint32_t);
        if (report)
            hipLaunchKernelGGL(seg_one_kernel<true>, grid, block, lds, c->stream, tok, T, bitmap, vocab, seg_id, sent_off, sent_len,
                               c->d.max_sentences, n_sent_dev, c->seg_arrive, c->n_sent_host_dev);
        else
            hipLaunchKernelGGL(seg_one_kernel<false>, grid, block, lds, c->stream, tok, T, bitmap, vocab, seg_id, sent_off, sent_len,
                               c->d.max_sentences, n_sent_dev, nullptr, nullptr);
        return hipGetLastError();
    }
    const int nb = (T + kSegTokPerBlock - 1) / kSegTokPerBlock;
    if (nb > 0) {
        hipLaunchKernelGGL(seg_count_kernel, dim3(nb), dim3(kSegThreads), 0, c->stream, tok, T, bitmap, vocab,
                           c->seg_part);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(seg_scan_kernel, dim3(nb > 0 ? nb : 1), dim3(kSegThreads), 0, c->stream, tok, T, bitmap, vocab,
                       c->seg_part, seg_id, sent_off, sent_len, c->d.max_sentences, n_sent_dev);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// Eq. 1: one wave per (layer * head, bucket).  A bucket's rows are contiguous in the pool, a row is
// D * EB bytes = LPR lanes of 16 bytes, so one wave-wide load instruction covers RPW = 64 / LPR
// consecutive rows fully coalesced.  Four or eight such loads are kept in flight per lane.
// ------------------------------------------------------------------------------------------------

// Nearest E4M3 code (8-bit float of the OCP specification: bias 7, no infinities, largest value 448) of a finite float,
// ties to the even code, magnitudes that do not fit saturate at 448.
__device__ __forceinline__ uint32_t f32_to_e4m3(float f) {
    const uint32_t u = __float_as_uint(f), sign = (u >> 24) & 0x80u, a = u & 0x7fffffffu;
    uint32_t code;
    if (a < 0x3c800000u) {                                   // below 2^-6, the smallest normal: multiples of 2^-9
        code = (uint32_t)__builtin_rintf(__uint_as_float(a) * 512.0f);         // round half to even; 8 is 2^-6 itself
    } else {
        const uint32_t r = a + 0x7ffffu + ((a >> 20) & 1u);  // 23 -> 3 fraction bits, round half to even
        code = min((r >> 20) - (120u << 3), 0x7eu);          // exponent bias 127 -> 7; 0x7e = 448
    }
    return sign | code;
}

// nearest bf16 of a finite float, ties to even
__device__ __forceinline__ uint32_t f32_to_bf16(float f) {
    const uint32_t u = __float_as_uint(f);
    return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}

// One lane's EPL means (sums / n) of a bucket to element `o` of the table.  SVB: bytes per stored element (4 = fp32, 2 = bf16,
// 1 = E4M3; rounded to nearest even).
template <int EPL, int SVB>
__device__ __forceinline__ void store_means(char* __restrict__ semvec, int64_t o, const float* acc, float n) {
#pragma unroll
    for (int i = 0; i < EPL; i += 4) {
        const float m[4] = {acc[i] / n, acc[i + 1] / n, acc[i + 2] / n, acc[i + 3] / n};
        if (SVB == 4)
            *reinterpret_cast<uint4*>(semvec + (o + i) * 4) = make_uint4(__float_as_uint(m[0]), __float_as_uint(m[1]), __float_as_uint(m[2]), __float_as_uint(m[3]));
        else if (SVB == 1)
            *reinterpret_cast<uint32_t*>(semvec + (o + i)) = f32_to_e4m3(m[0]) | (f32_to_e4m3(m[1]) << 8) |
                                                             (f32_to_e4m3(m[2]) << 16) | (f32_to_e4m3(m[3]) << 24);
        else
            *reinterpret_cast<uint2*>(semvec + (o + i) * 2) = make_uint2(f32_to_bf16(m[0]) | (f32_to_bf16(m[1]) << 16), f32_to_bf16(m[2]) | (f32_to_bf16(m[3]) << 16));
    }
}
// Two of them.
template <int SVB, bool STREAM>
__device__ __forceinline__ void store_pair(char* __restrict__ semvec, int64_t o, float m0, float m1) {
    auto put = [&](auto v) {
        auto* p = reinterpret_cast<decltype(v)*>(semvec + o * SVB);
        if (STREAM) __builtin_nontemporal_store(v, p);
        else *p = v;
    };
    if (SVB == 4) put((unsigned long long)__float_as_uint(m0) | ((unsigned long long)__float_as_uint(m1) << 32));
    else if (SVB == 2) put((uint32_t)(f32_to_bf16(m0) | (f32_to_bf16(m1) << 16)));
    else put((uint16_t)(f32_to_e4m3(m0) | (f32_to_e4m3(m1) << 8)));
}

// Bound by HBM: the pool once in, the table once out.  A wave per bucket, one-shot waves with all the rows of a bucket of
// average length requested at once.  LARGE: 8 waves per block (contiguous 40 KB) and non-temporal stores, else 4 and plain ones; see the launch.
// The keys' loads are non-temporal in both: a plain read takes a place in the memory-side cache, whose lines may have to be written
// back first.  32 layers x 8 heads, us, plain / non-temporal loads, after other work has filled the cache with written lines and
// after the keys themselves have just been written: 1000 tokens 30.4 / 19.0, 16.4 / 16.4; 3000 79 / 44, 43 / 37; 8192 164 / 115, 136 / 115;
// 32768 491 / 394, 469 / 394 (only keys that a table was built from just before are read again faster with plain ones: 1531 tokens 26 / 29).
template <int EB, int SVB, bool LARGE>
__global__ __launch_bounds__((LARGE ? 8 : 4) * kWave) void semvec_kernel(const char* __restrict__ K, int32_t T,
                                                                         const int32_t* __restrict__ sent_off_all,
                                                                         int32_t off_layer_stride, int32_t Hkv,
                                                                         int32_t S, char* __restrict__ semvec, bool runs) {
    using R = Row<EB>;
    const int lane = threadIdx.x & 63;
    // runs: blocks in runs of an XCD, see the launch.  Us, blocks as they come / runs of 32, 32 layers x 8 heads: 32768 tokens in lognormal lengths, fp32 table 416 / 370, E4M3 375 / 344,
    // geometric lengths 380 / 376 (runs of 4 381, 16 379, 64 380, 256 375, an eighth of the grid 425), 8192 tokens, lognormal, fp32 109.5 / 105, E4M3 95 / 90, 1531 the same.
    uint32_t bx = blockIdx.x, by = blockIdx.y;
    if (runs) {
        const uint32_t at = xcd_run(bx + gridDim.x * by, gridDim.x * gridDim.y);
        by = at / gridDim.x;
        bx = at - by * gridDim.x;
    }
    const int32_t s = bx * (LARGE ? 8 : 4) + (threadIdx.x >> 6);
    if (s >= S) return;                                   // wave-uniform
    const int64_t lh = by;
    const int32_t* sent_off = sent_off_all + (int64_t)(by / Hkv) * off_layer_stride;   // the layer's table
    const int32_t b = max(sent_off[s], 0), e = min(sent_off[s + 1], T);   // never read outside the pool
    const int r = lane / R::LPR, cc = lane % R::LPR;
    const char* base = K + (lh * T) * (int64_t)(kHeadDim * EB) + (int64_t)cc * 16;

    float acc[R::EPL];
#pragma unroll
    for (int i = 0; i < R::EPL; ++i) acc[i] = 0.f;

    // Four loads a lane in flight, eight in the buckets of more than 48 rows, whose waves live longest.  Four in all / this, 32 layers x 8 heads, us: geometric
    // lengths of mean 20, 1531 tokens 23.4 / 21.8, 3000 41.6 / 39.7, 8192 101.4 / 99.0; lognormal 21.3 / 20.5, 38.9 / 37.8, 104.6 / 102.9; lengths of 8 to 40 the
    // same (eight from 17 rows on: 3000 tokens of those 41.7 / 43.6); fp32, geometric, 1531 tokens 41.9 / 39.5.
    auto add_rows = [&](auto loads) {
        constexpr int kUnroll = decltype(loads)::value;
        for (int32_t x0 = b + r; x0 < e; x0 += R::RPW * kUnroll) {
            uint4 v[kUnroll];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                const int32_t x = x0 + u * R::RPW;
                // clamped address + masked value keeps the loads independent of the bounds test
                const uint4 t = ld_stream(base + (int64_t)min(x, e - 1) * (kHeadDim * EB));
                v[u] = (x < e) ? t : make_uint4(0, 0, 0, 0);
            }
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                float f[R::EPL];
                R::unpack(v[u], f);
#pragma unroll
                for (int i = 0; i < R::EPL; ++i) acc[i] += f[i];
            }
        }
    };
    if (e - b > 48) add_rows(std::integral_constant<int, 8>{});
    else add_rows(std::integral_constant<int, 4>{});
    // The sums over the wave's rows, half of the elements left to each side of an exchange: every lane divides and stores two, and the vector leaves in one
    // whole piece.  Before, 16 (fp32: 32) lanes held all sums and stored eight (four) each, an fp32 vector in two pieces with gaps, reduced ones with plain stores
    // in large tables too, where a piece goes past the caches now like everything else there.  32 layers x 8 heads, us, before / now: 32768 tokens, table in fp32
    // 388 / 378, bf16 403 / 361, E4M3 379 / 347; 16384, E4M3 204 / 180; table and the scores of every layer: 494 / 483, 487 / 449, 467 / 445; 283 / 274.  Up to 8192
    // tokens the same within 1 %.  What carries it is the one piece past the caches (an fp32 table of 205056 KiB was written as 253048): with plain stores 16 layers of 32768 tokens
    // take 185 -> 199, bf16 177 -> 195, with shuffles for the swaps or 32 lanes of 16 bytes for the 64 of 8 the same as this.  Not kept: loads counted out by the bucket's length instead of masked, and 52 registers instead of more, 32768 tokens 388 / 405;
    // 24 or 16 waves on a compute unit 407, 475.
    float h[4];
    if constexpr (R::RPW == 4) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const auto x = __builtin_amdgcn_permlane16_swap(__float_as_uint(acc[i]), __float_as_uint(acc[i + 4]), false, false);
            h[i] = __uint_as_float(x[0]) + __uint_as_float(x[1]);
        }
    } else {
        static_assert(R::RPW == 2 && R::EPL == 4);
#pragma unroll
        for (int i = 0; i < 4; ++i) h[i] = acc[i];
    }
    float m[2];
    const float n = (e > b) ? (float)(e - b) : 1.f;          // a bucket without tokens yields zeros
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(h[i]), __float_as_uint(h[i + 2]), false, false);
        m[i] = (__uint_as_float(x[0]) + __uint_as_float(x[1])) / n;
    }
    const int first = cc * R::EPL + (R::RPW == 4 ? (r & 1) * 4 + (r >> 1) * 2 : r * 2);
    store_pair<SVB, LARGE>(semvec, (lh * S + s) * (int64_t)kHeadDim + first, m[0], m[1]);
}

// Short buckets (a retained pool keeps a few tokens of each): the row's LPR lanes own a bucket, RPW buckets per wave, and walk
// its rows; no sum across lanes, and the table's rows are stored RPW at a time.  A wave per bucket is bound by the number of
// waves here: 32 x 8 x 4096 retained tokens in 1654 buckets (485 MB), 161-169 us with a wave per bucket, 90 us with this.  The pool has usually just been written by
// skv_compact_pool: the last heads are read first, while the memory-side cache still holds them, and with non-temporal loads, which leave the others their
// places.  Compaction and mean keys, first to last / last to first, us: 16 layers x 8 heads x 16384 retained tokens 526 / 511, smaller pools the same; plain /
// non-temporal loads there 536 / 511, 32 layers x 6000 tokens 371 / 370, x 4096 297 / 286, x 2048 with an E4M3 table 139 / 133, x 1024 119 / 120.
template <int EB, int SVB>
__global__ __launch_bounds__(kSemvecShortWaves * kWave) void semvec_short_kernel(const char* __restrict__ K, int32_t T,
                                                                                    const int32_t* __restrict__ sent_off_all,
                                                                                    int32_t off_layer_stride, int32_t Hkv,
                                                                                    int32_t S, char* __restrict__ semvec) {
    using R = Row<EB>;
    constexpr int kUnroll = 4;
    const int lane = threadIdx.x & 63, cc = lane % R::LPR;
    const int32_t s = ((int32_t)(gridDim.x - 1 - blockIdx.x) * kSemvecShortWaves + (threadIdx.x >> 6)) * R::RPW + lane / R::LPR;
    if (s >= S) return;
    const int64_t lh = gridDim.y - 1 - blockIdx.y;
    const int32_t* sent_off = sent_off_all + (int64_t)((gridDim.y - 1 - blockIdx.y) / Hkv) * off_layer_stride;   // the layer's table
    const int32_t b = max(sent_off[s], 0), e = min(sent_off[s + 1], T);   // never read outside the pool
    const char* base = K + (lh * T) * (int64_t)(kHeadDim * EB) + (int64_t)cc * 16;
    float acc[R::EPL];
#pragma unroll
    for (int i = 0; i < R::EPL; ++i) acc[i] = 0.f;
    for (int32_t x0 = b; x0 < e; x0 += kUnroll) {
        uint4 v[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const uint4 t = ld_stream(base + (int64_t)min(x0 + u, e - 1) * (kHeadDim * EB));
            v[u] = (x0 + u < e) ? t : make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            float f[R::EPL];
            R::unpack(v[u], f);
#pragma unroll
            for (int i = 0; i < R::EPL; ++i) acc[i] += f[i];
        }
    }
    const float n = (e > b) ? (float)(e - b) : 1.f;          // a bucket without tokens yields zeros
    store_means<R::EPL, SVB>(semvec, (lh * S + s) * (int64_t)kHeadDim + cc * R::EPL, acc, n);
}

template <int EB, int SVB>
static void launch_semvec_t(Ctx* c, const void* K_pool, int32_t T, const int32_t* sent_off, int32_t off_layer_stride, int32_t S,
                            void* semvec) {
    // By the bytes of a bucket's rows: 16 layers x 8 heads x 32768 tokens in buckets of n tokens, wave per bucket against several
    // per wave, us: bf16 pool, fp32 table, n = 6: 323 / 248, 8: 255 / 242, 10: 221 / 233, 24: 186 / 222; fp32 pool, n = 2:
    // 738 / 530, 4: 460 / 490, 8: 378 / 464.  Smaller tables move the line up a little (E4M3, n = 10: 225 / 202).
    const int LH = c->d.n_layers * c->d.n_kv_heads;
    const auto grid = [&](int per_block) { return dim3((S + per_block - 1) / per_block, LH); };
    if ((int64_t)T * (kHeadDim * EB) < kSemvecShortBytes * (int64_t)S) {
        hipLaunchKernelGGL((semvec_short_kernel<EB, SVB>), grid(kSemvecShortWaves * Row<EB>::RPW), dim3(kSemvecShortWaves * kWave), 0, c->stream,
                           (const char*)K_pool, T, sent_off, off_layer_stride, c->d.n_kv_heads, S, (char*)semvec);
        return;
    }
    // By the number of table rows (of 512 bytes in fp32).  The scores read the table next, from the memory-side cache while it fits there beside
    // the keys just read, and a short prompt is spread more evenly in small blocks.  fp32 table, 32 layers x 8 heads, keys not in any cache, us,
    // table / table and the scores of every layer, small against LARGE: 1531 tokens (15000 rows) 25.6 / 101 against 30.6 / 111,
    // 8192 (105000) 104 / 183 against 111 / 197, 11000 (142000) 137 / 217 against 139 / 225, 16384 (206000) 201 / 284 against 200 / 286 and, keys
    // just written, 212 / 298 against 198 / 288, 32768 426 / 528 against 397 / 503.
    // Blocks are dealt in runs where a head has 6000 tokens and more, a launch 4096 blocks and a bucket fewer than 128 tokens on average.  fp32 table, 8 heads, us, as they
    // come / in runs: 32 layers of 2048 tokens 26.5 / 27.05, 4 of 4096 10.2 / 10.5; one of 32768 (2736 blocks) 15.0 / 15.5, 32 heads of 8192 (3296) 14.5 / 14.8, 8 layers of 8192 in buckets of 12 tokens (10900) 31.0 / 29.95, of 20 the same, 2 layers of
    // 32768 (5500) 28.05 / 27.5; 16 layers of 32768 in buckets of 50 tokens 214 / 193, 100 192.8 / 187.9, 200 188.1 / 189.1, 500 192.7 / 201, 2000 223.5 / 229.7,
    // fp32 keys, 100 371 / 365, 200 362.5 / 362.5, 500 370 / 380.
    const bool small = (int64_t)LH * S <= kSemvecSmallRows;
    const int64_t blocks = ((int64_t)S + (small ? 4 : 8) - 1) / (small ? 4 : 8) * LH;
    const bool runs = T >= kSemvecRunTokens && blocks >= kSemvecRunBlocks && T < kSemvecRunBucket * (int64_t)S;
    if (small)
        hipLaunchKernelGGL((semvec_kernel<EB, SVB, false>), grid(4), dim3(4 * kWave), 0, c->stream, (const char*)K_pool, T, sent_off, off_layer_stride,
                           c->d.n_kv_heads, S, (char*)semvec, runs);
    else
        hipLaunchKernelGGL((semvec_kernel<EB, SVB, true>), grid(8), dim3(8 * kWave), 0, c->stream, (const char*)K_pool, T, sent_off, off_layer_stride,
                           c->d.n_kv_heads, S, (char*)semvec, runs);
}

template <int EB>
static void launch_semvec_eb(Ctx* c, const void* K_pool, int32_t T, const int32_t* sent_off, int32_t off_layer_stride, int32_t S,
                             void* semvec) {
    if (c->d.semvec_dtype == SKV_BF16) launch_semvec_t<EB, 2>(c, K_pool, T, sent_off, off_layer_stride, S, semvec);
    else if (c->d.semvec_dtype == SKV_FP8_E4M3) launch_semvec_t<EB, 1>(c, K_pool, T, sent_off, off_layer_stride, S, semvec);
    else launch_semvec_t<EB, 4>(c, K_pool, T, sent_off, off_layer_stride, S, semvec);
}

hipError_t launch_semvec(Ctx* c, const void* K_pool, int32_t T, const int32_t* sent_off, int32_t off_layer_stride, int32_t S,
                         void* semvec) {
    if (S == 0) return hipSuccess;
    if (c->d.kv_dtype == SKV_BF16) launch_semvec_eb<2>(c, K_pool, T, sent_off, off_layer_stride, S, semvec);
    else launch_semvec_eb<4>(c, K_pool, T, sent_off, off_layer_stride, S, semvec);
    return hipGetLastError();
}

}  // namespace skv
