// Decode-step kernels (Sec. 4.2, Eq. 3, Alg. 1 decoding phase): bucket scores, ranking + budgeted
// retrieval, K/V row gather, split-K attention with an online-softmax combine.  gfx950, wave64.
#include "skv_internal.h"
#include "skv_device.h"
#include "skv_stamps.h"

#include <type_traits>

#ifdef SKV_PHASE_STAMPS
namespace skv {
__device__ unsigned long long g_stamps[kStampBlocks * kStampSlots];
}
// Copies the stamp table (kStampBlocks x kStampSlots 64-bit ticks of the 100 MHz clock, zero where nothing was
// recorded) to `host` and clears it on the device.  Profiling build only.
extern "C" int skv_stamps_read(unsigned long long* host, int n_words) {
    if (!host || n_words != skv::kStampBlocks * skv::kStampSlots) return -1;
    if (hipDeviceSynchronize() != hipSuccess) return -3;
    if (hipMemcpyFromSymbol(host, HIP_SYMBOL(skv::g_stamps), sizeof(unsigned long long) * n_words) != hipSuccess) return -3;
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(skv::g_stamps)) != hipSuccess) return -3;
    return hipMemset(p, 0, sizeof(unsigned long long) * n_words) == hipSuccess ? 0 : -3;
}
#endif

namespace skv {

// Per-sequence slice of a ragged batch.
struct Seq {
    int32_t tok_base, n_tok_ctx;     // first pool row and number of tokens of the sequence
    int32_t sent_base, n_sent;       // first bucket and number of buckets
    int32_t budget;
};

// Read of an int32 array that the running launch does not write (the caller's cu_tok, cu_sent, budgets; n_tok, which an
// earlier launch of the same call may have written), through
// the constant address space: with a wave-uniform index it is a scalar load whatever else the kernel contains (loads of
// a plain global pointer turn into vector loads once the compiler cannot prove that the kernel leaves the memory alone,
// which an inline asm statement is enough to cause).
__device__ __forceinline__ int32_t ld_const(const int32_t* p, int64_t i) {
    typedef const int32_t __attribute__((address_space(4))) * ConstI32;
    return ((ConstI32)(uintptr_t)p)[i];
}

__device__ __forceinline__ Seq seq_of(const SeqView& v, int b) {
    Seq s;
    s.sent_base = v.cu_sent ? ld_const(v.cu_sent, b) : 0;
    s.n_sent = v.cu_sent ? ld_const(v.cu_sent, b + 1) - s.sent_base : v.S_total;
    s.tok_base = v.cu_tok ? ld_const(v.cu_tok, b) : 0;
    s.n_tok_ctx = v.cu_tok ? ld_const(v.cu_tok, b + 1) - s.tok_base : v.T_total;
    s.budget = v.budget_arr ? ld_const(v.budget_arr, b) : v.budget;
    return s;
}
// The same for the decode step, which has budgets, and both boundary arrays or neither: one round of loads at most, and nobody waits for the budget yet.
__device__ __forceinline__ Seq seq_of_step(const SeqView& v, int b) {
    Seq s;
    s.budget = ld_const(v.budget_arr, b);
    if (v.cu_sent) {
        const int32_t s0 = ld_const(v.cu_sent, b), s1 = ld_const(v.cu_sent, b + 1), t0 = ld_const(v.cu_tok, b), t1 = ld_const(v.cu_tok, b + 1);
        asm volatile("" ::"s"(s0), "s"(s1), "s"(t0), "s"(t1));
        s.sent_base = s0; s.n_sent = s1 - s0;
        s.tok_base = t0; s.n_tok_ctx = t1 - t0;
    } else {
        s.sent_base = 0; s.n_sent = v.S_total;
        s.tok_base = 0; s.n_tok_ctx = v.T_total;
    }
    return s;
}

// ------------------------------------------------------------------------------------------------
// Sentence query cache (Eq. 2; Alg. 1 decoding phase): running sum and count per sequence, mean query
// out, state cleared when the generated token ends a sentence.  One thread per 4 elements.
// ------------------------------------------------------------------------------------------------
template <int EB>
__global__ __launch_bounds__(kBlockThreads) void query_update_kernel(const char* __restrict__ q_t, const int32_t* __restrict__ tok_t,
                                                                     const uint32_t* __restrict__ bitmap, int32_t vocab,
                                                                     int32_t per_seq /* Hq * D */, float* __restrict__ q_sum,
                                                                     int32_t* __restrict__ q_cnt, char* __restrict__ q_bar) {
    const int b = blockIdx.x;                                        // one block per sequence
    const int32_t id = tok_t[b];
    const bool term = id >= 0 && id < vocab && ((bitmap[id >> 5] >> (id & 31)) & 1u);
    const int32_t n = q_cnt[b] + 1;
    const float fn = (float)n;
    for (int i4 = threadIdx.x * 4; i4 < per_seq; i4 += kBlockThreads * 4) {
        const int64_t e = (int64_t)b * per_seq + i4;
        float4 s = *reinterpret_cast<const float4*>(q_sum + e);
        float x[4];
        if (EB == 4) {
            const float4 t = *reinterpret_cast<const float4*>(q_t + e * 4);
            x[0] = t.x; x[1] = t.y; x[2] = t.z; x[3] = t.w;
        } else {
            const uint2 t = *reinterpret_cast<const uint2*>(q_t + e * 2);
            x[0] = __uint_as_float(t.x << 16); x[1] = __uint_as_float(t.x & 0xffff0000u);
            x[2] = __uint_as_float(t.y << 16); x[3] = __uint_as_float(t.y & 0xffff0000u);
        }
        s.x += x[0]; s.y += x[1]; s.z += x[2]; s.w += x[3];
        const float m[4] = {s.x / fn, s.y / fn, s.z / fn, s.w / fn};
        if (EB == 4) {
            *reinterpret_cast<float4*>(q_bar + e * 4) = make_float4(m[0], m[1], m[2], m[3]);
        } else {
            uint32_t r[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {                             // round to nearest even bf16 (inputs are finite)
                uint32_t u = __float_as_uint(m[k]);
                u += 0x7fffu + ((u >> 16) & 1u);
                r[k] = u >> 16;
            }
            *reinterpret_cast<uint2*>(q_bar + e * 2) = make_uint2(r[0] | (r[1] << 16), r[2] | (r[3] << 16));
        }
        *reinterpret_cast<float4*>(q_sum + e) = term ? make_float4(0.f, 0.f, 0.f, 0.f) : s;
    }
    __syncthreads();                                                  // every thread has read q_cnt[b]
    if (threadIdx.x == 0) q_cnt[b] = term ? 0 : n;
}

hipError_t launch_query_update(Ctx* c, int32_t B, const void* q_t, const int32_t* tok_t, const uint32_t* bitmap,
                               int32_t vocab, float* q_sum, int32_t* q_cnt, void* q_bar) {
    const int per_seq = c->d.n_q_heads * kHeadDim;
    const dim3 grid(B), block(kBlockThreads);
    if (c->d.kv_dtype == SKV_BF16)
        hipLaunchKernelGGL(query_update_kernel<2>, grid, block, 0, c->stream, (const char*)q_t, tok_t, bitmap, vocab, per_seq,
                           q_sum, q_cnt, (char*)q_bar);
    else
        hipLaunchKernelGGL(query_update_kernel<4>, grid, block, 0, c->stream, (const char*)q_t, tok_t, bitmap, vocab, per_seq,
                           q_sum, q_cnt, (char*)q_bar);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// Scores.  score[h][s] = sum_g q[hG+g] . semvec[h][s]  =  (sum_g q[hG+g]) . semvec[h][s].
// A semantic vector is 512 bytes = 32 lanes x float4; a wave covers 2 buckets per load instruction
// and keeps RPWV / 2 loads in flight (RPWV = buckets per wave; 8 measured best from 1.3 k to 26 k
// buckets per head: 4 and 32 were both slower).  The group-summed query lives in registers.
// Blocks are aligned to sequences: block x -> (sequence b, local block) by walking cu_sent.
// ------------------------------------------------------------------------------------------------

// Tag of a launch of the single-launch step for one pair: the pair's epoch after this launch (1 .. 2^26 - 1, never 0, so
// zero-filled memory never looks valid) above the pair's number.  A word of memory carries a pair's current tag only if
// a block of that pair wrote it in this launch: other pairs differ in the low bits, earlier launches in the epoch (which
// repeats after 2^26 - 1 launches of the pair).
__device__ __forceinline__ uint32_t step_tag(uint32_t epoch, int pair) {
    uint32_t e = (epoch + 1u) & ((1u << (32 - kStepPairBits)) - 1u);
    if (e == 0u) e = 1u;
    return (e << kStepPairBits) | (uint32_t)pair;
}

// What a block knows of its pair when it begins: the epoch, on its way from memory, and the pair's number.  The tag is formed where it is needed: formed
// at the top, the wait for the epoch comes before the request for the mean keys.
struct StepState {
    unsigned int epoch;
    int pair;
    __device__ __forceinline__ uint32_t tag() const {
        unsigned int e = epoch;
        asm volatile("" : "+v"(e));
        return step_tag(e, pair);
    }
};

// Scores of the STEP * N buckets from row_w on: p[i] of the lanes (lane / (64 / STEP)) is the score of bucket row_w + lane / (64 / STEP) + STEP i; c: the lane's place
// among those of its bucket, negative where they hold no sum.  TAGGED: consecutive lanes take consecutive buckets, for one store of whole words of a line.
template <bool TAGGED, int STEP, int N>
__device__ __forceinline__ void store_scores(void* __restrict__ out_seq, const float (&p)[N], int c, int32_t row_w, int32_t n_sent, const StepState& st) {
    constexpr int kLanes = kWave / STEP, kFirst = STEP == 8 ? 4 : 0;      // lanes of a bucket, the first that holds its sum
    const int lane = threadIdx.x & 63;
    if constexpr (TAGGED) {
        float v = p[0];
#pragma unroll
        for (int i = 1; i < N; ++i) {
            float x = p[i];
            asm volatile("" : "+v"(x));                                  // (selects; else the compiler makes an array in LDS of p)
            v = c == i ? x : v;
        }
        v = __shfl(v, kLanes * (lane & (STEP - 1)) + kFirst + ((lane / STEP) & (N - 1)));
        const int32_t s = row_w + lane;
        const uint32_t tag = st.tag();
        if (lane < STEP * N && s < n_sent) st_tagged(static_cast<unsigned long long*>(out_seq) + s, v, tag);
    } else if (c == 0) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int32_t s = row_w + lane / kLanes + STEP * i;
            if (s < n_sent) static_cast<float*>(out_seq)[s] = p[i];
        }
    }
}

// One wave: the RPWV buckets [row_w, row_w + RPWV) of a sequence.  q_grp = the first query of the head's group,
// sv_seq / out_seq = the (head, sequence) slices of the table and of the scores.  TAGGED: out_seq holds 64-bit (score, tag)
// words that other blocks of the same launch read.
template <int EB, int G, int RPWV, bool TAGGED>
__device__ __forceinline__ void score_wave_f32(const char* __restrict__ q_grp, const float* __restrict__ sv_seq,
                                               int32_t n_sent, int32_t row_w, void* __restrict__ out_seq, const StepState& st = {}) {
    const int lane = threadIdx.x & 63;
    const int c = lane & 31, half = lane >> 5;
    float qs[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const char* qrow = q_grp + ((int64_t)g * kHeadDim + c * 4) * EB;
        if (EB == 4) {
            const float4 t = *reinterpret_cast<const float4*>(qrow);
            qs[0] += t.x; qs[1] += t.y; qs[2] += t.z; qs[3] += t.w;
        } else {
            const uint2 t = *reinterpret_cast<const uint2*>(qrow);
            qs[0] += __uint_as_float(t.x << 16); qs[1] += __uint_as_float(t.x & 0xffff0000u);
            qs[2] += __uint_as_float(t.y << 16); qs[3] += __uint_as_float(t.y & 0xffff0000u);
        }
    }
    constexpr int kIter = RPWV / 2;
    const int32_t row0 = row_w + half;
    const float* base = sv_seq + c * 4;
    // Addresses are clamped into the sequence instead of predicating the loads, so that all of a
    // lane's loads are issued back to back; rows past the end are computed and dropped.
    float4 x[kIter];
#pragma unroll
    for (int i = 0; i < kIter; ++i) {
        const int32_t s = min(row0 + 2 * i, n_sent - 1);
        x[i] = __builtin_bit_cast(float4, ld_stream(base + (int64_t)s * kHeadDim));
    }
    float p[kIter];
#pragma unroll
    for (int i = 0; i < kIter; ++i) p[i] = x[i].x * qs[0] + x[i].y * qs[1] + x[i].z * qs[2] + x[i].w * qs[3];
#pragma unroll
    for (int i = 0; i < kIter; ++i) {                     // sum over the 32 lanes of a bucket
        p[i] = dpp_add<0xB1>(p[i]);
        p[i] = dpp_add<0x4E>(p[i]);
        p[i] = dpp_add<0x124>(p[i]);
        p[i] = dpp_add<0x128>(p[i]);
        p[i] += __shfl_xor(p[i], 16);
    }
    store_scores<TAGGED, 2>(out_seq, p, c, row_w, n_sent, st);
}

// The same from a bf16 table: a vector is 256 bytes = 16 lanes x 16 bytes (8 dims per lane), a wave load covers
// 4 buckets, RPWV / 4 loads in flight; the sum over a bucket's 16 lanes stays inside a DPP row.
template <int EB, int G, int RPWV, bool TAGGED>
__device__ __forceinline__ void score_wave_bf16(const char* __restrict__ q_grp, const char* __restrict__ sv_seq,
                                                int32_t n_sent, int32_t row_w, void* __restrict__ out_seq, const StepState& st = {}) {
    const int lane = threadIdx.x & 63;
    const int c = lane & 15, sub = lane >> 4;
    float qs[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const char* qrow = q_grp + ((int64_t)g * kHeadDim + c * 8) * EB;
        if (EB == 4) {
            const float4 t0 = *reinterpret_cast<const float4*>(qrow), t1 = *reinterpret_cast<const float4*>(qrow + 16);
            qs[0] += t0.x; qs[1] += t0.y; qs[2] += t0.z; qs[3] += t0.w;
            qs[4] += t1.x; qs[5] += t1.y; qs[6] += t1.z; qs[7] += t1.w;
        } else {
            float f[8];
            Row<2>::unpack(*reinterpret_cast<const uint4*>(qrow), f);
#pragma unroll
            for (int i = 0; i < 8; ++i) qs[i] += f[i];
        }
    }
    constexpr int kIter = RPWV / 4;
    const int32_t row0 = row_w + sub;
    const char* base = sv_seq + c * 16;
    uint4 x[kIter];
#pragma unroll
    for (int i = 0; i < kIter; ++i) {                       // clamped addresses: all loads issued back to back
        const int32_t s = min(row0 + 4 * i, n_sent - 1);
        x[i] = ld_stream(base + (int64_t)s * (kHeadDim * 2));
    }
    float p[kIter];
#pragma unroll
    for (int i = 0; i < kIter; ++i) {
        float f[8];
        Row<2>::unpack(x[i], f);
        p[i] = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) p[i] += f[e] * qs[e];
    }
#pragma unroll
    for (int i = 0; i < kIter; ++i) {                       // sum over the 16 lanes of a bucket
        p[i] = dpp_add<0xB1>(p[i]);
        p[i] = dpp_add<0x4E>(p[i]);
        p[i] = dpp_add<0x124>(p[i]);
        p[i] = dpp_add<0x128>(p[i]);
    }
    store_scores<TAGGED, 4>(out_seq, p, c, row_w, n_sent, st);
}

// The same from an E4M3 table: a vector is 128 bytes = 8 lanes x 16 bytes (16 dims per lane), a wave load covers 8 buckets,
// RPWV / 8 loads in flight; the sum over a bucket's 8 lanes is two quad exchanges and a rotation by 4.
template <int EB, int G, int RPWV, bool TAGGED>
__device__ __forceinline__ void score_wave_e4m3(const char* __restrict__ q_grp, const char* __restrict__ sv_seq,
                                                int32_t n_sent, int32_t row_w, void* __restrict__ out_seq, const StepState& st = {}) {
    const int lane = threadIdx.x & 63;
    const int c = lane & 7, sub = lane >> 3;
    float qs[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) qs[i] = 0.f;
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const char* qrow = q_grp + ((int64_t)g * kHeadDim + c * 16) * EB;
        if (EB == 4) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float4 t = *reinterpret_cast<const float4*>(qrow + 16 * k);
                qs[4 * k] += t.x; qs[4 * k + 1] += t.y; qs[4 * k + 2] += t.z; qs[4 * k + 3] += t.w;
            }
            // eight fp32 queries: four at a time, else the single-launch step has no registers for what lives across the scores (8 spilled; one sequence of
            // 32768 tokens 16.8 -> 15.6 us per layer, seven and one 15.9)
            if (TAGGED && G == 8 && g == 3) __builtin_amdgcn_sched_barrier(0);
        } else {
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                float f[8];
                Row<2>::unpack(*reinterpret_cast<const uint4*>(qrow + 16 * k), f);
#pragma unroll
                for (int i = 0; i < 8; ++i) qs[8 * k + i] += f[i];
            }
        }
    }
    constexpr int kIter = RPWV / 8;
    const int32_t row0 = row_w + sub;
    const char* base = sv_seq + c * 16;
    uint4 x[kIter];
#pragma unroll
    for (int i = 0; i < kIter; ++i) {                       // clamped addresses: all loads issued back to back
        const int32_t s = min(row0 + 8 * i, n_sent - 1);
        x[i] = ld_stream(base + (int64_t)s * kHeadDim);
    }
    float p[kIter];
#pragma unroll
    for (int i = 0; i < kIter; ++i) {
        const uint32_t wd[4] = {x[i].x, x[i].y, x[i].z, x[i].w};
        p[i] = 0.f;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            // v_cvt_pk_f32_fp8: two codes of a dword -> two floats; gfx950 reads them as E4M3 of the OCP specification
            // (a parity test scores a table holding every code against the format's written-out definition)
            typedef float f32x2 __attribute__((ext_vector_type(2)));
            const f32x2 lo = __builtin_amdgcn_cvt_pk_f32_fp8((int)wd[k], false), hi = __builtin_amdgcn_cvt_pk_f32_fp8((int)wd[k], true);
            p[i] += lo[0] * qs[4 * k] + lo[1] * qs[4 * k + 1] + hi[0] * qs[4 * k + 2] + hi[1] * qs[4 * k + 3];
        }
    }
#pragma unroll
    for (int i = 0; i < kIter; ++i) {                       // sum over the 8 lanes of a bucket
        p[i] = dpp_add<0xB1>(p[i]);
        p[i] = dpp_add<0x4E>(p[i]);
        p[i] = dpp_add<0x124>(p[i]);                        // row_ror 4: lanes 4..7 of each group of 8 now hold the group's sum
    }
    store_scores<TAGGED, 8>(out_seq, p, c - 4, row_w, n_sent, st);        // (lanes 4 .. 7 of each group)
}

constexpr int kScoreRowsPerWave16 = 16;
constexpr int kScoreRowsPerWave8 = 32;
enum { kTableF32 = 4, kTableBf16 = 2, kTableE4m3 = 1 };       // bytes per element of the mean-key table

// Scores of one layer: grid (blocks over the S_total buckets of the concatenated batch, KV heads).  A wave owns RPWV
// consecutive buckets of that axis, wherever the sequence boundaries fall, and scores them in runs that belong to one
// sequence, each run with that sequence's queries: one run unless a boundary falls inside the wave's buckets; a sequence
// without buckets has no run.  The sequence of the wave's first bucket r0 is the last b with cu_sent[b] <= r0: bisection
// of cu_sent down to eight candidates (dependent scalar loads), then eight consecutive boundaries in one scalar load,
// which also gives the end of the first run; log2(B / 8) + 1 round trips, whatever the batch size.

// The RPWV buckets [r0, r0 + RPWV) of the concatenated bucket axis, head h, by one wave.
template <int EB, int G, int SVB, int RPWV>
__device__ __forceinline__ void score_group(const char* __restrict__ q, const char* __restrict__ semvec, const SeqView& v,
                                            int32_t Hq, int h, int32_t r0, float* __restrict__ out) {
    const int32_t r1 = min(r0 + RPWV, v.S_total);
    auto run = [&](int b, int32_t first, int32_t n) {      // buckets [first, first + n) of the batch axis, sequence b
        const char* qg = q + ((int64_t)(b * Hq + h * G) * kHeadDim) * EB;
        const int64_t row = (int64_t)h * v.S_total + first;
        float* dst = out + row;
        if (SVB == kTableF32)
            score_wave_f32<EB, G, RPWV, false>(qg, reinterpret_cast<const float*>(semvec) + row * kHeadDim, n, 0, dst);
        else if (SVB == kTableBf16)
            score_wave_bf16<EB, G, RPWV, false>(qg, semvec + row * kHeadDim * 2, n, 0, dst);
        else
            score_wave_e4m3<EB, G, RPWV, false>(qg, semvec + row * kHeadDim, n, 0, dst);
    };
    if (!v.cu_sent) {                                      // one sequence
        run(0, r0, r1 - r0);
        return;
    }
    auto cu = [&](int i) { return ld_const(v.cu_sent, i); };
    int b = 0, hi = v.B;                                   // cu(b) <= r0 < cu(hi)
    int32_t end;
    if (v.B >= 8) {
        while (hi - b > 8) {
            const int mid = (b + hi) >> 1;
            if (cu(mid) <= r0) b = mid; else hi = mid;
        }
        const int start = min(b + 1, v.B - 7);             // boundaries start .. start + 7 include hi
        int32_t w[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) w[j] = cu(start + j);
        int below = 0;
        end = w[7];
#pragma unroll
        for (int j = 7; j >= 0; --j) {
            below += w[j] <= r0;
            if (w[j] > r0) end = w[j];
        }
        b = start - 1 + below;
    } else {
        while (hi - b > 1) {
            const int mid = (b + hi) >> 1;
            if (cu(mid) <= r0) b = mid; else hi = mid;
        }
        end = cu(b + 1);
    }
    int32_t cur = r0;
    for (;;) {
        end = min(end, r1);
        if (end > cur) {
            run(b, cur, end - cur);
            cur = end;
        }
        if (cur >= r1 || ++b >= v.B) break;
        end = cu(b + 1);
    }
}

template <int EB, int G, int SVB, int RPWV>
__global__ __launch_bounds__(kScoreWavesPerBlock * kWave) void score_kernel(const char* __restrict__ q,
                                                                            const char* __restrict__ semvec, SeqView v,
                                                                            int32_t Hq, float* __restrict__ score) {
    // every argument is demanded here, so the kernel-argument loads go out together; left alone, the compiler loads
    // each one before its first use, a dependent round trip per branch below
    asm volatile("" ::"s"(q), "s"(semvec), "s"(v.cu_sent), "s"(v.S_total), "s"(v.B), "s"(Hq), "s"(score));
    // (In runs of an XCD where a head has 256 blocks and more: 64 sequences of 32768 tokens, two layers, 294.7 / 290.6 us; 16 ragged ones 198.8 either way.)
    const int32_t r0 = ((int32_t)xcd_run(blockIdx.x, gridDim.x) * kScoreWavesPerBlock + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * RPWV;
    if (r0 >= v.S_total) return;
    score_group<EB, G, SVB, RPWV>(q, semvec, v, Hq, blockIdx.y, r0, score);
}

template <int EB, int G>
static void launch_score_t(Ctx* c, const char* q, const char* sv, const SeqView& v, float* score) {
    const bool sv16 = c->d.semvec_dtype == SKV_BF16, sv8 = c->d.semvec_dtype == SKV_FP8_E4M3;
    const int rows_per_block = (sv8 ? kScoreRowsPerWave8 : sv16 ? kScoreRowsPerWave16 : kScoreRowsPerWave) * kScoreWavesPerBlock;
    const dim3 grid((v.S_total + rows_per_block - 1) / rows_per_block, c->d.n_kv_heads), block(kScoreWavesPerBlock * kWave);
    if (sv8)
        hipLaunchKernelGGL((score_kernel<EB, G, kTableE4m3, kScoreRowsPerWave8>), grid, block, 0, c->stream, q, sv, v,
                           c->d.n_q_heads, score);
    else if (sv16)
        hipLaunchKernelGGL((score_kernel<EB, G, kTableBf16, kScoreRowsPerWave16>), grid, block, 0, c->stream, q, sv, v,
                           c->d.n_q_heads, score);
    else
        hipLaunchKernelGGL((score_kernel<EB, G, kTableF32, kScoreRowsPerWave>), grid, block, 0, c->stream, q, sv, v,
                           c->d.n_q_heads, score);
}

template <int EB>
static hipError_t launch_score_g(Ctx* c, const void* q, const void* semvec_layer, const SeqView& v, float* score) {
    const char* qp = (const char*)q;
    const char* sv = (const char*)semvec_layer;
    switch (c->G) {
        case 1: launch_score_t<EB, 1>(c, qp, sv, v, score); break;
        case 2: launch_score_t<EB, 2>(c, qp, sv, v, score); break;
        case 4: launch_score_t<EB, 4>(c, qp, sv, v, score); break;
        case 8: launch_score_t<EB, 8>(c, qp, sv, v, score); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_score(Ctx* c, const void* q, const void* semvec_layer, const SeqView& v, float* score) {
    if (v.S_total == 0) return hipSuccess;
    return c->d.kv_dtype == SKV_BF16 ? launch_score_g<2>(c, q, semvec_layer, v, score)
                                     : launch_score_g<4>(c, q, semvec_layer, v, score);
}

// ------------------------------------------------------------------------------------------------
// Selection (Sec. 4.2 ranking + budgeted retrieval) as a block-level routine for kBlockThreads
// threads, used by the stand-alone select kernel (one block per sequence and KV head) and, redundantly
// per block, by the fused attention kernel.
//
// Buckets are ranked by (score descending, id ascending) and taken along the ranking until the first
// one that does not fit.  Because lengths are positive the running total along the ranking is
// increasing, so the retrieved set is {i : (total length ranked before i) + len_i <= budget}.  The
// first bucket that overflows (the "cut") is found without sorting, by a length-weighted radix select
// on an order-preserving 32-bit image of the score: 11 + 11 + 10 bit digits, most significant first.
// Per pass: LDS atomics build a histogram of (count, total length) per digit and the total lengths of
// groups of 64 digits; after the one barrier of the pass every wave finds the crossing digit by itself: two lanes
// per group, from the top one down, a scan and the lane that sees the budget crossed, then a lane per digit
// of that group.  (The block finding it together, thread t with digits 2047-2t and 2046-2t, a block scan
// and the crossing thread telling the others, takes two more barriers and trips to LDS a pass: keys in
// registers to cut known 1.1 us, this way 0.7; a layer of the single-launch step of 32768 tokens 11.3 -> 11.1 us.)
// Scores close to each other, as keys with a large common part give them, fall into a few groups (one spans 6 % of the best
// score), and the lanes of a wave that add to one word do so one after the other: a group has eight counters, for the lanes in turn, read 16 bytes a lane.
// Us, the block scan / 64 groups of one counter each / this, scores 3 %, 1 % and 0.3 % apart (standard deviation over mean), then normal scores: a layer of the single-launch
// step of 131072 tokens, 5461 buckets, 16.6, 16.7, 17.3; 16.1 / 17.4, 18.7, 20.9; 15.55 / 16.45, 16.6, 17.1; 15.6, of 32768 tokens 11.95, 11.9, 12.1; 11.45 / 11.4, 11.65, 12.2;
// 10.55 / 11.2, 11.15, 11.3; 10.55; skv_select of 1400 buckets 6.25, 6.25, 6.4; 5.8 / 6.2, 6.6, 7.2; 5.45 / 6.05, 6.1, 6.25; 5.55, of 5200 8.2, 8.3, 8.45; 8.0 / 9.0, 10.6, 12.4; 7.6 /
// 8.3, 8.3, 8.5; 7.95.  The last one, skv_select of more than 2048 buckets, takes the totals of 64 groups from the histogram, a wave four groups, with a barrier more (64 groups of
// eight counters: 8.2, 8.5, 8.7; 7.75); the steps, whose blocks have more to do, would lose by that (131072 tokens, normal scores 15.75 -> 16.0).  Not kept: 64 groups of four
// counters (131072 tokens 16.8, 17.2, 17.8; 15.75), of eight (16.5, 16.7, 17.15; 15.7), of sixteen (17.1, 17.3, 17.8; 16.35), neighbouring buckets of a thread added up first (18.1, 18.1, 18.6; 17.5).  The three
// histograms are zeroed up front.  The search stops as soon as the crossing digit holds a single bucket
// (typically after one pass); buckets with exactly the cut's score are resolved in id order by a scan.
//
// The routine is written for few instructions per wave (a wave issues one instruction every 4+
// cycles, so instruction count is latency) and 32-bit arithmetic throughout (token totals < 2^31):
// thread t owns the kpt = ceil(S / 1024) consecutive buckets [t*kpt, (t+1)*kpt); keys, lengths and
// offsets of the first KREG of them live in registers (one global round trip); buckets beyond KREG per
// thread are re-read from memory in every phase.  The blocked ownership makes the id-ordered
// compaction a thread-local walk plus one block scan.
// ------------------------------------------------------------------------------------------------

constexpr int kSelKreg = 6;                                   // 1024 threads x 6 buckets in registers: S <= 6144
constexpr int kBins = 2048;                                   // 11-bit digits (the last pass uses 1024)
constexpr int kGroupCounters = 8;                             // counters of a group's total: lane l adds to l % 8

struct SelectShared {
    __attribute__((aligned(16))) unsigned long long hist[3][kBins];           // packed (count << 32 | total length) per digit
    __attribute__((aligned(16))) uint32_t group[3][kWave / 2 * kGroupCounters];   // total length per group of digits, in parts
    uint32_t wave_tot[3][kBlockWaves];                        // one slot per block scan
    int32_t gave_up;                                          // tagged scores: set by a thread whose wait ran out
    __attribute__((aligned(16))) uint32_t wmax[kBlockWaves];  // largest key per wave
};

// emit(s, off_s, len_s, sel_pos, tok_pos) is called by the owner thread of every selected bucket,
// sel_pos / tok_pos being the number of selected buckets / tokens with lower ids (sel_pos is only
// computed when COUNT is set, else 0).  Every thread of the block must call this; *n_sel_out /
// *n_tok_out are block-uniform.
// TAGGED: `sc` points at 64-bit (score, tag) words that other blocks of the same launch are writing; every thread reads
// its words again and again until they carry `tag` (at most wait_limit times: *ok_out tells whether they all
// arrived; if not, the selection is made from whatever was read and is meaningless).
template <int KREG, bool COUNT, bool TAGGED, typename Emit>
__device__ __forceinline__ void select_block(const float* __restrict__ sc, const int32_t* __restrict__ len,
                                             const int32_t* __restrict__ off, int32_t S, int32_t budget,
                                             SelectShared& sh, Emit emit, int32_t* n_sel_out, int32_t* n_tok_out,
                                             uint32_t tag = 0, int32_t wait_limit = 0, bool* ok_out = nullptr,
                                             uint32_t* __restrict__ key_lds = nullptr /* TAGGED: KREG * kBlockThreads words */) {
    constexpr bool kByHist = COUNT && KREG > 2;                // the groups' totals: from the histogram, else counted beside it
    constexpr int kGroupBins = kByHist ? kBins / kWave : 2 * kBins / kWave;      // digits of a group: a lane for each group, or two
    static_assert(sizeof(sh.group) == 3 * kWave * 16, "16 bytes a lane and pass: half of a group's counters, or a group's total");
    const int tid = threadIdx.x;
    *n_sel_out = 0;
    *n_tok_out = 0;
    if (ok_out) *ok_out = true;
    if (S <= 0 || budget <= 0) return;
    const int kpt = (S + kBlockThreads - 1) / kBlockThreads;
    const int32_t s0 = tid * kpt;
    const unsigned long long* tw = reinterpret_cast<const unsigned long long*>(sc);
    auto ldsc = [&](int32_t i) -> float { return TAGGED ? val_of(ld_tagged(tw + i)) : sc[i]; };

    uint32_t rkey[KREG];
    int32_t rlen[KREG], roff[KREG];
    static_assert(KREG <= 2 || KREG % 2 == 0, "the register-held buckets are loaded in pairs");
#pragma unroll
    for (int i = 0; i < KREG; ++i) { rkey[i] = 0; rlen[i] = 0; roff[i] = 0; }
    if (KREG > 2 && S >= 2) {
        // Many buckets per thread: they are consecutive, so two per load instruction (8 bytes at 4-byte alignment; with
        // two buckets per thread single loads measured slightly faster).  The pair is moved back so that it ends inside
        // the arrays; a slot past the end gets some in-range value and is dropped below.
        struct __attribute__((aligned(4))) Pair { uint32_t x, y; };
#pragma unroll
        for (int j = 0; j < KREG / 2; ++j) {
            if (2 * j < kpt) {                             // block-uniform; loads unconditional
                const int32_t idx = s0 + 2 * j, bse = min(idx, S - 2);
                Pair k{0u, 0u};
                if (!TAGGED) k = *reinterpret_cast<const Pair*>(sc + bse);
                const Pair l = *reinterpret_cast<const Pair*>(len + bse);
                const Pair o = *reinterpret_cast<const Pair*>(off + bse);
                const bool tail = idx == S - 1;            // the pair was moved back by one: the last bucket sits in .y
                rkey[2 * j] = tail ? k.y : k.x; rkey[2 * j + 1] = k.y;
                rlen[2 * j] = (int32_t)(tail ? l.y : l.x); rlen[2 * j + 1] = (int32_t)l.y;
                roff[2 * j] = (int32_t)(tail ? o.y : o.x); roff[2 * j + 1] = (int32_t)o.y;
            }
        }
    } else {
#pragma unroll
        for (int i = 0; i < KREG; ++i) {
            if (i < kpt) {                                 // block-uniform; addresses clamped, loads unconditional
                const int32_t sidx = min(s0 + i, S - 1);
                if (!TAGGED) rkey[i] = __float_as_uint(sc[sidx]);
                rlen[i] = len[sidx];
                roff[i] = off[sidx];
            }
        }
    }
    // zero the histograms while the loads are in flight
    auto zero_hist = [&]() {
        unsigned long long* h = &sh.hist[0][0];
#pragma unroll
        for (int i = 0; i < 3 * kBins / kBlockThreads; ++i) h[i * kBlockThreads + tid] = 0;
        if (!kByHist && tid < 3 * kWave) reinterpret_cast<uint4*>(sh.group)[tid] = make_uint4(0, 0, 0, 0);
    };
    zero_hist();
    if (tid == 0) sh.gave_up = 0;
    // The largest key of the block (over all buckets read, with or without tokens: an upper bound of the keys that take
    // part is all that is needed): a wave's maximum goes to LDS ahead of a barrier that is there anyway.
    uint32_t my_max = 0;
    auto share_max = [&]() {
        const uint32_t wm = (uint32_t)__builtin_amdgcn_readlane((int)wave_scan_max_u32(my_max), kWave - 1);
        if ((tid & (kWave - 1)) == 0) sh.wmax[tid >> 6] = wm;
    };
    if (!TAGGED) {
#pragma unroll
        for (int i = 0; i < KREG; ++i) {
            rkey[i] = score_key(__uint_as_float(rkey[i]));
            if (s0 + i >= S) rlen[i] = 0;                  // slots past the end take part in nothing
            if (i < kpt) my_max = max(my_max, rkey[i]);
        }
        for (int i = KREG; i < kpt; ++i)
            if (s0 + i < S) my_max = max(my_max, score_key(sc[s0 + i]));
        share_max();
        __syncthreads();
    } else {
        __syncthreads();                                   // the flag is clear
        // Every thread reads its own words until all of them carry the tag (bounded), without talking to anyone; the
        // block meets at one barrier afterwards.  A thread whose wait ran out raises the block's flag.
        const bool strided = kpt <= KREG;                  // every bucket of the pair is held in registers
        bool mine = false;
        if (strided) {
            // The words are read with consecutive lanes on consecutive words (thread t: words t, t + 1024, ...: whole
            // cache lines per wave instruction; a thread's own consecutive buckets would cost kpt times the memory
            // requests), and the keys reach their owners through LDS.
            // A wave asks again only for those of its instructions that found a word missing.
            uint32_t kk[KREG];
            unsigned int open = (1u << min(kpt, KREG)) - 1u;       // wave-uniform: instructions still to be asked
#pragma unroll
            for (int i = 0; i < KREG; ++i) kk[i] = 0u;
            for (int32_t round = 0; open != 0u && round < wait_limit; ++round) {
                unsigned long long wd[KREG];
#pragma unroll
                for (int i = 0; i < KREG; ++i) {
                    wd[i] = 0ull;
                    if ((open >> i) & 1u) wd[i] = ld_tagged(tw + min(i * kBlockThreads + tid, S - 1));
                }
#pragma unroll
                for (int i = 0; i < KREG; ++i) {
                    if ((open >> i) & 1u) {
                        kk[i] = (uint32_t)wd[i];
                        if (__all(tag_of(wd[i]) == tag)) open &= ~(1u << i);
                    }
                }
            }
            mine = open == 0u;
#pragma unroll
            for (int i = 0; i < KREG; ++i) {
                if (i < kpt) {
                    if constexpr (KREG == 1) rkey[i] = kk[i];          // a thread's word is its bucket's
                    else key_lds[i * kBlockThreads + tid] = kk[i];
                    my_max = max(my_max, score_key(__uint_as_float(kk[i])));
                }
            }
        } else {
            for (int32_t round = 0; !mine && round < wait_limit; ++round) {
                mine = true;
#pragma unroll
                for (int i = 0; i < KREG; ++i) {
                    const unsigned long long wd = ld_tagged(tw + min(s0 + i, S - 1));
                    rkey[i] = (uint32_t)wd;
                    mine = mine && tag_of(wd) == tag;
                }
                for (int i = KREG; i < kpt; ++i) {         // buckets beyond the registers are re-read in every phase below
                    if (s0 + i < S) {
                        const unsigned long long wd = ld_tagged(tw + s0 + i);
                        mine = mine && tag_of(wd) == tag;
                        my_max = max(my_max, score_key(val_of(wd)));
                    }
                }
            }
#pragma unroll
            for (int i = 0; i < KREG; ++i) my_max = max(my_max, score_key(__uint_as_float(rkey[i])));
        }
        share_max();
        if (!mine) sh.gave_up = 1;
        __syncthreads();
        if (sh.gave_up != 0 && ok_out) *ok_out = false;
        if (KREG > 1 && strided) {
#pragma unroll
            for (int i = 0; i < KREG; ++i)
                if (i < kpt) rkey[i] = key_lds[s0 + i];    // s0 + i < kpt * 1024 <= KREG * 1024
        }
#pragma unroll
        for (int i = 0; i < KREG; ++i) {
            rkey[i] = score_key(__uint_as_float(rkey[i]));
            if (s0 + i >= S) rlen[i] = 0;                  // slots past the end take part in nothing
        }
    }
    // the 16 waves' maxima, one a lane of every row of 16
    static_assert(kBlockWaves == 16, "a wave's maximum per lane of a DPP row");
    uint32_t kmax = sh.wmax[tid & (kBlockWaves - 1)];
    kmax = dpp_max_u32<0x128, 0xf>(kmax);                      // row_ror 8, 4, 2, 1
    kmax = dpp_max_u32<0x124, 0xf>(kmax);
    kmax = dpp_max_u32<0x122, 0xf>(kmax);
    kmax = dpp_max_u32<0x121, 0xf>(kmax);
    kmax = (uint32_t)__builtin_amdgcn_readfirstlane((int)kmax);
    SKV_T(1);

    // ---- weighted radix select of the cut ----------------------------------------------------------
    // Two attempts.  The first ranks the buckets by their distance below the best key, r = ~(kmax - key) (the same order
    // as the key), and looks only at those within 2^24 key steps of it (two binades of score; the others cannot be told
    // apart there and stay out of the histograms): digits of 11, 11 and 2 bits from bit 23 down, so that the first
    // histogram already resolves 2^13 key steps and the crossing digit mostly holds a single bucket: one pass instead of
    // two.  If those near buckets all fit the budget, the cut lies further down (or nowhere) and the second attempt runs
    // the plain digits 11, 11, 10 of the key over all buckets.
    uint32_t prefix = 0;        // resolved high bits of the cut's key
    int shift = 32;             // number of unresolved low bits
    int32_t carry = 0;          // total length of the buckets ranked strictly above the current digit range
    int32_t cut_cnt = 0;        // number of buckets sharing the resolved prefix
    bool select_all = false;
    bool near = true;           // first attempt: keys are distances below kmax
    auto to_rank = [&](uint32_t k) -> uint32_t { return near ? ~(kmax - k) : k; };
#pragma unroll
    for (int i = 0; i < KREG; ++i) rkey[i] = ~(kmax - rkey[i]);
    for (int attempt = 0; attempt < 2; ++attempt) {
        bool found_none = false;
        prefix = near ? 0xffu : 0u;
        shift = near ? 24 : 32;
        carry = 0;
#pragma unroll
        for (int pass = 0; pass < 3; ++pass) {
            const int bits = pass < 2 ? 11 : (near ? 2 : 10), nbins = 1 << bits, nshift = shift - bits;
            unsigned long long* H = sh.hist[pass];
            auto count = [&](uint32_t k, int32_t ln) {
                const uint32_t digit = (k >> nshift) & (nbins - 1);
                atomicAdd(&H[digit], (1ull << 32) | (unsigned long long)(uint32_t)ln);
                if (!kByHist) atomicAdd(&sh.group[pass][digit / kGroupBins * kGroupCounters + tid % kGroupCounters], (uint32_t)ln);
            };
#pragma unroll
            for (int i = 0; i < KREG; ++i)
                if (i < kpt && rlen[i] > 0 && (shift == 32 || (rkey[i] >> shift) == prefix)) count(rkey[i], rlen[i]);
            for (int i = KREG; i < kpt; ++i) {
                if (s0 + i < S && len[s0 + i] > 0) {           // a bucket without tokens takes part in nothing
                    const uint32_t k = to_rank(score_key(ldsc(s0 + i)));
                    if (shift == 32 || (k >> shift) == prefix) count(k, len[s0 + i]);
                }
            }
            __syncthreads();
            if constexpr (kByHist) {                               // 16 lanes a group, two digits each
                static_assert(2 * kBlockThreads == kBins && kGroupBins == 32);
                const uint4 two = *reinterpret_cast<const uint4*>(H + 2 * tid);
                uint32_t sum = two.x + two.z;
                sum = dpp_add_u32<0x128, 0xf>(sum);                // row_ror 8, 4, 2, 1
                sum = dpp_add_u32<0x124, 0xf>(sum);
                sum = dpp_add_u32<0x122, 0xf>(sum);
                sum = dpp_add_u32<0x121, 0xf>(sum);
                if (tid % 16 == 0) sh.group[pass][tid / 16] = sum;
                __syncthreads();
            }
            // The lane whose digits, `own` tokens of them, take the running total past the budget (none: -1); carry: the total above it.
            const int lane = tid & (kWave - 1);
            auto crossing = [&](uint32_t own) -> int {
                const uint32_t above = (uint32_t)carry + wave_scan_u32(own) - own;
                const unsigned long long at = __ballot(above <= (uint32_t)budget && above + own > (uint32_t)budget);
                if (at == 0ull) return -1;
                const int l = __builtin_ctzll(at);
                carry = __builtin_amdgcn_readlane((int)above, l);
                return l;
            };
            uint32_t in_group;
            if constexpr (kByHist) {
                in_group = sh.group[pass][kWave - 1 - lane];
            } else {                                               // the first of a group's two lanes stands for it
                const uint4 x = *reinterpret_cast<const uint4*>(&sh.group[pass][4 * (kWave - 1 - lane)]);
                in_group = dpp_add_u32<0xB1, 0xf>((x.x + x.y) + (x.z + x.w));
                if (lane & 1) in_group = 0;
            }
            const int at = crossing(in_group);
            if (at < 0) { found_none = true; break; }              // the buckets of this attempt all fit (only possible in pass 0)
            const int grp = kByHist ? kWave - 1 - at : (kWave - 1 - at) / 2, top = (grp + 1) * kGroupBins - 1;      // its highest digit
            const unsigned long long v = lane < kGroupBins ? H[top - lane] : 0ull;
            const int sub = crossing((uint32_t)v);
            const int digit = top - sub;
            cut_cnt = __builtin_amdgcn_readlane((int)(v >> 32), sub);
            prefix = (shift == 32) ? (uint32_t)digit : ((prefix << bits) | (uint32_t)digit);
            shift = nshift;
            if (cut_cnt == 1) break;                               // the cut is unique: it is the bucket that overflows
        }
        if (!found_none) break;
        if (!near) { select_all = true; break; }                   // every bucket was seen and they all fit: no cut
        // The buckets near the best key all fit: the cut, if there is one, is among the others.
        near = false;
#pragma unroll
        for (int i = 0; i < KREG; ++i) rkey[i] = kmax - ~rkey[i];  // back to the plain keys
        __syncthreads();                                           // every wave is past its reads of the first attempt
        zero_hist();
        __syncthreads();
    }
    const bool ties = !select_all && cut_cnt > 1;              // then shift == 0: several buckets share the cut's score
    SKV_T(2);

    // ---- compaction in id order --------------------------------------------------------------------
    // fn(i, s, key, len, off) for every bucket the thread owns, in id order
    auto for_items = [&](auto&& fn) {
#pragma unroll
        for (int i = 0; i < KREG; ++i)
            if (i < kpt && rlen[i] > 0) fn(i, s0 + i, rkey[i], rlen[i], roff[i]);
        for (int i = KREG; i < kpt; ++i)
            if (s0 + i < S && len[s0 + i] > 0) fn(i, s0 + i, to_rank(score_key(ldsc(s0 + i))), len[s0 + i], off[s0 + i]);
    };
    uint32_t tie_run = 0;          // length of tied buckets with lower ids (starts at the thread's base)
    if (ties) {
        uint32_t mine = 0;
        for_items([&](int, int32_t, uint32_t k, int32_t ln, int32_t) { if (k == prefix) mine += (uint32_t)ln; });
        uint32_t tot;
        tie_run = block_scan_u32(mine, sh.wave_tot[0], &tot) - mine;
    }
    auto chosen = [&](uint32_t k, int32_t ln, uint32_t& tie_acc) -> bool {
        if (select_all) return true;
        if ((k >> shift) > prefix) return true;                // shift < 32 here: at least one pass ran
        if (ties && k == prefix) {
            tie_acc += (uint32_t)ln;
            return (uint32_t)carry + tie_acc <= (uint32_t)budget;
        }
        return false;
    };
    // first walk: count; the register-held buckets that are chosen are remembered in a mask, so that the second walk
    // does not evaluate the rule again (buckets beyond the registers, re-read from memory, are evaluated in both walks)
    uint32_t my_tok = 0, my_cnt = 0, sel_mask = 0, tie_after_regs = tie_run;
    {
        uint32_t t = tie_run;
#pragma unroll
        for (int i = 0; i < KREG; ++i)
            if (i < kpt && rlen[i] > 0 && chosen(rkey[i], rlen[i], t)) { my_tok += (uint32_t)rlen[i]; my_cnt += 1; sel_mask |= 1u << i; }
        tie_after_regs = t;
        for (int i = KREG; i < kpt; ++i)
            if (s0 + i < S && len[s0 + i] > 0 && chosen(to_rank(score_key(ldsc(s0 + i))), len[s0 + i], t)) { my_tok += (uint32_t)len[s0 + i]; my_cnt += 1; }
    }
    uint32_t tot_tok, tot_cnt = 0;
    uint32_t pos_tok = block_scan_u32(my_tok, sh.wave_tot[1], &tot_tok) - my_tok;
    uint32_t pos_cnt = 0;
    if (COUNT) pos_cnt = block_scan_u32(my_cnt, sh.wave_tot[2], &tot_cnt) - my_cnt;
    if (my_cnt != 0) {
#pragma unroll
        for (int i = 0; i < KREG; ++i) {
            if ((sel_mask >> i) & 1u) {
                emit(s0 + i, roff[i], rlen[i], (int32_t)pos_cnt, (int32_t)pos_tok);
                pos_tok += (uint32_t)rlen[i];
                pos_cnt += 1;
            }
        }
        uint32_t t = tie_after_regs;
        for (int i = KREG; i < kpt; ++i) {
            if (s0 + i < S && len[s0 + i] > 0 && chosen(to_rank(score_key(ldsc(s0 + i))), len[s0 + i], t)) {
                emit(s0 + i, off[s0 + i], len[s0 + i], (int32_t)pos_cnt, (int32_t)pos_tok);
                pos_tok += (uint32_t)len[s0 + i];
                pos_cnt += 1;
            }
        }
    }
    *n_sel_out = (int32_t)tot_cnt;
    *n_tok_out = (int32_t)tot_tok;
    SKV_T(3);
}

// Stand-alone selection: the selected buckets go through an LDS list so that the token positions of
// each bucket are written by a whole wave, coalesced.
constexpr int kSelListCap = 2048;

__global__ __launch_bounds__(kBlockThreads) void select_kernel(const float* __restrict__ score,
                                                               const int32_t* __restrict__ sent_off,
                                                               const int32_t* __restrict__ sent_len, SeqView v,
                                                               int32_t Hkv, int32_t max_sel,
                                                               int32_t* __restrict__ sel_sent, int32_t* __restrict__ n_sel,
                                                               int32_t* __restrict__ tok_idx, int32_t idx_stride,
                                                               int32_t budget_cap, int32_t* __restrict__ n_tok) {
    __shared__ SelectShared sh;
    __shared__ int4 list[kSelListCap];                        // (bucket, offset, length, first output slot)
    const int bh = blockIdx.x, b = bh / Hkv, h = bh % Hkv;
    const Seq sq = seq_of(v, b);
    const int32_t budget = min(sq.budget, min(idx_stride, budget_cap));   // tok_idx holds at most idx_stride positions
    const float* sc = score + (int64_t)h * v.S_total + sq.sent_base;
    const int32_t* len = sent_len + sq.sent_base;
    const int32_t* off = sent_off + sq.sent_base + (v.cu_sent ? b : 0);
    int32_t* my_sel = sel_sent + (int64_t)bh * max_sel;
    int32_t* my_idx = tok_idx + (int64_t)bh * idx_stride;
    int32_t nsel, ntok;
    auto emit = [&](int32_t s, int32_t o, int32_t ln, int32_t sel_pos, int32_t tok_pos) {
        if (sel_pos < max_sel) my_sel[sel_pos] = s;
        if (sel_pos < kSelListCap) {
            list[sel_pos] = make_int4(s, o, ln, tok_pos);
        } else {                                              // list full: the owner writes its bucket's positions itself
            for (int32_t t = 0; t < ln && tok_pos + t < idx_stride; ++t) my_idx[tok_pos + t] = o + t;
        }
    };
    if (sq.n_sent <= 2 * kBlockThreads) select_block<2, true, false>(sc, len, off, sq.n_sent, budget, sh, emit, &nsel, &ntok);
    else select_block<kSelKreg, true, false>(sc, len, off, sq.n_sent, budget, sh, emit, &nsel, &ntok);
    if (threadIdx.x == 0) { n_sel[bh] = min(nsel, max_sel); n_tok[bh] = ntok; }
    __syncthreads();
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int listed = min(nsel, kSelListCap);
    for (int e = w; e < listed; e += kBlockWaves) {
        const int4 it = list[e];
        for (int32_t t = lane; t < it.z && it.w + t < idx_stride; t += kWave) my_idx[it.w + t] = it.y + t;
    }
}

hipError_t launch_select(Ctx* c, const float* score, const int32_t* sent_off, const int32_t* sent_len,
                         const SeqView& v, int32_t* sel_sent, int32_t* n_sel, int32_t* tok_idx, int32_t idx_stride,
                         int32_t budget_cap, int32_t* n_tok) {
    hipLaunchKernelGGL(select_kernel, dim3(v.B * c->d.n_kv_heads), dim3(kBlockThreads), 0, c->stream, score, sent_off,
                       sent_len, v, c->d.n_kv_heads, c->max_sel, sel_sent, n_sel, tok_idx, idx_stride, budget_cap, n_tok);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// Gather.  One 16-byte lane chunk per thread per row; a block copies RPB rows of K (blockIdx.z == 0) or V
// (blockIdx.z == 1) of one KV head with all its loads issued before its stores.  The pool pointer may be
// device-mapped pinned host memory: the same loads then cross PCIe.  RPB = 32 for a pool in HBM (16.7 MB per layer
// at a 2048-token budget: 6.3 us against 7.1 with 64 rows and 8.9 with 128), 64 for a host pool (53 GB/s over PCIe
// against 52 with 32 rows and 47 with 16).
// ------------------------------------------------------------------------------------------------
constexpr int kGatherRowsHbm = 32, kGatherRowsHost = kGatherRowsPerBlock;

template <int EB, int RPB>
__global__ __launch_bounds__(kGatherThreads) void gather_kernel(const char* __restrict__ Kl, const char* __restrict__ Vl,
                                                                int32_t T, const int32_t* __restrict__ tok_idx,
                                                                const int32_t* __restrict__ n_tok, int32_t budget,
                                                                char* __restrict__ Ks, char* __restrict__ Vs) {
    using R = Row<EB>;
    constexpr int kRowsPerIter = kGatherThreads / R::LPR;
    constexpr int kIter = RPB / kRowsPerIter;
    constexpr int kRowBytes = kHeadDim * EB;
    static_assert(kIter >= 1 && RPB % kRowsPerIter == 0, "block shape of the gather");
    const int h = blockIdx.y;
    const int32_t n = min(n_tok[h], budget);
    const int32_t j0 = blockIdx.x * RPB;
    if (j0 >= n) return;
    const char* src = (blockIdx.z == 0 ? Kl : Vl) + (int64_t)h * T * kRowBytes;
    char* dst = (blockIdx.z == 0 ? Ks : Vs) + (int64_t)h * budget * kRowBytes;
    const int r = threadIdx.x / R::LPR, cc = threadIdx.x % R::LPR;
    if (T <= 0) return;
    // Branch-free: indices and rows are clamped into range so every load can be issued up front
    // (two dependent rounds: all indices, then all rows); only the stores are predicated.
    int32_t x[kIter];
#pragma unroll
    for (int i = 0; i < kIter; ++i) {
        const int32_t j = min(j0 + i * kRowsPerIter + r, n - 1);
        x[i] = tok_idx[(int64_t)h * budget + j];
    }
    uint4 val[kIter];
#pragma unroll
    for (int i = 0; i < kIter; ++i) {
        const int32_t xc = min(max(x[i], 0), T - 1);
        val[i] = *reinterpret_cast<const uint4*>(src + (int64_t)xc * kRowBytes + cc * 16);
    }
#pragma unroll
    for (int i = 0; i < kIter; ++i) {
        const int32_t j = j0 + i * kRowsPerIter + r;
        if (j < n && x[i] >= 0 && x[i] < T) *reinterpret_cast<uint4*>(dst + (int64_t)j * kRowBytes + cc * 16) = val[i];
    }
}

template <int EB, int RPB>
static hipError_t launch_gather_g(Ctx* c, const void* K_layer, const void* V_layer, int32_t T, const int32_t* tok_idx,
                                  const int32_t* n_tok, int32_t budget, void* K_sel, void* V_sel) {
    const dim3 grid((budget + RPB - 1) / RPB, c->d.n_kv_heads, 2), block(kGatherThreads);
    hipLaunchKernelGGL((gather_kernel<EB, RPB>), grid, block, 0, c->stream, (const char*)K_layer, (const char*)V_layer, T, tok_idx,
                       n_tok, budget, (char*)K_sel, (char*)V_sel);
    return hipGetLastError();
}

hipError_t launch_gather(Ctx* c, const void* K_layer, const void* V_layer, int32_t T, bool host_pool, const int32_t* tok_idx,
                         const int32_t* n_tok, int32_t budget, void* K_sel, void* V_sel) {
    if (budget == 0) return hipSuccess;
    if (c->d.kv_dtype == SKV_BF16)
        return host_pool ? launch_gather_g<2, kGatherRowsHost>(c, K_layer, V_layer, T, tok_idx, n_tok, budget, K_sel, V_sel)
                         : launch_gather_g<2, kGatherRowsHbm>(c, K_layer, V_layer, T, tok_idx, n_tok, budget, K_sel, V_sel);
    return host_pool ? launch_gather_g<4, kGatherRowsHost>(c, K_layer, V_layer, T, tok_idx, n_tok, budget, K_sel, V_sel)
                     : launch_gather_g<4, kGatherRowsHbm>(c, K_layer, V_layer, T, tok_idx, n_tok, budget, K_sel, V_sel);
}

// ------------------------------------------------------------------------------------------------
// Attention (Eq. 3), split-K flash decoding.  A 1024-thread block (split, sequence * KV head) handles CHUNK consecutive retrieved
// tokens for the G query heads of its KV head, a wave for every 16 of them (Tile, below).
//   kDirect   : rows come from K_sel/V_sel and n_tok from memory (skv_attend).
//   kDirectDims : as kDirect, all tokens and 32 dims of the output to a block: there is nothing to merge.
//   kIndirect : rows of the pool through tok_idx, n_tok from memory.
//   kFused, kStep : the block first runs the selection for its (sequence, head) from the scores (redundantly with the other splits: the
//               scores are a few KB in L2, and it saves a launch plus a round trip through tok_idx) and reads
//               K/V straight from the pool (skv_decode_step).
//   1. every K and V piece is requested up front on clamped addresses (no load waits for a bounds test);
//   2. per wave: logits, max, weights, P V;   3. one barrier, then the block's sums relative to a common reference;
//   4. the un-normalised partial (reference, normaliser, sums) goes to the workspace with write-through stores; the last
//      block to arrive for the (sequence, KV head) -- a device-scope counter, no spinning -- merges the
//      partials with one round of independent loads and an online-softmax merge (kStep: see there).  A split that is
//      the only one writes the result.
// ------------------------------------------------------------------------------------------------

// ds_read_b64_tr_b16 (gfx950): within each group of 16 lanes, lane i receives element i % 4 of the 8-byte pieces that
// lanes i / 4, i / 4 + 4, i / 4 + 8 and i / 4 + 12 of the group point at, in that order.  With lane s of the group
// pointing at dims 4 (s % 4) .. + 3 of row s / 4 of a row-major 4 x 16 block of bf16, lane i gets column i of the
// block's four rows: the B fragment of a 16x16x16 MFMA whose k index runs over the rows (one read instead of four
// 2-byte reads).
typedef short bf16x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ bf16x4_t lds_read_tr16(const char* p) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((bf16x4_t __attribute__((address_space(3)))*)(p));
}

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
// A wave's weights are relative to its largest logit (log2 units), so that its largest weight is 1, which bf16 holds exactly: relative to a rounded
// maximum the error of out is 1.2 to 8 times as large (logits of standard deviation 0.5 to 8).  Where sums of waves and blocks meet they are
// relative to whole numbers: they then move from one reference to another by an exact power of two, which costs no more than a
// bare exp2 and reaches below the normal range of a float.
// 2^d for whole d <= 0; 0 for -infinity and for NaN (the difference of two references of nothing)
__device__ __forceinline__ float pow2_whole(float d) { return ldexpf(1.f, (int)fmaxf(d, -512.f)); }
// x <- 2^(x - ref), four weights of a lane (-infinity: 0).  The bare instruction flushes results below the normal range to zero; a wave
// that has such arguments (masked ones count) takes the full function: in every wave that one costs 2-3 % of the step of one sequence.
__device__ __forceinline__ void exp2_weights(float (&x)[4], float ref) {
    if (__any(fminf(fminf(x[0], x[1]), fminf(x[2], x[3])) < ref - 126.f)) {
#pragma unroll
        for (int j = 0; j < 4; ++j) x[j] = exp2f(x[j] - ref);
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) x[j] = __builtin_amdgcn_exp2f(x[j] - ref);
    }
}
// over the four lanes t16, t16 + 16, t16 + 32, t16 + 48 of a tile column; every lane gets the result
__device__ __forceinline__ float max_quads(float x) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    const float y = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(y), __float_as_uint(y), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float sum_quads(float x) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    const float y = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(y), __float_as_uint(y), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// of lane (t + 16 - N) % 16 of the row of 16
template <int N> __device__ __forceinline__ float of_row_turned(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x120 + N /* row_ror */, 0xf, 0xf, false));
}
// of the lane l ^ 8
__device__ __forceinline__ float other_eight(float x) { return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x128 /* row_ror:8 */, 0xf, 0xf, false)); }
// the larger of the lanes l and l ^ 32, in both
__device__ __forceinline__ float max_halves(float x) {
    const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
}

// A wave's tile of 16 tokens on the matrix cores.  With t16 = lane % 16 and qd = lane / 16:
//  * S^T = K Q^T: the A fragment is a 16-byte piece (at byte 64 s + 16 qd, s < kPieces) of token t16's key, the B fragment the same dims
//    of head t16's query (heads >= G are zero).  The order of the dims inside the contraction is free as long as A and B agree,
//    so a piece loaded from a row is one 32-deep step of v_mfma_f32_16x16x32_bf16, or four 4-deep steps of
//    v_mfma_f32_16x16x4_f32, one for each of its floats.  The accumulator holds logit(token 4 qd + j, head t16), j = 0..3.
//  * O = P V: that accumulator layout IS the A fragment layout of P (head t16, tokens 4 qd + j), for bf16 of one
//    v_mfma_f32_16x16x16_bf16, for fp32 of four 4-deep steps, step j on the tokens 4 qd + j.  The B fragments V[token 4 qd + j][16 dt + t16]
//    are read from a wave-private LDS copy of the 16 value rows, laid out so that the four token groups of a read fall into
//    different banks (bf16: 16 bytes between rows; fp32: 64-byte groups exchanged, no gaps, for rows that come by load_lds_stream).
//  * bf16 weights are rounded to bf16 (nearest even) and the normaliser sums the rounded weights; fp32 ones are used as they are.
//  * A NaN among a head's live logits makes its normaliser NaN, and with it out and lse, through every sum and merge below.
// fp32 through the vector pipe (rows over lanes, sums of the logits over 32 lanes by exchanges) took 3.7 us from the loads to
// the logits of 128 tokens and 1.7 to the partial result, budget 512, 4 heads; see launch_step for what it takes now.
template <int EB, int DIMS = kHeadDim> struct Tile {                // DIMS: dims of the value rows (bf16: 32, or all)
    static_assert(EB == 2 || DIMS == kHeadDim, "fp32 pieces are exchanged over the whole row");
    static constexpr int kPieces = kHeadDim * EB / 64;                // key pieces of a lane
    static constexpr int LPR = DIMS * EB / 16, RPL = kWave / LPR; // lanes of a value row, value rows of a load
    static constexpr int kLoads = 16 / RPL;                           // value loads of a lane: rows RPL i + lane / LPR
    static constexpr int kPitch = DIMS * EB + (EB == 2 ? 16 : 0); // bytes of a value row in LDS
    // place of 16-byte piece `piece` of value row `row` in the tile
    __device__ static __forceinline__ int place(int row, int piece) { return row * kPitch + 16 * (EB == 2 ? piece : piece ^ (4 * (row >> 2))); }

    // query(s): this lane's piece s of the queries
    template <typename Query>
    __device__ static __forceinline__ f32x4_t logits(const uint4 (&k)[kPieces], Query query) {
        f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
        if constexpr (EB == 2) {
#pragma unroll
            for (int s = 0; s < kPieces; ++s)
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, k[s]), __builtin_bit_cast(bf16x8_t, query(s)), acc, 0, 0, 0);
        } else {
            f32x4_t acc2 = {0.f, 0.f, 0.f, 0.f};                      // two chains: a step's latency is longer than its issue
#pragma unroll
            for (int s = 0; s < kPieces; ++s) {
                const uint4 q = query(s);
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(k[s].x), __uint_as_float(q.x), acc, 0, 0, 0);
                acc2 = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(k[s].y), __uint_as_float(q.y), acc2, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(k[s].z), __uint_as_float(q.z), acc, 0, 0, 0);
                acc2 = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(k[s].w), __uint_as_float(q.w), acc2, 0, 0, 0);
            }
            acc += acc2;
        }
        return acc;
    }
    // weights as P V takes them; the return value is what the normaliser sums
    __device__ static __forceinline__ float weight(float& p) {
        if constexpr (EB == 2) {
            uint32_t u = __float_as_uint(p);
            u += 0x7fffu + ((u >> 16) & 1u);
            p = p == p ? __uint_as_float(u & 0xffff0000u) : p;            // (the carry could leave a NaN's bits as a number)
        }
        return p;
    }
    // o[dt] += P V of the tile at `v` (16 rows of pitch kPitch); element j of o[dt]: head 4 qd + j, dim 16 dt + t16
    __device__ static __forceinline__ void output(const float (&p)[4], const char* v, int lane, f32x4_t (&o)[DIMS / 16]) {
        const int t16 = lane & 15, qd = lane >> 4;
        if constexpr (EB == 2) {
            const bf16x4_t pa = {(short)(__float_as_uint(p[0]) >> 16), (short)(__float_as_uint(p[1]) >> 16), (short)(__float_as_uint(p[2]) >> 16),
                                 (short)(__float_as_uint(p[3]) >> 16)};
            // B fragments by the LDS transpose read: this lane points at dims 4 (t16 % 4) .. + 3 of value row 4 qd + t16 / 4
            const char* vtr = v + (4 * qd + (t16 >> 2)) * kPitch + 8 * (t16 & 3);
#pragma unroll
            for (int dt = 0; dt < DIMS / 16; ++dt) o[dt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(pa, lds_read_tr16(vtr + 32 * dt), o[dt], 0, 0, 0);
        } else {
#pragma unroll
            for (int dt = 0; dt < DIMS / 16; ++dt) {
                const char* col = v + 4 * qd * kPitch + 64 * (dt ^ qd) + 4 * t16;
#pragma unroll
                for (int j = 0; j < 4; ++j) o[dt] = __builtin_amdgcn_mfma_f32_16x16x4f32(p[j], *reinterpret_cast<const float*>(col + j * kPitch), o[dt], 0, 0, 0);
            }
        }
    }
};

constexpr int max_of(int a, int b) { return a > b ? a : b; }

// orders a wave's LDS accesses before it against those after it (other lanes of the wave wrote or will write the same words)
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A wave leaves its sums of P V (element j of o[dt]: head 4 qd + j, dim 16 dt + t16) in the space of its value tile, head fastest (dim d,
// head g at [d * G + g]), so that a lane stores its heads of one dim with a single instruction.
template <int G, int NDT>
__device__ __forceinline__ void leave_sums(char* tile, const f32x4_t (&o)[NDT]) {
    const int lane = threadIdx.x & 63, t16 = lane & 15, qd = lane >> 4;
    if (4 * qd < G) {
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt) {
            float* dst = reinterpret_cast<float*>(tile) + (16 * dt + t16) * G + 4 * qd;
            if constexpr (G >= 4) *reinterpret_cast<float4*>(dst) = make_float4(o[dt][0], o[dt][1], o[dt][2], o[dt][3]);
            else if constexpr (G == 2) *reinterpret_cast<float2*>(dst) = make_float2(o[dt][0], o[dt][1]);
            else dst[0] = o[dt][0];
        }
    }
}
// What a wave leaves of its softmax for the block: its largest logit m as 2^m = factor * 2^reference, and the sum of its weights.
template <int NT> struct WaveSums {
    __attribute__((aligned(16))) float reference[16][NT], factor[16][NT], sum[16][NT];      // per head and wave
    // `base`: m, or 0 where there is no logit to speak of (m == -infinity)
    __device__ __forceinline__ void leave(int head, int w, float m, float base, float l) {
        reference[head][w] = rintf(m);
        factor[head][w] = __builtin_amdgcn_exp2f(base - rintf(base));
        sum[head][w] = l;
    }
};
// lane N of the lane's row of 16
template <int N> __device__ __forceinline__ float of_row(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x150 + N /* row_newbcast */, 0xf, 0xf, false));
}
// A barrier later: the block's output relative to its common reference, from the sums that NT waves left `stride` bytes apart, each relative to
// the wave's own max.  put(g, d, sum, reference, normaliser) for every head and dim, consecutive lanes on consecutive dims; norm(2 g, reference) and
// norm(2 g + 1, normaliser) of all heads, by lanes of the first wave together.
// A wave makes 16 dims of up to four heads: row r of its lanes adds up a quarter of the NT waves, a lane one dim of the four heads, 16 bytes at a time as the sums lie, and
// the rows meet in registers, where row r keeps head r.  What the weights of the NT waves and four heads take (differences of references, powers of two) is formed
// once a wave, lane 4 j + g of row r for wave NT / 4 r + j and head g, and handed out along the row.  (A lane per output, or two, each with all of the weights, and with sums
// read four lanes to a bank, and the references in a store of their own behind another barrier, with the queries as below: us per layer 131072 tokens 16.1 -> 15.9, 6
// sequences of 1900 to 21001 16.3 -> 15.9, 16 of 64 heads 50.1 -> 49.6.)
template <int G, int NT, int DIMS = kHeadDim, typename Put, typename Norm>
__device__ __forceinline__ void block_sums(const char* tiles, int stride, const WaveSums<NT>& ws, Put put, Norm norm) {
    constexpr int kHeads = G < 4 ? G : 4, kPer = NT / 4, kSlices = DIMS / 16;
    static_assert(NT % 4 == 0 && kPer <= 4 && DIMS % 16 == 0 && (G <= 4 || G == 8), "a weight per lane, a row of lanes per head");
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, t = lane & 15, row = lane >> 4;
    if (w >= kSlices * (G / kHeads)) return;
    const int h0 = G > 4 ? w / kSlices * 4 : 0, d = w % kSlices * 16 + t;
    // (reference, normaliser) of head h + t % 4, and the lane's weight
    auto head_sums = [&](int h, float& mb, float& lb) -> float {
        const int g = h + min(t & 3, kHeads - 1), k = kPer * row + ((t >> 2) & (kPer - 1));
        const float m = ws.reference[g][k], f = ws.factor[g][k], l = ws.sum[g][k];
        mb = m;
        if constexpr (kPer == 4) mb = fmaxf(mb, other_eight(mb));
        if constexpr (kPer >= 2) mb = fmaxf(mb, of_row_turned<4>(mb));
        mb = max_quads(mb);
        const float c = f * pow2_whole(m - mb);
        lb = c * l;
        if constexpr (kPer == 4) lb += other_eight(lb);
        if constexpr (kPer >= 2) lb += of_row_turned<4>(lb);
        lb = sum_quads(lb);
        if (lb != lb) mb = 0.f;                                       // NaN, perhaps with no other logit: merges pass over a reference of -infinity
        return c;
    };
    float mb, lb;
    const float c = head_sums(h0, mb, lb);
    float o[4] = {0.f, 0.f, 0.f, 0.f};
    auto add = [&](auto jj) {
        constexpr int j = decltype(jj)::value;
        if constexpr (j < kPer) {
            const char* src = tiles + (kPer * row + j) * stride + (d * G + h0) * 4;
            float x[kHeads];
            __builtin_memcpy(x, __builtin_assume_aligned(src, 4 * kHeads), sizeof(x));
            o[0] += of_row<4 * j>(c) * x[0];
            if constexpr (kHeads >= 2) o[1] += of_row<4 * j + 1>(c) * x[1];
            if constexpr (kHeads >= 4) { o[2] += of_row<4 * j + 2>(c) * x[2]; o[3] += of_row<4 * j + 3>(c) * x[3]; }
        }
    };
    add(std::integral_constant<int, 0>{});
    add(std::integral_constant<int, 1>{});
    add(std::integral_constant<int, 2>{});
    add(std::integral_constant<int, 3>{});
    // two exchanges: halves of the wave add heads (0, 1 | 2, 3), rows of a half one each
    auto halves = [](float x, float y) { const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false); return __uint_as_float(s[0]) + __uint_as_float(s[1]); };
    auto rows = [](float x, float y) { const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false); return __uint_as_float(s[0]) + __uint_as_float(s[1]); };
    const float sum = rows(halves(o[0], o[2]), halves(o[1], o[3]));
    auto of_head = [&](float x) {                                     // head r's in row r
        int v = __builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x00 /* quad_perm */, 0x1, 0xf, false);
        v = __builtin_amdgcn_update_dpp(v, __float_as_int(x), 0x55, 0x2, 0xf, false);
        v = __builtin_amdgcn_update_dpp(v, __float_as_int(x), 0xAA, 0x4, 0xf, false);
        return __int_as_float(__builtin_amdgcn_update_dpp(v, __float_as_int(x), 0xFF, 0x8, 0xf, false));
    };
    const float mr = of_head(mb), lr = of_head(lb);
    if (row < kHeads) put(h0 + row, d, sum, mr, lr);
    if (w == 0) {
        float m2 = mb, l2 = lb;
        if constexpr (G > 4) (void)head_sums(4, m2, l2);
        const int g = (t & 3) + 4 * (t >> 3);
        const float v = t < 8 ? (t < 4 ? mb : lb) : (t < 12 ? m2 : l2);
        if (row == 0 && (t & 3) < kHeads && g < G) norm(2 * g + ((t >> 2) & 1), v);
    }
}

// kStep: blocks of a pair that merge
__device__ __forceinline__ int merging_blocks(int G, int lg_merge) { return lg_merge >= 0 ? G << lg_merge : G >> -lg_merge; }

// In the order in which the single-launch step needs them: what it takes to ask for the mean keys in the first two lines.
struct AttArgs {
    // kStep: the blocks of a (sequence, head) pair first score the pair's buckets between them
    const char* q_score;      // [B][Hq][D]
    const char* semvec;       // the layer's table [Hkv][S_total][D]
    unsigned int* step_epoch; // [pairs][kStepEpochStride]: launches of the single-launch step each pair has been through
    unsigned long long* step_score;   // [pairs][score_stride] (score, tag) words
    const char* q;            // [B][Hq][D]
    float* out;
    SeqView v;
    int32_t Hkv;
    int32_t sv_bytes;         // bytes per element of the table: 4, 2 or 1
    int32_t score_stride;
    int32_t lg_parts;         // kStep: log2 of the blocks per pair
    int32_t parts;            // kStepRagged: blocks per pair, and 2^32 / that, rounded up
    uint32_t per_part;
    int32_t chunk;            // kStepRagged: tokens of an attending block (a multiple of 16, at most CHUNK), and 2^32 / that, rounded up
    uint32_t per_chunk;
    int32_t lg_merge;         // log2 of the blocks that merge one query head; -1: a block merges two heads
    int32_t budget_cap;       // budgets are clamped to this (the context's budget hint, at most max_budget)
    const int32_t* sent_off;  // kFused
    const int32_t* sent_len;  // kFused
    int32_t* n_tok_out;       // kFused, nullable: [B*Hkv]
    const char* Kb;           // kDirect: K_sel [B*Hkv][row_stride][D]; else the layer's pool [Hkv][T_total][D]
    const char* Vb;
    int32_t* tok_idx_out;     // kFused, nullable: [B*Hkv][idx_stride]
    unsigned long long* step_part;    // [blocks][step_part_words(G)] (value, tag) words: a block's sums [G][kHeadDim], then (reference, normaliser) [G]
    float* lse;
    int32_t idx_stride;       // kFused, kIndirect: max_budget (positions per pair in tok_idx / tok_idx_out)
    int32_t wait_limit;       // rounds of polling before a block gives up
    unsigned int* err_dev;    // set to 1 by a block that gave up
    unsigned int* err_host;   // the same word in pinned host memory (device address), nullable
    // the other forms
    const int32_t* n_tok;     // kDirect, kIndirect: [B*Hkv]
    const int32_t* tok_idx;   // kIndirect: [B*Hkv][idx_stride] positions local to the sequence
    const float* score;       // kFused: [Hkv][S_total]
    int32_t row_stride;       // kDirect
    int32_t max_splits;       // partial slots per query head (counted in 64-token chunks)
    float* part;
    float* ml;
    unsigned int* counter;
};

enum { kDirect = 0, kFused = 1, kIndirect = 2, kStep = 3, kStepRagged = 4, kDirectDims = 5 };      // kStepRagged: any number of blocks, any share of the budget

// Arguments are demanded together, so that their loads go out in one batch; left alone, the compiler loads each argument before its first use: one
// dependent round trip per branch, and a scalar-cache miss for each new 64-byte line of the argument block.
__device__ __forceinline__ void demand_seq_args(const AttArgs& a) {
    asm volatile("" ::"s"(a.v.cu_tok), "s"(a.v.cu_sent), "s"(a.v.budget_arr), "s"(a.v.T_total), "s"(a.v.S_total), "s"(a.v.budget), "s"(a.Hkv), "s"(a.q), "s"(a.out));
}
template <int MODE> __device__ __forceinline__ void demand_args(const AttArgs& a) {
    if constexpr (MODE != kDirect && MODE != kDirectDims) demand_seq_args(a);
    if constexpr (MODE == kFused)
        asm volatile("" ::"s"(a.score), "s"(a.sent_off), "s"(a.sent_len), "s"(a.tok_idx_out), "s"(a.n_tok_out), "s"(a.idx_stride), "s"(a.budget_cap));
    else
        asm volatile("" ::"s"(a.q), "s"(a.n_tok), "s"(a.tok_idx), "s"(a.row_stride), "s"(a.idx_stride), "s"(a.Hkv), "s"(a.out));
    asm volatile("" ::"s"(a.Kb), "s"(a.Vb), "s"(a.lse), "s"(a.max_splits), "s"(a.part), "s"(a.ml), "s"(a.counter));
}
// kStep, first: what the scores need, and a word of each line of the rest, which is on its way to the scalar cache then
template <bool RAGGED> __device__ __forceinline__ void demand_score_args(const AttArgs& a) {
    demand_seq_args(a);
    if constexpr (RAGGED) asm volatile("" ::"s"(a.parts), "s"(a.per_part), "s"(a.chunk));
    else asm volatile("" ::"s"(a.lg_parts));
    asm volatile("" ::"s"(a.q_score), "s"(a.semvec), "s"(a.step_epoch), "s"(a.step_score), "s"(a.score_stride), "s"(a.sv_bytes), "s"(a.lg_merge), "s"(a.budget_cap),
                 "s"(a.idx_stride));
}
// ... and after the scores, while others may still be at theirs, all the rest.  They are read through a pointer formed there, else the compiler asks for them with
// the first ones, has no registers for them and waits for them to move them away.
__device__ __forceinline__ void load_attend_args(AttArgs& a) {
    const AttArgs __attribute__((address_space(4))) * p = (const AttArgs __attribute__((address_space(4)))*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    a.sent_off = p->sent_off; a.sent_len = p->sent_len; a.n_tok_out = p->n_tok_out; a.Kb = p->Kb; a.Vb = p->Vb; a.tok_idx_out = p->tok_idx_out;
    a.step_part = p->step_part; a.lse = p->lse; a.idx_stride = p->idx_stride; a.wait_limit = p->wait_limit; a.err_dev = p->err_dev; a.err_host = p->err_host;
    asm volatile("" ::"s"(a.sent_off), "s"(a.sent_len), "s"(a.n_tok_out), "s"(a.Kb), "s"(a.Vb), "s"(a.tok_idx_out), "s"(a.step_part), "s"(a.lse), "s"(a.idx_stride),
                 "s"(a.wait_limit), "s"(a.err_dev), "s"(a.err_host));
}

// 16 bytes of a K/V row.  POOL: rows straight from the pool are read once (non-temporal: 32 layers of one 32K sequence 456 ->
// 445 us with the keys' loads, 461 -> 456 with the values' and the mean keys'); rows of K_sel/V_sel have just been written.
template <bool POOL>
__device__ __forceinline__ uint4 ld_row(const char* p) {
    return POOL ? ld_stream(p) : *reinterpret_cast<const uint4*>(p);
}

constexpr int kDimsPerBlock = 32, kMaxDirectDims = 416, kMaxDirectDims1 = 320;       // kDirectDims: dims of a block, tokens of a call (of one query head per KV head)
// kDirectDims, blocks of 16 waves: pair fastest in the grid, so that the blocks of a pair find their common keys in one L2, and each begins at another quarter of
// them.  Us a call, 32 query heads on 8: 257 tokens 6.02 -> 5.92 (5.98 without the quarters); with two lanes an output in block_sums, as it was then, 200 5.45 -> 4.97, 256 5.70 -> 5.22,
// 257 6.05 -> 5.78, 384 6.86 -> 6.34; 64 on 8: 256 6.15 -> 5.82; 32 on 32: 256 5.57 -> 5.37.  Fewer waves, heads first: 8 on 8, 64 tokens 3.03 -> 3.15, 128 3.54 -> 3.70; 32
// on 32, 64 tokens 3.57 -> 3.25.
template <int MODE, int CHUNK> constexpr bool kPairFirst = MODE == kStep || MODE == kStepRagged || (MODE == kDirectDims && CHUNK / 16 >= kBlockWaves);
// ceil(n / d) with `per` = 2^32 / d rounded up; exact while n + d <= 2^32 / d
__device__ __forceinline__ int32_t ceil_div(int32_t n, int32_t d, uint32_t per) { return (int32_t)__umulhi((uint32_t)(n + d - 1), per); }

// CHUNK = retrieved tokens per block, a tile of 16 for each of CHUNK / 16 waves (512: two tiles a wave): the smallest whose blocks all run
// at once, see launch_step, launch_select_attend and launch_attend.
template <int EB, int G, int MODE, int CHUNK>
__global__ __launch_bounds__(kBlockThreads) void attend_kernel(AttArgs args) {
    AttArgs a = args;
    constexpr int kDims = MODE == kDirectDims ? kDimsPerBlock : kHeadDim;         // dims of the output that a block makes
    constexpr bool kRowsDirect = MODE == kDirect || MODE == kDirectDims;
    using X = Tile<EB, kDims>;
    constexpr bool kStepping = MODE == kStep || MODE == kStepRagged;
    constexpr int kRowBytes = kHeadDim * EB;
    constexpr float kLog2e = 1.4426950408889634f, kLn2 = 0.6931471805599453f;
    constexpr int kTiles = CHUNK / 16 < kBlockWaves ? CHUNK / 16 : kBlockWaves;    // waves with 16-token tiles
    constexpr int kPasses = CHUNK / 16 / kTiles;              // tiles of such a wave: w, w + 16
    static_assert(kTiles * kPasses * 16 == CHUNK && CHUNK % kWave == 0 && kPasses <= (EB == 2 ? 2 : 1), "the rows of a wave's tiles are in registers together");
    constexpr int kOut = G * kDims;                        // outputs of the block
    constexpr int kCol2 = kOut / 2;                           // float pairs over the G heads
    constexpr int kGroups = kBlockThreads / kCol2;            // split groups of the merge: 16, 8, 4, 2 for G = 1, 2, 4, 8

    // One region of LDS, used in turn by the selection (SelectShared, and the pair's scores on their way to the owning threads), by the
    // waves' value tiles and, in each wave's own tile, its partial sums (dim d, head g at [d * G + g]), and by the merge.
    constexpr bool kSel = MODE == kFused || kStepping;    // the block runs the selection itself
    constexpr int kTileBytes = 16 * X::kPitch;
    static_assert(kOut * 4 <= kTileBytes, "a wave's partial sums fit in its value tile");
    constexpr int kSelBytes = kSel ? (int)((sizeof(SelectShared) + 15) / 16 * 16) : 0;
    constexpr int kKeyBytes = kStepping ? kSelKreg * kBlockThreads * 4 : 0;
    constexpr int kShBytes = max_of(max_of(kTiles * kTileBytes, kSelBytes + kKeyBytes), kStepping ? 0 : 16 * kBlockThreads);
    __shared__ __attribute__((aligned(16))) char sm[kShBytes];
    __shared__ WaveSums<kTiles> sm_waves;
    __shared__ int sm_last;                                                 // kStep: set by a thread of the merge whose wait ran out
    // The group's queries, requested first of all and once a block: the tile waves read their fragments from here.  (Every tile wave with fragments of its own from memory,
    // four 1 KB requests each, eight in fp32: see block_sums.)
    constexpr int kQueryPitch = kRowBytes + 64;                               // the four heads that a fragment read meets lie in different banks
    __shared__ __attribute__((aligned(16))) char sm_q[G * kQueryPitch];
    __shared__ int32_t sm_row[CHUNK];
    constexpr int kMergeWords = kStepping ? 3 * (kBlockThreads + kWave) : 1;
    __shared__ float sm_merge[kMergeWords];                                   // kStep: the merging block's scratch

    // Heads, sequences and splits are the dimensions of the grid (nothing has to be divided); where head and sequence are fastest (kPairFirst), the hardware's
    // round-robin of consecutive blocks over the XCDs keeps the blocks of a pair together whenever the number of pairs is a multiple of the number of XCDs.
    constexpr bool kFirst = kPairFirst<MODE, CHUNK>;
    const int h = (int)(kFirst ? blockIdx.x : blockIdx.y), b = (int)(kFirst ? blockIdx.y : blockIdx.z), part = (int)(kFirst ? blockIdx.z : blockIdx.x);
    const int split = MODE == kDirectDims ? 0 : part;
    const int dim0 = MODE == kDirectDims ? part * kDims : 0;        // first of the block's dims
    const int bh = b * a.Hkv + h;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int t16 = lane & 15, qd = lane >> 4;
    const int n_pairs = a.v.B * a.Hkv;
    const int64_t qhead0 = (int64_t)bh * G;                       // first query head of the group
    if constexpr (kStepping) demand_score_args<MODE == kStepRagged>(a);
    else demand_args<MODE>(a);
    // What the block does before it asks for its first mean keys is on the way of every launch.  Us per layer, grids of one dimension (two divisions), the sequence's
    // numbers one after the other, all arguments at once (there is no room for them: their waits came first too) and the tag formed here / this: 4096 tokens, fp32
    // 10.4 / 9.9, 32768 11.7 / 11.25, 131072 16.45 / 16.4, 6 sequences of 1900 to 21001 18.0 / 17.35, 3 of 8192 15.9 / 15.6.
    // kStep: the tag of this launch for this pair.  Every launch of the pair ends with its epoch advanced by one (block 0,
    // after it has seen the partial of every attending block, each of which had seen every score of the pair: so every
    // block whose tag matters has read the epoch by then), and the pair's number makes tags of different pairs differ.
    uint32_t tag = 0;
    StepState state = {};
    if constexpr (kStepping) {
        state = {ld_agent(a.step_epoch + bh * kStepEpochStride), bh};
    }
    Seq sq = {};
    if constexpr (!kRowsDirect) sq = seq_of_step(a.v, b);
    const int32_t chunk = MODE == kStepRagged ? a.chunk : CHUNK;        // tokens of a block
    auto blocks_of = [&](int32_t tokens) { return MODE == kStepRagged ? ceil_div(tokens, chunk, a.per_chunk) : (tokens + CHUNK - 1) / CHUNK; };
    const int32_t j0 = split * chunk;
    const int slot = split * (CHUNK / kWave);                     // partial slot (slots are counted in 64-token units)
    SKV_T(0);

    constexpr int kQueryPieces = G * kRowBytes / 16;                  // a thread each
    static_assert(kQueryPieces <= kTiles * kWave, "by tile waves");
    // Where no selection lies between the request and the rows, the queries' way through LDS is a barrier behind the rows' requests.  Every wave has its own fragments from memory
    // there, bf16 ones requested first of all, fp32 ones, twice the registers, just ahead of the keys; but for eight heads in bf16 and blocks of dims with a tile a wave,
    // where a wave would ask for as much as for its keys, and positions (kIndirect).  Us per call, once a block / own: 32 query heads on 8, 257 tokens 6.03 / 5.57, 400 7.06 /
    // 6.48, 1000 7.62 / 7.52, 2048 8.49 / 8.28, 4096 10.3 / 10.0, fp32, 257 9.8 / 9.4, 2048 11.5 / 11.1, 4096 16.7 / 14.6; 64 on 8 fp32, 4096 18.2 / 16.6; bf16, 500 7.27 / 7.40,
    // 1000 7.73 / 7.81, 2048 9.84 / 9.78; 24 on 3, 448 7.08 / 7.20; 64 sequences through positions 88.9 / 89.3, fp32 74.9 / 68.7.  (bf16 ones just ahead of the keys: 1000 7.70,
    // 2048 8.55.)
    constexpr bool kOwnQueries = !kSel && (EB == 4 || (MODE == kDirect && G < 8) || (MODE == kDirectDims && kPasses > 1));
    uint4 qB[X::kPieces];                                             // lane (t16, qd): pieces of head t16
    auto own_queries = [&]() {
#pragma unroll
        for (int s2 = 0; s2 < X::kPieces; ++s2)
            qB[s2] = *reinterpret_cast<const uint4*>(a.q + (qhead0 + min(t16, G - 1)) * kRowBytes + 64 * s2 + 16 * qd);
    };
    if constexpr (kOwnQueries && EB == 2) { if (w < kTiles) own_queries(); }
    uint4 q_piece = make_uint4(0, 0, 0, 0);
    if (!kOwnQueries && tid < kQueryPieces) q_piece = *reinterpret_cast<const uint4*>(a.q + qhead0 * kRowBytes + 16 * tid);
    auto leave_queries = [&]() {                                      // a barrier must follow
        if (tid < kQueryPieces) *reinterpret_cast<uint4*>(sm_q + tid / (kRowBytes / 16) * kQueryPitch + tid % (kRowBytes / 16) * 16) = q_piece;
    };

    int32_t n;                                                    // retrieved tokens of this (sequence, head)
    bool step_ok = true;                                          // kStep: every wait of this block ended in time
    if constexpr (kSel) {
        SelectShared& sel_sh = *reinterpret_cast<SelectShared*>(sm);
        const int32_t budget = min(sq.budget, a.budget_cap);
        if constexpr (kStepping) {
            // ---- 0. scores of this block's share of the pair's buckets, published to the pair's other blocks ---------
            // Part `split` of the pair's blocks owns the buckets [split * per, (split + 1) * per); wave
            // w takes RPWV consecutive buckets at a time.  The arithmetic per bucket is that of score_kernel (same
            // lanes, same order), so skv_score returns the very floats that are ranked here.  Each score is stored
            // with the launch tag in one 64-bit word; the blocks that go on read the pair's words until all carry it.
            const int32_t S = sq.n_sent;
            // From kStepLineRows buckets a block on, shares are whole lines of the exchange (16 words), each written by one store: a line that others poll and that is
            // written in pieces, by several stores or several blocks, costs its readers a trip through memory for each.  Us per layer, shares as
            // they come, a store for every two words / this: one sequence of 49152 tokens 13.5 / 12.5, 131072 17.8 / 17.2, two of 32768 15.4 / 14.6, four of
            // 16384 17.7 / 17.1; 32768 tokens (41 buckets a block, 28 of 32 blocks would score) 11.9 / 12.0, 8192 (11) 10.4 / 10.5.
            int32_t per = MODE == kStep ? (S + (1 << a.lg_parts) - 1) >> a.lg_parts : ceil_div(S, a.parts, a.per_part);
            const bool lines = per > kStepLineRows;
            if (lines) per = (per + 15) & ~15;
            const int32_t lo = split * per, hi = min(lo + per, S);
            const char* qg = a.q_score + ((qhead0 * kHeadDim) * EB);
            const int64_t row0 = (int64_t)h * a.v.S_total + sq.sent_base;
            unsigned long long* sc_out = a.step_score + (int64_t)bh * a.score_stride;
            // few buckets per block: 4 per wave visit (8 from an E4M3 table; two loads in flight per lane, all 16 waves busy from 64 buckets on);
            // more: 16 per visit (eight loads in flight per lane), a line of the exchange
            auto score_rows = [&](auto rows, auto score) {
                constexpr int R = decltype(rows)::value;
                for (int32_t rw = lo + w * R; rw < hi; rw += kBlockWaves * R) score(rows, rw);
            };
            auto score_table = [&](auto few, auto score) {
                if (lines) score_rows(std::integral_constant<int, 16>{}, score);
                else score_rows(few, score);
            };
            if (a.sv_bytes == kTableF32)
                score_table(std::integral_constant<int, 4>{}, [&](auto rows, int32_t rw) {
                    score_wave_f32<EB, G, decltype(rows)::value, true>(qg, reinterpret_cast<const float*>(a.semvec) + row0 * kHeadDim, hi, rw, sc_out, state);
                });
            else if (a.sv_bytes == kTableBf16)
                score_table(std::integral_constant<int, 4>{}, [&](auto rows, int32_t rw) {
                    score_wave_bf16<EB, G, decltype(rows)::value, true>(qg, a.semvec + row0 * kHeadDim * 2, hi, rw, sc_out, state);
                });
            else
                score_table(std::integral_constant<int, 8>{}, [&](auto rows, int32_t rw) {
                    score_wave_e4m3<EB, G, decltype(rows)::value, true>(qg, a.semvec + row0 * kHeadDim, hi, rw, sc_out, state);
                });
            SKV_T(12);
            tag = state.tag();
            // Blocks that neither attend (no position of theirs can hold a token: n <= budget) nor merge are done.
            if (split >= merging_blocks(G, a.lg_merge) && j0 >= budget) return;
            load_attend_args(a);
        } else {
            if (split > 0 && j0 >= budget) return;                // n <= budget: nothing for this split
        }
        if (tid < CHUNK) sm_row[tid] = -1;
        if (kStepping && tid == 0) sm_last = 0;
        leave_queries();
        int32_t nsel, ntok;
        // Each selected bucket that reaches into this block's positions marks, in every 64-position piece it touches,
        // where it starts there and which pool row that is; the waves then fill the positions in between.
        auto mark = [&](int32_t, int32_t o, int32_t ln, int32_t, int32_t tok_pos) {
#pragma unroll
            for (int pc = 0; pc < CHUNK / kWave; ++pc) {
                const int32_t lo = max(tok_pos, j0 + pc * kWave);
                if (lo < min(tok_pos + ln, j0 + (pc + 1) * kWave)) sm_row[lo - j0] = o + (lo - tok_pos);
            }
        };
        const float* sc = a.score + (int64_t)h * a.v.S_total + sq.sent_base;
        const int32_t* len = a.sent_len + sq.sent_base;
        const int32_t* off = a.sent_off + sq.sent_base + (a.v.cu_sent ? b : 0);
        if constexpr (kStepping) {                            // the scores are being written by the pair's blocks
            const float* tsc = reinterpret_cast<const float*>(a.step_score + (int64_t)bh * a.score_stride);
            uint32_t* sm_keys = reinterpret_cast<uint32_t*>(sm + kSelBytes);
            // at most one bucket a thread: no keys through LDS, a third of the walks.  With the search above, us per layer: 4096 tokens, fp32, 10.1 -> 9.45, 6 sequences
            // of 1900 to 21001 tokens 17.2 -> 16.3
            if (sq.n_sent <= kBlockThreads)
                select_block<1, false, true>(tsc, len, off, sq.n_sent, budget, sel_sh, mark, &nsel, &ntok, tag, a.wait_limit, &step_ok);
            else if (sq.n_sent <= 2 * kBlockThreads)
                select_block<2, false, true>(tsc, len, off, sq.n_sent, budget, sel_sh, mark, &nsel, &ntok, tag, a.wait_limit, &step_ok, sm_keys);
            else
                select_block<kSelKreg, false, true>(tsc, len, off, sq.n_sent, budget, sel_sh, mark, &nsel, &ntok, tag, a.wait_limit, &step_ok, sm_keys);
        } else if (sq.n_sent <= 2 * kBlockThreads) {
            select_block<2, false, false>(sc, len, off, sq.n_sent, budget, sel_sh, mark, &nsel, &ntok);
        } else {
            select_block<kSelKreg, false, false>(sc, len, off, sq.n_sent, budget, sel_sh, mark, &nsel, &ntok);
        }
        n = ntok;
        if (split == 0 && tid == 0 && a.n_tok_out) a.n_tok_out[bh] = n;
        __syncthreads();                                          // bucket starts are marked; the selection's LDS is free
    } else {
        n = min(ld_const(a.n_tok, bh), kRowsDirect ? a.row_stride : a.idx_stride);
    }
    // kStep: every block of the pair that ran the selection (and so used the epoch it read at its start) tells block 0 so
    // in the (reference, tag) word of its partial: the attending blocks with their partial, the others as soon as they
    // know that they hold no retrieved tokens.  Block 0 advances the epoch only after it has seen all of them, so that no
    // block of this launch can read the advanced epoch.
    auto presence = [&]() {
        if constexpr (kStepping) {
            if (tid == 0)                                         // a block that gave up publishes nothing valid
                st_tagged(a.step_part + (int64_t)(split * n_pairs + bh) * step_part_words(G) + G * kHeadDim, -INFINITY, step_ok ? tag : 0u);
        }
    };
    // block 0: the words of blocks first .. (blocks of the pair that run the selection) - 1 carry the tag (bounded wait);
    // every thread of the block calls this
    auto others_were_here = [&](int first) -> bool {
        if constexpr (kStepping) {
            const int n_cand = min(MODE == kStep ? 1 << a.lg_parts : a.parts, max(merging_blocks(G, a.lg_merge), blocks_of(max(min(sq.budget, a.budget_cap), 0))));
            if (n_cand <= first) return true;                     // block-uniform: the usual case, the budget is filled
            // the flag lives in the first word of the merge's scratch (thread 0, the only reader of that
            // word in the merge, is past its reads when it clears it)
            volatile uint32_t* missing = reinterpret_cast<uint32_t*>(sm_merge);
            if (tid == 0) *missing = 0u;
            __syncthreads();
            if (tid >= first && tid < n_cand) {
                const unsigned long long* src = a.step_part + (int64_t)(tid * n_pairs + bh) * step_part_words(G) + G * kHeadDim;
                bool there = false;
                for (int32_t round = 0; !there && round < a.wait_limit; ++round) there = tag_of(ld_tagged(src)) == tag;
                if (!there) *missing = 1u;
            }
            __syncthreads();
            return *missing == 0u;
        }
        return true;
    };
    if (n <= 0) {
        if (split == 0) {
            step_ok = others_were_here(1) && step_ok;
            for (int i = tid; i < kOut; i += kBlockThreads)
                a.out[MODE == kDirectDims ? (qhead0 + i / kDims) * kHeadDim + dim0 + i % kDims : qhead0 * kHeadDim + i] = step_ok ? 0.f : __builtin_nanf("");
            if (a.lse && tid < G && dim0 == 0) a.lse[qhead0 + tid] = -INFINITY;
            if constexpr (kStepping) {
                if (tid == 0) {
                    st_agent(a.step_epoch + bh * kStepEpochStride, tag >> kStepPairBits);     // this launch of the pair is over
                    if (!step_ok) { st_agent(a.err_dev, 1u); if (a.err_host) st_agent(a.err_host, 1u); }
                }
            }
        } else {
            presence();
        }
        return;
    }
    const int nsplit = MODE == kDirectDims ? 1 : blocks_of(n);
    // kStep: the first merging_blocks() blocks merge, whether or not they hold retrieved tokens themselves
    const bool has_work = split < nsplit;
    if (!has_work) {
        presence();
        if (!(kStepping && split < merging_blocks(G, a.lg_merge))) return;
    }
    unsigned long long* my_part = nullptr;
    uint32_t part_tag = 0;
    if constexpr (kStepping) {
        my_part = a.step_part + (int64_t)(split * n_pairs + bh) * step_part_words(G);
        part_tag = step_ok ? tag : 0u;                            // a block that gave up publishes nothing valid
    }
    if (has_work) {
        const int32_t cnt = min(chunk, n - j0);
        SKV_T(4);

        // ---- 1. issue every load of the chunk ------------------------------------------------------------
        const char* Kh;
        const char* Vh;
        if (kRowsDirect) {
            Kh = a.Kb + ((int64_t)bh * a.row_stride + j0) * kRowBytes;
            Vh = a.Vb + ((int64_t)bh * a.row_stride + j0) * kRowBytes + dim0 * EB;
        } else {
            Kh = a.Kb + ((int64_t)h * a.v.T_total + sq.tok_base) * kRowBytes;
            Vh = a.Vb + ((int64_t)h * a.v.T_total + sq.tok_base) * kRowBytes;
        }
        const float scale = kLog2e * rsqrtf((float)kHeadDim);
        // Shares of 80 to 112 and 144 to 240 tokens leave waves without a token (wave-uniform): these do nothing but say so.  Us per layer, with their loads and
        // matrix instructions on zeros / without: 3 sequences, budget 800 (80 tokens) 12.24 / 12.08, 1440 (144) 14.87 / 14.44, 5 sequences, 860 15.3 / 14.8; where
        // every wave has tokens the question costs 0.3 % (5 sequences, 1500: 17.35 / 17.41).
        const bool none = MODE == kStepRagged && kPasses == 1 && CHUNK > kAttChunk && 16 * __builtin_amdgcn_readfirstlane(w) >= __builtin_amdgcn_readfirstlane(cnt);
        if (w < kTiles && none) {
            f32x4_t o[kDims / 16];
#pragma unroll
            for (int dt = 0; dt < kDims / 16; ++dt) o[dt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            if (qd == 0) sm_waves.leave(t16, w, -INFINITY, 0.f, 0.f);
            leave_sums<G>(sm + w * kTileBytes, o);
        } else if (w < kTiles) {
            char* sm_v = sm + w * kTileBytes;                         // this wave's value tile
            if constexpr (kOwnQueries && EB == 4) own_queries();
            uint4 kA[kPasses][X::kPieces], vR[kPasses][X::kLoads];
            unsigned long long vm[kPasses];                           // bit t (t < 16): token t of the tile is real
#pragma unroll
            for (int ps = 0; ps < kPasses; ++ps) {
                // Pool row of the tile's token t16 (K) and of the tokens whose value row this lane loads; rows past the chunk's end (and
                // positions outside the sequence) are clamped to a valid row, loaded anyway and masked afterwards.
                const int tile = (MODE == kDirectDims && kFirst ? (w + part * (kTiles * kDims / kHeadDim)) % kTiles : w) + kTiles * ps, jj = 16 * tile + t16;
                if (ps > 0 && 16 * tile >= cnt) {                     // (wave-uniform) no second tile
                    vm[ps] = 0;
#pragma unroll
                    for (int s2 = 0; s2 < X::kPieces; ++s2) kA[ps][s2] = make_uint4(0, 0, 0, 0);
#pragma unroll
                    for (int i = 0; i < X::kLoads; ++i) vR[ps][i] = make_uint4(0, 0, 0, 0);
                    continue;
                }
                bool liveK = jj < cnt;
                int32_t rowK, rowV[X::kLoads];
                if constexpr (kRowsDirect) {
                    rowK = min(jj, cnt - 1);
#pragma unroll
                    for (int i = 0; i < X::kLoads; ++i) rowV[i] = min(16 * tile + X::RPL * i + lane / X::LPR, cnt - 1);
                } else {
                    // pool row of token t of the tile (t <= the chunk's last), -1: none
                    // (kSel: found in the piece's mask of starts and read there.  By a running maximum over the piece, an exchange for the start and one for the token, four
                    // trips one after the other: 32768 tokens 11.04 -> 10.91 us per layer, 131072 16.2 -> 16.1.)
                    [[maybe_unused]] const int32_t* piece = sm_row + (tile >> 2) * kWave;      // kSel: the tile's 64-position piece, its positions from `base` on
                    [[maybe_unused]] const int base = 16 * (tile & 3);
                    unsigned long long starts = 0;
                    if constexpr (kSel) starts = __ballot(piece[lane] >= 0);
                    auto row_of = [&](int t) -> int32_t {
                        if constexpr (kSel) {                         // the last bucket start at or before the position, and the way from there
                            const int p = base + t;
                            const unsigned long long upto = starts & (~0ull >> (63 - p));
                            const int hp = 63 - __builtin_clzll(upto | 1ull);
                            const int32_t start = piece[hp];
                            return start >= 0 ? start + (p - hp) : -1;     // (none before it: hp = 0, no start there)
                        } else {
                            return a.tok_idx[(int64_t)bh * a.idx_stride + j0 + 16 * tile + t];
                        }
                    };
                    if constexpr (kSel) {
                        if ((tile & 3) == 0 && a.tok_idx_out && (tile >> 2) * kWave + lane < cnt)
                            a.tok_idx_out[(int64_t)bh * a.idx_stride + j0 + (tile >> 2) * kWave + lane] = row_of(lane);
                    }
                    const int last = max(min(cnt - 1 - 16 * tile, 15), kSel ? -base : -16 * tile);
                    const int32_t xk = row_of(min(t16, last));
                    liveK = liveK && xk >= 0 && xk < sq.n_tok_ctx;        // the token lies in the sequence
                    rowK = min(max(xk, 0), max(sq.n_tok_ctx - 1, 0));
#pragma unroll
                    for (int i = 0; i < X::kLoads; ++i) rowV[i] = __shfl(rowK, X::RPL * i + lane / X::LPR);
                }
#pragma unroll
                for (int s2 = 0; s2 < X::kPieces; ++s2) kA[ps][s2] = ld_row<!kRowsDirect>(Kh + (int64_t)rowK * kRowBytes + 64 * s2 + 16 * qd);
#pragma unroll
                for (int i = 0; i < X::kLoads; ++i) vR[ps][i] = ld_row<!kRowsDirect>(Vh + (int64_t)rowV[i] * kRowBytes + 16 * (lane % X::LPR));
                vm[ps] = __ballot(liveK);
            }
            if constexpr (!kSel && !kOwnQueries) {                    // behind the rows' requests
                leave_queries();
                __syncthreads();
            }
#pragma unroll
            for (int s2 = 0; s2 < X::kPieces; ++s2) {
                if constexpr (!kOwnQueries) qB[s2] = *reinterpret_cast<const uint4*>(sm_q + min(t16, G - 1) * kQueryPitch + 64 * s2 + 16 * qd);
                if (t16 >= G) qB[s2] = make_uint4(0, 0, 0, 0);
            }
            SKV_T(5);
            float p[kPasses][4], mw = -INFINITY;
#pragma unroll
            for (int ps = 0; ps < kPasses; ++ps) {
                const f32x4_t acc = X::logits(kA[ps], [&](int s2) { return qB[s2]; });
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    p[ps][j] = ((vm[ps] >> (4 * qd + j)) & 1ull) ? acc[j] * scale : -INFINITY;
                    mw = fmaxf(mw, p[ps][j]);
                }
            }
            mw = max_quads(mw);
            const float ref = mw > -INFINITY ? mw : 0.f;              // (no live token, or logits of NaN only: those weights are NaN)
            f32x4_t o[kDims / 16];
#pragma unroll
            for (int dt = 0; dt < kDims / 16; ++dt) o[dt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            float lw = 0.f;
#pragma unroll
            for (int ps = 0; ps < kPasses; ++ps) {
                // the tile's value rows go to LDS (rows of masked tokens as zeros)
#pragma unroll
                for (int i = 0; i < X::kLoads; ++i) {
                    const int row = X::RPL * i + lane / X::LPR;
                    *reinterpret_cast<uint4*>(sm_v + X::place(row, lane % X::LPR)) = ((vm[ps] >> row) & 1ull) ? vR[ps][i] : make_uint4(0, 0, 0, 0);
                }
                SKV_T(6);
                exp2_weights(p[ps], ref);                             // masked: 2^-inf = 0
#pragma unroll
                for (int j = 0; j < 4; ++j) lw += X::weight(p[ps][j]);
                wave_lds_sync();                                      // the tile is the wave's own: order only
                X::output(p[ps], sm_v, lane, o);
                wave_lds_sync();
            }
            lw = sum_quads(lw);
            if (qd == 0) sm_waves.leave(t16, w, mw, ref, lw);
            leave_sums<G>(sm_v, o);
        } else if constexpr (!kSel && !kOwnQueries) {
            __syncthreads();                                          // the queries'
        }
        __syncthreads();
        block_sums<G, kTiles, kDims>(sm, kTileBytes, sm_waves, [&](int g, int d, float sum, float mb, float lb) {
            if constexpr (kStepping) {
                st_tagged(my_part + g * kHeadDim + d, sum, part_tag);
            } else if (nsplit == 1) {                                 // the only block: its sums are the result
                const bool empty = lb == 0.f;                       // every retrieved position was out of range
                a.out[(qhead0 + g) * kHeadDim + dim0 + d] = empty ? 0.f : sum / lb;
                if (a.lse && dim0 + d == 0) a.lse[qhead0 + g] = empty ? -INFINITY : (mb + log2f(lb)) * kLn2;
            } else {
                st_agent(a.part + (((qhead0 + g) * a.max_splits) + slot) * kHeadDim + d, sum);
                if (d < 2) st_agent(a.ml + (((qhead0 + g) * a.max_splits) + slot) * 2 + d, d == 0 ? mb : lb);
            }
        }, [&](int i, float v) {
            if constexpr (kStepping) st_tagged(my_part + G * kHeadDim + i, v, part_tag);      // one store: see step_part_words
        });
        SKV_T(7);
    }

    if constexpr (kStepping) {
        // ---- 5'. merge without an arrival counter ---------------------------------------------------------------
        // Block m of the pair merges 128 >> lg_merge dims of query head m >> lg_merge, or two heads.  Thread (grp, col) -- consecutive
        // lanes on consecutive words of a partial row -- reads dim `col` of the partials of the splits grp, grp + groups, ...
        // (value and tag in one word) and their (reference, normaliser) words, again and again until all carry the launch tag
        // (bounded; no barrier, no sleep: a wave leaves as soon as its own words are there), folds them into a running
        // (reference, normaliser, output), and the groups meet once in LDS.  No block waits for a store
        // acknowledgement and nothing is counted.
        if (split >= merging_blocks(G, a.lg_merge)) return;
        const int lg_dims = 7 - a.lg_merge, groups = kBlockThreads >> lg_dims;                            // 4 groups of 256 dims .. 32 of 32
        // column `col` of the block's 1 << lg_dims: dim (at % 128) of query head (at / 128)
        auto at_of = [&](int col) { return (split << lg_dims) + col; };
        const int at = at_of(tid & ((1 << lg_dims) - 1)), grp = tid >> lg_dims, g = at / kHeadDim;
        float M = -INFINITY, L = 0.f, o = 0.f;
        bool ok = step_ok;
        for (int base = 0; base < nsplit && ok; base += 2 * groups) {
            unsigned long long pv[2] = {0, 0}, mv[2] = {0, 0}, lv[2] = {0, 0};
            bool mine = false;
            for (int32_t round = 0; !mine && round < a.wait_limit; ++round) {
                mine = true;
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int sp = base + grp + u * groups;
                    if (sp < nsplit) {
                        const unsigned long long* src = a.step_part + (int64_t)(sp * n_pairs + bh) * step_part_words(G);
                        pv[u] = ld_tagged(src + at);
                        mv[u] = ld_tagged(src + G * kHeadDim + 2 * g);
                        lv[u] = ld_tagged(src + G * kHeadDim + 2 * g + 1);
                        mine = mine && tag_of(pv[u]) == tag && tag_of(mv[u]) == tag && tag_of(lv[u]) == tag;
                    }
                }
            }
            ok = mine;
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                if (ok && base + grp + u * groups < nsplit) {
                    const float ms = val_of(mv[u]), ls = val_of(lv[u]), ps = val_of(pv[u]);
                    const float nm = fmaxf(M, ms), ca = pow2_whole(M - nm), cb = pow2_whole(ms - nm);     // M == -inf gives ca == 0
                    L = L * ca + ls * cb;
                    o = o * ca + ps * cb;
                    M = nm;
                }
            }
        }
        SKV_T(10);
        // The groups meet in LDS, where every column's are taken by lanes of one wave, two groups each, that fold them with exchanges in registers; 32 columns: the
        // two groups of a wave meet before that.  (LDS rows have a pitch that lets these lanes read from different banks.)  One to four lanes a column, eight groups each,
        // and exchanges through LDS / this, us per layer: 8192 tokens, budget 1000, 10.82 / 10.48, 32768 (2048) 11.9 / 11.75, 131072 16.9 / 16.5, fp32 32768 14.3 / 14.0.
        if (!ok) { M = __builtin_nanf(""); sm_last = 1; }                     // a thread whose wait ran out
        auto finish = [&](auto lg) {
            constexpr int kCols = 1 << decltype(lg)::value, kHalves = kCols < kWave ? 2 : 1, kRows = kBlockThreads / kCols / kHalves;
            constexpr int kLanes = kRows / 2, kPitch = kCols + 32 / kLanes, kPlane = kRows * kPitch, kPer = kWave / kLanes;      // lanes of a column; columns of a wave
            static_assert(3 * kPlane <= kMergeWords && kLanes * kCols <= kBlockThreads, "");
            if constexpr (kHalves == 2) {
                const float nm = max_halves(M), c = pow2_whole(M - nm);
                o = sum_halves(o * c);
                L = sum_halves(L * c);
                M = nm;
            }
            if (kHalves == 1 || lane < kCols) {
                float* dst = sm_merge + (kHalves == 2 ? w : grp) * kPitch + (tid & (kCols - 1));
                dst[0] = o; dst[kPlane] = M; dst[2 * kPlane] = L;
            }
            __syncthreads();
            SKV_T(11);
            if (w >= kCols / kPer) return;
            const int col = w * kPer + lane % kPer, part = lane / kPer;
            const float* src = sm_merge + 2 * part * kPitch + col;
            const float o0 = src[0], o1 = src[kPitch], m0 = src[kPlane], m1 = src[kPlane + kPitch], l0 = src[2 * kPlane], l1 = src[2 * kPlane + kPitch];
            float Mx = fmaxf(m0, m1);
            if constexpr (kLanes == 8) Mx = fmaxf(Mx, other_eight(Mx));
            if constexpr (kLanes >= 4) Mx = max_quads(Mx);
            else Mx = max_halves(Mx);
            const float c0 = pow2_whole(m0 - Mx), c1 = pow2_whole(m1 - Mx);
            float Ls = c0 * l0 + c1 * l1, os = c0 * o0 + c1 * o1;
            if constexpr (kLanes == 8) { Ls += other_eight(Ls); os += other_eight(os); }
            if constexpr (kLanes >= 4) { Ls = sum_quads(Ls); os = sum_quads(os); }
            else { Ls = sum_halves(Ls); os = sum_halves(os); }
            const bool bad = sm_last != 0;                                    // a wait of this launch ran out
            if (part == 0) {
                const int to = at_of(col);
                const bool empty = Ls == 0.f;                               // every retrieved position was out of range
                a.out[qhead0 * kHeadDim + to] = bad ? __builtin_nanf("") : empty ? 0.f : os / Ls;
                if (a.lse && to % kHeadDim == 0) a.lse[qhead0 + to / kHeadDim] = empty ? -INFINITY : (Mx + log2f(Ls)) * kLn2;
            }
            if (bad && tid == 0) { st_agent(a.err_dev, 1u); if (a.err_host) st_agent(a.err_host, 1u); }
        };
        if (lg_dims == 5) finish(std::integral_constant<int, 5>{});
        else if (lg_dims == 6) finish(std::integral_constant<int, 6>{});
        else if (lg_dims == 7) finish(std::integral_constant<int, 7>{});
        else finish(std::integral_constant<int, 8>{});
        // Block 0 ends the pair's launch by advancing its epoch: its threads have seen the partial of every attending
        // block (the barrier above) and now make sure of the word of every other block that ran the selection; all of
        // them, and through the scores they waited for every scoring block, have read the epoch by then.
        if (split == 0) {
            const bool all_here = others_were_here(nsplit);
            if (tid == 0) {
                st_agent(a.step_epoch + bh * kStepEpochStride, tag >> kStepPairBits);
                if (!all_here) { st_agent(a.err_dev, 1u); if (a.err_host) st_agent(a.err_host, 1u); }
            }
        }
        SKV_T(9);
        return;
    }

    if (nsplit == 1) return;
    // ---- 5. last arrival combines ------------------------------------------------------------------
    // Every wave waits for its own write-through partial stores, then the barrier: only after both does thread 0
    // issue the device-scope increment, so whoever reads nsplit - 1 knows every partial is there.
    block_sync_after_stores();
    if (tid == 0) {
        const unsigned int old = __hip_atomic_fetch_add(&a.counter[bh], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        sm_last = (old == (unsigned int)(nsplit - 1));
    }
    __syncthreads();
    SKV_T(8);
    if (!sm_last) return;
    // A thread owns one pair of output floats and every kGroups-th split: one batch of independent 8-byte
    // loads, merged online (running max M, normaliser L, outputs) in registers; groups merge through LDS.
    float4* scratch = reinterpret_cast<float4*>(sm);                        // (o0, o1, M, L) per thread
    {
        const int col = tid % kCol2, grp = tid / kCol2;
        const int g = col / (kHeadDim / 2);
        const float* mlg = a.ml + ((qhead0 + g) * a.max_splits) * 2;
        const float* pg = a.part + ((qhead0 + g) * a.max_splits) * kHeadDim + (col % (kHeadDim / 2)) * 2;
        float M = -INFINITY, L = 0.f, o0 = 0.f, o1 = 0.f;
        constexpr int kU = CHUNK >= 2 * kWave ? 4 : 8;       // loads in flight per thread: sized for a 2048-token budget
        for (int s0 = grp; s0 < nsplit; s0 += kGroups * kU) {
            unsigned long long pv[kU], mv[kU];
#pragma unroll
            for (int u = 0; u < kU; ++u) {                   // clamped, unconditional loads
                const int sidx = min(s0 + u * kGroups, nsplit - 1) * (CHUNK / kWave);
                pv[u] = ld_agent64(pg + (int64_t)sidx * kHeadDim);
                mv[u] = ld_agent64(mlg + 2 * sidx);
            }
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const float ms = (s0 + u * kGroups < nsplit) ? lo_f(mv[u]) : -INFINITY;
                const float nm = fmaxf(M, ms), ca = pow2_whole(M - nm), cb = pow2_whole(ms - nm);      // M == -inf gives ca == 0
                L = L * ca + hi_f(mv[u]) * cb;
                o0 = o0 * ca + lo_f(pv[u]) * cb;
                o1 = o1 * ca + hi_f(pv[u]) * cb;
                M = nm;
            }
        }
        SKV_T(10);
        __syncthreads();                                     // the partial sums are no longer read by anyone
        scratch[grp * kCol2 + col] = make_float4(o0, o1, M, L);
    }
    __syncthreads();
    SKV_T(11);
    if (tid < kCol2) {
        float M = -INFINITY;
#pragma unroll
        for (int grp = 0; grp < kGroups; ++grp) M = fmaxf(M, scratch[grp * kCol2 + tid].z);
        float L = 0.f, o0 = 0.f, o1 = 0.f;
#pragma unroll
        for (int grp = 0; grp < kGroups; ++grp) {
            const float4 t = scratch[grp * kCol2 + tid];
            const float c = pow2_whole(t.z - M);
            L += c * t.w; o0 += c * t.x; o1 += c * t.y;
        }
        const bool empty = L == 0.f;                       // every retrieved position was out of range
        const float inv = empty ? 0.f : 1.f / L;
        reinterpret_cast<float2*>(a.out + qhead0 * kHeadDim)[tid] = make_float2(o0 * inv, o1 * inv);
        if (a.lse && (tid % (kHeadDim / 2)) == 0)
            a.lse[qhead0 + tid / (kHeadDim / 2)] = empty ? -INFINITY : (M + log2f(L)) * kLn2;
    }
    if (tid == 0) __hip_atomic_store(&a.counter[bh], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // for the next call
    SKV_T(9);
}

// ------------------------------------------------------------------------------------------------
// Streaming form of the attention for batches.  Measured on the 1024-thread kernel above with 16 sequences
// x 8 heads in bf16: all blocks start together, load together (memory saturated for 5 us) and then compute together
// (memory idle for 7 us), twice.  Here a wave owns 64 consecutive retrieved tokens and walks them in four 16-token
// MFMA tiles -- the next tile's K and V rows are requested as soon as the current ones have been consumed (K by the
// logit MFMAs, V by its copy to LDS) -- carrying a running (max, normaliser, output) per head as in flash decoding;
// all blocks of the launch are resident at once (16 waves per CU, each with 8 KB in flight).
// Tile arithmetic is that of the kernel above (Tile).
// A block is 16 waves and CHUNK = 1024 (or 512, or 2048) retrieved tokens of one (sequence, KV head).  It first runs the
// selection itself from the scores (as the single-sequence kernel does, redundantly with the head's other blocks) and
// keeps the pool rows of its positions in LDS: no selection launch, no tok_idx round trip, two partials per 2048-token
// budget with 1024-token blocks, none when one block covers the budget.
// Measured against select_kernel + a 4-wave form of this kernel that read tok_idx (16 sequences x 8 heads, budget
// 2048): 8.7 + 37.1 us -> 39 us per layer; equal or better from 8 to 48 sequences.
// ------------------------------------------------------------------------------------------------
constexpr int kStreamTiles = 4;                                   // 16-token tiles per wave
constexpr int kStreamWaves = kBlockWaves;                         // the block-level selection needs kBlockThreads threads
constexpr int kStreamChunk = kStreamWaves * kStreamTiles * 16;    // 1024 tokens per block, one position per thread
static_assert(kStreamChunk == kBlockThreads, "the usual block: one retrieved position per thread");

constexpr int kStreamMaxChunk = 2 * kStreamChunk;                 // the largest block: two positions per thread

template <int EB, int CHUNK> struct StreamShared {
    __attribute__((aligned(16))) char v[kStreamWaves][16 * Tile<EB>::kPitch];    // the selection's, then value tiles, then the waves' partial sums
    __attribute__((aligned(16))) char q[16][kHeadDim * EB];                      // the group's queries, rows >= G zero
    WaveSums<kStreamWaves> waves;
    int32_t row[max_of(CHUNK, kBlockThreads)];                                   // pool row of every position of the block (-1: none)
    int next_tile;
    int last;
};

// queries of the group -> LDS (16 rows, 16 bytes per thread); a barrier must follow before they are read
template <int EB, int G, int CHUNK>
__device__ __forceinline__ void stream_load_queries(const AttArgs& a, StreamShared<EB, CHUNK>& ss, int64_t qhead0) {
    constexpr int LPR = Tile<EB>::LPR;
    const int tid = threadIdx.x;
    if (tid < 16 * LPR) {
        const int row = tid / LPR, piece = tid % LPR;
        uint4 t = make_uint4(0, 0, 0, 0);
        if (row < G) t = *reinterpret_cast<const uint4*>(a.q + ((qhead0 + row) * kHeadDim) * EB + 16 * piece);
        *reinterpret_cast<uint4*>(&ss.q[row][16 * piece]) = t;
    }
}

// Attention of one block of CHUNK (512, 1024 or 2048) positions once the selection is known: n = retrieved tokens of the
// (sequence, head); ss.row holds the pool row of position split * CHUNK + i at i (-1: no such token) for i < CHUNK.
// The queries are on their way to ss.q.  Every thread of the block calls this.
template <int EB, int G, int CHUNK>
__device__ __forceinline__ void stream_attend(const AttArgs& a, StreamShared<EB, CHUNK>& ss, int bh, int b, int h, int split, const Seq& sq,
                                              int32_t n) {

    constexpr int NW = kStreamWaves;
    constexpr int kThreads = kBlockThreads;
    using X = Tile<EB>;
    constexpr int kRowBytes = kHeadDim * EB;
    constexpr float kLog2e = 1.4426950408889634f, kLn2 = 0.6931471805599453f;
    constexpr int kOut = G * kHeadDim, kCol2 = kOut / 2;
    constexpr int kColsPerThread = (kCol2 + kThreads - 1) / kThreads;
    static_assert(G * kHeadDim * 4 <= 16 * X::kPitch, "a wave's partial sums fit in its value tile");
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int t16 = lane & 15, qd = lane >> 4;
    const int64_t qhead0 = (int64_t)b * (a.Hkv * G) + (int64_t)h * G;
    const int32_t j0 = split * CHUNK;
    const int slot = split * (CHUNK / kWave);
    if (n <= 0) {
        if (split == 0) {
            for (int i = tid; i < kOut; i += kThreads) a.out[qhead0 * kHeadDim + i] = 0.f;
            if (a.lse && tid < G) a.lse[qhead0 + tid] = -INFINITY;
        }
        return;
    }
    const int nsplit = (n + CHUNK - 1) / CHUNK;
    if (split >= nsplit) return;
    const int32_t cnt = min(CHUNK, n - j0);

    // The block's positions are walked in 16-token tiles.  bf16: handed out dynamically, a wave starts with tile w and takes the
    // next free one from an LDS counter whenever it finishes one, so the waves that memory serves first do more tiles
    // and all 16 keep loads in flight until the block's last tile (with four fixed tiles per wave the slowest wave ran
    // about 5 us behind the first).  fp32: every 16th tile, so that a result is the same in every call.  Rows of unreal positions are
    // stored as -1.
    if (tid == 0) ss.next_tile = NW;
    const int ntiles = (cnt + 15) / 16;
    const char* Kh = a.Kb + ((int64_t)h * a.v.T_total + sq.tok_base) * kRowBytes;
    const char* Vh = a.Vb + ((int64_t)h * a.v.T_total + sq.tok_base) * kRowBytes;
    const float scale = kLog2e * rsqrtf((float)kHeadDim);
    __syncthreads();                                              // rows and the tile counter are in LDS
    SKV_T(4);

    uint4 kA[X::kPieces], vR[EB == 2 ? X::kLoads : 1];
    char* vt_b = ss.v[w];
    // rows of a tile: lanes with the same t16 hold the row of the tile's token t16 (-1: not real)
    auto rows_of = [&](int tile) { return ss.row[16 * tile + t16]; };
    // Requests on 32-bit byte offsets from the (head, sequence) base: the host only uses this kernel for pools of less than 4 GB a head.
    // Value rows are requested whole and go non-temporal; a key instruction takes 64 bytes of each of
    // 16 rows, so two of them share every 128-byte line, which must stay until the second (non-temporal key loads:
    // 6 sequences in 512-token blocks 720 -> 790 us for 32 layers).
    auto issue_keys = [&](int32_t rowt, int ln) {
        const uint32_t offK = (uint32_t)max(rowt, 0) * kRowBytes + 16u * (ln >> 4);
#pragma unroll
        for (int s2 = 0; s2 < X::kPieces; ++s2) kA[s2] = *reinterpret_cast<const uint4*>(Kh + (offK + 64u * s2));
    };
    // bf16: to registers, as early as the keys; fp32: straight to the value tile (registers would spill), once that is free
    auto issue_values = [&](int32_t rowt, int ln) {
        const int32_t rc = max(rowt, 0);
#pragma unroll
        for (int ii = 0; ii < X::kLoads; ++ii) {
            const uint32_t offV = (uint32_t)__shfl(rc, X::RPL * ii + ln / X::LPR) * kRowBytes;
            if constexpr (EB == 2) vR[ii] = ld_stream(Vh + (offV + 16u * (ln % X::LPR)));
            else load_lds_stream(Vh, offV + 16u * ((ln % X::LPR) ^ (4 * ((X::RPL * ii) >> 2))), vt_b + 1024 * ii);
        }
    };
    int tile = w;                                                 // wave-uniform
    int32_t row_cur = tile < ntiles ? rows_of(tile) : -1;
    if (tile < ntiles) { issue_keys(row_cur, lane); issue_values(row_cur, lane); }
    SKV_T(5);

    float m_run = -INFINITY, l_run = 0.f;                         // per head t16; l_run covers this lane's tokens only
    f32x4_t o[kHeadDim / 16];
#pragma unroll
    for (int dt = 0; dt < kHeadDim / 16; ++dt) o[dt] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    while (tile < ntiles) {
        // fp32: addresses that depend on the lane are formed anew for every tile (kept across the loop they would be spilled)
        int ln = lane;
        if constexpr (EB == 4) asm volatile("" : "+v"(ln));
        // the wave's next tile, asked for early so that its rows are known when this tile's registers come free
        int nxt = tile + NW;
        if constexpr (EB == 2) {
            if (lane == 0) nxt = atomicAdd(&ss.next_tile, 1);
            nxt = __builtin_amdgcn_readfirstlane(nxt);
        }
        const unsigned int tm = (unsigned int)__ballot(row_cur >= 0) & 0xffffu;   // bit t: token t of the tile is real
        const f32x4_t acc = X::logits(kA, [&](int s2) { return *reinterpret_cast<const uint4*>(&ss.q[ln & 15][64 * s2 + 16 * (ln >> 4)]); });
        if constexpr (EB == 2) {
            // the tile's value rows go to the wave's LDS tile (rows of masked tokens as zeros) ...
#pragma unroll
            for (int ii = 0; ii < X::kLoads; ++ii) {
                const int row = X::RPL * ii + lane / X::LPR;
                *reinterpret_cast<uint4*>(vt_b + X::place(row, lane % X::LPR)) = ((tm >> row) & 1u) ? vR[ii] : make_uint4(0, 0, 0, 0);
            }
        }
        // ... which frees the row registers for the next tile: its loads fly during this tile's softmax and P.V
        row_cur = nxt < ntiles ? rows_of(nxt) : -1;
        if (nxt < ntiles) {
            issue_keys(row_cur, ln);
            if constexpr (EB == 2) issue_values(row_cur, ln);
        }
        tile = nxt;
        float p[4], mt = -INFINITY;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            p[j] = ((tm >> (4 * qd + j)) & 1u) ? acc[j] * scale : -INFINITY;
            mt = fmaxf(mt, p[j]);
        }
        const float m_new = fmaxf(m_run, max_quads(mt));
        const float alpha = m_new > -INFINITY ? exp2f(m_run - m_new) : 1.f;   // m_run == -inf gives 0
        const float ref = m_new > -INFINITY ? m_new : 0.f;        // (no live token yet, or logits of NaN only: those weights are NaN)
        float lw = 0.f;
        exp2_weights(p, ref);                                     // masked: 2^-inf = 0
#pragma unroll
        for (int j = 0; j < 4; ++j) lw += X::weight(p[j]);
        l_run = l_run * alpha + lw;
        m_run = m_new;
        // running outputs: row 4qd+j of o is head 4qd+j, whose factor sits in lane 4qd+j
        float ar[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) ar[j] = __shfl(alpha, 4 * qd + j);
#pragma unroll
        for (int dt = 0; dt < kHeadDim / 16; ++dt)
#pragma unroll
            for (int j = 0; j < 4; ++j) o[dt][j] *= ar[j];
        if constexpr (EB == 4) {
            // this tile's values have landed (the next tile's keys, requested after them, may be outstanding); rows of masked tokens as zeros
            if (nxt < ntiles) wait_loads<X::kPieces>();
            else wait_loads<0>();
            if (tm != 0xffffu) {
#pragma unroll 1
                for (int row = 0; row < 16; ++row)
                    if (!((tm >> row) & 1u) && ln < X::LPR) *reinterpret_cast<uint4*>(vt_b + X::place(row, ln)) = make_uint4(0, 0, 0, 0);
            }
        }
        wave_lds_sync();                                          // the tile is private to the wave: order only
        X::output(p, vt_b, ln, o);
        wave_lds_sync();                                          // reads of this tile precede the next tile's writes
        if constexpr (EB == 4) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            if (nxt < ntiles) issue_values(row_cur, ln);
        }
    }
    SKV_T(6);

    // ---- the block's waves combine -------------------------------------------------------------------------------
    l_run = sum_quads(l_run);
    if (qd == 0) ss.waves.leave(t16, w, m_run, m_run > -INFINITY ? m_run : 0.f, l_run);
    leave_sums<G>(vt_b, o);
    __syncthreads();
    block_sums<G, NW>(ss.v[0], sizeof(ss.v[0]), ss.waves, [&](int g, int d, float sum, float mb, float lb) {
        if (nsplit == 1) {                                        // the only block of this (sequence, head): no partials, no arrival, no merge
            const bool empty = lb == 0.f;                       // every retrieved position was out of range
            a.out[(qhead0 + g) * kHeadDim + d] = empty ? 0.f : sum / lb;
            if (a.lse && d == 0) a.lse[qhead0 + g] = empty ? -INFINITY : (mb + log2f(lb)) * kLn2;
        } else {
            st_agent(a.part + (((qhead0 + g) * a.max_splits) + slot) * kHeadDim + d, sum);
            if (d < 2) st_agent(a.ml + (((qhead0 + g) * a.max_splits) + slot) * 2 + d, d == 0 ? mb : lb);
        }
    }, [](int, float) {});
    if (nsplit == 1) return;
    SKV_T(7);

    // ---- last arrival combines (same protocol as attend_kernel) ------------------------------------------------
    block_sync_after_stores();
    if (tid == 0) {
        const unsigned int old = __hip_atomic_fetch_add(&a.counter[bh], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        ss.last = (old == (unsigned int)(nsplit - 1));
    }
    __syncthreads();
    SKV_T(8);
    if (!ss.last) return;
#pragma unroll
    for (int c = 0; c < kColsPerThread; ++c) {
        const int col = tid + c * kThreads;
        if (col >= kCol2) break;
        const int g = col / (kHeadDim / 2);
        const float* mlg = a.ml + ((qhead0 + g) * a.max_splits) * 2;
        const float* pg = a.part + ((qhead0 + g) * a.max_splits) * kHeadDim + (col % (kHeadDim / 2)) * 2;
        float M = -INFINITY, L = 0.f, o0 = 0.f, o1 = 0.f;
        constexpr int kU = 2;                                     // loads in flight per thread: sized for a 2048-token budget
        for (int s0 = 0; s0 < nsplit; s0 += kU) {
            unsigned long long pv[kU], mv[kU];
#pragma unroll
            for (int u = 0; u < kU; ++u) {                        // clamped, unconditional loads
                const int sidx = min(s0 + u, nsplit - 1) * (CHUNK / kWave);
                pv[u] = ld_agent64(pg + (int64_t)sidx * kHeadDim);
                mv[u] = ld_agent64(mlg + 2 * sidx);
            }
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const float ms = (s0 + u < nsplit) ? lo_f(mv[u]) : -INFINITY;
                const float nm = fmaxf(M, ms), ca = pow2_whole(M - nm), cb = pow2_whole(ms - nm);
                L = L * ca + hi_f(mv[u]) * cb;
                o0 = o0 * ca + lo_f(pv[u]) * cb;
                o1 = o1 * ca + hi_f(pv[u]) * cb;
                M = nm;
            }
        }
        const bool empty = L == 0.f;                            // every retrieved position was out of range
        const float inv = empty ? 0.f : 1.f / L;
        reinterpret_cast<float2*>(a.out + qhead0 * kHeadDim)[col] = make_float2(o0 * inv, o1 * inv);
        if (a.lse && (col % (kHeadDim / 2)) == 0) a.lse[qhead0 + g] = empty ? -INFINITY : (M + log2f(L)) * kLn2;
    }
    if (tid == 0) __hip_atomic_store(&a.counter[bh], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // for the next call
    SKV_T(9);
}

template <int EB, int G, int CHUNK>
__global__ __launch_bounds__(kBlockThreads) __attribute__((amdgpu_waves_per_eu(4, 4))) void select_attend_stream_kernel(AttArgs a) {
    static_assert(CHUNK % kWave == 0 && CHUNK <= kStreamMaxChunk, "the row table holds kStreamMaxChunk positions");
    __shared__ StreamShared<EB, CHUNK> ss;
    const int h = blockIdx.y, b = blockIdx.z, bh = b * a.Hkv + h, split = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63;
    demand_args<kFused>(a);
    const Seq sq = seq_of_step(a.v, b);
    const int32_t j0 = split * CHUNK;
    SKV_T(0);

    int32_t n;                    // retrieved tokens of this (sequence, head)
    {
        static_assert(sizeof(SelectShared) <= sizeof(ss.v), "the selection works in the value tiles' space");
        SelectShared& sel_sh = *reinterpret_cast<SelectShared*>(ss.v);
        const int32_t budget = min(sq.budget, a.budget_cap);
        if (split > 0 && j0 >= budget) return;                    // n <= budget: nothing for this split
        stream_load_queries<EB, G, CHUNK>(a, ss, (int64_t)b * (a.Hkv * G) + (int64_t)h * G);
        for (int p = tid; p < (CHUNK > kBlockThreads ? CHUNK : kBlockThreads); p += kBlockThreads)
            ss.row[p] = -1;                                       // bucket-start marks first, the rows of all positions later
        // A selected bucket that reaches into this block's positions marks, in every 64-position piece it touches,
        // where it starts there and which pool row that is; each wave then fills the positions of its own piece.
        auto mark = [&](int32_t, int32_t o, int32_t ln, int32_t, int32_t tok_pos) {
            const int32_t hi = min(tok_pos + ln, j0 + CHUNK);
            int32_t lo = max(tok_pos, j0);
            while (lo < hi) {
                ss.row[lo - j0] = o + (lo - tok_pos);
                lo = j0 + (((lo - j0) >> 6) + 1) * kWave;
            }
        };
        const float* sc = a.score + (int64_t)h * a.v.S_total + sq.sent_base;
        const int32_t* len = a.sent_len + sq.sent_base;
        const int32_t* off = a.sent_off + sq.sent_base + (a.v.cu_sent ? b : 0);
        int32_t nsel, ntok;
        if (sq.n_sent <= 2 * kBlockThreads) select_block<2, false, false>(sc, len, off, sq.n_sent, budget, sel_sh, mark, &nsel, &ntok);
        else select_block<kSelKreg, false, false>(sc, len, off, sq.n_sent, budget, sel_sh, mark, &nsel, &ntok);
        n = ntok;
        if (split == 0 && tid == 0 && a.n_tok_out) a.n_tok_out[bh] = n;
        __syncthreads();                                          // bucket starts are marked, queries are in LDS
        for (int pc = tid >> 6; pc < CHUNK / kWave; pc += kStreamWaves) {    // a wave fills 64-position pieces, in place
            const int32_t v = ss.row[pc * kWave + lane];
            // position of the last bucket start at or before this lane (-1: none): running maximum of lane + 1 over the starts
            const int32_t hp = (int32_t)wave_scan_max_u32(v >= 0 ? (uint32_t)lane + 1u : 0u) - 1;
            const int32_t base = __shfl(v, max(hp, 0));
            const int32_t xi = hp >= 0 ? base + (lane - hp) : -1;
            const int32_t pos = j0 + pc * kWave + lane;
            if (a.tok_idx_out && pos < n) a.tok_idx_out[(int64_t)bh * a.idx_stride + pos] = xi;
            ss.row[pc * kWave + lane] = (pos < n && xi >= 0 && xi < sq.n_tok_ctx) ? xi : -1;
        }
    }
    stream_attend<EB, G, CHUNK>(a, ss, bh, b, h, split, sq, n);
}

template <int EB, int CHUNK>
static hipError_t launch_select_attend_stream_g(Ctx* c, const AttArgs& a) {
    int n_splits = (c->budget_cap + CHUNK - 1) / CHUNK;
    if (n_splits < 1) n_splits = 1;       // block 0 still writes the empty-selection result
    const dim3 grid(n_splits, c->d.n_kv_heads, a.v.B), block(kBlockThreads);
    switch (c->G) {
        case 1: hipLaunchKernelGGL((select_attend_stream_kernel<EB, 1, CHUNK>), grid, block, 0, c->stream, a); break;
        case 2: hipLaunchKernelGGL((select_attend_stream_kernel<EB, 2, CHUNK>), grid, block, 0, c->stream, a); break;
        case 4: hipLaunchKernelGGL((select_attend_stream_kernel<EB, 4, CHUNK>), grid, block, 0, c->stream, a); break;
        case 8: hipLaunchKernelGGL((select_attend_stream_kernel<EB, 8, CHUNK>), grid, block, 0, c->stream, a); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int EB, int MODE, int CHUNK>
static hipError_t launch_attend_g(Ctx* c, const AttArgs& a, int32_t n_splits) {
    const int H = c->d.n_kv_heads, B = a.v.B;
    const dim3 grid = kPairFirst<MODE, CHUNK> ? dim3(H, B, n_splits) : dim3(n_splits, H, B), block(kBlockThreads);
    switch (c->G) {
        case 1: hipLaunchKernelGGL((attend_kernel<EB, 1, MODE, CHUNK>), grid, block, 0, c->stream, a); break;
        case 2: hipLaunchKernelGGL((attend_kernel<EB, 2, MODE, CHUNK>), grid, block, 0, c->stream, a); break;
        case 4: hipLaunchKernelGGL((attend_kernel<EB, 4, MODE, CHUNK>), grid, block, 0, c->stream, a); break;
        case 8: hipLaunchKernelGGL((attend_kernel<EB, 8, MODE, CHUNK>), grid, block, 0, c->stream, a); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

static AttArgs att_common(Ctx* c, const void* q, const void* Kbase, const void* Vbase, const SeqView& v, float* out,
                          float* lse) {
    AttArgs a{};
    a.q = (const char*)q; a.Kb = (const char*)Kbase; a.Vb = (const char*)Vbase;
    a.v = v; a.Hkv = c->d.n_kv_heads; a.max_splits = c->max_splits;
    a.part = c->att_part; a.ml = c->att_ml; a.counter = c->att_counter; a.out = out; a.lse = lse;
    a.budget_cap = c->budget_cap;
    return a;
}

// Many (sequence, head) pairs fill the GPU with 256-token blocks; below that 128-token blocks.
static bool wide_chunks(const Ctx* c, const SeqView& v) { return v.B * c->d.n_kv_heads >= kWideChunkMinHeads; }

hipError_t launch_attend(Ctx* c, const void* q, const void* K_sel, const void* V_sel, int32_t row_stride,
                         const int32_t* n_tok, int32_t budget, const SeqView& v, float* out, float* lse) {
    AttArgs a = att_common(c, q, K_sel, V_sel, v, out, lse);
    a.n_tok = n_tok; a.row_stride = row_stride;
    // bf16, up to 416 tokens (one query head per KV head: 320) of few heads: blocks that take all tokens and a quarter of the dims each (kDirectDims), so that nothing is merged and
    // a compute unit, which gets its rows at about 34 bytes a nanosecond, reads the keys and a quarter of the values.  Us per call, 4 query heads
    // per KV head, before / now: 64 tokens 3.9 / 3.2, 128: 4.31 / 3.94, 256 (one block) 6.2 / 5.2, 257 (three blocks and a merge) 6.8 / 5.8, 384:
    // 6.9 / 6.3; 8 query heads, 128: 5.2 / 4.2, 257: 7.8 / 6.4; one query head, 64: 3.5 / 3.1; halves of the dims, 257 tokens: 6.6.  Around the lines, blocks of tokens /
    // of dims, 400 tokens: 32 heads on 8 7.15 / 6.57, 64 on 8 8.06 / 7.17, 12 on 3 6.84 / 6.77; 448: 7.13 / 6.92, 8.00 / 7.54, 6.82 / 6.97; 512: 7.35 / 7.53, 8.19 / 8.23,
    // 6.88 / 7.47; 8 heads on 8, 32 on 32, 320 tokens: 5.97 / 5.82, 6.69 / 6.30; 352: 6.00 / 6.07, 6.78 / 6.57; 400: 6.14 / 6.46, 6.79 / 6.89.
    constexpr int parts = kHeadDim / kDimsPerBlock;
    if (c->d.kv_dtype == SKV_BF16 && budget <= (c->G > 1 ? kMaxDirectDims : kMaxDirectDims1) && v.B * c->d.n_kv_heads * parts <= c->n_cu) {
        if (budget <= kAttChunk) return launch_attend_g<2, kDirectDims, kAttChunk>(c, a, parts);
        if (budget <= kAttChunkMid) return launch_attend_g<2, kDirectDims, kAttChunkMid>(c, a, parts);
        if (budget <= kAttChunkWide) return launch_attend_g<2, kDirectDims, kAttChunkWide>(c, a, parts);
        return launch_attend_g<2, kDirectDims, 2 * kAttChunkWide>(c, a, parts);
    }
    // Else bf16, 129 to 256 tokens: one block, which writes the result itself (fp32 tiles keep the matrix cores of a compute unit busy too long for that: 16
    // tiles 0.9 us behind 8).  Else, for few (sequence, head) pairs, 128-token blocks.  The merging block's uncached reads of the partials cost about
    // 0.1 us per split, more than a 64-token block saves on its K/V rows (budget 2048: 11.0 us with 64-token blocks,
    // 9.2 with 128, 10.8 with 256; from a budget of 4096 on 256-token blocks are ahead).
    const bool wide = wide_chunks(c, v) || budget >= 4096 ||
                      (c->d.kv_dtype == SKV_BF16 && budget > kAttChunkMid && budget <= kAttChunkWide);
    const int chunk = wide ? kAttChunkWide : kAttChunkMid;
    int n_splits = (budget + chunk - 1) / chunk;
    if (n_splits < 1) n_splits = 1;       // block 0 still writes the empty-selection result
    if (wide)
        return c->d.kv_dtype == SKV_BF16 ? launch_attend_g<2, kDirect, kAttChunkWide>(c, a, n_splits)
                                         : launch_attend_g<4, kDirect, kAttChunkWide>(c, a, n_splits);
    return c->d.kv_dtype == SKV_BF16 ? launch_attend_g<2, kDirect, kAttChunkMid>(c, a, n_splits)
                                     : launch_attend_g<4, kDirect, kAttChunkMid>(c, a, n_splits);
}

hipError_t launch_attend_indirect(Ctx* c, const void* q, const void* K_layer, const void* V_layer, const int32_t* tok_idx,
                                  const int32_t* n_tok, const SeqView& v, float* out, float* lse) {
    AttArgs a = att_common(c, q, K_layer, V_layer, v, out, lse);
    a.n_tok = n_tok; a.tok_idx = tok_idx; a.idx_stride = c->d.max_budget;
    const int n_splits = (c->budget_cap + kAttChunkWide - 1) / kAttChunkWide;
    return c->d.kv_dtype == SKV_BF16 ? launch_attend_g<2, kIndirect, kAttChunkWide>(c, a, n_splits)
                                     : launch_attend_g<4, kIndirect, kAttChunkWide>(c, a, n_splits);
}

// Batch form of the fused step: blocks that select, then stream.  Rows are addressed with 32-bit byte offsets inside a (head, sequence)
// slab.
bool can_stream(const Ctx* c, int32_t T_total) { return T_total < (c->d.kv_dtype == SKV_BF16 ? 1 << 24 : 1 << 23); }
hipError_t launch_select_attend_stream(Ctx* c, const void* q, const void* K_layer, const void* V_layer, const float* score,
                                       const int32_t* sent_off, const int32_t* sent_len, const SeqView& v, float* out,
                                       float* lse, int32_t* tok_idx_out, int32_t* n_tok_out) {
    if (!can_stream(c, v.T_total)) return hipErrorInvalidValue;
    AttArgs a = att_common(c, q, K_layer, V_layer, v, out, lse);
    a.score = score; a.sent_off = sent_off; a.sent_len = sent_len;
    a.tok_idx_out = tok_idx_out; a.n_tok_out = n_tok_out; a.idx_stride = c->d.max_budget;
    // Block size by rounds of blocks (one block per compute unit).  While 512-token blocks still run in one round they
    // are ahead: two tiles per wave instead of four and twice the compute units busy (8 sequences x 8 heads, budget 2048:
    // 36.7 -> 33.0 us per layer); in two rounds they lose (16 sequences: 50.8 -> 58.1).  With several rounds of 1024-token
    // blocks, 2048-token blocks halve the selections and, up to a budget of 2048, need no merge: a round of them takes
    // about 5/3 of a 1024-token round (32 sequences: 94.7 -> 87.0 us, 64: 180.2 -> 166.3; 48: 137.8 either way).
    const int pairs = v.B * c->d.n_kv_heads;
    const int blocks = pairs * ((c->budget_cap + kStreamChunk - 1) / kStreamChunk);
    const bool bf16 = c->d.kv_dtype == SKV_BF16;
    if (2 * blocks <= c->n_cu) return bf16 ? launch_select_attend_stream_g<2, kStreamChunk / 2>(c, a) : launch_select_attend_stream_g<4, kStreamChunk / 2>(c, a);
    const int big_blocks = pairs * ((c->budget_cap + kStreamMaxChunk - 1) / kStreamMaxChunk);
    const int rounds = (blocks + c->n_cu - 1) / c->n_cu, big_rounds = (big_blocks + c->n_cu - 1) / c->n_cu;
    if (5 * big_rounds < 3 * rounds) return bf16 ? launch_select_attend_stream_g<2, kStreamMaxChunk>(c, a) : launch_select_attend_stream_g<4, kStreamMaxChunk>(c, a);
    return bf16 ? launch_select_attend_stream_g<2, kStreamChunk>(c, a) : launch_select_attend_stream_g<4, kStreamChunk>(c, a);
}

hipError_t launch_select_attend(Ctx* c, const void* q, const void* K_layer, const void* V_layer, const float* score,
                                const int32_t* sent_off, const int32_t* sent_len, const SeqView& v, float* out,
                                float* lse, int32_t* tok_idx_out, int32_t* n_tok_out) {
    AttArgs a = att_common(c, q, K_layer, V_layer, v, out, lse);
    a.score = score; a.sent_off = sent_off; a.sent_len = sent_len;
    a.tok_idx_out = tok_idx_out; a.n_tok_out = n_tok_out; a.idx_stride = c->d.max_budget;
    // One block per compute unit fits (value tiles + selection histograms in LDS), so the block size is the
    // smallest whose blocks all run at once; a second round of blocks costs more than the larger blocks' longer K/V phase
    // (4 sequences of 32K, 8 heads, budget 2048, bf16: 25.9 us in 128-token blocks, 17 in 256-token blocks).
    const int pairs = v.B * c->d.n_kv_heads;
    auto blocks = [&](int chunk) { return pairs * ((c->budget_cap + chunk - 1) / chunk); };
    if (blocks(kAttChunkMid) > c->n_cu) {
        const int n_splits = (c->budget_cap + kAttChunkWide - 1) / kAttChunkWide;
        return c->d.kv_dtype == SKV_BF16 ? launch_attend_g<2, kFused, kAttChunkWide>(c, a, n_splits)
                                         : launch_attend_g<4, kFused, kAttChunkWide>(c, a, n_splits);
    }
    // Every split block of a head repeats the selection; with thousands of buckets per sequence that repetition
    // (bucket loads from L2, histogram passes) outweighs the shorter K/V phase of 64-token blocks.
    if (v.S_total / (v.B > 0 ? v.B : 1) > kMidChunkMinSentences || blocks(kAttChunk) > c->n_cu) {
        const int n_splits = (c->budget_cap + kAttChunkMid - 1) / kAttChunkMid;
        return c->d.kv_dtype == SKV_BF16 ? launch_attend_g<2, kFused, kAttChunkMid>(c, a, n_splits)
                                         : launch_attend_g<4, kFused, kAttChunkMid>(c, a, n_splits);
    }
    const int n_splits = (c->budget_cap + kAttChunk - 1) / kAttChunk;
    return c->d.kv_dtype == SKV_BF16 ? launch_attend_g<2, kFused, kAttChunk>(c, a, n_splits)
                                     : launch_attend_g<4, kFused, kAttChunk>(c, a, n_splits);
}

// Single-launch step.  Blocks per pair: the largest power of two that keeps pairs x blocks within the compute units (every
// block must be resident for the per-pair wait to end: one 1024-thread block per compute unit).  All of them score; the
// first ceil(max_budget / CHUNK) of them attend.
// Blocks of the single-launch kernel a compute unit can hold at once (registers, LDS), asked of the runtime once per
// instantiation: the kernel's waits need every block of the grid resident, so the launcher refuses grids beyond
// compute units x this number.
template <int EB, int G, int MODE, int CHUNK>
static int step_blocks_per_cu() {
    static int cached = -1;
    if (cached < 0) {
        int n = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, attend_kernel<EB, G, MODE, CHUNK>, kBlockThreads, 0) != hipSuccess) {
            (void)hipGetLastError();
            n = 0;
        }
        cached = n;
    }
    return cached;
}

template <int EB, int MODE, int CHUNK>
static hipError_t launch_step_g(Ctx* c, const AttArgs& a, int parts, bool* launched) {
    const dim3 grid(c->d.n_kv_heads, a.v.B, parts), block(kBlockThreads);
    const int n_blocks = c->d.n_kv_heads * a.v.B * parts;
    int per_cu = 0;
    switch (c->G) {
        case 1: per_cu = step_blocks_per_cu<EB, 1, MODE, CHUNK>(); break;
        case 2: per_cu = step_blocks_per_cu<EB, 2, MODE, CHUNK>(); break;
        case 4: per_cu = step_blocks_per_cu<EB, 4, MODE, CHUNK>(); break;
        case 8: per_cu = step_blocks_per_cu<EB, 8, MODE, CHUNK>(); break;
        default: return hipErrorInvalidValue;
    }
    if (per_cu < 1 || n_blocks > c->n_cu * per_cu) return hipSuccess;       // not every block would be resident: other forms
    *launched = true;
    switch (c->G) {
        case 1: hipLaunchKernelGGL((attend_kernel<EB, 1, MODE, CHUNK>), grid, block, 0, c->stream, a); break;
        case 2: hipLaunchKernelGGL((attend_kernel<EB, 2, MODE, CHUNK>), grid, block, 0, c->stream, a); break;
        case 4: hipLaunchKernelGGL((attend_kernel<EB, 4, MODE, CHUNK>), grid, block, 0, c->stream, a); break;
        case 8: hipLaunchKernelGGL((attend_kernel<EB, 8, MODE, CHUNK>), grid, block, 0, c->stream, a); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_step(Ctx* c, const void* q_score, const void* q_attn, const void* semvec_layer, const void* K_layer,
                       const void* V_layer, const int32_t* sent_off, const int32_t* sent_len, const SeqView& v, float* out,
                       float* lse, int32_t* tok_idx_out, int32_t* n_tok_out, bool* launched) {
    *launched = false;
    const int pairs = v.B * c->d.n_kv_heads;
    const int max_blocks = c->n_cu < kStepMaxBlocks ? c->n_cu : kStepMaxBlocks;
    if (pairs < 1 || pairs > kStepMaxPairs || pairs > max_blocks || c->step_score_stride <= 0) return hipSuccess;
    if (v.S_total > c->step_score_stride || (int64_t)pairs * c->step_score_stride > c->step_score_words) return hipSuccess;
    int parts = max_blocks / pairs, pow2 = 1;
    while (2 * pow2 <= parts) pow2 *= 2;
    if (c->budget_cap <= pow2 * kAttChunk) parts = pow2;
    const int sv_bytes = c->d.semvec_dtype == SKV_BF16 ? kTableBf16 : c->d.semvec_dtype == SKV_FP8_E4M3 ? kTableE4m3 : kTableF32;
    // Attention blocks of 64 or 128 tokens where a pair has a power of two of them and they cover the budget (MODE kStep; constants where the other
    // form has arguments, 0.5 % of a step; shares of exactly 256 tokens too, 8 sequences, budget 1024: 19.55 / 19.45).  A block's K/V rows pass its compute unit at 34
    // bytes a nanosecond, so that small blocks are faster until there are too many partials to merge: one sequence, us per layer in 128- / 64-token blocks: bf16 budget 512:
    // 10.9 / 10.0, 1000: 11.5 / 10.8, 2048: 13.1 / 12.8; fp32 13.6 / 11.9, 14.5 / 12.7, 15.9 / 15.0; budget 2500 in 20 blocks of 128 / 32 of 80: 13.0 / 14.1.
    // Otherwise (kStepRagged) every block of the pair takes an equal share.  Us per layer, powers of two of blocks of 128, 256 or 512 tokens / this: 3 sequences,
    // budget 2048, eight blocks / ten: 19.2 / 18.2; 6 sequences, budget 1500, three blocks of four / five: 22.2 / 18.1; 8 sequences, budget 1100, two
    // launches / four blocks: 22.2 / 18.8; 4 sequences, budget 1100, five of eight / eight: 19.3 / 18.6; budget 2500, two launches / eight: 23.2 / 19.9.
    // Budgets that a power of two of 64-token blocks covers leave the pair's other blocks out; equal shares of 64 / this: 5 sequences of 8192 tokens, budget 128 11.68 / 11.40,
    // fp32, 256 14.4 / 14.0, 64 query heads, 256 13.3 / 12.8; 6 sequences, 256 12.1 / 11.85 (of 32768 tokens 17.4 / 17.9); 3 sequences 10.58 / 10.61.
    const int share = max((c->budget_cap + 16 * parts - 1) / (16 * parts) * 16, kAttChunk);
    const bool even = parts == pow2 && (c->budget_cap <= parts * kAttChunkMid || share == kAttChunkWide);
    const int chunk = !even || share == kAttChunkWide ? share : c->budget_cap <= parts * kAttChunk ? kAttChunk : kAttChunkMid;
    const int most = c->d.kv_dtype == SKV_BF16 ? 2 * kAttChunkWide : kAttChunkWide;
    if (chunk > most || parts < 2 || v.S_total >= (1 << 24)) return hipSuccess;
    // More than 256 tokens, bf16 only: two tiles a wave.  Every attending block waits for all the scores of its pair, and the two-launch form spreads
    // the rows over all compute units: where a sequence has more than 1024 buckets on average, the mean-key rows have to take at most half the
    // bytes of the retrieved ones.  Two launches / one, us per layer: 6 sequences, budget 1500, 960 buckets, 0.64 of the bytes: 24.4 / 21.3; 8 sequences,
    // budget 1300, 960, 0.74: 25.6 / 23.6; budget 2048, 1310, 0.64: 30.0 / 29.0; past the line: 6 sequences, budget 2048, 2621, 0.64: 27.2 / 28.8;
    // budget 2048, 1600, 0.78: 27.3 / 27.7; 4 sequences, budget 2600, 2621, 1.0: 28.0 / 28.7.
    if (chunk > kAttChunkWide && v.S_total > 1024ll * v.B && (int64_t)v.S_total * sv_bytes > (int64_t)v.B * c->budget_cap * 2) return hipSuccess;
    const int att_parts = (c->budget_cap + chunk - 1) / chunk;
    if (c->G > 2 * parts) return hipSuccess;                                     // mergers do not fit
    AttArgs a = att_common(c, q_attn, K_layer, V_layer, v, out, lse);
    a.sent_off = sent_off; a.sent_len = sent_len;
    a.tok_idx_out = tok_idx_out; a.n_tok_out = n_tok_out; a.idx_stride = c->d.max_budget;
    a.q_score = (const char*)q_score; a.semvec = (const char*)semvec_layer;
    // Up to four blocks merge a head, 32 dims each, so that a thread has one word of a partial row to wait for instead of four (one sequence,
    // budget 2048, per layer: 12.8 -> 12.55 us, fp32 14.9 -> 14.5), as long as they all attend themselves: a block that runs the
    // selection only to merge costs more than it saves (budget 512, 8 query heads per KV head: 10.5 -> 12.0 with 32 of them).
    int lg_merge = 0;
    while (lg_merge < 2 && (c->G << (lg_merge + 1)) <= att_parts) ++lg_merge;
    // two heads per merging block where a pair has fewer blocks that attend than heads: 8 query heads per KV head, 16 layers, 5 to 8
    // sequences 319 -> 278 us and 347 -> 304 (which had to take two launches), one sequence at a budget of 200 178 -> 173
    if (c->G > att_parts && c->G > 1 && (c->G > parts || c->G <= 2 * att_parts)) lg_merge = -1;
    auto per = [](int n) { return (uint32_t)(((1ull << 32) + (unsigned long long)n - 1) / (unsigned long long)n); };
    a.sv_bytes = sv_bytes; a.lg_parts = even ? __builtin_ctz(parts) : 0; a.lg_merge = lg_merge;
    a.parts = parts; a.chunk = chunk; a.per_part = per(parts); a.per_chunk = per(chunk);
    a.step_epoch = c->step_epoch; a.step_score = c->step_score; a.score_stride = c->step_score_stride;
    a.step_part = c->step_part; a.wait_limit = c->wait_limit;
    a.err_dev = c->err_dev; a.err_host = c->err_host_dev;
    const bool bf16 = c->d.kv_dtype == SKV_BF16;
    auto go = [&](auto mode, auto cap) {
        constexpr int M = decltype(mode)::value, C = decltype(cap)::value;
        return bf16 ? launch_step_g<2, M, C>(c, a, parts, launched) : launch_step_g<4, M, C>(c, a, parts, launched);
    };
    using std::integral_constant;
    if (even && chunk == kAttChunk) return go(integral_constant<int, kStep>{}, integral_constant<int, kAttChunk>{});
    if (even && chunk == kAttChunkMid) return go(integral_constant<int, kStep>{}, integral_constant<int, kAttChunkMid>{});
    if (even) return go(integral_constant<int, kStep>{}, integral_constant<int, kAttChunkWide>{});
    if (chunk == kAttChunk) return go(integral_constant<int, kStepRagged>{}, integral_constant<int, kAttChunk>{});
    if (chunk <= kAttChunkMid) return go(integral_constant<int, kStepRagged>{}, integral_constant<int, kAttChunkMid>{});
    if (chunk <= kAttChunkWide) return go(integral_constant<int, kStepRagged>{}, integral_constant<int, kAttChunkWide>{});
    return launch_step_g<2, kStepRagged, 2 * kAttChunkWide>(c, a, parts, launched);
}

// ------------------------------------------------------------------------------------------------
// Merge of two partial attention results over disjoint token sets (Eq. 3 over their union): the retrieved tokens and,
// for instance, a contiguous window of recent tokens attended with skv_attend.  One thread per output pair.
// ------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void merge_lse_kernel(const float* __restrict__ out_a, const float* __restrict__ lse_a,
                                                        const float* __restrict__ out_b, const float* __restrict__ lse_b,
                                                        int32_t n_heads, float* __restrict__ out, float* __restrict__ lse) {
    const int32_t i = blockIdx.x * 256 + threadIdx.x;                  // pair index: head * (D / 2) + pair
    if (i >= n_heads * (kHeadDim / 2)) return;
    const int32_t j = i / (kHeadDim / 2);
    const float la = lse_a[j], lb = lse_b[j];
    const float m = fmaxf(la, lb);
    float2 r = make_float2(0.f, 0.f);
    float l = -INFINITY;
    if (m > -INFINITY || la != la || lb != lb) {                       // (NaN is not an empty side)
        const float za = expf(la - m), zb = expf(lb - m);              // an empty side has lse = -inf: weight 0
        const float inv = 1.f / (za + zb);
        const float2 a = reinterpret_cast<const float2*>(out_a)[i], b = reinterpret_cast<const float2*>(out_b)[i];
        r.x = ((za > 0.f ? za * a.x : 0.f) + (zb > 0.f ? zb * b.x : 0.f)) * inv;
        r.y = ((za > 0.f ? za * a.y : 0.f) + (zb > 0.f ? zb * b.y : 0.f)) * inv;
        l = m + logf(za + zb);
    }
    reinterpret_cast<float2*>(out)[i] = r;
    if (lse && (i % (kHeadDim / 2)) == 0) lse[j] = l;
}

hipError_t launch_merge_lse(Ctx* c, const float* out_a, const float* lse_a, const float* out_b, const float* lse_b,
                            int32_t n_heads, float* out, float* lse) {
    const int n = n_heads * (kHeadDim / 2);
    hipLaunchKernelGGL(merge_lse_kernel, dim3((n + 255) / 256), dim3(256), 0, c->stream, out_a, lse_a, out_b, lse_b, n_heads, out,
                       lse);
    return hipGetLastError();
}

}  // namespace skv
