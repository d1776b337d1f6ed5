// Prefill-side token retention (Sec. 4.1 "Token importance measurement", "Token selection within sentence
// buckets"; App. "Effect of Sentence Length"; Alg. 1 prefilling phase): observation-window importance on the
// matrix cores, global top-k of the importance, buckets of the retained tokens, compaction of the K/V pool.
// gfx950, wave64, bf16 and fp32 inputs.
#include "skv_internal.h"
#include "skv_device.h"

#include <atomic>
#include <type_traits>

namespace skv {

// ------------------------------------------------------------------------------------------------
// Importance.  For one layer and KV head h the window's R = G*N query rows (row = g*N + n: query head
// h*G+g, window token n, contiguous in q_obs) meet all T keys on v_mfma_f32_32x32x16_bf16.  fp32 inputs are split
// exactly into three bf16 terms -- see Frag -- so that the products keep fp32 accuracy.
//   pass 1 (stats):   per row, a whole reference r near the largest logit s (log2 units) and the sum of exp2(s - r) over the
//                     keys visible to it (positions <= Tp + n), per block of keys; the block of the (layer, head) that
//                     arrives last combines the partials per row;
//   pass 2 (colsum):  per KV head, the column sums of exp2(s - r_row) * (1 / sum_row) over the head's rows, for the Tp
//                     prefix keys; the head whose block arrives last for a range of keys adds the heads in ascending
//                     order (deterministic).
// References are whole numbers so that sums change from one to another by exact powers of two, and reference and sum stay apart up
// to the last multiplication: s - r is then rounded once, at the size of the result.  (Their logarithm in one float, r + log2(sum), has only the
// fraction bits that the logit's magnitude leaves: from exact logits of 166 to 423, a relative error of 1e-5 instead of 4.6e-7.)
// Each pass covers all layers in one launch (grid z = layer).  Its one read of the keys takes 300 us for 32 layers x 8 heads x 32768 keys (a
// second read within reach of the memory-side cache is no faster, 7.1 TB/s either way), its matrix instructions and
// exp2 take 260-310 us by themselves at the clock (1.6-2.1 GHz) that the power limit leaves, and the two overlap: 350-400 us a pass.
//   * The keys go to LDS by asynchronous whole-row non-temporal loads, a ring of stages; the query fragments stay in registers: a wave
//     owns a row tile and a key tile of every stage.
//   * Tiles of 32 x 32: a matrix instruction keeps the vector pipe from issuing for 8 cycles, of 32 that it runs (of 16 in the
//     16 x 16 form).  Next to it a wave issues little more than exp2, fma and add of every logit.
//   * One key tile's sums are taken while the matrix cores work on the next.
// Window of 32 tokens, 4 query heads per KV head, 32K tokens: 912-940 us -> 800 us; 1.1K tokens: 55 -> 45; fp32, 8K tokens: 1250 -> 845, 8
// query heads: 2920 -> 1540.  (Before: fragments straight from memory by 64-byte pieces of 16 rows per load instruction at 5 TB/s,
// queries from LDS and for fp32 split again for every tile, four launches.)
// ------------------------------------------------------------------------------------------------
template <int EB, int RT> struct Imp {                          // RT: 32-row tiles of the window's rows
    static constexpr int RS = RT;                              // waves that share the rows, a tile each
    static constexpr int NW = EB == 2 ? (RT == 1 ? 2 : RT == 8 ? 8 : 4) : (RT == 1 ? 4 : 8);     // waves of a block
    static constexpr int KSP = NW / RS;                        // 32-key tiles of a stage, one for each wave of a row tile
    static constexpr int kThreads = NW * kWave, kRows = 32 * RT;
    static constexpr int kStageKeys = 32 * KSP, kStageBytes = kStageKeys * kHeadDim * EB;
    static constexpr int kPerCu = EB == 4 ? 1 : RT == 8 ? 2 : 3;     // blocks on a compute unit
    static constexpr int kRingBytes = EB == 4 ? 128 * 1024 : RT == 8 ? 72 * 1024 : 48 * 1024;
    static constexpr int NB = kRingBytes / kStageBytes;        // stages in the ring
    static constexpr int kLoads = kStageBytes / (NW * kWave * 16);   // load instructions of a wave per stage
    static constexpr int kWavesPerSimd = (kPerCu * NW + 3) / 4;
    static_assert(RS * KSP == NW && NB >= 2 && kLoads >= 1 && NB * kLoads < 64, "every wave has its rows, keys and loads");
};

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x16 mfma_bf16(const uint4& a, const uint4& b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
// 2^x: the bare instruction; results below the normal range flush to zero
__device__ __forceinline__ float exp2_neg(float x) { return __builtin_amdgcn_exp2f(x); }

// the upper halves of two words in one
__device__ __forceinline__ uint32_t high_halves(uint32_t lo, uint32_t hi) { return __builtin_amdgcn_perm(hi, lo, 0x07060302u); }

// 8 consecutive elements of a row as bf16 fragments.  bf16 storage: 16 bytes as they are.  fp32 storage: each value
// is split exactly into three bf16 terms by truncation (8 + 8 + 8 mantissa bits: x = a + b + c), and x*y is evaluated
// as aa' + ab' + ba' + ac' + bb' + ca' by six MFMAs; the dropped terms are below 2^-23 of the product.
template <int EB> struct Frag;
template <> struct Frag<2> {
    uint4 t0;
    __device__ __forceinline__ void set(const uint4& lo, const uint4&) { t0 = lo; }
};
template <> struct Frag<4> {
    uint4 t0, t1, t2;
    __device__ __forceinline__ void set(const uint4& lo4, const uint4& hi4) {
        const uint32_t x[8] = {lo4.x, lo4.y, lo4.z, lo4.w, hi4.x, hi4.y, hi4.z, hi4.w};
        uint32_t a[8], b[8], c[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            a[i] = x[i];
            const float r1 = __uint_as_float(x[i]) - __uint_as_float(x[i] & 0xffff0000u);          // exact
            b[i] = __float_as_uint(r1);
            c[i] = __float_as_uint(r1 - __uint_as_float(b[i] & 0xffff0000u));                      // exact, at most 8 significant bits
        }
        t0 = make_uint4(high_halves(a[0], a[1]), high_halves(a[2], a[3]), high_halves(a[4], a[5]), high_halves(a[6], a[7]));
        t1 = make_uint4(high_halves(b[0], b[1]), high_halves(b[2], b[3]), high_halves(b[4], b[5]), high_halves(b[6], b[7]));
        t2 = make_uint4(high_halves(c[0], c[1]), high_halves(c[2], c[3]), high_halves(c[4], c[5]), high_halves(c[6], c[7]));
    }
};

template <int EB>
__device__ __forceinline__ f32x16 frag_mma(const Frag<EB>& k, const Frag<EB>& q, f32x16 c) {
    if constexpr (EB == 4) {                                  // small terms first
        c = mfma_bf16(k.t2, q.t0, c);
        c = mfma_bf16(k.t1, q.t1, c);
        c = mfma_bf16(k.t0, q.t2, c);
        c = mfma_bf16(k.t1, q.t0, c);
        c = mfma_bf16(k.t0, q.t1, c);
    }
    return mfma_bf16(k.t0, q.t0, c);
}

// Query fragments of a wave's row tile: lane (r, g) = (lane % 32, lane / 32), step d holds dims 16d+8g .. +7 of row row0 + r (rows
// >= R are zero).
template <int EB>
__device__ __forceinline__ void load_queries(Frag<EB> (&qf)[8], const char* __restrict__ q_head /* [R][D] */, int R, int row0) {
    const int lane = threadIdx.x & 63, row = row0 + (lane & 31);
    const char* src = q_head + (int64_t)min(row, R - 1) * (kHeadDim * EB) + 8 * EB * (lane >> 5);
    const uint32_t live = row < R ? ~0u : 0u;
#pragma unroll
    for (int d = 0; d < 8; ++d) {
        uint4 lo = *reinterpret_cast<const uint4*>(src + 16 * EB * d);
        uint4 hi = EB == 4 ? *reinterpret_cast<const uint4*>(src + 16 * EB * d + 16) : make_uint4(0, 0, 0, 0);
        lo = make_uint4(lo.x & live, lo.y & live, lo.z & live, lo.w & live);
        hi = make_uint4(hi.x & live, hi.y & live, hi.z & live, hi.w & live);
        qf[d].set(lo, hi);
    }
}

// this lane's key fragment of step d for key row `row` of a stage
template <int EB>
__device__ __forceinline__ void stage_frag(Frag<EB>& f, const char* stage, int row, int d, int g) {
    const char* base = stage + row * (kHeadDim * EB);
    if constexpr (EB == 2) {
        const uint4 lo = *reinterpret_cast<const uint4*>(base + 16 * ((2 * d + g) ^ (row & 15)));
        f.set(lo, lo);
    } else {
        f.set(*reinterpret_cast<const uint4*>(base + 16 * ((4 * d + 2 * g) ^ (row & 15))),
              *reinterpret_cast<const uint4*>(base + 16 * ((4 * d + 2 * g + 1) ^ (row & 15))));
    }
}

// The ring of stages of one head's keys base0 .. of a block.  A wave requests its share of a stage's rows (its own tile where it has all
// rows of the window), each instruction whole rows.  The 16-byte piece p of row r lands at piece p ^ (r % 16), so that fragment reads
// (two pieces of 32 rows) spread over the banks.
template <int EB, int RT>
struct KeyRing {
    using P = Imp<EB, RT>;
    static constexpr int kRowBytes = kHeadDim * EB, kPieces = kRowBytes / 16, kRows = kWave / kPieces;      // rows per instruction
    const char* Kh;
    char* ring;
    int32_t base0, last;      // keys past `last` are replaced by it: never out of bounds
    int n, slot, ahead;
    int row;                  // stage row of this lane's first load, its byte offset in the stage
    uint32_t off[P::kLoads];

    __device__ __forceinline__ KeyRing(const char* Kh_, char* ring_, int32_t base0_, int32_t last_, int n_)
        : Kh(Kh_), ring(ring_), base0(base0_), last(last_), n(n_) {
        const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
        row = kRows * P::kLoads * w + lane / kPieces;
#pragma unroll
        for (int i = 0; i < P::kLoads; ++i) {
            const int r = row + kRows * i;
            off[i] = (uint32_t)(r * kRowBytes + 16 * ((lane % kPieces) ^ (r & 15)));
        }
        slot = 0;
        ahead = P::NB - 1;
        for (int s = 0; s < P::NB - 1 && s < n; ++s) request(s, s);
    }
    __device__ __forceinline__ void request(int s, int to) {
        const int32_t key0 = base0 + s * P::kStageKeys;
        const char* src = Kh + (int64_t)key0 * kRowBytes;               // wave-uniform
        char* dst = ring + to * P::kStageBytes + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * (P::kLoads * 1024);
        if (key0 + P::kStageKeys - 1 <= last) {
#pragma unroll
            for (int i = 0; i < P::kLoads; ++i) load_lds_stream(src, off[i], dst + 1024 * i);
        } else {
#pragma unroll
            for (int i = 0; i < P::kLoads; ++i) {
                const int r = row + kRows * i, beyond = max(r - (last - key0), 0);
                load_lds_stream(src, off[i] - (uint32_t)(beyond * kRowBytes), dst + 1024 * i);
            }
        }
    }
    // Stage s, in turn: landed, and one more requested into the place of the stage before it.  Where a wave has all rows it reads only
    // keys that it requested itself and asks for the next before it waits; otherwise the block meets here.
    __device__ __forceinline__ const char* next(int s) {
        auto more = [&]() { request(s + P::NB - 1, ahead); };
        if constexpr (P::RS == 1) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            if (s + P::NB - 1 < n) { more(); wait_loads<(P::NB - 1) * P::kLoads>(); }
            else wait_loads<0>();
        } else {
            if (s + P::NB - 2 < n) wait_loads<(P::NB - 2) * P::kLoads>();
            else wait_loads<0>();
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            if (s + P::NB - 1 < n) more();
        }
        const char* stage = ring + slot * P::kStageBytes;
        slot = slot + 1 == P::NB ? 0 : slot + 1;
        ahead = ahead + 1 == P::NB ? 0 : ahead + 1;
        return stage;
    }
};

// A 32-key tile against a wave's row tile.  KEYS_A: keys as the A operand (element i of a lane: key 8 (i / 4) + 4 g + i % 4, row r), else
// the queries (that row, key r).
template <int EB, bool KEYS_A>
__device__ __forceinline__ void tile_logits(f32x16& acc, const Frag<EB> (&qf)[8], const char* stage, int row, int g) {
    f32x16 c = {};
#pragma unroll
    for (int d = 0; d < 8; ++d) {
        Frag<EB> kf;
        stage_frag<EB>(kf, stage, row, d, g);
        c = KEYS_A ? frag_mma<EB>(kf, qf[d], c) : frag_mma<EB>(qf[d], kf, c);
    }
    acc = c;
}
__device__ __forceinline__ int tile_pos(int i, int g) { return 8 * (i >> 2) + 4 * g + (i & 3); }

// The waves that the ring leaves room for, no more: with fewer registers the compiler reads one key fragment at a time.
#define SKV_IMP_WAVES __attribute__((amdgpu_waves_per_eu(Imp<EB, RT>::kWavesPerSimd, Imp<EB, RT>::kWavesPerSimd)))

// sum * 2^(from - to) for whole from <= to (from == -infinity: a sum of nothing, or of NaN)
__device__ __forceinline__ float move_reference(float sum, float from, float to) {
    return from > -INFINITY ? ldexpf(sum, (int)fmaxf(from - to, -512.f)) : 0.f * sum;
}

// alpha[l][i] = sum over the heads of alpha_h[l][h][i] in ascending order; grid (any, Hkv, L)
__device__ __forceinline__ void add_heads(const float* __restrict__ alpha_h, float* __restrict__ alpha, int32_t Tp) {
    const int Hkv = gridDim.y, l = blockIdx.z;
    const float* src = alpha_h + (int64_t)l * Hkv * Tp;
    const int32_t step = gridDim.x * gridDim.y * blockDim.x;
    for (int32_t i = (blockIdx.x * gridDim.y + blockIdx.y) * blockDim.x + threadIdx.x; i < Tp; i += step) {
        float v = 0.f;
        for (int hh = 0; hh < Hkv; hh += 8) {
            float y[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) y[u] = src[(int64_t)min(hh + u, Hkv - 1) * Tp + i];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (hh + u < Hkv) v += y[u];
        }
        alpha[(int64_t)l * Tp + i] = v;
    }
}

// pass 1, a block: chunk `chunk` of `nchunks` (kpb keys each) of a (layer, head); part [L][Hkv][chunks][rows] (reference, sum); rowstat
// [L][Hkv][rows] (reference, 1 / sum) over all keys with 1 <= sum < 2 ((+infinity, 0) for rows >= R), written by the (layer, head)'s last block, which
// gets true.
template <int EB, int RT>
__device__ __forceinline__ bool importance_stats(const char* __restrict__ q_obs, const char* __restrict__ K_pool, int32_t T, int32_t N, int32_t G,
                                                 int32_t kpb, float2* part, float2* rowstat, unsigned int* arrive, int chunk, int nchunks,
                                                 int64_t lh) {
    using P = Imp<EB, RT>;
    constexpr int kRowBytes = kHeadDim * EB, kRows = P::kRows;
    constexpr float kLog2e = 1.4426950408889634f;
    extern __shared__ __attribute__((aligned(16))) char sm_ring[];
    __shared__ float sm_m[P::KSP][kRows], sm_l[P::KSP][kRows];
    __shared__ int sm_last;

    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, r = lane & 31, g = lane >> 5;
    const int rs = w / P::KSP, ks = w % P::KSP;
    const int R = G * N, Tp = T - N;
    const char* Kh = K_pool + lh * T * kRowBytes;
    const int32_t base0 = chunk * kpb, n = (min(kpb, T - base0) + P::kStageKeys - 1) / P::kStageKeys;
    KeyRing<EB, RT> keys(Kh, sm_ring, base0, T - 1, n);                  // before the queries: both are on their way together
    Frag<EB> qf[8];
    load_queries<EB>(qf, q_obs + lh * R * kRowBytes, R, 32 * rs);
    const float scale = kLog2e * rsqrtf((float)kHeadDim);

    // Sums are kept per LANE (a lane sees half of the keys of every tile of its row); the two lanes of a row meet once, after the last
    // stage.  While every key of a stage is visible to every row, the reference stays what it is until a tile's sum reaches
    // kFar: any reference near the largest logit gives the same sum, and a running maximum would take a third of the
    // instructions.  It is set kAbove over the largest logit, so that a later one seldom is too far above (a tile's keys are mostly of one
    // sentence and have like logits: with 0 and 32 for the two, every third tile of a wave had a row to move, 418 us
    // instead of 374 for the pass); both together keep the arguments of exp2 that matter within -8 .. 8.
    constexpr float kFar = 256.f, kAbove = 4.f;
    float ref = -INFINITY, l_run = 0.f;
    auto add_relative = [&](const f32x16& x, float m) {                  // reference: the largest logit so far, `m` among them
        const float to = fmaxf(ref, rintf(m * scale) + kAbove), base = to > -INFINITY ? to : 0.f;   // (nothing visible yet: every term is exp2(-inf) = 0)
        float sum = 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i) sum += exp2_neg(fmaf(x[i], scale, -base));
        l_run = move_reference(l_run, ref, base) + sum;
        ref = to;
    };
    auto sum_tile = [&](const f32x16& x) {
        float sum[2] = {0.f, 0.f};
#pragma unroll
        for (int i = 0; i < 16; ++i) sum[i & 1] += exp2_neg(fmaf(x[i], scale, -ref));
        float both = sum[0] + sum[1];
        asm volatile("" : "+v"(both));                                   // here, next to the matrix instructions, not behind the next barrier
        return both;
    };
    auto settle = [&](const f32x16& x, float sum) {                      // adds sum_tile's result, if need be to another reference
        if (sum < kFar) {
            l_run += sum;
        } else {                                                         // the row's first tile, and rarely a later one
            float m = -INFINITY;
#pragma unroll
            for (int i = 0; i < 16; ++i) m = fmaxf(m, x[i]);
            add_relative(x, m);
        }
    };
    auto add_tile_masked = [&](f32x16& x, int32_t key0) {
        const int32_t limit = min(Tp + (32 * rs + r) % N, T - 1);        // last position visible to this lane's row
        float m = -INFINITY;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            if (key0 + tile_pos(i, g) > limit) x[i] = -INFINITY;
            m = fmaxf(m, x[i]);
        }
        add_relative(x, m);
    };
    const int row0 = 32 * ks + r;                                        // this lane's key row in a stage
    const int n_open = min(max((Tp - base0) / P::kStageKeys, 0), n);     // stages whose keys are all visible to all rows
    if (n_open > 0) {
        // the sums of a tile are taken while the matrix cores work on the next one, and settled a barrier later (a branch in between
        // would keep the two apart)
        f32x16 acc[2];
        float sum = 0.f;
        tile_logits<EB, true>(acc[0], qf, keys.next(0), row0, g);
        int s = 1;
        for (; s + 1 < n_open; s += 2) {
            const char* stage = keys.next(s);
            settle(acc[1], sum);
            tile_logits<EB, true>(acc[1], qf, stage, row0, g);
            sum = sum_tile(acc[0]);
            stage = keys.next(s + 1);
            settle(acc[0], sum);
            tile_logits<EB, true>(acc[0], qf, stage, row0, g);
            sum = sum_tile(acc[1]);
        }
        if (s < n_open) {
            const char* stage = keys.next(s);
            settle(acc[1], sum);
            tile_logits<EB, true>(acc[1], qf, stage, row0, g);
            settle(acc[0], sum_tile(acc[0]));
            sum = sum_tile(acc[1]);
        }
        settle(acc[1], sum);
        if (n_open & 1) settle(acc[0], sum_tile(acc[0]));
    }
#pragma unroll 1
    for (int s = n_open; s < n; ++s) {
        f32x16 x;
        tile_logits<EB, true>(x, qf, keys.next(s), row0, g);
        add_tile_masked(x, base0 + s * P::kStageKeys + 32 * ks);
    }
    // the two lanes of a row, then the block's waves
    {
        const float m = fmaxf(ref, __shfl_xor(ref, 32));
        float l = move_reference(l_run, ref, m);
        l += __shfl_xor(l, 32);
        if (g == 0) { sm_m[ks][32 * rs + r] = m; sm_l[ks][32 * rs + r] = l; }
    }
    __syncthreads();
    if (tid < kRows) {
        float m = -INFINITY;
#pragma unroll
        for (int k = 0; k < P::KSP; ++k) m = fmaxf(m, sm_m[k][tid]);
        float l = 0.f;
#pragma unroll
        for (int k = 0; k < P::KSP; ++k) l += move_reference(sm_l[k][tid], sm_m[k][tid], m);
        st_agent64(part + (lh * nchunks + chunk) * kRows + tid, m, l);
    }
    // ---- the last block of the (layer, head): combined statistics ------------------------------------------------
    block_sync_after_stores();
    if (tid == 0) sm_last = __hip_atomic_fetch_add(&arrive[lh], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (unsigned int)(nchunks - 1);
    __syncthreads();
    if (!sm_last) return false;
    constexpr int kGroups = P::kThreads / kRows;                         // chunks grp, grp + kGroups, ... by thread (grp, row)
    const int row = tid % kRows, grp = tid / kRows;
    float M = -INFINITY, L = 0.f;
    constexpr int kU = 12;                                               // loads in flight (8: the same, 32768 keys of 128 rows 844 / 839 us, of 256 685 / 692)
    for (int c = grp; c < nchunks; c += kU * kGroups) {
        unsigned long long v[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) v[u] = ld_agent64(&part[(lh * nchunks + min(c + u * kGroups, nchunks - 1)) * kRows + row].x);
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const float pm = c + u * kGroups < nchunks ? lo_f(v[u]) : -INFINITY;
            const float nm = fmaxf(M, pm);
            L = move_reference(L, M, nm) + move_reference(hi_f(v[u]), pm, nm);
            M = nm;
        }
    }
    float* sm_g = reinterpret_cast<float*>(sm_ring);                     // the ring is no longer read
    sm_g[tid] = M;
    sm_g[P::kThreads + tid] = L;
    __syncthreads();
    if (tid < kRows) {
#pragma unroll
        for (int g = 1; g < kGroups; ++g) {
            const float m2 = sm_g[g * kRows + row], l2 = sm_g[P::kThreads + g * kRows + row], nm = fmaxf(M, m2);
            L = move_reference(L, M, nm) + move_reference(l2, m2, nm);
            M = nm;
        }
        const bool adds = row < R && L > 0.f;
        const int e = adds ? ilogbf(L) : 0;
        rowstat[lh * kRows + row] = adds ? make_float2(M + (float)e, 1.f / ldexpf(L, -e)) : make_float2(INFINITY, 0.f);
    }
    if (tid == 0) __hip_atomic_store(&arrive[lh], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // for the next call
    return true;
}

// grid (chunks, Hkv, L)
template <int EB, int RT>
__global__ __launch_bounds__((Imp<EB, RT>::kThreads)) SKV_IMP_WAVES void importance_stats_kernel(
    const char* __restrict__ q_obs, const char* __restrict__ K_pool, int32_t T, int32_t N, int32_t G, int32_t kpb, float2* part,
    float2* __restrict__ rowstat, unsigned int* arrive) {
    (void)importance_stats<EB, RT>(q_obs, K_pool, T, N, G, kpb, part, rowstat, arrive, blockIdx.x, gridDim.x,
                                   (int64_t)blockIdx.z * gridDim.y + blockIdx.y);
}

// pass 2, a block: chunk `chunk` of `nchunks` of the Tp prefix keys (kpb each) of head h; alpha_h [L][Hkv][Tp], alpha [L][Tp].  Here the queries are
// the A operand: a lane gets half of the rows of one key, and the sum over the rows is in-lane but for one exchange.
template <int EB, int RT>
__device__ __forceinline__ void importance_colsum(const char* __restrict__ q_obs, const char* __restrict__ K_pool, int32_t T, int32_t N, int32_t G,
                                                  int32_t kpb, const float2* rowstat, float* alpha_h, float* __restrict__ alpha,
                                                  unsigned int* arrive, int chunk, int nchunks, int h, int Hkv, int l) {
    using P = Imp<EB, RT>;
    constexpr int kRowBytes = kHeadDim * EB, kRows = P::kRows;
    constexpr float kLog2e = 1.4426950408889634f;
    extern __shared__ __attribute__((aligned(16))) char sm_ring[];
    __shared__ float sm_col[2][P::RS][P::kStageKeys];
    __shared__ int sm_last;

    const int64_t lh = (int64_t)l * Hkv + h;                             // (layer, KV head)
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, r = lane & 31, g = lane >> 5;
    const int rs = w / P::KSP, ks = w % P::KSP;
    const int R = G * N, Tp = T - N;
    const char* Kh = K_pool + lh * T * kRowBytes;
    const int32_t base0 = chunk * kpb, cnt = min(kpb, Tp - base0), n = (cnt + P::kStageKeys - 1) / P::kStageKeys;
    KeyRing<EB, RT> keys(Kh, sm_ring, base0, Tp - 1, n);
    Frag<EB> qf[8];
    load_queries<EB>(qf, q_obs + lh * R * kRowBytes, R, 32 * rs);
    float2 st[16];                                                       // this lane's rows of the tile
#pragma unroll
    for (int i = 0; i < 16; ++i) st[i] = rowstat[lh * kRows + 32 * rs + tile_pos(i, g)];
    const float scale = kLog2e * rsqrtf((float)kHeadDim);
    const int row0 = 32 * ks + r;                                        // this lane's key in a stage
    float* dst = alpha_h + lh * Tp + base0;
    // sums over the wave's rows of its tile of stage s; with the rows on several waves they meet in LDS, and `put` adds and stores them
    // a barrier later
    auto sum_tile = [&](const f32x16& x, int s) {
        float p[2] = {0.f, 0.f};
#pragma unroll
        for (int i = 0; i < 16; ++i) p[i & 1] = fmaf(exp2_neg(fmaf(x[i], scale, -st[i].x)), st[i].y, p[i & 1]);      // prefix keys: at most 1
        const float v = sum_halves(p[0] + p[1]);
        if constexpr (P::RS == 1) {
            if (g == 0 && s * P::kStageKeys + row0 < cnt) st_agent(dst + s * P::kStageKeys + row0, v);
        } else {
            if (g == 0) sm_col[s & 1][rs][row0] = v;
        }
    };
    auto put = [&](int s) {
        if constexpr (P::RS > 1) {
            if (tid < P::kStageKeys) {
                float v = sm_col[s & 1][0][tid];
#pragma unroll
                for (int k = 1; k < P::RS; ++k) v += sm_col[s & 1][k][tid];
                if (s * P::kStageKeys + tid < cnt) st_agent(dst + s * P::kStageKeys + tid, v);
            }
        }
    };

    // the sums of a tile are taken while the matrix cores work on the next one
    f32x16 acc[2];
    tile_logits<EB, false>(acc[0], qf, keys.next(0), row0, g);
    for (int s = 1; s < n; s += 2) {
        const char* stage = keys.next(s);
        if (s > 1) put(s - 2);
        tile_logits<EB, false>(acc[1], qf, stage, row0, g);
        sum_tile(acc[0], s - 1);
        if (s + 1 < n) {
            stage = keys.next(s + 1);
            put(s - 1);
            tile_logits<EB, false>(acc[0], qf, stage, row0, g);
            sum_tile(acc[1], s);
        }
    }
    if (n & 1) sum_tile(acc[0], n - 1);
    else sum_tile(acc[1], n - 1);
    __syncthreads();
    if (n > 1) put(n - 2);
    put(n - 1);
    // ---- the last of the heads' blocks for these keys: their sum in ascending order ---------------------------------
    block_sync_after_stores();
    unsigned int* mine = arrive + (int64_t)l * nchunks + chunk;
    if (tid == 0) sm_last = __hip_atomic_fetch_add(mine, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (unsigned int)(Hkv - 1);
    __syncthreads();
    if (!sm_last) return;
    const float* src = alpha_h + (int64_t)l * Hkv * Tp + base0;
    for (int i = tid; i < cnt; i += P::kThreads) {
        float v = 0.f;
        for (int hh = 0; hh < Hkv; hh += 8) {
            float x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) x[u] = ld_agent(src + (int64_t)min(hh + u, Hkv - 1) * Tp + i);
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (hh + u < Hkv) v += x[u];
        }
        alpha[(int64_t)l * Tp + base0 + i] = v;
    }
    if (tid == 0) __hip_atomic_store(mine, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);            // for the next call
}

// grid (chunks, Hkv, L)
template <int EB, int RT>
__global__ __launch_bounds__((Imp<EB, RT>::kThreads)) SKV_IMP_WAVES void importance_colsum_kernel(
    const char* __restrict__ q_obs, const char* __restrict__ K_pool, int32_t T, int32_t N, int32_t G, int32_t kpb,
    const float2* __restrict__ rowstat, float* alpha_h, float* __restrict__ alpha, unsigned int* arrive) {
    importance_colsum<EB, RT>(q_obs, K_pool, T, N, G, kpb, rowstat, alpha_h, alpha, arrive, blockIdx.x, gridDim.x, blockIdx.y, gridDim.y, blockIdx.z);
}

// ------------------------------------------------------------------------------------------------
// Importance in one sweep over the keys, bf16, up to 128 rows.  The two passes read every key, multiply it and take its exp2 twice,
// because a row's normaliser is known only once all keys have been seen.  Here the exp2 values of a chunk of keys stay in the
// registers of the block that made them (64 a lane: half of the chip's registers) until the blocks that hold the other chunks of the
// (layer, head) have published their sums of every row.
//   Blocks of eight waves, two on a compute unit, as many as some whole heads have chunks: a block takes the same chunk of one head after another.
//   Per chunk:  logits of its keys, tile by tile on the matrix cores (the keys of the next chunk are requested as the places in LDS come free), exp2 of
//   a tile and the sums of its rows beside the next tile's logits, relative to a whole reference from the wave's first tile -> published ->
//   the blocks of the head combine a share of its rows each and publish 1 / sum -> column sums of the values held.
// A wave whose logits rise far above its references (kFar) in some tile moves them up and the values that it holds down.  (The chunk's logits taken from memory once
// more instead, with its own maxima, while all blocks of the head wait: with a key in every chunk 45 nats above the others 32768 keys of 128 rows 2680 -> 750 us,
// 64 rows 1460 -> 452, 32 rows 928 -> 378; every tile 45 nats above the one before it 1370, 656, 407; none far above: the same.  That code and the masks of the
// last keys lie behind the kernel's end: between the tiles 705, there 694, where the form without it took 699.)
// The exchange passes tagged words: nothing is cleared, drained or counted.  A block publishes its next chunk only after it has seen
// every row of the present one combined, so one place per block is enough.  While one block of a compute unit waits for the
// others, its neighbour computes.  Some of a block's waves request keys, others talk to the other blocks: a wave's loads return in
// order, and a polled word would come only after the keys requested before it.
// Waiting needs the blocks of a head to be resident together.  A block that has polled `limit` times, or sees that another gave up, marks the
// launch as failed and ends; the kernel behind the sweep, which otherwise adds up the heads, then does all of the work in two passes.
// Bound by HBM for 32 rows (a chunk is 1024 keys, 5.7 TB/s), by the exchange for 128 (256 keys): a block by itself takes 7.5 us for such a chunk, 2.5 until its
// exp2 values are there, 0.8 until its sums are published, 3.3 for two trips through memory, 0.9 for the column sums; two on a compute unit take 10.6 us each.
// us, 32 layers x 8 heads, two passes / waves of 32 rows that took the maximum of the whole chunk first, all exp2 after all logits, four waves a block / now:
// 32768 keys 812 / 815 / 680, 64 rows 713 / 515 / 442, 32 rows 727 / 417 / 382; 4096 keys 131 / 110 / 85, 64 rows 105 / 73 / 62, 32 rows 100 / 61 / 51.
// What the way there gave, 32768 keys of 128 rows: the chunk that holds the last keys masks its last tile only, the limits from LDS (every block of the head
// waited 1.5 us for it), and exp2 beside the matrix instructions 815 -> 720; waves of 16 rows, eight a block 730 -> 690; stages of 64 keys for every width
// (64 rows 490 -> 450).  Not kept: polls one instruction at a time (each waits for its own trip: 840), a row a wave to combine (many writers to a line of the
// combined words: 830), the next chunk's keys requested together behind the sums or the exchange (770, 790), priorities for all waves behind the
// logits (the same), heads confined to two of the chip's dies (the same).
// ------------------------------------------------------------------------------------------------
template <int RT> struct Sweep {                               // RT: 32-row tiles of the window's rows
    static constexpr int NW = 8, RS = 2 * RT, KSP = NW / RS;   // waves of a block: 16 rows each, KSP beside each other along the keys
    static constexpr int KT = 16;                              // 16-key tiles of a wave in a chunk, 4 registers each
    static constexpr int TPS = RT;                             // of these, in a stage of 64 keys
    static constexpr int SC = KT / TPS, NS = 4;                // stages of a chunk, stages that LDS holds
    static constexpr int kThreads = NW * kWave, kRows = 32 * RT;
    static constexpr int kStageKeys = 16 * KSP * TPS, kStageBytes = kStageKeys * kHeadDim * 2, kChunkKeys = kStageKeys * SC;
    static constexpr int kRingBytes = NS * kStageBytes;
    static constexpr int kPollers = 2, kStorers = 4, kLoaders = 4;     // waves 0, 1; 0 to 3; 4 to 7
    static constexpr int kLoads = kStageBytes / (kLoaders * 1024);     // load instructions of a loader per stage
    static_assert(RS * KSP == NW && kStorers + kLoaders == NW && SC % NS == 0 && NS * kLoads < 64, "a stage has one place in LDS, the load counter holds them all");
};

struct SweepArgs {
    const char* q_obs;
    const char* K_pool;
    float* alpha_h;              // [heads][Tp]
    unsigned long long* part;    // [blocks][rows] a chunk's sums
    unsigned long long* stat;    // [stat_heads][rows] 1 / sum of all chunks
    unsigned int* state;         // number of the heads so far, the last failed launch, the last launch, its blocks that are done
    int64_t part_words, stat_words;      // all there are
    int32_t T, N, G, nch, total, stat_heads, limit;
    int32_t heads_at_once;               // the grid is this many times nch blocks
};

struct MaxOp { __device__ static __forceinline__ float of(float a, float b) { return fmaxf(a, b); } };
struct AddOp { __device__ static __forceinline__ float of(float a, float b) { return a + b; } };
template <int CTRL> __device__ __forceinline__ int dpp_move(int x) { return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xf, 0xf, false); }
template <int CTRL> __device__ __forceinline__ float dpp_move(float x) { return __int_as_float(dpp_move<CTRL>(__float_as_int(x))); }
// x of the lane l ^ N, N = 16 or 32
template <int N> __device__ __forceinline__ int other_half(int x) {
    const auto s = N == 16 ? __builtin_amdgcn_permlane16_swap((uint32_t)x, (uint32_t)x, false, false)
                           : __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)x, false, false);
    return (int)(s[0] ^ s[1] ^ (uint32_t)x);
}
// over the 16 lanes of a row of lanes, in all of them
template <class Op> __device__ __forceinline__ float reduce_16(float x) {
    x = Op::of(x, dpp_move<0x128>(x));                                   // row_ror 8, 4, 2, 1
    x = Op::of(x, dpp_move<0x124>(x));
    x = Op::of(x, dpp_move<0x122>(x));
    return Op::of(x, dpp_move<0x121>(x));
}
// a + (a of lane l ^ N) in the lanes without bit N, b + (b of lane l ^ N) in the others; N = 16 or 32
template <int N> __device__ __forceinline__ float add_swap(float a, float b) {
    const auto s = N == 16 ? __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false)
                           : __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}
// A number m * 2^x, 1 <= m < 2, and the tag of the (layer, head) it belongs to in one 64-bit word: 24 bits, 17 of the exponent, 23 of m.
constexpr int kExpBias = 1 << 16, kExpNone = -kExpBias, kExpNan = kExpBias - 1;       // exponents that stand for zero and NaN
__device__ __forceinline__ unsigned long long tagged_number(float v, int exponent, uint32_t tag) {       // v * 2^exponent, v >= 0
    const int e = v != v ? kExpNan : v > 0.f ? exponent + __builtin_amdgcn_frexp_expf(v) - 1 : kExpNone;
    const uint32_t m = __float_as_uint(__builtin_amdgcn_frexp_mantf(v)) & 0x7fffffu;
    return ((unsigned long long)tag << 40) | ((unsigned long long)(uint32_t)(e + kExpBias) << 23) | m;
}
__device__ __forceinline__ uint32_t number_tag(unsigned long long w) { return (uint32_t)(w >> 40); }
__device__ __forceinline__ int number_exp(unsigned long long w) { return (int)((uint32_t)(w >> 23) & 0x1ffffu) - kExpBias; }
__device__ __forceinline__ float number_mant(unsigned long long w) {
    const int e = number_exp(w);
    return e == kExpNone ? 0.f : e == kExpNan ? NAN : __uint_as_float(0x3f800000u | ((uint32_t)w & 0x7fffffu));
}

// A block's stages in LDS, across its chunks: stage k of a chunk at place k % NS, filled again (with stage k + NS, of the next chunk at the end) when
// every wave has read it.
template <int RT>
struct SweepStages {
    using P = Sweep<RT>;
    static constexpr int kRowBytes = kHeadDim * 2, kPieces = kRowBytes / 16, kRows = kWave / kPieces;      // rows per instruction
    int loader;               // which of the loading waves, negative: none
    uint32_t lds;             // where the ring begins
    __device__ __forceinline__ SweepStages(char* ring, int loader_) : loader(loader_) {
        lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)ring;
    }
    // Stage k (compile time) of the chunk whose first key is `src`, `keys` of the head's keys from there on; a loader takes its share of the rows, four to
    // an instruction; piece p of row r lands at piece p ^ (r % 16).
    __device__ __forceinline__ void request(const char* src, int keys, int k) const {
        static_assert(kRows * P::kLoads % 16 == 0, "a loader begins at a multiple of 16 rows");
        if (loader < 0) return;
        int lane = threadIdx.x & 63;
        asm volatile("" : "+v"(lane));                                   // offsets made here, not kept in registers
        const int row = lane / kPieces, at = loader * P::kLoads * 1024;
        const uint32_t piece = (uint32_t)(16 * ((lane % kPieces) ^ row));
        if (keys >= (k + 1) * P::kStageKeys) {
            const uint32_t first = (uint32_t)(row * kRowBytes) + piece;
#pragma unroll
            for (int i = 0; i < P::kLoads; ++i)
                load_lds_stream_at(src + (k * P::kStageBytes + 1024 * i) + at, first ^ (uint32_t)(16 * (kRows * i & 15)), lds + (uint32_t)(k % P::NS * P::kStageBytes + 1024 * i + at));
        } else {                                                         // keys past the last: that one again
#pragma unroll
            for (int i = 0; i < P::kLoads; ++i)
                load_lds_stream_at(src, (uint32_t)(min(k * P::kStageKeys + kRows * (P::kLoads * loader + i) + row, keys - 1) * kRowBytes) + (piece ^ (uint32_t)(16 * (kRows * i & 15))),
                                   lds + (uint32_t)(k % P::NS * P::kStageBytes + 1024 * i + at));
        }
    }
    // stage k has landed: at most this many stages were requested after it
    template <int AFTER> __device__ __forceinline__ void landed() const {
        if (loader >= 0) wait_loads<AFTER * P::kLoads>();
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    }
};

// Words of other blocks, asked for until they carry the tag.
struct Waiter {
    const unsigned int* failed;
    unsigned int failed_if;
    int limit;
    bool ok;
    // word u of a lane: base[at(u, lane)], where need(u, lane)
    template <int U, class At, class Need>
    __device__ __forceinline__ void get(const unsigned long long* base, At at, Need need, uint32_t tag, unsigned long long (&v)[U]) {
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = 0;
        for (int n = 0; ok; ++n) {
            bool all = true;
            int lane = threadIdx.x & 63;
            asm volatile("" : "+v"(lane));                               // addresses made in every round, not kept in registers
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = ld_tagged(base + at(u, lane));
#pragma unroll
            for (int u = 0; u < U; ++u) all = all && (!need(u, lane) || number_tag(v[u]) == tag);
            if (__all(all)) return;
            if (n >= limit || ((n & 31) == 31 && ld_agent(failed) == failed_if)) ok = false;
        }
    }
};

template <int RT>
__global__ __launch_bounds__((Sweep<RT>::kThreads)) __attribute__((amdgpu_waves_per_eu(kSweepPerCu * Sweep<RT>::NW / 4, kSweepPerCu * Sweep<RT>::NW / 4))) void importance_sweep_kernel(SweepArgs x) {
    using P = Sweep<RT>;
    constexpr int kRowBytes = kHeadDim * 2, kRows = P::kRows;
    constexpr float kLog2e = 1.4426950408889634f, kAbove = 4.f, kFar = 24.f;
    // Reference of a row that has shown a wave nothing: below every other, so that it is not the largest of a block's waves, and the first finite logit that comes
    // to it rises far above it.  exp2(-infinity + 3.4e38) = 0.
    constexpr float kNothing = -3.402823466e38f;
    constexpr float kLeast = -4.f * kExpBias;                            // a reference as low as this next to any that a word holds: the values weigh nothing
    extern __shared__ __attribute__((aligned(16))) char sm_ring[];
    __shared__ __attribute__((aligned(16))) float sm_m[P::KSP][kRows], sm_l[P::KSP][kRows];
    __shared__ float sm_col[P::RS][P::kChunkKeys];
    __shared__ int sm_ok[P::kPollers], sm_last;
    __shared__ __attribute__((aligned(16))) int32_t sm_limit[kRows];     // last key that a row sees

    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // what depends on the lane is made where it is used: kept for the whole loop it would take registers from the chunk's values
    int lane_of = threadIdx.x & 63;
    auto this_lane = [&]() { int l = lane_of; asm volatile("" : "+v"(l)); return l; };
    const int rs = w / P::KSP, ks = w % P::KSP;
    const int R = x.G * x.N, Tp = x.T - x.N, nblk = gridDim.x;
    const int loader = w - P::kStorers;                                  // negative: none
    const float scale = kLog2e * rsqrtf((float)kHeadDim);
    const unsigned int epoch = ld_agent(x.state);
    int lh = blockIdx.x / x.nch, chunk = blockIdx.x - lh * x.nch;
    auto chunk_src = [&](int head, int ch) { return x.K_pool + ((int64_t)head * x.T + ch * P::kChunkKeys) * kRowBytes; };
    for (int row = threadIdx.x; row < kRows; row += P::kThreads) sm_limit[row] = min(Tp + row % x.N, x.T - 1);      // (the first stage's barrier follows)
    const SweepStages<RT> stages(sm_ring, loader);
#pragma unroll
    for (int k = 0; k < P::NS; ++k) stages.request(chunk_src(lh, chunk), x.T - chunk * P::kChunkKeys, k);
    // Lane (t16, qd) = (lane % 16, lane / 16).  Queries are the A operand of v_mfma_f32_16x16x32_bf16, keys the B operand, the 16 bytes 4 s + qd of a row for
    // step s; element j of a tile is (row 4 qd + j, key t16).
    uint4 qf[4];
    auto load_q = [&](int head) {
        const int lane = this_lane(), t16 = lane & 15, qd = lane >> 4;
        // rows past the last repeat it: they get a factor of zero
        const char* q = x.q_obs + ((int64_t)head * R + min(16 * rs + t16, R - 1)) * kRowBytes + 16 * qd;
#pragma unroll
        for (int st = 0; st < 4; ++st) qf[st] = *reinterpret_cast<const uint4*>(q + 64 * st);
    };
    load_q(lh);

    for (int left = ((int)x.total - (int)blockIdx.x + nblk - 1) / nblk - 1; left >= 0; --left) {         // chunks after this one
        const int32_t base0 = chunk * P::kChunkKeys;
        const uint32_t tag = epoch + 1 + (uint32_t)lh;
        const int lh_next = lh + x.heads_at_once;
        const char *src = chunk_src(lh, chunk), *src_next = chunk_src(lh_next, chunk);
        const int keys = x.T - base0;
        f32x4 acc[P::KT];
        float ref[4], sum[4];
        const int lane = this_lane(), tid = lane + w * kWave, t16 = lane & 15, qd = lane >> 4;
        const int row_of = 16 * rs + 4 * qd;                             // row of a tile's first element
        // keys that a row does not see  (here and below: inlined though it is rarely run, or the tiles would not stay in registers)
        auto mask_tile = [&](f32x4& v, int t) __attribute__((always_inline)) {
            const int key = base0 + 16 * (P::KSP * t + ks) + t16;
            const int4 limit = *reinterpret_cast<const int4*>(sm_limit + row_of);
            if (key > limit.x) v[0] = -INFINITY;
            if (key > limit.y) v[1] = -INFINITY;
            if (key > limit.z) v[2] = -INFINITY;
            if (key > limit.w) v[3] = -INFINITY;
        };
        // whole references, kAbove over the largest logit of the wave's first tile
        auto set_references = [&]() {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float top = rintf(reduce_16<MaxOp>(acc[0][j]) * scale) + kAbove;
                ref[j] = top > -INFINITY ? top : kNothing;
                sum[j] = 0.f;
            }
        };
        // Some row's logits in tile t rise kFar and more above its reference, which moves up to them; the values in registers move down with it (an exact factor).
        auto raise_references = [&](int t) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float top = fmaxf(rintf(reduce_16<MaxOp>(acc[t][j]) * scale) + kAbove, ref[j]);
                const float f = exp2_neg(ref[j] < top ? ref[j] - top : 0.f);
                ref[j] = top;
                sum[j] = sum[j] == INFINITY ? 0.f : sum[j] * f;            // (of logits that a float does not hold: see below)
#pragma unroll
                for (int u = 0; u < P::KT; ++u)
                    if (u < t) acc[u][j] = acc[u][j] == INFINITY ? 0.f : acc[u][j] * f;
            }
        };
        // the exp2 values of tile t and its part of the sums, here and not behind a later barrier
        auto exps = [&](int t) {
            f32x4 v = acc[t];
            float x0 = fmaf(v[0], scale, -ref[0]), x1 = fmaf(v[1], scale, -ref[1]), x2 = fmaf(v[2], scale, -ref[2]), x3 = fmaf(v[3], scale, -ref[3]);
            if (t > 0 && __builtin_expect(__any(fmaxf(fmaxf(x0, x1), fmaxf(x2, x3)) > kFar), 0)) {
                raise_references(t);
                x0 = fmaf(v[0], scale, -ref[0]); x1 = fmaf(v[1], scale, -ref[1]); x2 = fmaf(v[2], scale, -ref[2]); x3 = fmaf(v[3], scale, -ref[3]);
            }
            acc[t] = f32x4{exp2_neg(x0), exp2_neg(x1), exp2_neg(x2), exp2_neg(x3)};
#pragma unroll
            for (int j = 0; j < 4; ++j) sum[j] += acc[t][j];
            asm volatile("" : "+v"(sum[0]), "+v"(sum[1]), "+v"(sum[2]), "+v"(sum[3]));
        };
#pragma unroll
        for (int k = 0; k < P::SC; ++k) {
            // one stage was requested after each that has been read, but the last of a chunk already behind the barrier after it
            if (k == 0) stages.template landed<P::NS - 1>();
            else if (k + P::NS - 2 < P::SC || left > 0) stages.template landed<P::NS - 2>();
            else stages.template landed<0>();
            if (k > 0) {
                if (k - 1 + P::NS < P::SC) stages.request(src, keys, k - 1 + P::NS);
                else if (left > 0) stages.request(src_next, keys, k - 1 + P::NS - P::SC);
            }
            const char* stage = sm_ring + k % P::NS * P::kStageBytes;
            // a fragment of the next tile is read behind the matrix instruction that used its registers
            uint4 kf[4];
            auto key_frag = [&](int u, int st) {
                const int row = 16 * (P::KSP * u + ks) + t16;
                kf[st] = *reinterpret_cast<const uint4*>(stage + row * kRowBytes + 16 * ((4 * st + qd) ^ t16));
            };
#pragma unroll
            for (int st = 0; st < 4; ++st) key_frag(0, st);
#pragma unroll
            for (int u = 0; u < P::TPS; ++u) {
                const int t = k * P::TPS + u;
                f32x4 c = {};
#pragma unroll
                for (int st = 0; st < 4; ++st) {
                    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, qf[st]), __builtin_bit_cast(bf16x8, kf[st]), c, 0, 0, 0);
                    if (u + 1 < P::TPS) key_frag(u + 1, st);
                }
                if (t == 1) set_references();
                if (t >= 1) exps(t - 1);
                acc[t] = c;
                if (__builtin_expect(base0 + 16 * P::KSP * (t + 1) > Tp, 0)) mask_tile(acc[t], t);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        exps(P::KT - 1);
#pragma unroll
        for (int j = 0; j < 4; ++j) sum[j] = reduce_16<AddOp>(sum[j]);
        // Logits that a float does not hold (from 2^31 on) can lie 2^128 above the reference that is rounded from them.  Such a row's values weigh nothing next to
        // a wave's that the words hold; where there is none, the launch is left to the passes.
        if (__builtin_expect(__any(fmaxf(fmaxf(sum[0], sum[1]), fmaxf(sum[2], sum[3])) == INFINITY), 0)) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool nothing = sum[j] == INFINITY;
                sum[j] = nothing ? 0.f : sum[j];
#pragma unroll
                for (int t = 0; t < P::KT; ++t) acc[t][j] = nothing ? 0.f : acc[t][j];
            }
        }
        if (t16 == 0) {
            *reinterpret_cast<float4*>(&sm_m[ks][row_of]) = make_float4(ref[0], ref[1], ref[2], ref[3]);
            *reinterpret_cast<float4*>(&sm_l[ks][row_of]) = make_float4(sum[0], sum[1], sum[2], sum[3]);
        }
        __syncthreads();
        if (left > 0) stages.request(src_next, keys, P::NS - 1);
        if (w < P::kPollers) {
            __builtin_amdgcn_s_setprio(3);
            // published: the sum of every row; four rows of a chunk side by side, then those of the next chunk
            unsigned long long* part = x.part + ((int64_t)blockIdx.x - chunk) * kRows;
            Waiter wait{x.state + 1, epoch + 1, x.limit, true};
            for (int row = tid; row < kRows; row += P::kPollers * kWave) {
                float m = sm_m[0][row];
#pragma unroll
                for (int k = 1; k < P::KSP; ++k) m = fmaxf(m, sm_m[k][row]);
                float l = 0.f;
#pragma unroll
                for (int k = 0; k < P::KSP; ++k) l += ldexpf(sm_l[k][row], (int)fmaxf(sm_m[k][row] - m, -512.f));
                const bool fits = fabsf(m) < (float)(kExpBias - 256);                        // within the words' exponents
                if (l == l && m > kNothing && !fits) wait.ok = false;
                __hip_atomic_store(part + ((row >> 2) * x.nch + chunk) * 4 + (row & 3), tagged_number(l, l > 0.f && fits ? (int)m : 0, tag), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            }
            wait.ok = __all(wait.ok);
            // combined: four rows a wave, 16 lanes to a row, U words of a lane asked for together
            unsigned long long* stat = x.stat + (int64_t)(lh % x.stat_heads) * kRows;
            auto combine = [&](auto words) {
                constexpr int U = decltype(words)::value;
                for (int row0 = 4 * (chunk * P::kPollers + w); row0 < kRows; row0 += 4 * P::kPollers * x.nch) {
                    const int row = row0 + (lane & 3);
                    int X = kExpNone;
                    float L = 0.f;
                    for (int c0 = 0; c0 < x.nch; c0 += 16 * U) {
                        unsigned long long v[U];
                        auto need = [&](int u, int l) { return c0 + 16 * u + (l >> 2) < x.nch; };
                        wait.get<U>(part, [&](int u, int l) { return (uint32_t)(row0 * x.nch + min(c0 + 16 * u + (l >> 2), x.nch - 1) * 4 + (l & 3)); }, need, tag, v);
                        // Mostly every number is one that a float holds, and so is their sum: its bits are then those of the word, but for the bias.
                        bool plain = x.nch <= 16 * U;
#pragma unroll
                        for (int u = 0; u < U; ++u) plain = plain && (uint32_t)(number_exp(v[u]) + 100) <= 200u;
                        if (__all(plain)) {
                            X = 0;
#pragma unroll
                            for (int u = 0; u < U; ++u) L += need(u, lane) ? __uint_as_float((uint32_t)v[u] + (127u << 23)) : 0.f;
                        } else {
                            int top = X;
#pragma unroll
                            for (int u = 0; u < U; ++u) top = max(top, need(u, lane) ? number_exp(v[u]) : kExpNone);
                            L = ldexpf(L, max(X - top, -512));
#pragma unroll
                            for (int u = 0; u < U; ++u) L += need(u, lane) ? ldexpf(number_mant(v[u]), max(number_exp(v[u]) - top, -512)) : 0.f;
                            X = top;
                        }
                    }
                    int top = max(X, dpp_move<0x124>(X));                // row_ror 4, 8: the lanes of the row
                    top = max(top, dpp_move<0x128>(top));
                    top = max(top, other_half<16>(top));
                    top = max(top, other_half<32>(top));
                    L = ldexpf(L, max(X - top, -512));
                    L += dpp_move<0x124>(L);
                    L += dpp_move<0x128>(L);
                    L = sum_rows16(L);
                    L = sum_halves(L);
                    if (wait.ok && lane < 4)
                        __hip_atomic_store(stat + row, tagged_number(row < R && L > 0.f ? 1.f / L : 0.f, -top, tag), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            };
            if (x.nch <= 16) combine(std::integral_constant<int, 1>{});
            else if (x.nch <= 64) combine(std::integral_constant<int, 4>{});
            else combine(std::integral_constant<int, 8>{});
            // all rows: the factor that makes this chunk's values probabilities
            for (int row = tid; row - lane < kRows; row += P::kPollers * kWave) {
                unsigned long long v[1];
                wait.get<1>(stat, [&](int, int l) { return (uint32_t)min(row - lane + l, kRows - 1); }, [&](int, int) { return row < kRows; }, tag, v);
                if (row < kRows) {
#pragma unroll
                    for (int k = 0; k < P::KSP; ++k)
                        sm_l[k][row] = ldexpf(number_mant(v[0]), min(max((int)fmaxf(sm_m[k][row], kLeast) + number_exp(v[0]), -512), 512));
                }
            }
            if (lane == 0) sm_ok[w] = wait.ok;
            __builtin_amdgcn_s_setprio(0);
        }
        load_q(left > 0 ? lh_next : lh);                                 // (always: until here no register holds queries)
        __syncthreads();
        bool ok = true;
#pragma unroll
        for (int i = 0; i < P::kPollers; ++i) ok = ok && sm_ok[i];
        if (!ok) {                                                       // the passes that follow do it
            if (tid == 0) st_agent(x.state + 1, epoch + 1);
            break;
        }
        __builtin_amdgcn_sched_barrier(0);
        {
            const float4 f = *reinterpret_cast<const float4*>(&sm_l[ks][row_of]);
#pragma unroll
            for (int t = 0; t < P::KT; t += 4) {
                float y[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) y[u] = fmaf(acc[t + u][3], f.w, fmaf(acc[t + u][2], f.z, fmaf(acc[t + u][1], f.y, acc[t + u][0] * f.x)));
                // the four lanes of a key, for four tiles together: lanes qd end with tile t + qd
                const float z0 = add_swap<32>(y[0], y[2]), z1 = add_swap<32>(y[1], y[3]);
                sm_col[rs][16 * (P::KSP * (t + qd) + ks) + t16] = add_swap<16>(z0, z1);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        __syncthreads();
        if (loader < 0) {
            float* dst = x.alpha_h + (int64_t)lh * Tp + base0;
            for (int i = tid; i < P::kChunkKeys && base0 + i < Tp; i += P::kStorers * kWave) {
                float v = sm_col[0][i];
#pragma unroll
                for (int k = 1; k < P::RS; ++k) v += sm_col[k][i];
                dst[i] = v;
            }
        }
        lh = lh_next;
        asm volatile("" : "+s"(chunk));                                  // what depends on it is made in every round (made once: 4096 keys of 32 rows 59.4 -> 59.8 us)
    }
    wait_loads<0>();                                                     // nothing lands in LDS after the block's end
    // The last block to end moves the numbers on.  Before a tag comes again the words are cleared.  (Not in the place of sm_ok: behind the
    // `break` there is no barrier, and a wave may still be reading that.)
    if (threadIdx.x == 0)
        sm_last = __hip_atomic_fetch_add(x.state + 3, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (unsigned int)(nblk - 1);
    __syncthreads();
    if (!sm_last) return;
    const unsigned int heads = (unsigned int)(x.total / x.nch), next = epoch + heads;
    const bool again = next + heads > kSweepTags;
    if (threadIdx.x == 0) {
        st_agent(x.state + 2, epoch + 1);
        st_agent(x.state + 3, 0u);
        st_agent(x.state, again ? 0u : next);
    }
    if (again) {
        for (int64_t i = threadIdx.x; i < x.part_words; i += P::kThreads) __hip_atomic_store(x.part + i, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        for (int64_t i = threadIdx.x; i < x.stat_words; i += P::kThreads) __hip_atomic_store(x.stat + i, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// Behind the sweep, grid (chunks of pass 1, Hkv, L): the heads added up, or, if it failed, all of the work: pass 1, and pass 2 of a (layer, head) by
// its last block.
template <int RT>
__global__ __launch_bounds__((Imp<2, RT>::kThreads)) void importance_finish_kernel(
    const char* __restrict__ q_obs, const char* __restrict__ K_pool, int32_t T, int32_t N, int32_t G, int32_t kpb, float2* part, float2* rowstat,
    unsigned int* arrive, float* alpha_h, float* alpha, const unsigned int* state) {
    if (ld_agent(state + 1) != ld_agent(state + 2)) {
        add_heads(alpha_h, alpha, T - N);
        return;
    }
    const int h = blockIdx.y, Hkv = gridDim.y, l = blockIdx.z;
    if (!importance_stats<2, RT>(q_obs, K_pool, T, N, G, kpb, part, rowstat, arrive, blockIdx.x, gridDim.x, (int64_t)l * Hkv + h)) return;
    block_sync_after_stores();
    const int n = (T - N + kpb - 1) / kpb;
    for (int chunk = 0; chunk < n; ++chunk) {
        importance_colsum<2, RT>(q_obs, K_pool, T, N, G, kpb, rowstat, alpha_h, alpha, arrive + (int64_t)gridDim.z * Hkv, chunk, n, h, Hkv, l);
        __syncthreads();
    }
}

// Keys per block, in units of 128: the number that gives the least rounds x (units + 2), two units being about what a block's
// start and end take.
constexpr int kImpUnit = 128;
static int importance_rows(int rows) { return rows <= 32 ? 32 : rows <= 64 ? 64 : rows <= 128 ? 128 : 256; }
static int importance_keys_per_block(const Ctx* c, int32_t T, int32_t N) {
    const int per_cu = c->d.kv_dtype != SKV_BF16 ? Imp<4, 8>::kPerCu : importance_rows(c->G * N) == 256 ? Imp<2, 8>::kPerCu : Imp<2, 4>::kPerCu;
    static_assert(Imp<4, 1>::kPerCu == Imp<4, 8>::kPerCu && Imp<2, 1>::kPerCu == Imp<2, 4>::kPerCu && Imp<2, 2>::kPerCu == Imp<2, 4>::kPerCu, "by type and 256 rows");
    const int64_t heads = (int64_t)c->d.n_layers * c->d.n_kv_heads, resident = (int64_t)c->n_cu * per_cu;
    const int64_t units = (T + kImpUnit - 1) / kImpUnit;
    int64_t best = 0, best_cost = 0;
    for (int64_t per = 1; per <= 256 && per <= units; ++per) {
        const int64_t rounds = (heads * ((units + per - 1) / per) + resident - 1) / resident, cost = rounds * (per + 2);
        if (best == 0 || cost < best_cost) { best = per; best_cost = cost; }
    }
    return kImpUnit * (int)best;
}

// LDS above 64 KB needs the opt-in once per kernel
template <class F> static hipError_t raise_lds(F kernel, int bytes, std::atomic<bool>& raised) {
    if (raised.load(std::memory_order_acquire)) return hipSuccess;
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e == hipSuccess) raised.store(true, std::memory_order_release);
    return e;
}

static int sweep_blocks(const Ctx* c) { return min(kSweepPerCu * c->n_cu, kSweepMaxBlocks); }

// Where the sweep is the faster form (us, two passes / one sweep): the chunks of a head fit the chip at once, and the launch has chunks enough (96; 64
// chunks: 512 keys a chunk 14.8 / 15.4, 1024: 17.5 / 16.9, 256: 15.7 / 14.6; 96 chunks of 256 keys 16.8 / 13.9, 20.2 / 16.0 with 192).
// 32 and 64 rows gain at every length (131072 keys, 8 layers: 737 / 390, 715 / 538).  128 rows gain up to 64 chunks a head (1024 keys of 32 layers 44 / 34.5, of 8 layers
// 22.6 / 17.6; 9465 keys, 32, 16, 8, 4 layers: 250 / 227, 136 / 118, 77 / 63, 48 / 37; 14585 keys, 57 chunks, whole heads fill 89 % of the chip's blocks: 373 / 364,
// 200 / 185, 112 / 96, 63 / 51), and up to 128, whose words a wave combines in one round of loads, as long as whole heads fill the blocks: 93 % of them in launches of more
// than 64 heads, where the start and end of the two passes weigh less, 84 % in smaller ones.  16, 8, 4 layers of 8 heads: 18937 keys (74 chunks, 87 %) 254 / 258, 142 / 129,
// 75 / 72; 20473 (94 %) 270 / 262, 151 / 133, 79 / 73; 22521 (86 %) 296 / 308, 163 / 154, 85 / 81; 23545 (90 %) 305 / 315, 172 / 158, 86 / 82; 26105 (99.6 %) 338 / 325, 181 / 166,
// 94 / 84; 26361 (103 chunks, 80 %) 339 / 377, 189 / 186, 98 / 95; 27641 (84.4 %) 355 / 382, 190 / 197, 102 / 97; 29689 (91 %) 378 / 393, 210 / 192, 111 / 99; 30713 (94 %) 391 / 391,
// 210 / 197, 112 / 102; 32761 (100 %) 416 / 392, 226 / 199, 120 / 104; 32 layers, 74 chunks 487 / 495, 80 515 / 507, 85 547 / 507.  Keys without structure draw more power: 20473 keys
// 250 / 267, 136 / 127, 74 / 68; 26361 323 / 374, 170 / 185, 89 / 91; 32761 397 / 390, 203 / 197, 108 / 99.  More chunks: 40000 keys, 16 layers 499 / 538, 65536 807 / 848.
bool importance_may_sweep(const skv_desc& d) {
    const int64_t heads = (int64_t)d.n_layers * d.n_kv_heads;
    static_assert(Sweep<1>::kChunkKeys >= kSweepMinChunk && Sweep<2>::kChunkKeys >= kSweepMinChunk && Sweep<4>::kChunkKeys >= kSweepMinChunk && Sweep<4>::kRows <= kSweepMaxRows, "");
    return d.kv_dtype == SKV_BF16 && heads <= kSweepMostHeads && heads * ((d.max_tokens + kSweepMinChunk - 1) / kSweepMinChunk) >= kSweepMinChunks;
}

template <int RT>
static bool importance_sweeps(const Ctx* c, int32_t T) {
    using P = Sweep<RT>;
    const int64_t heads = (int64_t)c->d.n_layers * c->d.n_kv_heads, nch = (T + P::kChunkKeys - 1) / P::kChunkKeys, most = sweep_blocks(c);
    if (!c->single_launch || !c->imp_part || nch > most || heads > kSweepMostHeads || heads * nch > (1 << 30) || heads * nch < kSweepMinChunks) return false;
    return RT < 4 || nch <= 64 || (nch <= 128 && most / nch * nch * 100 >= (heads > 64 ? 93 : 84) * most);
}

template <int RT>
static hipError_t launch_sweep(Ctx* c, const char* q_obs, const char* K_pool, int32_t T, int32_t N, float* alpha, float2* part, float2* rowstat,
                               float* alpha_h) {
    using P = Sweep<RT>;
    static std::atomic<bool> raised{false}, raised_finish{false};
    hipError_t e = raise_lds(&importance_sweep_kernel<RT>, P::kRingBytes, raised);
    if (e == hipSuccess) e = raise_lds(&importance_finish_kernel<RT>, Imp<2, RT>::kRingBytes, raised_finish);
    if (e != hipSuccess) return e;
    const int Hkv = c->d.n_kv_heads, L = c->d.n_layers, kpb = importance_keys_per_block(c, T, N);
    SweepArgs x;
    x.q_obs = q_obs;
    x.K_pool = K_pool;
    x.alpha_h = alpha_h;
    x.part = c->imp_part;
    x.stat = c->imp_stat;
    x.state = c->imp_state;
    x.part_words = c->imp_part_words;
    x.stat_words = c->imp_stat_words;
    x.T = T;
    x.N = N;
    x.G = c->G;
    x.nch = (T + P::kChunkKeys - 1) / P::kChunkKeys;
    x.total = L * Hkv * x.nch;
    x.stat_heads = min(L * Hkv, kSweepStatHeads);
    x.limit = min(c->wait_limit, kSweepWaitLimit);
    x.heads_at_once = min(sweep_blocks(c) / x.nch, L * Hkv);               // whole heads: else every head's blocks wait for those of the next ones
    const int blocks = x.heads_at_once * x.nch;
    hipLaunchKernelGGL((importance_sweep_kernel<RT>), dim3(blocks), dim3(P::kThreads), P::kRingBytes, c->stream, x);
    hipLaunchKernelGGL((importance_finish_kernel<RT>), dim3((T + kpb - 1) / kpb, Hkv, L), dim3(Imp<2, RT>::kThreads), (Imp<2, RT>::kRingBytes), c->stream,
                       q_obs, K_pool, T, N, c->G, kpb, part, rowstat, c->imp_arrive, alpha_h, alpha, c->imp_state);
    return hipGetLastError();
}

template <int EB, int RT>
static hipError_t launch_importance_rt(Ctx* c, const char* q_obs, const char* K_pool, int32_t T, int32_t N, float* alpha, float2* part,
                                       float2* rowstat, float* alpha_h) {
    using P = Imp<EB, RT>;
    if constexpr (EB == 2 && RT <= 4)
        if (importance_sweeps<RT>(c, T)) return launch_sweep<RT>(c, q_obs, K_pool, T, N, alpha, part, rowstat, alpha_h);
    const int Hkv = c->d.n_kv_heads, L = c->d.n_layers, G = c->G, Tp = T - N, kpb = importance_keys_per_block(c, T, N);
    constexpr int lds = P::kRingBytes;
    static std::atomic<bool> raised_stats{false}, raised_colsum{false};
    hipError_t e = raise_lds(&importance_stats_kernel<EB, RT>, lds, raised_stats);
    if (e == hipSuccess) e = raise_lds(&importance_colsum_kernel<EB, RT>, lds, raised_colsum);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((importance_stats_kernel<EB, RT>), dim3((T + kpb - 1) / kpb, Hkv, L), dim3(P::kThreads), lds, c->stream, q_obs,
                       K_pool, T, N, G, kpb, part, rowstat, c->imp_arrive);
    hipLaunchKernelGGL((importance_colsum_kernel<EB, RT>), dim3((Tp + kpb - 1) / kpb, Hkv, L), dim3(P::kThreads), lds, c->stream, q_obs,
                       K_pool, T, N, G, kpb, rowstat, alpha_h, alpha, c->imp_arrive + (int64_t)L * Hkv);
    return hipGetLastError();
}

template <int EB>
static hipError_t launch_importance_eb(Ctx* c, const char* q_obs, const char* K_pool, int32_t T, int32_t N, float* alpha, float2* part,
                                       float2* rowstat, float* alpha_h) {
    const int R = c->G * N;
    if (R <= 32) return launch_importance_rt<EB, 1>(c, q_obs, K_pool, T, N, alpha, part, rowstat, alpha_h);
    if (R <= 64) return launch_importance_rt<EB, 2>(c, q_obs, K_pool, T, N, alpha, part, rowstat, alpha_h);
    if (R <= 128) return launch_importance_rt<EB, 4>(c, q_obs, K_pool, T, N, alpha, part, rowstat, alpha_h);
    if (R <= 256) return launch_importance_rt<EB, 8>(c, q_obs, K_pool, T, N, alpha, part, rowstat, alpha_h);
    return hipErrorInvalidValue;
}

static int64_t importance_chunks(const Ctx* c, int32_t T, int32_t N) {
    const int per = importance_keys_per_block(c, T, N);
    return (T + per - 1) / per;
}

// arrival counters of both passes: one per (layer, head), one per (layer, block of keys): at most a block for every unit of max_tokens
int64_t importance_counters(const skv_desc& d) {
    return (int64_t)d.n_layers * (d.n_kv_heads + (d.max_tokens + kImpUnit - 1) / kImpUnit);
}

// work = part [L][Hkv][chunks][rows][2] | rowstat [L][Hkv][rows][2] | alpha_h [L][Hkv][Tp], floats
int64_t importance_work_bytes(const Ctx* c, int32_t T, int32_t N) {
    const int64_t rows = importance_rows(c->G * N), LH = (int64_t)c->d.n_layers * c->d.n_kv_heads;
    return (LH * importance_chunks(c, T, N) * rows * 2 + LH * rows * 2 + LH * (int64_t)(T - N)) * (int64_t)sizeof(float);
}

// Two launches cover all layers: the rows' statistics, and the column sums with them.
hipError_t launch_importance(Ctx* c, const void* q_obs, const void* K_pool, int32_t T, int32_t N, float* alpha, void* work) {
    const int64_t rows = importance_rows(c->G * N), LH = (int64_t)c->d.n_layers * c->d.n_kv_heads;
    float2* part = (float2*)work;
    float2* rowstat = part + LH * importance_chunks(c, T, N) * rows;
    float* alpha_h = (float*)(rowstat + LH * rows);
    return c->d.kv_dtype == SKV_BF16
               ? launch_importance_eb<2>(c, (const char*)q_obs, (const char*)K_pool, T, N, alpha, part, rowstat, alpha_h)
               : launch_importance_eb<4>(c, (const char*)q_obs, (const char*)K_pool, T, N, alpha, part, rowstat, alpha_h);
}

// ------------------------------------------------------------------------------------------------
// Retention.  One 1024-thread block per layer: radix select (11 + 11 + 10 bits of the order-preserving
// key) of the k-th largest importance, tokens with equal importance by lower position, compaction of
// the kept positions in ascending order, then the retained buckets: kept tokens of one bucket are
// consecutive in keep_idx (positions ascend, bucket ids do not decrease), so ret_off[s] is the index of
// the first kept token whose bucket id is >= s.
// Bound by latency and by what one compute unit can load and count.  A wave owns consecutive tokens, a lane every 64th of them:
// whole lines per load, and ranks within a wave by ballots.  (A thread with 32 consecutive tokens made every load
// instruction touch 64 lines: 32 layers of 32768 tokens 47 us.)
// ------------------------------------------------------------------------------------------------
struct RetainShared {
    uint32_t hist[2048];
    uint32_t wave_tot[8][kBlockWaves];
    int32_t res[3][4];
};

template <int kRetainKreg>
__global__ __launch_bounds__(kBlockThreads) void retain_kernel(const float* __restrict__ alpha_all, int32_t Tp, int32_t k,
                                                               const int32_t* __restrict__ seg_id, int32_t S,
                                                               int32_t* __restrict__ keep_all, int32_t keep_stride,
                                                               int32_t* __restrict__ n_keep, int32_t* __restrict__ ret_off_all,
                                                               int32_t* __restrict__ ret_len_all) {
    __shared__ RetainShared sh;
    const int l = blockIdx.x, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const float* alpha = alpha_all + (int64_t)l * Tp;
    int32_t* keep = keep_all + (int64_t)l * keep_stride;
    int32_t* ret_off = ret_off_all + (int64_t)l * (S + 1);
    int32_t* ret_len = ret_len_all + (int64_t)l * S;
    const int32_t need = max(min(k, Tp), 0);
    if (tid == 0) n_keep[l] = need;
    if (need == 0) {
        for (int s = tid; s <= S; s += kBlockThreads) ret_off[s] = 0;
        for (int s = tid; s < S; s += kBlockThreads) ret_len[s] = 0;
        return;
    }
    const int kpt = (Tp + kBlockThreads - 1) / kBlockThreads;
    const int32_t i0 = w * kpt * kWave + lane;                         // this lane's tokens: i0, i0 + 64, ..., kpt of them

    // Up to kRetainKreg tokens per thread keep their keys in registers: one batch of loads on
    // clamped addresses instead of a load per token in each of the sweeps below.
    const bool in_regs = kpt <= kRetainKreg;                           // block-uniform
    uint32_t rk[kRetainKreg];
    if (in_regs) {
#pragma unroll
        for (int j = 0; j < kRetainKreg; ++j) rk[j] = __float_as_uint(alpha[min(i0 + j * kWave, Tp - 1)]);
#pragma unroll
        for (int j = 0; j < kRetainKreg; ++j) rk[j] = score_key(__uint_as_float(rk[j]));
    }
    // fn(i, key, exists) for the 64 tokens of every step of the wave, in position order
    auto for_keys = [&](auto&& fn) {
        if (in_regs) {
#pragma unroll
            for (int j = 0; j < kRetainKreg; ++j)
                if (j < kpt) fn(i0 + j * kWave, rk[j], i0 + j * kWave < Tp);
        } else {
            for (int j = 0; j < kpt; j += 8) {
                float x[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) x[u] = alpha[min(i0 + (j + u) * kWave, Tp - 1)];
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if (j + u < kpt) fn(i0 + (j + u) * kWave, score_key(x[u]), i0 + (j + u) * kWave < Tp);
            }
        }
    };

    // ---- key of the need-th largest importance ---------------------------------------------------------
    uint32_t prefix = 0;
    int shift = 32;
    uint32_t above = 0;                                                // tokens ranked strictly above the current digit range
#pragma unroll 1
    for (int pass = 0; pass < 3; ++pass) {
        const int bits = pass < 2 ? 11 : 10, nbins = 1 << bits, nshift = shift - bits;
        for (int i = tid; i < 2048; i += kBlockThreads) sh.hist[i] = 0;
        if (tid == 0) sh.res[pass][0] = -1;
        __syncthreads();
        for_keys([&](int32_t, uint32_t key, bool exists) {
            if (exists && (pass == 0 || (key >> shift) == prefix)) atomicAdd(&sh.hist[(key >> nshift) & (nbins - 1)], 1u);
        });
        __syncthreads();
        // thread order == descending digit order: thread t owns digits nbins-1-2t and nbins-2-2t
        const int d1 = nbins - 1 - 2 * tid;
        const uint32_t c1 = d1 >= 0 ? sh.hist[d1] : 0u, c0 = d1 >= 1 ? sh.hist[d1 - 1] : 0u;
        uint32_t total;
        const uint32_t incl = block_scan_u32(c1 + c0, sh.wave_tot[pass], &total);
        const uint32_t above1 = above + incl - c1 - c0, above0 = above1 + c1;
        if (c1 > 0 && above1 < (uint32_t)need && above1 + c1 >= (uint32_t)need) { sh.res[pass][0] = d1; sh.res[pass][1] = (int32_t)above1; }
        if (c0 > 0 && above0 < (uint32_t)need && above0 + c0 >= (uint32_t)need) { sh.res[pass][0] = d1 - 1; sh.res[pass][1] = (int32_t)above0; }
        __syncthreads();
        const int digit = sh.res[pass][0];                             // always found: need <= Tp
        prefix = (pass == 0) ? (uint32_t)digit : ((prefix << bits) | (uint32_t)digit);
        above = (uint32_t)sh.res[pass][1];
        shift = nshift;
    }
    // prefix is the full key of the cut; `above` tokens have a larger key; need - above of the equal ones are kept
    const uint32_t take_equal = (uint32_t)need - above;

    // ---- compaction in position order ------------------------------------------------------------------
    // counts of the wave, exclusive over the waves before it; every lane holds them
    auto before_wave = [&](uint32_t mine, uint32_t* slot) -> uint32_t {
        uint32_t tot;
        const uint32_t own = lane == 0 ? mine : 0u;
        return (uint32_t)__builtin_amdgcn_readfirstlane((int)(block_scan_u32(own, slot, &tot) - own));
    };
    auto lower = [&](unsigned long long m) { return (uint32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u)); };
    uint32_t my_gt = 0, my_eq = 0;
    for_keys([&](int32_t, uint32_t key, bool exists) {
        my_gt += (uint32_t)__popcll(__ballot(exists && key > prefix));
        my_eq += (uint32_t)__popcll(__ballot(exists && key == prefix));
    });
    uint32_t eq = before_wave(my_eq, sh.wave_tot[3]);                  // equal ones before the wave, later before the step
    const uint32_t eq_kept = min(eq + my_eq, take_equal) - min(eq, take_equal);
    uint32_t pos = before_wave(my_gt + eq_kept, sh.wave_tot[4]);
    for_keys([&](int32_t i, uint32_t key, bool exists) {
        const unsigned long long m_eq = __ballot(exists && key == prefix);
        const bool kept = exists && (key > prefix || (key == prefix && eq + lower(m_eq) < take_equal));
        const unsigned long long m = __ballot(kept);
        if (kept) keep[pos + lower(m)] = i;
        eq += (uint32_t)__popcll(m_eq);
        pos += (uint32_t)__popcll(m);
    });
    __syncthreads();                                                   // keep[0 .. need) is written (block-visible)

    // ---- buckets of the retained tokens ------------------------------------------------------------------
    // kept tokens of a thread whose loads are out together (us per call, 32 layers, with 4 / 12: 1531 tokens, 500 kept 7.3 / 7.7; 2500, 2000 8.2 / 9.1; 4096,
    // 1024 8.5 / 9.3; 16384, 4096 21.4 / 22.3; 20000, 10000 24.9 / 25.2)
    constexpr int kU = 4;
    for (int32_t j0 = tid; j0 < need; j0 += kU * kBlockThreads) {
        int32_t s_cur[kU], s_prev[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int32_t j = min(j0 + u * kBlockThreads, need - 1);
            s_cur[u] = keep[j];
            s_prev[u] = keep[max(j - 1, 0)];
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            s_cur[u] = seg_id[s_cur[u]];
            s_prev[u] = seg_id[s_prev[u]];
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int32_t j = j0 + u * kBlockThreads;
            if (j >= need) break;
            const int32_t cur = min(max(s_cur[u], 0), S - 1), prev = j > 0 ? min(max(s_prev[u], 0), S - 1) : -1;
            for (int32_t s = prev + 1; s <= cur; ++s) ret_off[s] = j;
            if (j == need - 1)
                for (int32_t s = cur + 1; s <= S; ++s) ret_off[s] = need;
        }
    }
    __syncthreads();
    for (int s = tid; s < S; s += kBlockThreads) ret_len[s] = ret_off[s + 1] - ret_off[s];
}

// ------------------------------------------------------------------------------------------------
// Retention of long prompts: the same in four launches of several blocks per layer, 8192 or 4096 tokens each.  One block per layer reads
// its tokens' importances five times at what one compute unit gets, from 32769 tokens on from memory.
//   digit:      counts by the top 11 bits of the key; the layer's last block finds the digit that holds the cut; once more with the next 11 bits
//               where too many tokens share that digit;
//   candidates: the tokens of that digit go to a list, those above it are counted per block; the layer's last block finds the cut among the
//               listed ones (more than kRetList of them: among all tokens, as the single block would), the last position kept of those that equal
//               it, and the kept tokens before every block;
//   compact:    kept positions, ret_off at the first token of every bucket (the kept tokens before it), ret_len by the layer's last block.
// Bound by latency: an arrival and the last block's block scans in each launch, 5 to 8 us apiece (2 where the second digit is not needed).  Us per call, one
// block a layer / this with 8192 tokens a block, importances spread over 2^+-6 and, in brackets, within 10 %: 32 layers x 16500 tokens 21.2 / 22.7 (26.7 / 28.0), 20000 22.5 /
// 22.6 (29.3 / 28.1), the line, 32768 27.6 / 24.5 (38.9 / 29.6), 16 x 65536 68 / 26 (87 / 32), 8 x 131072 127 / 27 (166 / 31).
// ------------------------------------------------------------------------------------------------
template <int TOK> constexpr int kRetChunk = TOK * kBlockThreads;       // tokens of a block, TOK of each thread
constexpr int kRetTok = 8, kRetTokFew = 4, kRetFewTok = 65536;          // tokens of a thread, of one of a layer of up to kRetFewTok tokens
struct RetainWork {
    unsigned int* hist;           // [L][2048], zero between calls
    unsigned long long* list;     // [L][kRetList] (key, position)
    unsigned int* count;          // [L][4] arrivals, length of the list; zero between calls
    int32_t* cut;                 // [L][4] leading bits, tokens above them, bits left, tokens that share them; then (2, 3) key of the cut, last position kept of
                                  // those that equal it
    int32_t* chunk;               // [L][kRetMaxChunks] tokens above the digit, then kept tokens before the block
};

// this wave's tokens of its block, i0 + 64 j, and their keys (0 past the end)
template <int TOK> struct RetainTokens {
    int32_t i0;
    uint32_t key[TOK];
    __device__ __forceinline__ RetainTokens(const float* __restrict__ alpha, int32_t Tp) {
        const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
        i0 = blockIdx.x * kRetChunk<TOK> + w * (TOK * kWave) + lane;
        float x[TOK];
#pragma unroll
        for (int j = 0; j < TOK; ++j) x[j] = alpha[min(i0 + j * kWave, Tp - 1)];
#pragma unroll
        for (int j = 0; j < TOK; ++j) key[j] = score_key(x[j]);
    }
};
// true in the block of the layer that arrives last (all of the layer's stores before it are visible to it)
__device__ __forceinline__ bool retain_last(unsigned int* arrive, int* sm_last) {
    block_sync_after_stores();
    if (threadIdx.x == 0) {
        *sm_last = __hip_atomic_fetch_add(arrive, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
        if (*sm_last) __hip_atomic_store(arrive, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);       // for the next launch
    }
    __syncthreads();
    return *sm_last != 0;
}
// The digit (of nbins <= 2048, counts by `count`) that holds the need-th largest; res = digit, number above it, its count.  Every thread calls it.
template <typename Count>
__device__ __forceinline__ void retain_cross(int nbins, uint32_t need, Count count, uint32_t* slot, int32_t* res) {
    const int d1 = nbins - 1 - 2 * (int)threadIdx.x;
    const uint32_t c1 = d1 >= 0 ? count(d1) : 0u, c0 = d1 >= 1 ? count(d1 - 1) : 0u;
    uint32_t total;
    const uint32_t above1 = block_scan_u32(c1 + c0, slot, &total) - c1 - c0, above0 = above1 + c1;
    if (c1 > 0 && above1 < need && above0 >= need) { res[0] = d1; res[1] = (int32_t)above1; res[2] = (int32_t)c1; }
    if (c0 > 0 && above0 < need && above0 + c0 >= need) { res[0] = d1 - 1; res[1] = (int32_t)above0; res[2] = (int32_t)c0; }
    __syncthreads();
}

// SECOND: the 11 bits behind the first digit, where more tokens share it than the list takes (importances of like tokens: 32768 tokens in three or four
// digits); else nothing.
template <bool SECOND, int TOK>
__global__ __launch_bounds__(kBlockThreads) void retain_digit_kernel(const float* __restrict__ alpha_all, int32_t Tp, int32_t k, RetainWork wk) {
    __shared__ uint32_t hist[2048], wave_tot[kBlockWaves];
    __shared__ int32_t res[3];
    __shared__ int sm_last;
    const int l = blockIdx.y, tid = threadIdx.x;
    int32_t* cut = wk.cut + 4 * l;
    const int32_t digit = SECOND ? ld_agent(cut) : 0, above = SECOND ? ld_agent(cut + 1) : 0;
    if (SECOND && ld_agent(cut + 3) <= kRetList) return;
    const RetainTokens<TOK> t(alpha_all + (int64_t)l * Tp, Tp);
    for (int i = tid; i < 2048; i += kBlockThreads) hist[i] = 0;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < TOK; ++j)
        if (t.i0 + j * kWave < Tp && (!SECOND || (int32_t)(t.key[j] >> 21) == digit)) atomicAdd(&hist[SECOND ? (t.key[j] >> 10) & 2047u : t.key[j] >> 21], 1u);
    __syncthreads();
    unsigned int* all = wk.hist + (int64_t)l * 2048;
    for (int i = tid; i < 2048; i += kBlockThreads)
        if (hist[i] != 0) __hip_atomic_fetch_add(all + i, hist[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (!retain_last(wk.count + 4 * l, &sm_last)) return;             // (every block of the layer has read `cut`)
    retain_cross(2048, (uint32_t)(min(k, Tp) - above), [&](int d) { return ld_agent(all + d); }, wave_tot, res);
    if (tid == 0) {
        st_agent(cut, SECOND ? (digit << 11) | res[0] : res[0]);
        st_agent(cut + 1, above + res[1]);
        st_agent(cut + 2, SECOND ? 10 : 21);
        st_agent(cut + 3, res[2]);
    }
    for (int i = tid; i < 2048; i += kBlockThreads) st_agent(all + i, 0u);
}

template <int TOK>
__global__ __launch_bounds__(kBlockThreads) void retain_candidates_kernel(const float* __restrict__ alpha_all, int32_t Tp, int32_t k, RetainWork wk) {
    __shared__ uint32_t hist[2048], wave_tot[2][kBlockWaves], before[kRetMaxChunks];
    __shared__ int32_t equal[kRetList];
    __shared__ int32_t res[3], tie, n_equal;
    __shared__ uint32_t sm_base;
    __shared__ int sm_last;
    const int l = blockIdx.y, tid = threadIdx.x, lane = tid & 63, w = tid >> 6, nchunk = gridDim.x;
    const float* alpha = alpha_all + (int64_t)l * Tp;
    const uint32_t digit = (uint32_t)ld_agent(wk.cut + 4 * l), above = (uint32_t)ld_agent(wk.cut + 4 * l + 1);
    const int open = ld_agent(wk.cut + 4 * l + 2);                     // bits of the key behind the digits
    const RetainTokens<TOK> t(alpha, Tp);
    auto lower = [&](unsigned long long m) { return (uint32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u)); };
    uint32_t n_above = 0, n_cand = 0;
#pragma unroll
    for (int j = 0; j < TOK; ++j) {
        const bool exists = t.i0 + j * kWave < Tp;
        n_above += (uint32_t)__popcll(__ballot(exists && (t.key[j] >> open) > digit));
        n_cand += (uint32_t)__popcll(__ballot(exists && (t.key[j] >> open) == digit));
    }
    uint32_t all_above, all_cand;
    (void)block_scan_u32(lane == 0 ? n_above : 0u, wave_tot[0], &all_above);
    uint32_t at = block_scan_u32(lane == 0 ? n_cand : 0u, wave_tot[1], &all_cand);
    at = (uint32_t)__builtin_amdgcn_readfirstlane((int)(at - n_cand));                 // candidates of the block's waves before this one
    if (tid == 0) {
        sm_base = __hip_atomic_fetch_add(wk.count + 4 * l + 1, all_cand, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        st_agent(wk.chunk + (int64_t)l * kRetMaxChunks + blockIdx.x, (int32_t)all_above);
    }
    __syncthreads();
    at += sm_base;
    unsigned long long* list = wk.list + (int64_t)l * kRetList;
#pragma unroll
    for (int j = 0; j < TOK; ++j) {
        const bool cand = t.i0 + j * kWave < Tp && (t.key[j] >> open) == digit;
        const unsigned long long m = __ballot(cand);
        const uint32_t to = at + lower(m);
        if (cand && to < (uint32_t)kRetList)
            __hip_atomic_store(list + to, ((unsigned long long)t.key[j] << 32) | (uint32_t)(t.i0 + j * kWave), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        at += (uint32_t)__popcll(m);
    }
    if (!retain_last(wk.count + 4 * l, &sm_last)) return;

    // ---- the layer's last block ----------------------------------------------------------------------------
    const uint32_t listed = ld_agent(wk.count + 4 * l + 1);
    const bool fits = listed <= (uint32_t)kRetList;
    uint32_t need = (uint32_t)min(k, Tp) - above;                     // of the candidates, at least one
    constexpr int kMine = kRetList / kBlockThreads;
    unsigned long long mine[kMine];
#pragma unroll
    for (int j = 0; j < kMine; ++j) mine[j] = __hip_atomic_load(list + j * kBlockThreads + tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // fn(key, position) for every candidate: the listed ones, or those among all tokens
    auto for_candidates = [&](auto&& fn) {
        if (fits) {
#pragma unroll
            for (int j = 0; j < kMine; ++j)
                if ((uint32_t)(j * kBlockThreads + tid) < listed) fn((uint32_t)(mine[j] >> 32), (int32_t)(uint32_t)mine[j]);
        } else {
            for (int32_t i = tid; i < Tp; i += kBlockThreads) {
                const uint32_t key = score_key(alpha[i]);
                if ((key >> open) == digit) fn(key, i);
            }
        }
    };
    uint32_t prefix = digit;
    for (int shift = open; shift > 0;) {                               // 11 and 10 bits, or 10
        const int bits = shift == 21 ? 11 : 10;
        for (int i = tid; i < 2048; i += kBlockThreads) hist[i] = 0;
        __syncthreads();
        for_candidates([&](uint32_t key, int32_t) {
            if ((key >> shift) == prefix) atomicAdd(&hist[(key >> (shift - bits)) & ((1u << bits) - 1u)], 1u);
        });
        __syncthreads();
        retain_cross(1 << bits, need, [&](int d) { return hist[d]; }, wave_tot[shift == 21], res);
        prefix = (prefix << bits) | (uint32_t)res[0];
        need -= (uint32_t)res[1];
        shift -= bits;
        __syncthreads();
    }
    // `need` of the tokens whose key is `prefix` are kept, those of the lowest positions
    const uint32_t n_eq = hist[prefix & 1023u];
    if (tid == 0) { tie = Tp; n_equal = 0; }
    for (int i = tid; i < nchunk; i += kBlockThreads) before[i] = fits ? (uint32_t)ld_agent(wk.chunk + (int64_t)l * kRetMaxChunks + i) : 0u;
    __syncthreads();
    if (need < n_eq) {
        if (n_eq <= (uint32_t)kRetList) {
            // The need-th lowest position.  A few are compared with each other; more by two digits of ten bits, the lowest position the highest digit, whose
            // block scans cost 1.2 us.  (Us per call, compared / by digits, 32 layers x 32768 tokens, equal ones at the cut: 64 24.6 / 25.2, 500 30.6 / 26.3,
            // 2001 101 / 32, 4096 329 / 37.)
            for_candidates([&](uint32_t key, int32_t i) { if (key == prefix) equal[atomicAdd(&n_equal, 1)] = i; });
            if (n_eq <= 128u) {
                __syncthreads();
                if (tid < (int)n_eq) {
                    uint32_t rank = 0;
                    for (int o = 0; o < (int)n_eq; ++o) rank += equal[o] < equal[tid];
                    if (rank == need - 1) tie = equal[tid];
                }
            } else {
                static_assert((int64_t)kRetMaxChunks * kRetChunk<kRetTok> <= 1 << 20, "20 bits of a position");
                constexpr uint32_t kLast = (1u << 20) - 1u;
                uint32_t lead = 0, left = need;
#pragma unroll
                for (int shift = 10; shift >= 0; shift -= 10) {
                    for (int i = tid; i < 1024; i += kBlockThreads) hist[i] = 0;
                    __syncthreads();
                    for (int e = tid; e < (int)n_eq; e += kBlockThreads) {
                        const uint32_t place = kLast - (uint32_t)equal[e];
                        if (shift == 10 || place >> 10 == lead) atomicAdd(&hist[(place >> shift) & 1023u], 1u);
                    }
                    __syncthreads();
                    retain_cross(1024, left, [&](int d) { return hist[d]; }, wave_tot[shift == 10], res);
                    lead = (lead << 10) | (uint32_t)res[0];
                    left -= (uint32_t)res[1];
                    __syncthreads();
                }
                if (tid == 0) tie = (int32_t)(kLast - lead);
            }
        } else {                                                       // a plateau: in position order, 1024 tokens at a time
            uint32_t seen = 0;
            for (int32_t g = 0; g < Tp && seen < need; g += kBlockThreads) {
                const uint32_t eq = g + tid < Tp && score_key(alpha[min(g + tid, Tp - 1)]) == prefix;
                uint32_t total;
                const uint32_t rank = seen + block_scan_u32(eq, wave_tot[0], &total);
                if (eq && rank == need) tie = g + tid;
                seen += total;
                __syncthreads();
            }
        }
        __syncthreads();
    }
    if (fits) {
        for_candidates([&](uint32_t key, int32_t i) { if (key > prefix || (key == prefix && i <= tie)) atomicAdd(&before[i / kRetChunk<TOK>], 1u); });
    } else {
        for (int32_t g = 0; g < Tp; g += kBlockThreads) {
            const int32_t i = g + tid;
            const uint32_t key = score_key(alpha[min(i, Tp - 1)]);
            const unsigned long long m = __ballot(i < Tp && (key > prefix || (key == prefix && i <= tie)));
            if (lane == 0 && m != 0) atomicAdd(&before[(g + w * kWave) / kRetChunk<TOK>], (uint32_t)__popcll(m));
        }
    }
    __syncthreads();
    if (w == 0) {                                                      // kRetMaxChunks = 128: two a lane
        const uint32_t a = 2 * lane < nchunk ? before[2 * lane] : 0u, b = 2 * lane + 1 < nchunk ? before[2 * lane + 1] : 0u;
        const uint32_t ex = wave_scan_u32(a + b) - a - b;
        int32_t* dst = wk.chunk + (int64_t)l * kRetMaxChunks + 2 * lane;
        if (2 * lane < nchunk) dst[0] = (int32_t)ex;
        if (2 * lane + 1 < nchunk) dst[1] = (int32_t)(ex + a);
    }
    if (tid == 0) {
        wk.cut[4 * l + 2] = (int32_t)prefix;
        wk.cut[4 * l + 3] = tie;
        st_agent(wk.count + 4 * l + 1, 0u);                            // for the next call
    }
}

template <int TOK>
__global__ __launch_bounds__(kBlockThreads) void retain_compact_kernel(const float* __restrict__ alpha_all, int32_t Tp, int32_t k,
                                                                       const int32_t* __restrict__ seg_id, int32_t S, int32_t* __restrict__ keep_all,
                                                                       int32_t keep_stride, int32_t* __restrict__ n_keep, int32_t* ret_off_all,
                                                                       int32_t* __restrict__ ret_len_all, RetainWork wk) {
    __shared__ uint32_t wave_tot[kBlockWaves];
    __shared__ int sm_last;
    const int l = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
    int32_t* keep = keep_all + (int64_t)l * keep_stride;
    int32_t* ret_off = ret_off_all + (int64_t)l * (S + 1);
    const int32_t need = min(k, Tp);
    const uint32_t cut = (uint32_t)wk.cut[4 * l + 2];
    const int32_t tie = wk.cut[4 * l + 3];
    const RetainTokens<TOK> t(alpha_all + (int64_t)l * Tp, Tp);
    int32_t cur[TOK], prev[TOK];
#pragma unroll
    for (int j = 0; j < TOK; ++j) {
        const int32_t i = min(t.i0 + j * kWave, Tp - 1);
        cur[j] = seg_id[i];
        prev[j] = seg_id[max(i - 1, 0)];
    }
    unsigned long long kept[TOK];
    uint32_t mine = 0;
#pragma unroll
    for (int j = 0; j < TOK; ++j) {
        const int32_t i = t.i0 + j * kWave;
        kept[j] = __ballot(i < Tp && (t.key[j] > cut || (t.key[j] == cut && i <= tie)));
        mine += (uint32_t)__popcll(kept[j]);
    }
    uint32_t total;
    uint32_t pos = block_scan_u32(lane == 0 ? mine : 0u, wave_tot, &total) - mine;
    pos = (uint32_t)__builtin_amdgcn_readfirstlane((int)pos) + (uint32_t)wk.chunk[(int64_t)l * kRetMaxChunks + blockIdx.x];
#pragma unroll
    for (int j = 0; j < TOK; ++j) {
        const int32_t i = t.i0 + j * kWave;
        const uint32_t at = pos + (uint32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(kept[j] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)kept[j], 0u));
        if ((kept[j] >> lane) & 1ull) keep[at] = i;
        if (i < Tp) {
            const int32_t c = min(max(cur[j], 0), S - 1), p = i > 0 ? min(max(prev[j], 0), S - 1) : -1;
            for (int32_t s = p + 1; s <= c; ++s) st_agent(ret_off + s, (int32_t)at);
            if (i == Tp - 1)
                for (int32_t s = c + 1; s <= S; ++s) st_agent(ret_off + s, need);
        }
        pos += (uint32_t)__popcll(kept[j]);
    }
    if (blockIdx.x == 0 && tid == 0) n_keep[l] = need;
    if (!retain_last(wk.count + 4 * l, &sm_last)) return;
    for (int s = tid; s < S; s += kBlockThreads) ret_len_all[(int64_t)l * S + s] = ld_agent(ret_off + s + 1) - ld_agent(ret_off + s);
}

template <int TOK>
static void launch_retain_long(Ctx* c, const float* alpha, int32_t Tp, int32_t k, const int32_t* seg_id, int32_t S, int32_t* keep_idx,
                               int32_t* n_keep, int32_t* ret_off, int32_t* ret_len) {
    static_assert((kRetFewTok + kRetChunk<kRetTokFew> - 1) / kRetChunk<kRetTokFew> <= kRetMaxChunks, "");
    const RetainWork wk = {c->ret_hist, c->ret_list, c->ret_count, c->ret_cut, c->ret_chunk};
    const dim3 chunks((Tp + kRetChunk<TOK> - 1) / kRetChunk<TOK>, c->d.n_layers), block(kBlockThreads);
    hipLaunchKernelGGL((retain_digit_kernel<false, TOK>), chunks, block, 0, c->stream, alpha, Tp, k, wk);
    hipLaunchKernelGGL((retain_digit_kernel<true, TOK>), chunks, block, 0, c->stream, alpha, Tp, k, wk);
    hipLaunchKernelGGL(retain_candidates_kernel<TOK>, chunks, block, 0, c->stream, alpha, Tp, k, wk);
    hipLaunchKernelGGL(retain_compact_kernel<TOK>, chunks, block, 0, c->stream, alpha, Tp, k, seg_id, S, keep_idx, max(k, 1), n_keep, ret_off, ret_len, wk);
}

hipError_t launch_retain(Ctx* c, const float* alpha, int32_t Tp, int32_t k, const int32_t* seg_id, int32_t S, int32_t* keep_idx,
                         int32_t* n_keep, int32_t* ret_off, int32_t* ret_len) {
    const dim3 grid(c->d.n_layers), block(kBlockThreads);
    if (k > 0 && c->ret_hist && Tp > kRetainLongTok && (Tp + kRetChunk<kRetTok> - 1) / kRetChunk<kRetTok> <= kRetMaxChunks) {
        // Shorter blocks for few tokens, as long as the chip holds them all at once.  Us per call, 8192 / 4096 tokens a block, importances spread over 2^+-6 and, in
        // brackets, within 10 %: 32 layers x 20500 tokens 22.3 / 20.2 (30.8 / 26.1), 32768 23.0 / 21.0 (31.6 / 27.3), 2 x 65536 22.0 / 20.1 (30.1 / 25.0), 16 x 65536
        // 24.4 / 23.8 (32.6 / 30.0), 8 x 131072 25.2 / 25.6 (34.1 / 32.2); more blocks than compute units: 64 x 32768 23.1 / 25.1, 32 x 49152 24.3 / 26.1, 32 x 65536
        // 24.8 / 28.1.
        const int few_blocks = (Tp + kRetChunk<kRetTokFew> - 1) / kRetChunk<kRetTokFew> * c->d.n_layers;
        if (Tp <= kRetFewTok && few_blocks <= c->n_cu) launch_retain_long<kRetTokFew>(c, alpha, Tp, k, seg_id, S, keep_idx, n_keep, ret_off, ret_len);
        else launch_retain_long<kRetTok>(c, alpha, Tp, k, seg_id, S, keep_idx, n_keep, ret_off, ret_len);
        return hipGetLastError();
    }
    if (Tp <= 4 * kBlockThreads)
        hipLaunchKernelGGL(retain_kernel<4>, grid, block, 0, c->stream, alpha, Tp, k, seg_id, S, keep_idx, max(k, 1), n_keep, ret_off, ret_len);
    else                                                               // up to 32768 tokens in registers; more only for contexts of many layers, and past 2^20
        hipLaunchKernelGGL(retain_kernel<32>, grid, block, 0, c->stream, alpha, Tp, k, seg_id, S, keep_idx, max(k, 1), n_keep, ret_off, ret_len);
    return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// Pool compaction: K_ret/V_ret [L][Hkv][k][D] = rows keep_idx[l][0 .. n_keep[l]) of K/V [L][Hkv][T][D].
// Same branch-free copy as the decode-side gather; the kept positions are shared by the heads of a layer.  The mean keys of the retained tokens
// are made of K_ret next: values go first and keys last, with plain stores, so that what fits the 256 MB memory-side cache of K_ret is still there.  Us for retention,
// compaction and mean keys together, keys first and non-temporal / this (and keys of semvec_short_kernel read last to first, non-temporal), 32 layers x 8 bf16 heads,
// kept of tokens: 1024 of 8192 87.2 / 81.4, 2048 of 4096 129.6 / 120.7, 1024 of 32768 136 / 120.5, 6000 of 16384 395 / 370, 4096 of 32768 295 / 286; 16 layers,
// 16384 of 65536 526 / 511, fp32 3000 of 20000 219 / 204; keys first with plain stores 32768 310.
// ------------------------------------------------------------------------------------------------
template <int EB, bool STREAM>
__global__ __launch_bounds__(kGatherThreads) void compact_pool_kernel(const char* __restrict__ Kp, const char* __restrict__ Vp, int32_t T,
                                                                     const int32_t* __restrict__ keep_all, int32_t k,
                                                                     const int32_t* __restrict__ n_keep, int32_t Hkv,
                                                                     char* __restrict__ Kr, char* __restrict__ Vr) {
    using R = Row<EB>;
    constexpr int kRowsPerIter = kGatherThreads / R::LPR;
    constexpr int kIter = kGatherRowsPerBlock / kRowsPerIter;
    constexpr int kRowBytes = kHeadDim * EB;
    const int lh = blockIdx.y, l = lh / Hkv;
    const int32_t n = min(n_keep[l], k);
    const int32_t j0 = blockIdx.x * kGatherRowsPerBlock;
    if (j0 >= n || T <= 0) return;
    const bool keys = blockIdx.z != 0;                                 // (dispatched last)
    const char* src = (keys ? Kp : Vp) + (int64_t)lh * T * kRowBytes;
    char* dst = (keys ? Kr : Vr) + (int64_t)lh * k * kRowBytes;
    const int32_t* keep = keep_all + (int64_t)l * k;
    const int r = threadIdx.x / R::LPR, cc = threadIdx.x % R::LPR;
    int32_t x[kIter];
#pragma unroll
    for (int i = 0; i < kIter; ++i) x[i] = keep[min(j0 + i * kRowsPerIter + r, n - 1)];
    uint4 val[kIter];
#pragma unroll
    for (int i = 0; i < kIter; ++i) {
        const char* p = src + (int64_t)min(max(x[i], 0), T - 1) * kRowBytes + cc * 16;
        val[i] = STREAM ? ld_stream(p) : *reinterpret_cast<const uint4*>(p);
    }
#pragma unroll
    for (int i = 0; i < kIter; ++i) {
        const int32_t j = j0 + i * kRowsPerIter + r;
        char* p = dst + (int64_t)j * kRowBytes + cc * 16;
        if (j < n && x[i] >= 0 && x[i] < T) {
            if (STREAM && !keys) st_stream(p, val[i]);
            else *reinterpret_cast<uint4*>(p) = val[i];
        }
    }
}

// Non-temporal loads and stores of values from this many bytes of output on (a smaller retained pool is read again from the caches): 32 layers x 8 heads, the whole
// retention, us, all plain / from here on: 134 MB 90.1 / 81.4, 269 MB 126.0 / 120.7, 537 MB 316 / 286; everywhere / from here on: 67 MB 42.0 / 41.7.
constexpr int64_t kCompactStreamBytes = 96ll << 20;
hipError_t launch_compact_pool(Ctx* c, const void* K_pool, const void* V_pool, int32_t T, const int32_t* keep_idx, int32_t k,
                               const int32_t* n_keep, void* K_ret, void* V_ret) {
    if (k == 0) return hipSuccess;
    const dim3 grid((k + kGatherRowsPerBlock - 1) / kGatherRowsPerBlock, c->d.n_layers * c->d.n_kv_heads, 2), block(kGatherThreads);
    const int64_t bytes = 2ll * c->d.n_layers * c->d.n_kv_heads * k * kHeadDim * (c->d.kv_dtype == SKV_BF16 ? 2 : 4);
    auto launch = [&](auto eb, auto stream) {
        hipLaunchKernelGGL((compact_pool_kernel<decltype(eb)::value, decltype(stream)::value>), grid, block, 0, c->stream, (const char*)K_pool,
                           (const char*)V_pool, T, keep_idx, k, n_keep, c->d.n_kv_heads, (char*)K_ret, (char*)V_ret);
    };
    using std::integral_constant;
    const bool streams = bytes > kCompactStreamBytes;
    if (c->d.kv_dtype == SKV_BF16) {
        if (streams) launch(integral_constant<int, 2>{}, std::true_type{});
        else launch(integral_constant<int, 2>{}, std::false_type{});
    } else {
        if (streams) launch(integral_constant<int, 4>{}, std::true_type{});
        else launch(integral_constant<int, 4>{}, std::false_type{});
    }
    return hipGetLastError();
}

}  // namespace skv
