// libdart: DART's policy-update hot path as hand-written HIP for gfx950 (CDNA4).
//
// Paper: DART, arXiv 2509.23866 — token entropy and step entropy (Sec. 4.3),
// high-entropy step selection (Sec. 4.3, indicator of Eq. 2), truncated
// importance sampling (Sec. 4.4), clipped surrogate (Eq. 1, Eq. 2).
//
// Kernels of the path, all launched on the caller's stream:
//   tok_stats_kernel    one workgroup per logits row; one streaming pass with an
//                       online (max, normaliser, entropy) triple in fp32 per lane,
//                       merged across lanes and waves; target logit gathered.
//   step_mean_kernel    one wave per step: mean entropy, fp64 sums in a fixed order.
//   step_select_kernel  one workgroup per group of steps: direct rank of the
//                       step keys (small groups) or radix select of the k-th
//                       largest 32-bit key with LDS histograms; index-ordered ties.
//   tis_coef_kernel     many workgroups: per-token ratio, TIS weight, clip gate and
//                       loss coefficient; partial sums of the loss in fp64
//                       (tis_coef_step_kernel: step-level ratios, one wave per step).
//   tis_loss_finalize_kernel  adds the partial sums in a fixed order.
//   select_coef_kernel  one workgroup: step_select_kernel's and tis_coef_kernel's
//                       device code back to back (up to 4096 tokens and 80 steps), the
//                       offsets and mask handed over in LDS.
//   tis_grad_kernel     one workgroup per 4 KB chunk of a row; second streaming
//                       pass writing coef * (onehot - softmax) in the logits dtype.
// The two streaming kernels are HBM-bound (no matrix contraction anywhere):
// 16-byte non-temporal loads and stores, several loads in flight per lane,
// base-2 exponentials.
#include <hip/hip_runtime.h>
#include <hip/hip_bf16.h>
#include <math.h>
#include <stdint.h>

#include <mutex>
#include <type_traits>

#include "internal.h"
#include "dart.h"

namespace {

constexpr float kLog2e = 1.44269504088896340736f;

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// ------------------------------------------------------------------------
// element access
// ------------------------------------------------------------------------

template <dart_dtype_t D>
struct Elt;
template <>
struct Elt<DART_BF16> {
    using T = uint16_t;
    static constexpr int kPerVec = 8;  // elements per 16-byte vector
};
template <>
struct Elt<DART_F32> {
    using T = float;
    static constexpr int kPerVec = 4;
};

template <dart_dtype_t D>
__device__ __forceinline__ void unpack(const u32x4 v, float* z);

template <>
__device__ __forceinline__ void unpack<DART_BF16>(const u32x4 v, float* z) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        z[2 * i] = __uint_as_float(v[i] << 16);
        z[2 * i + 1] = __uint_as_float(v[i] & 0xFFFF0000u);
    }
}

template <>
__device__ __forceinline__ void unpack<DART_F32>(const u32x4 v, float* z) {
#pragma unroll
    for (int i = 0; i < 4; ++i) z[i] = __uint_as_float(v[i]);
}

template <dart_dtype_t D>
__device__ __forceinline__ float load_one(const void* row, int64_t col) {
    if constexpr (D == DART_BF16)
        return __uint_as_float((uint32_t)static_cast<const uint16_t*>(row)[col] << 16);
    else
        return static_cast<const float*>(row)[col];
}

template <dart_dtype_t D>
__device__ __forceinline__ void store_one(void* row, int64_t col, float x) {
    if constexpr (D == DART_BF16) {
        __hip_bfloat16 b = __float2bfloat16(x);  // round to nearest even
        static_cast<__hip_bfloat16*>(row)[col] = b;
    } else {
        static_cast<float*>(row)[col] = x;
    }
}

template <dart_dtype_t D>
__device__ __forceinline__ u32x4 pack(const float* d);

template <>
__device__ __forceinline__ u32x4 pack<DART_BF16>(const float* d) {
    u32x4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        __hip_bfloat162 p = __float22bfloat162_rn(make_float2(d[2 * i], d[2 * i + 1]));
        v[i] = *reinterpret_cast<const uint32_t*>(&p);
    }
    return v;
}

template <>
__device__ __forceinline__ u32x4 pack<DART_F32>(const float* d) {
    u32x4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = __float_as_uint(d[i]);
    return v;
}

// ------------------------------------------------------------------------
// online (max, normaliser, entropy) triple
// ------------------------------------------------------------------------
// For the elements seen so far, with m their maximum and x_v = (z_v - m) log2(e):
//   s = sum_v 2^{x_v},   w = sum_v 2^{x_v} x_v.
// Then lse = m + ln2 log2(s) and H = ln2 (log2(s) - w / s). Two triples merge
// by rescaling to the larger maximum: s' = 2^{d} s, w' = 2^{d} (w + d s),
// d = (m - m_new) log2(e). An empty triple has s == 0 and m == -inf.
struct Triple {
    float m, s, w;
};

__device__ __forceinline__ Triple triple_empty() { return Triple{-INFINITY, 0.f, 0.f}; }

// Adds N elements exactly: the running maximum is updated once per call, then
// every element costs one FMA, one clamp, one exp2, one add and one FMA. The
// clamp keeps 2^x * x finite for -inf logits (2^-256 is 0 in fp32, so no finite
// value moves).
// The logits enter scaled by k = inv_temp * log2(e) (inv_temp > 0); m is kept
// in units of inv_temp * z.
template <int N>
__device__ __forceinline__ void triple_add_exact(Triple& a, const float* z, float inv_temp,
                                                 float k) {
    float cm = z[0];
#pragma unroll
    for (int i = 1; i < N; ++i) cm = fmaxf(cm, z[i]);
    cm *= inv_temp;
    if (cm > a.m) {
        if (a.s > 0.f) {
            const float d = (a.m - cm) * kLog2e;
            const float sc = __builtin_amdgcn_exp2f(d);
            a.w = sc * fmaf(d, a.s, a.w);
            a.s *= sc;
        }
        a.m = cm;
    }
    if (a.m == -INFINITY) return;
    const float mb = a.m * kLog2e;
    float s = 0.f, w = 0.f;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const float x = fmaxf(fmaf(z[i], k, -mb), -256.f);
        const float e = __builtin_amdgcn_exp2f(x);
        s += e;
        w = fmaf(e, x, w);
    }
    a.s += s;
    a.w += w;
}

// Adds N elements against a lazy reference: the triple's m need not be the
// maximum, only some value that keeps every 2^x term small. A lane takes its
// first finite element as the reference and keeps it while a chunk's terms sum
// below 2^30 (x <= ~30, so fp32 keeps H and lse to a few 1e-6) and are not NaN;
// otherwise (a much larger logit, or a -inf logit making 0 * -inf) the chunk is
// redone exactly, which also moves the reference to the chunk maximum. Per
// element this costs one FMA, one exp2, one add and one FMA: the per-element
// maximum and clamp leave the hot loop.
template <int N>
__device__ __forceinline__ void triple_add(Triple& a, const float* z, float inv_temp, float k) {
    if (a.m == -INFINITY) a.m = z[0] * inv_temp;
    if (a.m != -INFINITY) {
        const float mb = a.m * kLog2e;
        float s = 0.f, w = 0.f;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const float x = fmaf(z[i], k, -mb);
            const float e = __builtin_amdgcn_exp2f(x);
            s += e;
            w = fmaf(e, x, w);
        }
        if (s < 0x1p30f && w == w) {
            a.s += s;
            a.w += w;
            return;
        }
    }
    triple_add_exact<N>(a, z, inv_temp, k);
}

// Wave reductions in a fixed order on the DPP network (no LDS round trips): pairs
// (quad_perm 1,0,3,2), quads (quad_perm 2,3,0,1), half-rows (row_half_mirror),
// rows of 16 (row_mirror), then rows 0+1 and 2+3 (row_bcast15 into rows 1, 3)
// and all four (row_bcast31 into rows 2, 3); lane 63 holds the result, which
// every lane receives. The whole wave must be active.
template <int CTRL, int ROW_MASK, class F>
__device__ __forceinline__ float dpp_step(float x, float none, F f) {
    return f(x, __int_as_float(__builtin_amdgcn_update_dpp(
                    __float_as_int(none), __float_as_int(x), CTRL, ROW_MASK, 0xf, false)));
}

// none: what f leaves alone (lanes without a partner get it).
template <class F>
__device__ __forceinline__ float wave_reduce_f32(float x, float none, F f) {
    x = dpp_step<0xB1, 0xf>(x, none, f);
    x = dpp_step<0x4E, 0xf>(x, none, f);
    x = dpp_step<0x141, 0xf>(x, none, f);
    x = dpp_step<0x140, 0xf>(x, none, f);
    x = dpp_step<0x142, 0xa>(x, none, f);
    x = dpp_step<0x143, 0xc>(x, none, f);
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 63));
}

// The merge of a wave's triples: the largest reference first, each lane rescaled
// to it once, then two sums. (Merging pairs of triples, six rounds of three
// exchanges and two exponentials, then the waves one after the other, cost a row
// ~2 us behind its last load.)
__device__ __forceinline__ Triple triple_wave_merge(const Triple a) {
    const float M = wave_reduce_f32(a.s != 0.f ? a.m : -INFINITY, -INFINITY,
                                    [](float x, float y) { return fmaxf(x, y); });
    float s = 0.f, w = 0.f;
    if (a.s != 0.f) {
        const float d = (a.m - M) * kLog2e;
        const float c = __builtin_amdgcn_exp2f(d);
        s = c * a.s;
        w = c * fmaf(d, a.s, a.w);
    }
    auto add = [](float x, float y) { return x + y; };
    return Triple{M, wave_reduce_f32(s, 0.f, add), wave_reduce_f32(w, 0.f, add)};
}

// The statistics pass gives each row one workgroup and each lane kStatsUnroll
// 16-byte vectors at a time: vector j of the aligned body is read by lane
// j % THREADS in iteration j / (THREADS * kStatsUnroll), so every wave reads 1
// KiB contiguous per load, and the last, partial iteration is one batch too.
// THREADS follows the row's length, see stats_threads. The gradient pass runs
// one-shot workgroups of 128 threads x 2 vectors over 4 KB chunks of a bf16 row (best
// of 32..1024 threads x 1..8 vectors, ~15% faster than one 1024-thread workgroup
// per row and faster than a plain elementwise copy). Non-temporal loads and
// stores win in both (see kCachedLogits); register double-buffering does not. NTL
// / NTS select non-temporal loads / stores.
constexpr int kStatsUnroll = 4;
// rows per launch of the statistics (a dispatch holds at most 2^32 - 1 work-items)
constexpr int64_t kStatsMaxRows = int64_t(1) << 22;
constexpr int kGradThreads = 128;
constexpr int kGradUnroll = 2;
// fp32 rows of at least this many vectors that are no whole number of 128-byte lines
// apart go in 8 KB chunks, by twice the threads: the workgroups on both sides of a
// chunk's end share its line, and there are half as many ends. Measured against 4 KB (us;
// in brackets before a row's coefficient decided on its loads): 12000 x 32003 618 ->
// 545 [599], 3000 x 32003 143 -> 129 [139], 8000 x 50257 560 -> 534 [543], 2500 x 70001
// 232 -> 228 [225], 6000 x 17000 135 -> 133 [131]; but 20000 x 1000, where a row does not
// fill a chunk, 27.4 -> 28.3. Rows of whole lines go either way by V (152064 -6%, 32000
// -2%, 120000 +1%, 107392 +3 to +5%) and keep 4 KB, as bf16 rows do (4096 x 152064 384 ->
// 423).
constexpr int64_t kGradWideVectors = 1024;
constexpr int64_t kGradMaxBlocks = 1ll << 24;
constexpr bool kNtStore = true;
// Logits up to this size are loaded as any other data, larger ones
// non-temporally: what fits the caches beside the gradient is still there when
// the gradient pass reads it again. Measured for the two passes (us): 29 MB 24.0 ->
// 21.8, 64 MB 36.2 -> 34.0, 91 MB 53.8 -> 51.0; but the statistics alone lose 8%
// at 91 MB (23.0 -> 24.9, 12% at 1.2 GB) where they gain 5% at 29 MB.
constexpr int64_t kCachedLogits = int64_t(64) << 20;

template <bool NT>
__device__ __forceinline__ u32x4 vload(const u32x4* p) {
    if constexpr (NT)
        return __builtin_nontemporal_load(p);
    else
        return *p;
}

// The same load at any element alignment: gfx950 under HSA reads 16 bytes a
// lane at any address, in one instruction.
typedef u32x4 u32x4_any __attribute__((aligned(2)));
template <bool NT>
__device__ __forceinline__ u32x4 vload_any(const void* p) {
    const u32x4_any* q = static_cast<const u32x4_any*>(p);
    if constexpr (NT)
        return __builtin_nontemporal_load(q);
    else
        return *q;
}

template <bool NT>
__device__ __forceinline__ void vstore(const u32x4 v, u32x4* p) {
    if constexpr (NT)
        __builtin_nontemporal_store(v, p);
    else
        *p = v;
}

struct RowLayout {
    int64_t head;      // scalar elements before the first 16-byte boundary
    int64_t nvec;      // aligned 16-byte vectors
    int64_t body_end;  // first element after the vectors
};

// row is aligned to its elements (the entry points refuse others), so fewer than
// kPerVec elements lie before the first boundary and fewer than that after the last
// vector: the statistics load them one a lane.
template <dart_dtype_t D>
__device__ __forceinline__ RowLayout row_layout(const void* row, int64_t V) {
    using E = typename Elt<D>::T;
    constexpr int EPV = Elt<D>::kPerVec;
    RowLayout L;
    const uintptr_t addr = reinterpret_cast<uintptr_t>(row);
    const int64_t head = (int64_t)(((16 - (addr & 15)) & 15) / sizeof(E));
    L.head = head < V ? head : V;
    L.nvec = (V - L.head) / EPV;
    L.body_end = L.head + L.nvec * EPV;
    return L;
}

// ------------------------------------------------------------------------
// K1: token statistics
// ------------------------------------------------------------------------

template <dart_dtype_t D, int THREADS, int UNROLL, bool NTL>
__global__ void __launch_bounds__(THREADS, 8)  // 8 waves a SIMD: 64 registers
tok_stats_kernel(const void* __restrict__ logits, int64_t V, int64_t ld,
                 const int32_t* __restrict__ target, float inv_temp, float* __restrict__ logp,
                 float* __restrict__ entropy, float* __restrict__ lse) {
    using E = typename Elt<D>::T;
    constexpr int EPV = Elt<D>::kPerVec;
    constexpr int PER_IT = THREADS * UNROLL;
    constexpr int WAVES = THREADS / 64;
    static_assert(WAVES <= 64, "one wave merges the waves' triples");
    static_assert(2 * EPV <= THREADS, "a lane for every element beside the vectors");
    __shared__ Triple partial[WAVES];

    const int64_t t = blockIdx.x;
    const int tid = threadIdx.x;
    const E* row = static_cast<const E*>(logits) + t * ld;
    // an out-of-range target id (a broken precondition) yields NaN, never a stray read
    const int64_t y_in = target[t];
    const bool y_ok = y_in >= 0 && y_in < V;
    const int64_t y = y_ok ? y_in : -1;
    const RowLayout L = row_layout<D>(row, V);
    const u32x4* vrow = reinterpret_cast<const u32x4*>(row + L.head);

    // The target element is left out of the lane sums and added once at the
    // end, so that 1 - p_target (and logp near 0) keep full relative accuracy.
    const int64_t vy = (y >= L.head && y < L.body_end) ? (y - L.head) / EPV : -1;
    const int64_t it_y = vy >= 0 ? vy / PER_IT : -1;
    const int y_in_vec = (int)((y - L.head) % EPV);
    auto drop_target = [&](float* z, int64_t j) {
        if (j != vy) return;
#pragma unroll
        for (int e = 0; e < EPV; ++e)
            if (e == y_in_vec) z[e] = -INFINITY;
    };
    // the target's logit and the head and tail elements (fewer than 2 EPV, one
    // a lane) are asked for first and used last
    const float zy_raw = load_one<D>(row, y_ok ? y : 0);
    const int64_t nscalar = L.head + (V - L.body_end);
    float z1[1] = {-INFINITY};
    if (tid < nscalar) {
        const int64_t col = tid < L.head ? tid : L.body_end + (tid - L.head);
        if (col != y) z1[0] = load_one<D>(row, col);
    }

    const float k = inv_temp * kLog2e;
    Triple acc = triple_empty();
    const int64_t nfull = L.nvec / PER_IT;
    for (int64_t it = 0; it < nfull; ++it) {
        u32x4 v[UNROLL];
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) v[u] = vload<NTL>(vrow + it * PER_IT + u * THREADS + tid);
        float z[UNROLL * EPV];
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) unpack<D>(v[u], z + u * EPV);
        if (it == it_y)
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) drop_target(z + u * EPV, it * PER_IT + u * THREADS + tid);
        triple_add<UNROLL * EPV>(acc, z, inv_temp, k);
    }
    if (nfull * PER_IT < L.nvec) {
        const int64_t j0 = nfull * PER_IT + tid;
        u32x4 v[UNROLL];
#pragma unroll
        for (int u = 0; u < UNROLL; ++u)
            if (j0 + u * THREADS < L.nvec) v[u] = vload<NTL>(vrow + j0 + u * THREADS);
#pragma unroll
        for (int u = 0; u < UNROLL; ++u)
            if (j0 + u * THREADS < L.nvec) {
                float z[EPV];
                unpack<D>(v[u], z);
                drop_target(z, j0 + u * THREADS);
                triple_add<EPV>(acc, z, inv_temp, k);
            }
    }
    if (tid < nscalar) triple_add<1>(acc, z1, inv_temp, k);

    Triple x = triple_wave_merge(acc);
    if constexpr (WAVES > 1) {
        const int lane = tid & 63;
        if (lane == 0) partial[tid >> 6] = x;
        __syncthreads();
        if (tid >= 64) return;
        x = triple_wave_merge(lane < WAVES ? partial[lane] : triple_empty());
    }
    if (tid != 0) return;

    // add the target element
    const float zy = y_ok ? zy_raw * inv_temp : __builtin_nanf("");
    const float M = fmaxf(x.m, zy);
    float sx = 0.f, wx = 0.f;
    if (x.s > 0.f) {
        const float dx = (x.m - M) * kLog2e;
        const float cx = __builtin_amdgcn_exp2f(dx);
        sx = cx * x.s;
        wx = cx * fmaf(dx, x.s, x.w);
    }
    const float xy = (zy - M) * kLog2e;
    const float ey = zy == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(xy);
    const float s = sx + ey;
    const float w = ey > 0.f ? fmaf(ey, xy, wx) : wx;
    // log2(s) as exponent + log2 of a mantissa near 1, and w / s with its remainder,
    // combined in fp64: one log2f of the whole s is rounded to its magnitude (s is
    // some thousands against a lane's reference), which was most of the error that
    // lse's own rounding leaves. Root mean square of the difference from 64 bits at
    // V = 8000 and 2048, fp32: lse 3.7e-7 -> 2.9e-7 and 3.5e-7 -> 3.0e-7, entropy
    // 4.5e-7 -> 3.6e-7 and 4.4e-7 -> 3.8e-7; one work-item a row does this, and the
    // pass takes no longer.
    float mant = __builtin_amdgcn_frexp_mantf(s);
    int ex = __builtin_amdgcn_frexp_expf(s);
    if (mant < 0.70710678f) {
        mant *= 2.f;
        --ex;
    }
    const double log2s = (double)ex + (double)log2f(mant);
    const float q = w / s;
    const double mean_x = (double)q + (double)(isfinite(s) ? fmaf(-q, s, w) / s : 0.f);
    const double ln_s = log2s * 0.69314718055994530942;
    lse[t] = (float)((double)M + ln_s);
    entropy[t] = fmaxf((float)(0.69314718055994530942 * (log2s - mean_x)), 0.f);
    // p_y = ey / (sx + ey): -log1p(sx / ey) is exact to a few ulps when p_y -> 1
    logp[t] = sx < ey ? -log1pf(sx / ey) : (float)((double)zy - (double)M - ln_s);
}

// ------------------------------------------------------------------------
// K2: step entropy + top-k step selection
// ------------------------------------------------------------------------

constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / 64;
constexpr int kSelLdsKeys = 8192;  // groups up to this many steps keep their keys in LDS
constexpr int kSelLdsTokens = 16384;  // one group of up to this many tokens: means fused in,
// up to this many steps: the one workgroup takes ~1 us for every 16 of them, as long
// as a launch of step_mean_kernel at 48. Measured (fused against two launches, us, 3000
// tokens): 33 steps 3.9 and 4.5, 40 4.3 and 4.5, 49 4.7 and 4.6, 64 5.3 and 4.6; 512
// steps of 32 tokens 23.8 and 7.6
constexpr int64_t kSelFusedMaxS = 48;
constexpr int kSelRankMax = 256;   // groups up to this many steps are ranked directly

// Wave sums of 64-bit values in the order of wave_reduce_f32: a value moves as two
// 32-bit halves under the same control.
template <int CTRL, int ROW_MASK = 0xf>
__device__ __forceinline__ uint64_t dpp_u64(uint64_t x) {
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)x, CTRL, ROW_MASK, 0xf, false);
    const int hi =
        __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(x >> 32), CTRL, ROW_MASK, 0xf, false);
    return ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo;
}

__device__ __forceinline__ uint64_t lane63_u64(uint64_t x) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, 63);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), 63);
    return ((uint64_t)hi << 32) | lo;
}

template <class Add>
__device__ __forceinline__ uint64_t wave_reduce_u64(uint64_t x, Add add) {
    x = add(x, dpp_u64<0xB1>(x));
    x = add(x, dpp_u64<0x4E>(x));
    x = add(x, dpp_u64<0x141>(x));
    x = add(x, dpp_u64<0x140>(x));
    x = add(x, dpp_u64<0x142, 0xa>(x));
    x = add(x, dpp_u64<0x143, 0xc>(x));
    return lane63_u64(x);
}

__device__ __forceinline__ double wave_sum(double x) {
    const uint64_t r = wave_reduce_u64(__double_as_longlong(x), [](uint64_t a, uint64_t b) {
        return (uint64_t)__double_as_longlong(__longlong_as_double(a) + __longlong_as_double(b));
    });
    return __longlong_as_double(r);
}

__device__ __forceinline__ int64_t wave_sum_i64(int64_t x) {
    return (int64_t)wave_reduce_u64((uint64_t)x, [](uint64_t a, uint64_t b) { return a + b; });
}

// Workgroup barrier for data exchanged through LDS only: waits for the wave's
// LDS accesses (lgkmcnt) but not for its global stores, which the fence of
// __syncthreads would wait for (~1 us each time in the one-workgroup kernels);
// the empty asm statements keep the compiler from moving memory accesses
// across it.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_s_waitcnt(0xF | (0x7 << 4) | (0x3 << 14));  // lgkmcnt(0)
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Token range of step s, clamped to [0, T] so that malformed offsets (a broken
// precondition) give meaningless numbers but never an out-of-bounds access.
__device__ __forceinline__ void step_bounds(const int32_t* off, int64_t s, int64_t T, int64_t& b,
                                            int64_t& e) {
    b = min(max((int64_t)off[s], (int64_t)0), T);
    e = min(max((int64_t)off[s + 1], b), T);
}

// Order-preserving map of a float to uint32 (larger float -> larger key); -0 == +0.
__device__ __forceinline__ uint32_t float_key(float f) {
    uint32_t u = __float_as_uint(f == 0.f ? 0.f : f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Step means: one wave per step, lanes stride the step's tokens, fixed
// butterfly order (identical steps give identical means wherever they sit).
// Grid: ceil(S / waves per workgroup), so every step runs in parallel.
__global__ void __launch_bounds__(kSelThreads)
step_mean_kernel(const float* __restrict__ H, int64_t T, const int32_t* __restrict__ off,
                 int64_t S, float* __restrict__ step_H) {
    const int lane = threadIdx.x & 63;
    const int64_t s = (int64_t)blockIdx.x * kSelWaves + (threadIdx.x >> 6);
    if (s >= S) return;
    int64_t b, e;
    step_bounds(off, s, T, b, e);
    double sum = 0.0;
    for (int64_t i = b + lane; i < e; i += 64) sum += (double)H[i];
    sum = wave_sum(sum);
    if (lane == 0) step_H[s] = (float)(sum / (double)(e - b));
}

// k = clamp(ceil(rho * n - 1e-6), 0, n), with the two double operations
// rounded separately (no contraction) so that it equals the host's count.
__device__ __forceinline__ int64_t kept_steps_dev(int64_t n, double rho) {
    double k = ceil(__dsub_rn(__dmul_rn(rho, (double)n), 1e-6));
    k = fmin(fmax(k, 0.0), (double)n);
    return (int64_t)k;
}

// One workgroup per group of steps: group g is steps [grp[g], grp[g+1]) (or all
// S steps when grp is null, with k given); it keeps the ceil(rho S_g) steps of
// highest mean entropy (step_H, from step_mean_kernel) among its own, equal
// means lower step index first: by direct rank in small groups, else by a
// radix select of the k-th key and a scan over the keys equal to it.
// FUSED (one group, T <= kSelLdsTokens, S <= kSelFusedSteps): the workgroup first
// computes the step means itself, from the token entropies and offsets staged
// in LDS, in the order of step_mean_kernel (so with bit-identical results),
// and writes them to step_H.
// LDS of the selection for groups of up to KEYS steps staged there; with the
// means fused in, also the token entropies and the clamped offsets (off_l[s] =
// first token of step s, off_l[S] = end)
constexpr int kSelFusedSteps = 128;  // most steps of a fused launch
static_assert(kSelFusedMaxS <= kSelFusedSteps, "steps of a fused selection");
template <int KEYS>
struct SelLds {
    uint32_t keys[KEYS];
    uint32_t hist[256];
    uint32_t sel_bin;
    int64_t sel_remaining;
    int64_t wave_count[kSelWaves];
};

template <bool FUSED>
__device__ __forceinline__ void select_steps(const float* __restrict__ H, int64_t T,
                                             const int32_t* __restrict__ off, int64_t S,
                                             const int32_t* __restrict__ grp, double rho,
                                             int64_t k_all, float* __restrict__ step_H,
                                             uint8_t* __restrict__ mask,
                                             int32_t* __restrict__ n_kept,
                                             SelLds<FUSED ? kSelFusedSteps : kSelLdsKeys>& sl,
                                             float* H_l, int32_t* off_l,
                                             uint8_t* mask_l = nullptr) {
    uint32_t* keys = sl.keys;
    uint32_t* hist = sl.hist;
    uint32_t& sel_bin = sl.sel_bin;
    int64_t& sel_remaining = sl.sel_remaining;
    int64_t* wave_count = sl.wave_count;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    if constexpr (FUSED) {
#pragma unroll 4
        for (int64_t i = tid; i < T; i += kSelThreads) H_l[i] = H[i];
        for (int64_t s = tid; s < S; s += kSelThreads) {
            int64_t b, e;
            step_bounds(off, s, T, b, e);
            off_l[s] = (int32_t)b;
            if (s == S - 1) off_l[S] = (int32_t)e;
        }
        __syncthreads();
        for (int64_t s = wave; s < S; s += kSelWaves) {
            const int64_t b = off_l[s], e = max((int64_t)off_l[s + 1], b);
            double sum = 0.0;
            for (int64_t i = b + lane; i < e; i += 64) sum += (double)H_l[i];
            sum = wave_sum(sum);
            const float m = (float)(sum / (double)(e - b));
            if (lane == 0) {
                step_H[s] = m;
                keys[s] = float_key(m);
            }
        }
        lds_barrier();  // the keys; the step means in global memory are not read here
    }
    int64_t gs = 0, ge = S, k = k_all;
    if (grp) {
        gs = min(max((int64_t)grp[blockIdx.x], (int64_t)0), S);
        ge = min(max((int64_t)grp[blockIdx.x + 1], gs), S);
        k = kept_steps_dev(ge - gs, rho);
    }
    const int64_t Sg = ge - gs;

    if (k <= 0 || k >= Sg) {
        for (int64_t s = gs + tid; s < ge; s += kSelThreads) {
            mask[s] = k > 0 ? 1 : 0;
            if (mask_l) mask_l[s] = k > 0 ? 1 : 0;
        }
        if (tid == 0 && n_kept) n_kept[blockIdx.x] = (int32_t)(k > 0 ? Sg : 0);
        return;
    }

    // the group's keys, read once (LDS when they fit)
    const bool staged = FUSED || Sg <= kSelLdsKeys;
    if (staged && !FUSED) {
        for (int64_t i = tid; i < Sg; i += kSelThreads) keys[i] = float_key(step_H[gs + i]);
        __syncthreads();
    }
    auto key_at = [&](int64_t i) -> uint32_t {
        return staged ? keys[i] : float_key(step_H[gs + i]);
    };

    if (FUSED || Sg <= kSelRankMax) {
        // small group: the rank of each step among the group (higher key
        // first, equal keys lower index first) decides directly; beyond 16
        // steps four work-items (of four waves) share a step's comparisons
        // (one alone: 256 steps took 4 us longer than the radix select, 64 steps 5.7 us
        // in place of 4.6, 33 4.8 in place of 4.3; 16 steps alike)
        static_assert(kSelThreads == 4 * kSelRankMax, "four work-items a step");
        const int n = (int)Sg, i = tid % kSelRankMax, way = tid / kSelRankMax;
        auto rank_of = [&](auto ways) {
            const uint32_t ki = keys[i];
            uint32_t r = 0;
#pragma unroll 8
            for (int j = ways.value > 1 ? way : 0; j < n; j += ways.value) {
                const uint32_t kj = keys[j];
                r += (kj > ki || (kj == ki && j < i)) ? 1 : 0;
            }
            return r;
        };
        uint32_t rank = 0;
        if (n <= 16) {
            if (tid < n) rank = rank_of(std::integral_constant<int, 1>{});
        } else {
            if (i < n) rank = rank_of(std::integral_constant<int, 4>{});
            if (tid < n) hist[tid] = 0;
            __syncthreads();
            if (i < n) atomicAdd(&hist[i], rank);
            __syncthreads();
            if (tid < n) rank = hist[tid];
        }
        if (tid < n) {
            mask[gs + tid] = (int64_t)rank < k ? 1 : 0;
            if (mask_l) mask_l[gs + tid] = (int64_t)rank < k ? 1 : 0;
        }
        if (tid == 0 && n_kept) n_kept[blockIdx.x] = (int32_t)k;
        return;
    }

    // radix select of the k-th largest key, 8 bits per pass from the top
    uint32_t prefix = 0, pmask = 0;
    int64_t remaining = k;
    for (int shift = 24; shift >= 0; shift -= 8) {
        for (int i = tid; i < 256; i += kSelThreads) hist[i] = 0;
        __syncthreads();
        for (int64_t i = tid; i < Sg; i += kSelThreads) {
            const uint32_t key = key_at(i);
            if ((key & pmask) == prefix) atomicAdd(&hist[(key >> shift) & 255u], 1u);
        }
        __syncthreads();
        if (wave == 0) {
            // lane l holds bins 255-4l .. 252-4l (descending key order)
            const int b0 = 255 - 4 * lane;
            const uint32_t c0 = hist[b0], c1 = hist[b0 - 1], c2 = hist[b0 - 2], c3 = hist[b0 - 3];
            const int64_t local = (int64_t)c0 + c1 + c2 + c3;
            int64_t incl = local;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const int64_t o = __shfl_up(incl, d);
                if (lane >= d) incl += o;
            }
            const int64_t excl = incl - local;
            if (excl < remaining && remaining <= incl) {
                int64_t r = remaining - excl;
                int bin = b0;
                if (r > c0) {
                    r -= c0;
                    bin = b0 - 1;
                    if (r > c1) {
                        r -= c1;
                        bin = b0 - 2;
                        if (r > c2) {
                            r -= c2;
                            bin = b0 - 3;
                        }
                    }
                }
                sel_bin = (uint32_t)bin;
                sel_remaining = r;
            }
        }
        __syncthreads();
        prefix |= sel_bin << shift;
        pmask |= 255u << shift;
        remaining = sel_remaining;
        __syncthreads();
    }

    // keep keys above the k-th; of the keys equal to it keep the first
    // `remaining` in step order (block scan over tiles of kSelThreads steps)
    int64_t carry = 0;
    for (int64_t base = 0; base < Sg; base += kSelThreads) {
        const int64_t i = base + tid;
        const uint32_t key = i < Sg ? key_at(i) : 0u;
        const bool eq = i < Sg && key == prefix;
        const uint64_t ballot = __ballot(eq);
        const int before = __popcll(ballot & ((1ull << lane) - 1ull));
        if (lane == 0) wave_count[wave] = __popcll(ballot);
        __syncthreads();
        int64_t wave_before = 0, total = 0;
        for (int w = 0; w < kSelWaves; ++w) {
            if (w < wave) wave_before += wave_count[w];
            total += wave_count[w];
        }
        if (i < Sg) {
            const int64_t rank = carry + wave_before + before;
            const uint8_t m = (key > prefix || (eq && rank < remaining)) ? 1 : 0;
            mask[gs + i] = m;
            if (mask_l) mask_l[gs + i] = m;
        }
        carry += total;
        __syncthreads();
    }
    if (tid == 0 && n_kept) n_kept[blockIdx.x] = (int32_t)k;
}

template <bool FUSED>
__global__ void __launch_bounds__(kSelThreads)
step_select_kernel(const float* __restrict__ H, int64_t T, const int32_t* __restrict__ off,
                   int64_t S, const int32_t* __restrict__ grp, double rho, int64_t k_all,
                   float* __restrict__ step_H, uint8_t* __restrict__ mask,
                   int32_t* __restrict__ n_kept) {
    __shared__ SelLds<FUSED ? kSelFusedSteps : kSelLdsKeys> sl;
    if constexpr (FUSED) {
        __shared__ float H_l[kSelLdsTokens];
        __shared__ int32_t off_l[kSelFusedSteps + 1];
        select_steps<true>(H, T, off, S, grp, rho, k_all, step_H, mask, n_kept, sl, H_l, off_l);
    } else {
        select_steps<false>(H, T, off, S, grp, rho, k_all, step_H, mask, n_kept, sl, nullptr,
                            nullptr);
    }
}

// ------------------------------------------------------------------------
// step-wise GRPO advantage (Sec. 3.3)
// ------------------------------------------------------------------------

constexpr int kAdvThreads = 256;
constexpr int64_t kAdvTokens = 2048, kAdvMaxPer = 16;

// gridDim.y workgroups per group, one for every kAdvTokens tokens of the average
// group and at most kAdvMaxPer. Over the group's steps (each step counts its
// trajectory's reward once): mean and population standard deviation, summed
// per trajectory with weight = its step count, in fp64, in a fixed order, in each
// of them; then every token of trajectory i gets (R_i - mean) / sd (0 when sd == 0),
// runs of 64 tokens dealt out to the group's workgroups and the trajectory's waves.
// (One workgroup a group wrote 152,569 tokens of 4 groups in 9.6 us. One wave for the
// 1000 tokens of a group's only trajectory, 40 such groups, took 5.3 us, all four 3.7.)
__global__ void __launch_bounds__(kAdvThreads)
grpo_advantage_kernel(const float* __restrict__ reward, const int32_t* __restrict__ traj_off,
                      int64_t n_traj, const int32_t* __restrict__ grp_off,
                      const int32_t* __restrict__ off, int64_t S, int64_t T,
                      float* __restrict__ adv, float* __restrict__ group_mean,
                      float* __restrict__ group_std) {
    __shared__ double red[2][kAdvThreads / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t i0 = min(max((int64_t)grp_off[blockIdx.x], (int64_t)0), n_traj);
    const int64_t i1 = min(max((int64_t)grp_off[blockIdx.x + 1], i0), n_traj);
    auto steps_of = [&](int64_t i, int64_t& a, int64_t& b) {
        a = min(max((int64_t)traj_off[i], (int64_t)0), S);
        b = min(max((int64_t)traj_off[i + 1], a), S);
    };
    auto block_sum2 = [&](double& x, double& y) {
        x = wave_sum(x);
        y = wave_sum(y);
        if (lane == 0) {
            red[0][wave] = x;
            red[1][wave] = y;
        }
        __syncthreads();
        x = 0.0;
        y = 0.0;
        for (int i = 0; i < kAdvThreads / 64; ++i) {
            x += red[0][i];
            y += red[1][i];
        }
        __syncthreads();
    };
    double cnt = 0.0, sum = 0.0;
    for (int64_t i = i0 + tid; i < i1; i += kAdvThreads) {
        int64_t a, b;
        steps_of(i, a, b);
        cnt += (double)(b - a);
        sum += (double)(b - a) * (double)reward[i];
    }
    block_sum2(cnt, sum);
    const double mean = cnt > 0.0 ? sum / cnt : 0.0;
    double sq = 0.0, unused = 0.0;
    for (int64_t i = i0 + tid; i < i1; i += kAdvThreads) {
        int64_t a, b;
        steps_of(i, a, b);
        const double d = (double)reward[i] - mean;
        sq += (double)(b - a) * d * d;
    }
    block_sum2(sq, unused);
    const double sd = cnt > 0.0 ? sqrt(sq / cnt) : 0.0;
    if (tid == 0 && blockIdx.y == 0) {
        if (group_mean) group_mean[blockIdx.x] = (float)mean;
        if (group_std) group_std[blockIdx.x] = (float)sd;
    }
    // a wave a trajectory, or where the group has fewer than four, two or all waves
    const int ways = i1 - i0 >= kAdvThreads / 64 ? 1 : i1 - i0 > 1 ? 2 : kAdvThreads / 64;
    const int64_t part = (int64_t)blockIdx.y * ways + wave % ways, parts = (int64_t)gridDim.y * ways;
    for (int64_t i = i0 + wave / ways; i < i1; i += kAdvThreads / 64 / ways) {
        int64_t a, b;
        steps_of(i, a, b);
        const float A = sd > 0.0 ? (float)(((double)reward[i] - mean) / sd) : 0.f;
        const int64_t t0 = min(max((int64_t)off[a], (int64_t)0), T);
        const int64_t t1 = min(max((int64_t)off[b], t0), T);
        for (int64_t t = t0 + part * 64 + lane; t < t1; t += parts * 64) adv[t] = A;
    }
}

// ------------------------------------------------------------------------
// K3: per-token TIS / clip coefficient and the loss
// ------------------------------------------------------------------------

struct LossConfig {
    float eps_low, eps_high, C, log_C;
    int kl, agg, ratio;
    float beta;
};

// Per token t of step s (M = 1 if the step is kept, else 0):
//   loss term  l_t = -M om_t (w o - beta kl_t),  o = min(r A, clip(r) A)
//   coefficient g_t = dL/dlogp_t = -M (Om w [u <= c] r A dlog - om_t beta dkl_t)
// with om_t the aggregation weight (1/N, 1/T or 1/(K |s|)). Token ratios use
// r = exp(logp - lp_old) and w = min(exp(lp_old - lp_roll), C) per token
// (Om = om_t, dlog = 1); step ratios use the sum (product) or mean (geometric
// mean) of the token log-ratios of the step and its mean advantage, shared by
// all its tokens (Om = om |s|, dlog = 1 or 1/|s|).
//
// Token ratios run on many workgroups (one CU cannot keep enough loads in
// flight to read T tokens quickly); each writes the partial sums of its
// tokens to a small workspace, and tis_loss_finalize_kernel adds them in
// workgroup order. Step ratios run one wave per step, on many workgroups too.
// Every sum is in fp64 and in a fixed order: per lane in token order, then a
// fixed butterfly, then waves, then workgroups.

// partial sums per workgroup, in this order
enum { kPartLoss = 0, kPartW, kPartClip, kPartCap, kPartKl, kParts };

constexpr int kCoefThreads = 256;  // workgroup of the many-workgroup launch
constexpr int kCoefWaves = kCoefThreads / 64;
constexpr int kCoefOneThreads = 1024;  // workgroup of the one-workgroup launch
constexpr int kCoefBatch = 4;  // tokens per lane whose loads are in flight together
constexpr int kCoefChunk = kCoefThreads * kCoefBatch;  // tokens per workgroup iteration
constexpr int kCoefMaxBlocks = 1024;
// up to this many tokens the one-workgroup launch is used even with a
// workspace: one launch instead of two (the finalize kernel). Measured on
// MI355X: at T = 512 one workgroup saves ~2.5 us a step; at T = 4096 the
// many-workgroup launch saves ~5 us.
constexpr int64_t kCoefOneBlockMaxT = 2048;
// up to this many tokens and steps the selection and the loss run in one workgroup
// in dart_select_tis_loss_fwd (its arithmetic grows with T, its step means with
// S). Measured on MI355X against the two calls (us): T = 2048, S = 64 13.0 and
// 13.6; T = 4096, S = 42 12.5 and 13.7, S = 128 18.6 and 14.1; T = 3000, S = 93
// 16.1 and 14.0; T = 6000, S = 62 15.2 and 14.5.
constexpr int64_t kSelCoefMaxT = 4096, kSelCoefMaxS = 80;
constexpr int kCoefLdsSteps = 8192;  // offsets and mask of up to this many steps go to LDS
constexpr int kStepCoefThreads = 1024;
constexpr int kStepCoefWaves = kStepCoefThreads / 64;
// up to this many steps (two a wave) the step ratios run on one workgroup also
// with a workspace: beyond, the finalize kernel costs less than a third step
constexpr int64_t kStepCoefOneBlockMaxS = 2 * kStepCoefWaves;

// workgroups of the many-workgroup launch for T tokens
__host__ __device__ constexpr int64_t coef_blocks(int64_t T) {
    return (T + kCoefChunk - 1) / kCoefChunk < kCoefMaxBlocks ? (T + kCoefChunk - 1) / kCoefChunk
                                                                : kCoefMaxBlocks;
}

// workspace: kParts doubles per workgroup, then N and K
__host__ __device__ constexpr int64_t coef_workspace_doubles(int64_t nblocks) {
    return nblocks * kParts + 2;
}

// KL estimators of D_KL(pi_theta || pi_ref) from the sampled token, with
// delta = log pi_ref - log pi_theta: k1 = -delta, k2 = delta^2 / 2,
// k3 = exp(delta) - delta - 1 (GRPO's), and their derivatives w.r.t.
// log pi_theta. In double: k3 cancels to O(delta^2) for small delta.
__device__ __forceinline__ void kl_terms(int kl, double delta, double& value, double& dlogp) {
    value = 0.0;
    dlogp = 0.0;
    if (kl == DART_KL_K1) {
        value = -delta;
        dlogp = 1.0;
    } else if (kl == DART_KL_K2) {
        value = 0.5 * delta * delta;
        dlogp = -delta;
    } else if (kl == DART_KL_K3) {
        const double e = exp(delta);
        value = e - delta - 1.0;
        dlogp = 1.0 - e;
    }
}

// Kept tokens N and kept steps K over all S steps, block-wide; with
// off_l/mask_l non-null the (clamped) offsets and the mask are also staged.
template <int THREADS>
__device__ __forceinline__ void count_kept(const int32_t* __restrict__ off,
                                           const uint8_t* __restrict__ mask, int64_t S, int64_t T,
                                           int32_t* off_l, uint8_t* mask_l,
                                           int64_t (*red)[THREADS / 64], int64_t& N, int64_t& K) {
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    int64_t n_local = 0, k_local = 0;
#pragma unroll 4
    for (int64_t s = tid; s < S; s += THREADS) {
        int64_t b, e;
        step_bounds(off, s, T, b, e);
        const uint8_t m = mask[s];
        if (off_l) {
            off_l[s] = (int32_t)b;
            mask_l[s] = m;
            if (s == S - 1) off_l[S] = (int32_t)e;
        }
        if (m) {
            n_local += e - b;
            k_local += 1;
        }
    }
    n_local = wave_sum_i64(n_local);
    k_local = wave_sum_i64(k_local);
    if (lane == 0) {
        red[0][wave] = n_local;
        red[1][wave] = k_local;
    }
    __syncthreads();
    N = 0;
    K = 0;
    for (int i = 0; i < THREADS / 64; ++i) {
        N += red[0][i];
        K += red[1][i];
    }
}

// N and K from offsets and mask already in LDS (as count_kept stages them).
template <int THREADS>
__device__ __forceinline__ void count_kept_lds(const int32_t* off_l, const uint8_t* mask_l,
                                               int64_t S, int64_t (*red)[THREADS / 64],
                                               int64_t& N, int64_t& K) {
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    int64_t n_local = 0, k_local = 0;
    // step s ends at max(off_l[s + 1], off_l[s]): the clamped end of step_bounds
    for (int64_t s = tid; s < S; s += THREADS)
        if (mask_l[s]) {
            n_local += (int64_t)max(off_l[s + 1], off_l[s]) - off_l[s];
            k_local += 1;
        }
    n_local = wave_sum_i64(n_local);
    k_local = wave_sum_i64(k_local);
    if (lane == 0) {
        red[0][wave] = n_local;
        red[1][wave] = k_local;
    }
    lds_barrier();
    N = 0;
    K = 0;
    for (int i = 0; i < THREADS / 64; ++i) {
        N += red[0][i];
        K += red[1][i];
    }
}

// Sums the kParts per-lane values over the block in a fixed order (butterfly
// within each wave, then a butterfly over the wave totals in wave 0); the
// result is valid in thread 0.
template <int THREADS>
__device__ __forceinline__ void block_sum_parts(double (&acc)[kParts],
                                                double (*red)[THREADS / 64]) {
    constexpr int WAVES = THREADS / 64;
    static_assert(WAVES <= 64, "one wave adds the wave totals");
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
#pragma unroll
    for (int i = 0; i < kParts; ++i) acc[i] = wave_sum(acc[i]);
    if (lane == 0)
#pragma unroll
        for (int i = 0; i < kParts; ++i) red[i][wave] = acc[i];
    lds_barrier();
    if (wave == 0)
#pragma unroll
        for (int i = 0; i < kParts; ++i) acc[i] = wave_sum(lane < WAVES ? red[i][lane] : 0.0);
}

// Loss and stats = {clip fraction, mean TIS weight, capped fraction, N, mean
// KL, K} (the first nstats of them) from the summed parts.
__device__ __forceinline__ void write_loss(const double (&acc)[kParts], double N, double K,
                                           double* loss, float* stats, int nstats) {
    const double inv_n = N > 0 ? 1.0 / N : 0.0;
    loss[0] = acc[kPartLoss];
    if (stats) {
        const float out[6] = {(float)(acc[kPartClip] * inv_n), (float)(acc[kPartW] * inv_n),
                              (float)(acc[kPartCap] * inv_n), (float)N,
                              (float)(acc[kPartKl] * inv_n), (float)K};
        for (int j = 0; j < nstats; ++j) stats[j] = out[j];
    }
}

// Token ratios. Workgroup b takes chunks b, b + grid, ... of THREADS *
// kCoefBatch tokens; lane tokens are THREADS apart within a chunk (coalesced).
// The step of each token is found by binary search over the offsets. With
// part != null each workgroup writes its partial sums there (workgroup 0 also
// N and K); with part == null the grid is one workgroup, which writes the loss
// and stats itself.
template <int THREADS>
struct CoefRed {
    int64_t i[2][THREADS / 64];
    double d[kParts][THREADS / 64];
};

// The lane's tokens of one chunk of THREADS * kCoefBatch tokens (zeros past T).
struct CoefTokens {
    float A[kCoefBatch], lp[kCoefBatch], lpo[kCoefBatch], lpr[kCoefBatch], lpf[kCoefBatch];
};

template <int THREADS>
__device__ __forceinline__ void load_coef_tokens(CoefTokens& x, int64_t c, int64_t T,
                                                 const float* __restrict__ logp,
                                                 const float* __restrict__ lp_old,
                                                 const float* __restrict__ lp_roll,
                                                 const float* __restrict__ lp_ref,
                                                 const float* __restrict__ adv, bool with_kl) {
    constexpr int CHUNK = THREADS * kCoefBatch;
#pragma unroll
    for (int j = 0; j < kCoefBatch; ++j) {
        const int64_t t = c * CHUNK + threadIdx.x + (int64_t)j * THREADS;
        x.A[j] = x.lp[j] = x.lpo[j] = x.lpr[j] = x.lpf[j] = 0.f;
        if (t < T) {
            x.A[j] = adv[t];
            x.lp[j] = logp[t];
            x.lpo[j] = lp_old[t];
            x.lpr[j] = lp_roll[t];
            if (with_kl) x.lpf[j] = lp_ref[t];
        }
    }
}

// PRE: the caller has put the clamped offsets (off_l[s] = first token of step
// s, off_l[S] = T) and the mask in LDS (S <= kCoefLdsSteps) and loaded this
// workgroup's first chunk into x; else both happen here.
template <bool GENERAL, int THREADS, bool PRE = false>
__device__ __forceinline__ void coef_tokens(
    int64_t T, const float* __restrict__ logp, const float* __restrict__ lp_old,
    const float* __restrict__ lp_roll, const float* __restrict__ lp_ref,
    const float* __restrict__ adv, const int32_t* __restrict__ off, int64_t S,
    const uint8_t* __restrict__ mask, const LossConfig& cfg, float* __restrict__ coef,
    double* __restrict__ part, double* __restrict__ loss, float* __restrict__ stats, int nstats,
    int32_t* off_l, uint8_t* mask_l, CoefRed<THREADS>& red, CoefTokens& x) {
    constexpr int CHUNK = THREADS * kCoefBatch;
    auto& red_i = red.i;
    auto& red_d = red.d;

    const int tid = threadIdx.x;
    const bool with_kl = GENERAL && cfg.kl != DART_KL_NONE;
    const int64_t nchunks = (T + CHUNK - 1) / CHUNK;
    // the lane's tokens of a chunk: loaded before they are needed (the first
    // chunk's loads are in flight while the kept counts are taken)
    float(&A)[kCoefBatch] = x.A;
    float(&lp)[kCoefBatch] = x.lp;
    float(&lpo)[kCoefBatch] = x.lpo;
    float(&lpr)[kCoefBatch] = x.lpr;
    float(&lpf)[kCoefBatch] = x.lpf;
    auto load_chunk = [&](int64_t c) {
        load_coef_tokens<THREADS>(x, c, T, logp, lp_old, lp_roll, lp_ref, adv, with_kl);
    };
    if (!PRE && (int64_t)blockIdx.x < nchunks) load_chunk(blockIdx.x);

    const bool staged = PRE || S <= kCoefLdsSteps;
    int64_t N, K;
    if constexpr (PRE)
        count_kept_lds<THREADS>(off_l, mask_l, S, red_i, N, K);
    else
        count_kept<THREADS>(off, mask, S, T, staged ? off_l : nullptr, staged ? mask_l : nullptr,
                            red_i, N, K);
    if (part && blockIdx.x == 0 && tid == 0) {
        part[(int64_t)gridDim.x * kParts] = (double)N;
        part[(int64_t)gridDim.x * kParts + 1] = (double)K;
    }

    const double inv_n = N > 0 ? 1.0 / (double)N : 0.0;
    const float lo = 1.f - cfg.eps_low, hi = 1.f + cfg.eps_high;
    const double beta = (double)cfg.beta;
    auto weight = [&](int64_t len) -> double {
        if (GENERAL && cfg.agg == DART_AGG_TOKEN_MEAN_ALL) return 1.0 / (double)T;
        if (GENERAL && cfg.agg == DART_AGG_STEP_MEAN) return 1.0 / ((double)K * (double)len);
        return inv_n;
    };
    // largest power of two below S (binary search over step indices [0, S-1])
    int64_t top = 0;
    if (S > 1) {
        top = 1;
        while (top * 2 <= S - 1) top *= 2;
    }

    double acc[kParts] = {0.0, 0.0, 0.0, 0.0, 0.0};
    // the token loop, compiled twice: offsets and mask in LDS or in global
    // memory (a run-time choice per access would serialise the probes)
    auto token_loop = [&](auto staged_tag) {
        constexpr bool STAGED = decltype(staged_tag)::value;
        auto off_at = [&](int64_t i) -> int64_t {
            if constexpr (STAGED)
                return (int64_t)off_l[i];
            else
                return min(max((int64_t)off[i], (int64_t)0), T);
        };
        for (int64_t c = blockIdx.x; c < nchunks; c += gridDim.x) {
            if (c != (int64_t)blockIdx.x) load_chunk(c);
            const int64_t base = c * CHUNK + tid;
            // step of each token: the last s with off[s] <= t, the lane's tokens
            // searched together (every probe of a round issued before any is used)
            int64_t st[kCoefBatch];
#pragma unroll
            for (int j = 0; j < kCoefBatch; ++j) st[j] = 0;
            for (int64_t stride = top; stride > 0; stride >>= 1) {
                int64_t probe[kCoefBatch];
#pragma unroll
                for (int j = 0; j < kCoefBatch; ++j) probe[j] = off_at(min(st[j] + stride, S - 1));
#pragma unroll
                for (int j = 0; j < kCoefBatch; ++j) {
                    const int64_t t = base + (int64_t)j * THREADS;
                    st[j] = (st[j] + stride < S && probe[j] <= t) ? st[j] + stride : st[j];
                }
            }
#pragma unroll
            for (int j = 0; j < kCoefBatch; ++j) {
                const int64_t t = base + (int64_t)j * THREADS;
                if (t >= T) break;
                const bool kept = N > 0 && (STAGED ? mask_l[st[j]] : mask[st[j]]) != 0;
                if (!kept) {
                    coef[t] = 0.f;
                    continue;
                }
                const double om = weight(off_at(st[j] + 1) - off_at(st[j]));
                const float r = expf(lp[j] - lpo[j]);
                const float d = lpo[j] - lpr[j];
                const bool capped = d >= cfg.log_C;
                const float wf = capped ? cfg.C : fminf(expf(d), cfg.C);
                const float rc = fminf(fmaxf(r, lo), hi);
                const float u = r * A[j];
                const float cl = rc * A[j];
                const bool gate = u <= cl;
                const double w = (double)wf;
                const double obj = w * (double)fminf(u, cl);
                const double dobj = gate ? w * (double)A[j] * (double)r : 0.0;
                double klv = 0.0, kld = 0.0;
                if (with_kl) kl_terms(cfg.kl, (double)lpf[j] - (double)lp[j], klv, kld);
                acc[kPartLoss] -= om * (obj - beta * klv);
                coef[t] = (float)(-(om * dobj - om * beta * kld));
                acc[kPartW] += w;
                acc[kPartClip] += gate ? 0.0 : 1.0;
                acc[kPartCap] += capped ? 1.0 : 0.0;
                acc[kPartKl] += klv;
            }
        }
    };
    if (staged)
        token_loop(std::true_type{});
    else
        token_loop(std::false_type{});
    block_sum_parts<THREADS>(acc, red_d);
    if (tid != 0) return;
    if (part)
#pragma unroll
        for (int i = 0; i < kParts; ++i) part[(int64_t)blockIdx.x * kParts + i] = acc[i];
    else
        write_loss(acc, (double)N, (double)K, loss, stats, nstats);
}

template <bool GENERAL, int THREADS>
__global__ void __launch_bounds__(THREADS)
tis_coef_kernel(int64_t T, const float* __restrict__ logp, const float* __restrict__ lp_old,
                const float* __restrict__ lp_roll, const float* __restrict__ lp_ref,
                const float* __restrict__ adv, const int32_t* __restrict__ off, int64_t S,
                const uint8_t* __restrict__ mask, LossConfig cfg, float* __restrict__ coef,
                double* __restrict__ part, double* __restrict__ loss, float* __restrict__ stats,
                int nstats) {
    __shared__ int32_t off_l[kCoefLdsSteps + 1];
    __shared__ uint8_t mask_l[kCoefLdsSteps];
    __shared__ CoefRed<THREADS> red;
    CoefTokens x;
    coef_tokens<GENERAL, THREADS>(T, logp, lp_old, lp_roll, lp_ref, adv, off, S, mask, cfg, coef,
                                  part, loss, stats, nstats, off_l, mask_l, red, x);
}

// Step selection and token coefficients of one group in one workgroup (T <=
// kSelCoefMaxT <= kSelLdsTokens, S <= kSelCoefMaxS, token ratios, token mean
// over kept tokens): select_steps with the means fused in, then coef_tokens of the
// one-workgroup launch, the two sharing the staged offsets. Its outputs are
// those of step_select_kernel<true> followed by tis_coef_kernel<false,
// kCoefOneThreads>, bit for bit.
__global__ void __launch_bounds__(kSelThreads)
select_coef_kernel(const float* __restrict__ H, int64_t T, const int32_t* __restrict__ off,
                   int64_t S, double rho, int64_t k, float* __restrict__ step_H,
                   uint8_t* __restrict__ mask, int32_t* __restrict__ n_kept,
                   const float* __restrict__ logp, const float* __restrict__ lp_old,
                   const float* __restrict__ lp_roll, const float* __restrict__ adv,
                   LossConfig cfg, float* __restrict__ coef, double* __restrict__ loss,
                   float* __restrict__ stats, int nstats) {
    static_assert(kSelThreads == kCoefOneThreads, "one workgroup size for both parts");
    static_assert(kSelCoefMaxT <= kSelLdsTokens, "the entropies fit the selection's LDS");
    static_assert(kSelCoefMaxS <= kSelFusedSteps && kSelFusedSteps <= kCoefLdsSteps,
                  "the staged offsets serve both parts");
    __shared__ SelLds<kSelFusedSteps> sl;
    __shared__ float H_l[kSelCoefMaxT];
    __shared__ int32_t off_l[kSelFusedSteps + 1];
    __shared__ uint8_t mask_l[kSelFusedSteps];
    __shared__ CoefRed<kCoefOneThreads> red;
    // the first chunk of tokens is in flight during the selection
    CoefTokens x;
    load_coef_tokens<kCoefOneThreads>(x, 0, T, logp, lp_old, lp_roll, nullptr, adv, false);
    select_steps<true>(H, T, off, S, nullptr, rho, k, step_H, mask, n_kept, sl, H_l, off_l,
                       mask_l);
    lds_barrier();  // the staged offsets and the mask in LDS
    coef_tokens<false, kCoefOneThreads, true>(T, logp, lp_old, lp_roll, nullptr, adv, off, S,
                                              mask, cfg, coef, nullptr, loss, stats, nstats,
                                              off_l, mask_l, red, x);
}

// Step ratios: one wave per step, the step's sums first. Workgroup b takes
// steps b * kStepCoefWaves + wave, then every gridDim.x * kStepCoefWaves-th;
// with part != null it writes its partial sums there (workgroup 0 also N and
// K) for tis_loss_finalize_kernel, with part == null the grid is one workgroup,
// which writes the loss and stats itself.
// A step costs a wave ~2 us of dependent loads and fp64 arithmetic, whatever
// its length up to a few hundred tokens, so the steps have to run beside each
// other: 1600 steps of 95 tokens took 200 us on one workgroup (100 steps a
// wave). With BATCH a lane's next kStepBatch tokens are loaded together.
constexpr int kStepBatch = 4;
template <bool BATCH>
__global__ void __launch_bounds__(kStepCoefThreads)
tis_coef_step_kernel(int64_t T, const float* __restrict__ logp, const float* __restrict__ lp_old,
                     const float* __restrict__ lp_roll, const float* __restrict__ lp_ref,
                     const float* __restrict__ adv, const int32_t* __restrict__ off, int64_t S,
                     const uint8_t* __restrict__ mask, LossConfig cfg, float* __restrict__ coef,
                     double* __restrict__ part, double* __restrict__ loss,
                     float* __restrict__ stats, int nstats) {
    __shared__ int64_t red_i[2][kStepCoefWaves];
    __shared__ double red_d[kParts][kStepCoefWaves];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    int64_t N, K;
    count_kept<kStepCoefThreads>(off, mask, S, T, nullptr, nullptr, red_i, N, K);
    if (part && blockIdx.x == 0 && tid == 0) {
        part[(int64_t)gridDim.x * kParts] = (double)N;
        part[(int64_t)gridDim.x * kParts + 1] = (double)K;
    }

    const double inv_n = N > 0 ? 1.0 / (double)N : 0.0;
    const float lo = 1.f - cfg.eps_low, hi = 1.f + cfg.eps_high;
    const bool with_kl = cfg.kl != DART_KL_NONE;
    const double beta = (double)cfg.beta;
    double acc[kParts] = {0.0, 0.0, 0.0, 0.0, 0.0};
    // in a register: the grid's size would be loaded again for every step
    uint32_t stride = gridDim.x * kStepCoefWaves;
    asm volatile("" : "+s"(stride));
    for (int64_t s = (int64_t)blockIdx.x * kStepCoefWaves + wave; s < S; s += stride) {
        int64_t b, e;
        step_bounds(off, s, T, b, e);
        const int64_t len = e - b;
        const bool kept = mask[s] != 0 && N > 0;
        if (!kept) {
            for (int64_t t = b + lane; t < e; t += 64) coef[t] = 0.f;
            continue;
        }
        double om = inv_n;
        if (cfg.agg == DART_AGG_TOKEN_MEAN_ALL) om = 1.0 / (double)T;
        if (cfg.agg == DART_AGG_STEP_MEAN) om = 1.0 / ((double)K * (double)len);
        double slr = 0.0, slw = 0.0, sa = 0.0, dlog = 1.0;
        if constexpr (!BATCH) {
            for (int64_t t = b + lane; t < e; t += 64) {
                slr += (double)logp[t] - (double)lp_old[t];
                slw += (double)lp_old[t] - (double)lp_roll[t];
                sa += (double)adv[t];
            }
        } else {
            for (int64_t t0 = b + lane; t0 < e; t0 += 64 * kStepBatch) {
                float lp[kStepBatch], lpo[kStepBatch], lpr[kStepBatch], A[kStepBatch];
#pragma unroll
                for (int j = 0; j < kStepBatch; ++j) {
                    const int64_t t = t0 + 64 * j;
                    // tokens past the step's end add exact zeros
                    lp[j] = lpo[j] = lpr[j] = A[j] = 0.f;
                    if (t < e) {
                        lp[j] = logp[t];
                        lpo[j] = lp_old[t];
                        lpr[j] = lp_roll[t];
                        A[j] = adv[t];
                    }
                }
#pragma unroll
                for (int j = 0; j < kStepBatch; ++j) {
                    slr += (double)lp[j] - (double)lpo[j];
                    slw += (double)lpo[j] - (double)lpr[j];
                    sa += (double)A[j];
                }
            }
        }
        slr = wave_sum(slr);
        slw = wave_sum(slw);
        sa = wave_sum(sa);
        if (cfg.ratio == DART_RATIO_STEP_GEOMEAN) {
            slr /= (double)len;
            slw /= (double)len;
            dlog = 1.0 / (double)len;
        }
        const double r_s = exp(slr);
        const bool capped = slw >= (double)cfg.log_C;
        const double w = capped ? (double)cfg.C : fmin(exp(slw), (double)cfg.C);
        const double A_s = sa / (double)len;
        const double om_obj = om * (double)len;
        const double rc = fmin(fmax(r_s, (double)lo), (double)hi);
        const double u = r_s * A_s;
        const double cl = rc * A_s;
        const bool gate = u <= cl;
        const double obj = w * fmin(u, cl);
        const double dobj = gate ? w * r_s * A_s * dlog : 0.0;
        for (int64_t t = b + lane; t < e; t += 64) {
            double klv = 0.0, kld = 0.0;
            if (with_kl) kl_terms(cfg.kl, (double)lp_ref[t] - (double)logp[t], klv, kld);
            acc[kPartLoss] -= om * (obj - beta * klv);
            coef[t] = (float)(-(om_obj * dobj - om * beta * kld));
            acc[kPartW] += w;
            acc[kPartClip] += gate ? 0.0 : 1.0;
            acc[kPartCap] += capped ? 1.0 : 0.0;
            acc[kPartKl] += klv;
        }
    }
    block_sum_parts<kStepCoefThreads>(acc, red_d);
    if (tid != 0) return;
    if (part)
#pragma unroll
        for (int i = 0; i < kParts; ++i) part[(int64_t)blockIdx.x * kParts + i] = acc[i];
    else
        write_loss(acc, (double)N, (double)K, loss, stats, nstats);
}

// Adds the nblocks partial sums in workgroup order and writes the loss and
// stats.
__global__ void __launch_bounds__(kCoefThreads)
tis_loss_finalize_kernel(const double* __restrict__ part, int64_t nblocks,
                         double* __restrict__ loss, float* __restrict__ stats, int nstats) {
    __shared__ double red_d[kParts][kCoefWaves];
    double acc[kParts] = {0.0, 0.0, 0.0, 0.0, 0.0};
    for (int64_t b = threadIdx.x; b < nblocks; b += kCoefThreads)
#pragma unroll
        for (int i = 0; i < kParts; ++i) acc[i] += part[b * kParts + i];
    block_sum_parts<kCoefThreads>(acc, red_d);
    if (threadIdx.x == 0)
        write_loss(acc, part[nblocks * kParts], part[nblocks * kParts + 1], loss, stats, nstats);
}

// ------------------------------------------------------------------------
// K4: dlogits = coef * (onehot(target) - softmax(z))
// ------------------------------------------------------------------------

// dlogits[t, v] = it * g_t * (onehot(y_t)[v] - exp(it * z_tv - lse_t)), it the
// inverse temperature, written in the logits dtype (bf16 rounded to nearest
// even). The body of each row is cut into chunks of THREADS * UNROLL 16-byte
// vectors, and workgroup b takes chunk b % nchunk of row b / nchunk in one shot;
// chunk 0 also takes the row's unaligned head and tail elements. Small one-shot
// workgroups walking along the rows keep HBM busier than long per-row loops. (The
// compiler waits for a lane's first load ahead of its second, which is under a
// condition. With both out at once 6000 x 32003 bf16 takes 135 us in place of 143, but
// 4096 x 152064 400 in place of 384, and fp32 rows 0 to 5% longer.)
// The vectors are those of the output row (16-byte stores); where the logits row has
// another alignment (a padded head's logits cut to an odd vocabulary, the gradient
// contiguous) they are loaded as they lie, in the same instruction. (Such rows went
// element by element through chunk 0's workgroup: at T = 2000, V = 50257 in rows of
// 50304, 282 us; as vectors 69 us, the bytes alone at the rate of a copy 64 us.)
// The target element uses 1 - p_y = -expm1(logp_y), accurate when p_y -> 1. dlogits
// may be the logits buffer itself (in place): each element is read, then written, by
// the same lane.
// A row whose coefficient is zero (a dropped step's, a clipped token's) is written
// without reading its logits: with a finite lse, and logits that are finite or -inf,
// every 2^x is finite, so the product is the zero of -g's sign that is written
// (DART_GRAD_SKIP_ZERO_ROWS: +0, whatever lse). A NaN or +inf logit is not seen: the
// statistics drop it from the row's sums, so that lse need not tell of it, and where
// its product would be NaN a zero is written. At T = 16384, V = 151936 with a quarter
// of the steps kept the pass takes 1.00 ms against 1.58 for reading every row, at T =
// 4096, V = 152064 with four fifths kept 0.375 against 0.388.
template <dart_dtype_t D, int THREADS, int UNROLL, bool NTL, bool NTS>
__global__ void __launch_bounds__(THREADS)
tis_grad_kernel(const void* logits, int64_t V, int64_t ld,
                      const int32_t* __restrict__ target, const float* __restrict__ lse,
                      const float* __restrict__ logp, const float* __restrict__ coef,
                      float inv_temp, uint32_t flags, void* dlogits, int64_t ld_out, int64_t T,
                      int64_t nchunk) {
    using E = typename Elt<D>::T;
    constexpr int EPV = Elt<D>::kPerVec;
    constexpr int PER = THREADS * UNROLL;
    const int tid = threadIdx.x;
    const int64_t nblocks = T * nchunk;
    for (int64_t b = blockIdx.x; b < nblocks; b += gridDim.x) {
        const int64_t t = b / nchunk;
        const int64_t c = b - t * nchunk;
        const E* row = static_cast<const E*>(logits) + t * ld;
        E* orow = static_cast<E*>(dlogits) + t * ld_out;
        const int64_t y_in = target[t];
        const int64_t y = (y_in >= 0 && y_in < V) ? y_in : -1;
        const float g = coef[t] * inv_temp;
        const float neg_g = -g;
        const float k = inv_temp * kLog2e;
        const float l = lse[t], lb = l * kLog2e;
        const RowLayout L = row_layout<D>(orow, V);
        const bool skip = flags & DART_GRAD_SKIP_ZERO_ROWS;
        const bool zero_row = g == 0.f && (skip || fabsf(l) < INFINITY);
        const float fill = skip ? 0.f : neg_g;
        const float dy = zero_row && skip ? 0.f : g * -expm1f(logp[t]);

        const E* body = row + L.head;
        u32x4* vout = reinterpret_cast<u32x4*>(orow + L.head);
        const int64_t base = c * PER + tid;
        if (zero_row) {
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) {
                const int64_t j = base + (int64_t)u * THREADS;
                if (j >= L.nvec) continue;
                float z[EPV];
#pragma unroll
                for (int e = 0; e < EPV; ++e) z[e] = L.head + j * EPV + e == y ? dy : fill;
                vstore<NTS>(pack<D>(z), vout + j);
            }
        } else {
            u32x4 v[UNROLL];
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) {
                const int64_t j = base + (int64_t)u * THREADS;
                if (j < L.nvec) v[u] = vload_any<NTL>(body + j * EPV);
            }
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) {
                const int64_t j = base + (int64_t)u * THREADS;
                if (j >= L.nvec) continue;
                float z[EPV];
                unpack<D>(v[u], z);
#pragma unroll
                for (int e = 0; e < EPV; ++e) {
                    z[e] = neg_g * __builtin_amdgcn_exp2f(fmaf(z[e], k, -lb));
                    if (L.head + j * EPV + e == y) z[e] = dy;
                }
                vstore<NTS>(pack<D>(z), vout + j);
            }
        }
        if (c == 0) {
            const int64_t nscalar = L.head + (V - L.body_end);
            for (int64_t q = tid; q < nscalar; q += THREADS) {
                const int64_t col = q < L.head ? q : L.body_end + (q - L.head);
                float d = fill;
                if (!zero_row) d = neg_g * __builtin_amdgcn_exp2f(fmaf(load_one<D>(row, col), k, -lb));
                store_one<D>(orow, col, col == y ? dy : d);
            }
        }
    }
}

// ------------------------------------------------------------------------
// host helpers
// ------------------------------------------------------------------------

bool bad_dtype(dart_dtype_t d) { return d != DART_F32 && d != DART_BF16; }

size_t elem_size(dart_dtype_t d) { return d == DART_F32 ? 4 : 2; }

// dlogits may alias logits exactly (same base, same row stride); any other
// overlap of the two [T, ld] row ranges is rejected.
bool bad_overlap(const void* logits, int64_t ld, const void* dlogits, int64_t ld_out, int64_t T,
                 int64_t V, size_t es) {
    const uintptr_t a0 = reinterpret_cast<uintptr_t>(logits);
    const uintptr_t a1 = a0 + (uintptr_t)(((T - 1) * ld + V) * (int64_t)es);
    const uintptr_t b0 = reinterpret_cast<uintptr_t>(dlogits);
    const uintptr_t b1 = b0 + (uintptr_t)(((T - 1) * ld_out + V) * (int64_t)es);
    const bool alias = a0 == b0 && ld == ld_out;
    return !alias && a0 < b1 && b0 < a1;
}

dart_status_t launch_status() {
    return hipGetLastError() == hipSuccess ? DART_OK : DART_ERR_HIP;
}

// Threads per row of the statistics pass for rows of nvec vectors. A row is a
// chain of loads, reduction and finish, so short rows want many small workgroups
// on a compute unit and long ones enough loads in flight to need few iterations.
// Measured (us; 768 threads as every row had before, then the choice, its
// neighbours in brackets):
//   T 16384, V   2048 bf16 (256 vectors)   110 -> 128: 18 [256: 21]
//   T 16000, V   8000 bf16 (1000)          147 -> 256: 44 [128: 45, 512: 54]
//   T  6000, V  32003 bf16 (4000)           94 -> 512: 60 [256: 66, 768: 73]
//   T  4096, V 152064 bf16 (19008)         183 -> 768: 183 [512: 187, 1024: 184]
// The number of rows does not enter: the threads are the order of a row's sums, and
// the same row has the same statistics in a call of any size. (Few rows have a compute
// unit each and want its width, but not by much: T = 200, V = 32000 fp32, 8000
// vectors, 7.9 -> 512: 5.8 [768: 5.6].)
int stats_threads(int64_t nvec) {
    if (nvec <= 512) return 128;
    if (nvec <= 2048) return 256;
    return nvec <= 8192 ? 512 : 768;
}

// f(dtype, non-temporal loads) as compile-time constants.
template <class F>
void with_logits(dart_dtype_t dtype, int64_t T, int64_t V, F&& f) {
    using BF16 = std::integral_constant<dart_dtype_t, DART_BF16>;
    using F32 = std::integral_constant<dart_dtype_t, DART_F32>;
    const bool nt = V > kCachedLogits / (T * (int64_t)elem_size(dtype));
    if (dtype == DART_BF16)
        nt ? f(BF16{}, std::true_type{}) : f(BF16{}, std::false_type{});
    else
        nt ? f(F32{}, std::true_type{}) : f(F32{}, std::false_type{});
}

template <int THREADS>
void launch_tok_stats(const void* logits, dart_dtype_t dtype, int64_t T, int64_t V, int64_t ld,
                      const int32_t* target, float inv_temp, float* logp, float* entropy,
                      float* lse, hipStream_t stream) {
    constexpr int64_t most = kStatsMaxRows;
    static_assert(most * THREADS <= 0xFFFFFFFFll, "statistics grid");
    for (int64_t r0 = 0; r0 < T; r0 += most) {
        const dim3 grid((unsigned)(T - r0 < most ? T - r0 : most)), block(THREADS);
        const void* lr =
            static_cast<const char*>(logits) + (size_t)r0 * (size_t)ld * elem_size(dtype);
        auto go = [&](auto dt, auto nt) {
            hipLaunchKernelGGL((tok_stats_kernel<decltype(dt)::value, THREADS, kStatsUnroll,
                                                 decltype(nt)::value>),
                               grid, block, 0, stream, lr, V, ld, target + r0, inv_temp, logp + r0,
                               entropy + r0, lse + r0);
        };
        with_logits(dtype, T, V, go);
    }
}

// Workgroups of the step ratios, for which a workspace of the split size has room: one
// for every 16 tokens, that is, for every step a wave, however short the steps, and
// one a compute unit at most (each counts the kept steps for itself: 20,000 steps take
// 32 us on 149 workgroups and 45 on 1024).
constexpr int64_t kStepMaxBlocks = 256;
constexpr int64_t spare_blocks(int64_t T) {
    return T > int64_t(kStepCoefWaves) * kStepMaxBlocks ? kStepMaxBlocks
                                                       : (T + kStepCoefWaves - 1) / kStepCoefWaves;
}
static_assert(spare_blocks(1) >= coef_blocks(1) &&
                  spare_blocks(kSelCoefMaxT) >= coef_blocks(kSelCoefMaxT),
              "the spare part serves the token ratios of small fused selections too");

// Step ratios load a lane's tokens in batches from this many tokens a mean step on:
// below, most places of a batch are empty, and adding up their zeros is work. On one
// workgroup, batches and one token at a time: 5000 steps of 1 token 573 and 546 us,
// 20,000 of 8 2290 and 2210; 1600 of 95 229 either way.
constexpr int64_t kStepBatchTokens = 48;

// What a loss workspace of the split size has beyond the plain size, null where it is
// smaller. Step ratios and small fused selections leave their partial sums there: the
// plain part is untouched by them, so that a caller may share it with them unordered.
double* spare_part(void* workspace, size_t bytes, int64_t T) {
    return workspace && bytes >= dart_tis_loss_split_workspace_bytes(T)
               ? reinterpret_cast<double*>(static_cast<char*>(workspace) +
                                           dart_tis_loss_workspace_bytes(T))
               : nullptr;
}

// K3 and the loss reduction for one configuration: up to kCoefMaxBlocks
// workgroups plus the finalize kernel when a workspace (step ratios: a spare part) is
// given and T > kCoefOneBlockMaxT (token ratios) or S > kStepCoefOneBlockMaxS (step
// ratios), else one workgroup.
dart_status_t launch_tis_coef(bool general, int64_t T, const float* logp, const float* lp_old,
                              const float* lp_roll, const float* lp_ref, const float* adv,
                              const int32_t* off, int64_t S, const uint8_t* mask,
                              const LossConfig& cfg, float* coef, double* loss, float* stats,
                              int nstats, void* workspace, double* spare, hipStream_t stream) {
    if (general && cfg.ratio != DART_RATIO_TOKEN) {
        // never more workgroups than the spare part has room for
        const int64_t want = (S + kStepCoefWaves - 1) / kStepCoefWaves, room = spare_blocks(T);
        const int64_t nb = !spare || S <= kStepCoefOneBlockMaxS ? 1 : want < room ? want : room;
        double* part = nb > 1 ? spare : nullptr;
        auto launch = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3((unsigned)nb), dim3(kStepCoefThreads), 0, stream, T,
                               logp, lp_old, lp_roll, lp_ref, adv, off, S, mask, cfg, coef, part,
                               loss, stats, nstats);
        };
        if (T >= kStepBatchTokens * S)
            launch(tis_coef_step_kernel<true>);
        else
            launch(tis_coef_step_kernel<false>);
        if (part)
            hipLaunchKernelGGL(tis_loss_finalize_kernel, dim3(1), dim3(kCoefThreads), 0, stream,
                               part, nb, loss, stats, nstats);
        return launch_status();
    }
    if (!workspace || T <= kCoefOneBlockMaxT) {
        if (general)
            hipLaunchKernelGGL((tis_coef_kernel<true, kCoefOneThreads>), dim3(1),
                               dim3(kCoefOneThreads), 0, stream, T, logp, lp_old, lp_roll, lp_ref,
                               adv, off, S, mask, cfg, coef, nullptr, loss, stats, nstats);
        else
            hipLaunchKernelGGL((tis_coef_kernel<false, kCoefOneThreads>), dim3(1),
                               dim3(kCoefOneThreads), 0, stream, T, logp, lp_old, lp_roll, lp_ref,
                               adv, off, S, mask, cfg, coef, nullptr, loss, stats, nstats);
        return launch_status();
    }
    const int64_t nblocks = coef_blocks(T);
    double* part = static_cast<double*>(workspace);
    if (general)
        hipLaunchKernelGGL((tis_coef_kernel<true, kCoefThreads>), dim3((unsigned)nblocks),
                           dim3(kCoefThreads), 0, stream, T, logp, lp_old, lp_roll, lp_ref, adv,
                           off, S, mask, cfg, coef, part, nullptr, nullptr, 0);
    else
        hipLaunchKernelGGL((tis_coef_kernel<false, kCoefThreads>), dim3((unsigned)nblocks),
                           dim3(kCoefThreads), 0, stream, T, logp, lp_old, lp_roll, lp_ref, adv,
                           off, S, mask, cfg, coef, part, nullptr, nullptr, 0);
    hipLaunchKernelGGL(tis_loss_finalize_kernel, dim3(1), dim3(kCoefThreads), 0, stream, part,
                       nblocks, loss, stats, nstats);
    return launch_status();
}

// A workspace is either absent or large enough and 8-byte aligned.
bool bad_workspace(const void* workspace, size_t bytes, int64_t T) {
    if (!workspace) return false;
    return bytes < (size_t)coef_workspace_doubles(coef_blocks(T)) * sizeof(double) ||
           reinterpret_cast<uintptr_t>(workspace) % sizeof(double) != 0;
}

// Host-side argument rules of dart_tis_loss_fwd_bwd (both halves), workspace
// aside: true when the call must return DART_ERR_INVALID_ARG.
bool bad_fwd_bwd_args(const void* logits, dart_dtype_t dtype, int64_t T, int64_t V, int64_t ld,
                      const int32_t* target, const float* logp, const float* lse,
                      const float* logp_old, const float* logp_rollout, const float* adv,
                      const int32_t* step_offsets, int64_t S, const uint8_t* step_mask,
                      float eps_low, float eps_high, float C, const void* dlogits, int64_t ld_out,
                      const double* loss, const float* tok_coef) {
    if (!logits || !target || !lse || !dlogits) return true;
    if (bad_dtype(dtype) || V < 1 || ld < V || ld_out < V) return true;
    const size_t es = elem_size(dtype);
    if (reinterpret_cast<uintptr_t>(logits) % es || reinterpret_cast<uintptr_t>(dlogits) % es)
        return true;
    if (!logp || !logp_old || !logp_rollout || !adv || !step_offsets || !step_mask || !loss ||
        !tok_coef)
        return true;
    if (T < 1 || S < 1 || S > T || T > 0x7FFFFFFFll) return true;
    if (!(eps_low >= 0.f) || !(eps_high >= 0.f) || !(C > 0.f)) return true;
    return bad_overlap(logits, ld, dlogits, ld_out, T, V, es);
}

// The loss of dart_tis_loss_fwd: token ratios, token mean over kept tokens,
// no KL term.
LossConfig plain_loss_config(float eps_low, float eps_high, float C) {
    LossConfig cfg;
    cfg.eps_low = eps_low;
    cfg.eps_high = eps_high;
    cfg.C = C;
    cfg.log_C = isinf(C) ? INFINITY : (float)log((double)C);
    cfg.kl = DART_KL_NONE;
    cfg.beta = 0.f;
    cfg.agg = DART_AGG_TOKEN_MEAN;
    cfg.ratio = DART_RATIO_TOKEN;
    return cfg;
}

}  // namespace

// Scratch of dart_tis_loss_fwd_bwd_noalloc: the loss kernels' per-workgroup
// partial sums and the kept counts, sized for the largest many-workgroup
// launch (kCoefMaxBlocks workgroups, 40,976 bytes), so every T fits. Each
// device holds its own copy for the life of the process. Host code never
// passes the array's name to a kernel (on the host it is only a stand-in for
// the symbol): the device address comes from hipGetSymbolAddress, once per
// device, with that device current.
constexpr int64_t kNoAllocScratchDoubles = coef_workspace_doubles(kCoefMaxBlocks);
constexpr size_t kNoAllocScratchBytes = (size_t)kNoAllocScratchDoubles * sizeof(double);
static __device__ __align__(256) double scratch[kNoAllocScratchDoubles];

constexpr int kMaxScratchDevices = 64;
static std::mutex g_scratch_mu;
static void* g_scratch_ptr[kMaxScratchDevices] = {};

// The device address of dev's scratch array (null on a HIP error or a device
// index beyond kMaxScratchDevices).
static void* device_scratch(int dev) {
    if (dev < 0 || dev >= kMaxScratchDevices) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        DeviceGuard on_dev(dev);
        if (!on_dev.ok) return nullptr;
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return nullptr;
        g_scratch_ptr[dev] = ptr;
    }
    return g_scratch_ptr[dev];
}

extern "C" {

const char* dart_status_string(dart_status_t status) {
    switch (status) {
        case DART_OK: return "DART_OK";
        case DART_ERR_INVALID_ARG: return "DART_ERR_INVALID_ARG";
        case DART_ERR_UNSUPPORTED: return "DART_ERR_UNSUPPORTED";
        case DART_ERR_HIP: return "DART_ERR_HIP";
    }
    return "DART_ERR_UNKNOWN";
}

int64_t dart_kept_steps(int64_t S, double rho) {
    if (S < 0 || !(rho >= 0.0 && rho <= 1.0)) return -1;
    double k = ceil(rho * (double)S - 1e-6);
    if (k < 0.0) k = 0.0;
    if (k > (double)S) k = (double)S;
    return (int64_t)k;
}

size_t dart_tis_loss_workspace_bytes(int64_t T) {
    if (T < 1 || T > 0x7FFFFFFFll) return 0;
    return (size_t)coef_workspace_doubles(coef_blocks(T)) * sizeof(double);
}

size_t dart_tis_loss_split_workspace_bytes(int64_t T) {
    const size_t plain = dart_tis_loss_workspace_bytes(T);
    return plain ? plain + (size_t)coef_workspace_doubles(spare_blocks(T)) * sizeof(double) : 0;
}

dart_status_t dart_tok_stats_ex(const void* logits, dart_dtype_t dtype, int64_t T, int64_t V,
                                int64_t ld, const int32_t* target, float inv_temp, float* logp,
                                float* entropy, float* lse, hipStream_t stream) {
    if (!logits || !target || !logp || !entropy || !lse) return DART_ERR_INVALID_ARG;
    if (bad_dtype(dtype) || T < 1 || V < 1 || ld < V || T > 0x7FFFFFFFll)
        return DART_ERR_INVALID_ARG;
    if (!(inv_temp > 0.f) || isinf(inv_temp)) return DART_ERR_INVALID_ARG;
    if (reinterpret_cast<uintptr_t>(logits) % elem_size(dtype)) return DART_ERR_INVALID_ARG;
    if (const dart_status_t ck = dart_check::run(
            stream, {{dart_check::Item::Ids, target, T, V}}); ck != DART_OK)
        return ck;
    switch (stats_threads(V / (int64_t)(16 / elem_size(dtype)))) {
        case 128: launch_tok_stats<128>(logits, dtype, T, V, ld, target, inv_temp, logp, entropy, lse, stream); break;
        case 256: launch_tok_stats<256>(logits, dtype, T, V, ld, target, inv_temp, logp, entropy, lse, stream); break;
        case 512: launch_tok_stats<512>(logits, dtype, T, V, ld, target, inv_temp, logp, entropy, lse, stream); break;
        default: launch_tok_stats<768>(logits, dtype, T, V, ld, target, inv_temp, logp, entropy, lse, stream);
    }
    return launch_status();
}

dart_status_t dart_tok_stats(const void* logits, dart_dtype_t dtype, int64_t T, int64_t V,
                             int64_t ld, const int32_t* target, float* logp, float* entropy,
                             float* lse, hipStream_t stream) {
    return dart_tok_stats_ex(logits, dtype, T, V, ld, target, 1.f, logp, entropy, lse, stream);
}

dart_status_t dart_step_select(const float* entropy, int64_t T, const int32_t* step_offsets,
                               int64_t S, double rho, float* step_entropy, uint8_t* step_mask,
                               int32_t* n_kept_steps, hipStream_t stream) {
    if (!entropy || !step_offsets || !step_entropy || !step_mask) return DART_ERR_INVALID_ARG;
    if (T < 1 || S < 1 || S > T || T > 0x7FFFFFFFll) return DART_ERR_INVALID_ARG;
    const int64_t k = dart_kept_steps(S, rho);
    if (k < 0) return DART_ERR_INVALID_ARG;
    if (const dart_status_t ck = dart_check::run(
            stream, {{dart_check::Item::Offsets, step_offsets, S, T}}); ck != DART_OK)
        return ck;
    if (!grid_fits((S + kSelWaves - 1) / kSelWaves, kSelThreads)) return DART_ERR_UNSUPPORTED;
    if (T <= kSelLdsTokens && S <= kSelFusedMaxS) {
        hipLaunchKernelGGL(step_select_kernel<true>, dim3(1), dim3(kSelThreads), 0, stream,
                           entropy, T, step_offsets, S, nullptr, rho, k, step_entropy, step_mask,
                           n_kept_steps);
        return launch_status();
    }
    hipLaunchKernelGGL(step_mean_kernel, dim3((unsigned)((S + kSelWaves - 1) / kSelWaves)),
                       dim3(kSelThreads), 0, stream, entropy, T, step_offsets, S, step_entropy);
    hipLaunchKernelGGL(step_select_kernel<false>, dim3(1), dim3(kSelThreads), 0, stream, entropy,
                       T, step_offsets, S, nullptr, rho, k, step_entropy, step_mask, n_kept_steps);
    return launch_status();
}

dart_status_t dart_step_select_groups(const float* entropy, int64_t T,
                                     const int32_t* step_offsets, int64_t S,
                                     const int32_t* group_step_offsets, int64_t G, double rho,
                                     float* step_entropy, uint8_t* step_mask,
                                     int32_t* n_kept_steps, hipStream_t stream) {
    if (!entropy || !step_offsets || !group_step_offsets || !step_entropy || !step_mask)
        return DART_ERR_INVALID_ARG;
    if (T < 1 || S < 1 || S > T || T > 0x7FFFFFFFll || G < 1 || G > S || G > 0x7FFFFFFFll)
        return DART_ERR_INVALID_ARG;
    if (dart_kept_steps(S, rho) < 0) return DART_ERR_INVALID_ARG;
    if (!grid_fits((S + kSelWaves - 1) / kSelWaves, kSelThreads) || !grid_fits(G, kSelThreads))
        return DART_ERR_UNSUPPORTED;
    if (const dart_status_t ck = dart_check::run(
            stream, {{dart_check::Item::Offsets, step_offsets, S, T},
                     {dart_check::Item::Offsets, group_step_offsets, G, S}}); ck != DART_OK)
        return ck;
    hipLaunchKernelGGL(step_mean_kernel, dim3((unsigned)((S + kSelWaves - 1) / kSelWaves)),
                       dim3(kSelThreads), 0, stream, entropy, T, step_offsets, S, step_entropy);
    hipLaunchKernelGGL(step_select_kernel<false>, dim3((unsigned)G), dim3(kSelThreads), 0, stream,
                       entropy, T, step_offsets, S, group_step_offsets, rho, (int64_t)0,
                       step_entropy, step_mask, n_kept_steps);
    return launch_status();
}

dart_status_t dart_grpo_advantage(const float* reward, int64_t n_traj,
                                  const int32_t* traj_step_offsets,
                                  const int32_t* group_traj_offsets, int64_t G,
                                  const int32_t* step_offsets, int64_t S, int64_t T, float* adv,
                                  float* group_mean, float* group_std, hipStream_t stream) {
    if (!reward || !traj_step_offsets || !group_traj_offsets || !step_offsets || !adv)
        return DART_ERR_INVALID_ARG;
    if (n_traj < 1 || G < 1 || G > n_traj || S < 1 || S > T || T > 0x7FFFFFFFll ||
        G > 0x7FFFFFFFll)
        return DART_ERR_INVALID_ARG;
    if (!grid_fits(G, kAdvThreads)) return DART_ERR_UNSUPPORTED;
    if (const dart_status_t ck = dart_check::run(
            stream, {{dart_check::Item::Offsets, traj_step_offsets, n_traj, S},
                     {dart_check::Item::Offsets, group_traj_offsets, G, n_traj},
                     {dart_check::Item::Offsets, step_offsets, S, T}}); ck != DART_OK)
        return ck;
    // workgroups per group: one per kAdvTokens tokens of an average group, while
    // the dispatch holds them
    int64_t per = T / (G * kAdvTokens);
    per = per < 1 ? 1 : per > kAdvMaxPer ? kAdvMaxPer : per;
    if (!grid_fits(G * per, kAdvThreads)) per = 1;
    hipLaunchKernelGGL(grpo_advantage_kernel, dim3((unsigned)G, (unsigned)per), dim3(kAdvThreads), 0, stream,
                       reward, traj_step_offsets, n_traj, group_traj_offsets, step_offsets, S, T,
                       adv, group_mean, group_std);
    return launch_status();
}

dart_status_t dart_tis_loss_fwd_ex(int64_t T, const float* logp, const float* logp_old,
                                   const float* logp_rollout, const float* logp_ref,
                                   const float* adv, const int32_t* step_offsets, int64_t S,
                                   const uint8_t* step_mask, const dart_loss_config_t* config,
                                   double* loss, float* tok_coef, float* stats, void* workspace,
                                   size_t workspace_bytes, hipStream_t stream) {
    if (!config) return DART_ERR_INVALID_ARG;
    const dart_loss_config_t& c = *config;
    if (c.kl < DART_KL_NONE || c.kl > DART_KL_K3 || c.aggregation < DART_AGG_TOKEN_MEAN ||
        c.aggregation > DART_AGG_STEP_MEAN || c.ratio < DART_RATIO_TOKEN ||
        c.ratio > DART_RATIO_STEP_PRODUCT)
        return DART_ERR_INVALID_ARG;
    if (c.kl != DART_KL_NONE && (!logp_ref || !(c.beta >= 0.f) || isinf(c.beta)))
        return DART_ERR_INVALID_ARG;
    if (!logp || !logp_old || !logp_rollout || !adv || !step_offsets || !step_mask || !loss ||
        !tok_coef)
        return DART_ERR_INVALID_ARG;
    if (T < 1 || S < 1 || S > T || T > 0x7FFFFFFFll) return DART_ERR_INVALID_ARG;
    if (!(c.eps_low >= 0.f) || !(c.eps_high >= 0.f) || !(c.C > 0.f)) return DART_ERR_INVALID_ARG;
    if (bad_workspace(workspace, workspace_bytes, T)) return DART_ERR_INVALID_ARG;
    if (const dart_status_t ck = dart_check::run(
            stream, {{dart_check::Item::Offsets, step_offsets, S, T},
                     {dart_check::Item::Mask, step_mask, S, 0}}); ck != DART_OK)
        return ck;
    LossConfig cfg;
    cfg.eps_low = c.eps_low;
    cfg.eps_high = c.eps_high;
    cfg.C = c.C;
    cfg.log_C = isinf(c.C) ? INFINITY : (float)log((double)c.C);
    cfg.kl = c.kl;
    cfg.beta = c.kl == DART_KL_NONE ? 0.f : c.beta;
    cfg.agg = c.aggregation;
    cfg.ratio = c.ratio;
    return launch_tis_coef(true, T, logp, logp_old, logp_rollout,
                           c.kl == DART_KL_NONE ? nullptr : logp_ref, adv, step_offsets, S,
                           step_mask, cfg, tok_coef, loss, stats, 6, workspace,
                           spare_part(workspace, workspace_bytes, T), stream);
}

dart_status_t dart_tis_loss_fwd(int64_t T, const float* logp, const float* logp_old,
                                const float* logp_rollout, const float* adv,
                                const int32_t* step_offsets, int64_t S, const uint8_t* step_mask,
                                float eps_low, float eps_high, float C, double* loss,
                                float* tok_coef, float* stats, void* workspace,
                                size_t workspace_bytes, hipStream_t stream) {
    if (!logp || !logp_old || !logp_rollout || !adv || !step_offsets || !step_mask || !loss ||
        !tok_coef)
        return DART_ERR_INVALID_ARG;
    if (T < 1 || S < 1 || S > T || T > 0x7FFFFFFFll) return DART_ERR_INVALID_ARG;
    if (!(eps_low >= 0.f) || !(eps_high >= 0.f) || !(C > 0.f)) return DART_ERR_INVALID_ARG;
    if (bad_workspace(workspace, workspace_bytes, T)) return DART_ERR_INVALID_ARG;
    if (const dart_status_t ck = dart_check::run(
            stream, {{dart_check::Item::Offsets, step_offsets, S, T},
                     {dart_check::Item::Mask, step_mask, S, 0}}); ck != DART_OK)
        return ck;
    return launch_tis_coef(false, T, logp, logp_old, logp_rollout, nullptr, adv, step_offsets, S,
                           step_mask, plain_loss_config(eps_low, eps_high, C), tok_coef, loss,
                           stats, 4, workspace, nullptr, stream);
}

dart_status_t dart_select_tis_loss_fwd(int64_t T, const float* entropy, const float* logp,
                                       const float* logp_old, const float* logp_rollout,
                                       const float* adv, const int32_t* step_offsets, int64_t S,
                                       double rho, float eps_low, float eps_high, float C,
                                       float* step_entropy, uint8_t* step_mask,
                                       int32_t* n_kept_steps, double* loss, float* tok_coef,
                                       float* stats, void* workspace, size_t workspace_bytes,
                                       hipStream_t stream) {
    // the argument rules of dart_step_select and dart_tis_loss_fwd, all checked
    // before anything is enqueued
    if (!entropy || !step_offsets || !step_entropy || !step_mask || !logp || !logp_old ||
        !logp_rollout || !adv || !loss || !tok_coef)
        return DART_ERR_INVALID_ARG;
    if (T < 1 || S < 1 || S > T || T > 0x7FFFFFFFll) return DART_ERR_INVALID_ARG;
    const int64_t k = dart_kept_steps(S, rho);
    if (k < 0) return DART_ERR_INVALID_ARG;
    if (!(eps_low >= 0.f) || !(eps_high >= 0.f) || !(C > 0.f)) return DART_ERR_INVALID_ARG;
    if (bad_workspace(workspace, workspace_bytes, T)) return DART_ERR_INVALID_ARG;
    if (T > kSelCoefMaxT || S > kSelCoefMaxS) {
        // beyond what one workgroup does faster: the two calls in turn
        const dart_status_t st = dart_step_select(entropy, T, step_offsets, S, rho, step_entropy,
                                                  step_mask, n_kept_steps, stream);
        if (st != DART_OK) return st;
        void* part = workspace;
        size_t part_bytes = workspace_bytes;
        if (T <= kSelCoefMaxT && S <= kSelLdsKeys) {
            part = spare_part(workspace, workspace_bytes, T);
            part_bytes = part ? dart_tis_loss_workspace_bytes(T) : 0;
        }
        return dart_tis_loss_fwd(T, logp, logp_old, logp_rollout, adv, step_offsets, S, step_mask,
                                 eps_low, eps_high, C, loss, tok_coef, stats, part, part_bytes,
                                 stream);
    }
    if (const dart_status_t ck = dart_check::run(
            stream, {{dart_check::Item::Offsets, step_offsets, S, T}}); ck != DART_OK)
        return ck;
    hipLaunchKernelGGL(select_coef_kernel, dim3(1), dim3(kSelThreads), 0, stream, entropy, T,
                       step_offsets, S, rho, k, step_entropy, step_mask, n_kept_steps, logp,
                       logp_old, logp_rollout, adv, plain_loss_config(eps_low, eps_high, C),
                       tok_coef, loss, stats, 4);
    return launch_status();
}

dart_status_t dart_tis_grad_ex(const void* logits, dart_dtype_t dtype, int64_t T, int64_t V,
                               int64_t ld, const int32_t* target, const float* logp,
                               const float* lse, const float* tok_coef, float inv_temp,
                               uint32_t flags, void* dlogits, int64_t ld_out, hipStream_t stream) {
    if (!logits || !target || !logp || !lse || !tok_coef || !dlogits) return DART_ERR_INVALID_ARG;
    if (bad_dtype(dtype) || T < 1 || V < 1 || ld < V || ld_out < V || T > 0x7FFFFFFFll)
        return DART_ERR_INVALID_ARG;
    if (!(inv_temp > 0.f) || isinf(inv_temp) || (flags & ~DART_GRAD_SKIP_ZERO_ROWS))
        return DART_ERR_INVALID_ARG;
    const size_t es = elem_size(dtype);
    if (reinterpret_cast<uintptr_t>(logits) % es || reinterpret_cast<uintptr_t>(dlogits) % es)
        return DART_ERR_INVALID_ARG;
    if (bad_overlap(logits, ld, dlogits, ld_out, T, V, es)) return DART_ERR_INVALID_ARG;
    if (const dart_status_t ck = dart_check::run(
            stream, {{dart_check::Item::Ids, target, T, V}}); ck != DART_OK)
        return ck;
    const int64_t nvec = V / (int64_t)(16 / es);
    auto launch = [&](auto threads) {
        // chunks of threads * kGradUnroll vectors per row; a grid of at most
        // kGradMaxBlocks workgroups strides over the T * nchunk chunks
        constexpr int N = decltype(threads)::value;
        const int64_t per = (int64_t)N * kGradUnroll;
        const int64_t nchunk = nvec > 0 ? (nvec + per - 1) / per : 1;
        const int64_t nblocks = T * nchunk < kGradMaxBlocks ? T * nchunk : kGradMaxBlocks;
        with_logits(dtype, T, V, [&](auto dt, auto nt) {
            constexpr dart_dtype_t D = decltype(dt)::value;
            if constexpr (N == kGradThreads || D == DART_F32)
                hipLaunchKernelGGL((tis_grad_kernel<D, N, kGradUnroll, decltype(nt)::value, kNtStore>),
                                   dim3((unsigned)nblocks), dim3(N), 0, stream, logits, V, ld,
                                   target, lse, logp, tok_coef, inv_temp, flags, dlogits, ld_out, T,
                                   nchunk);
        });
    };
    const bool lines = (ld_out * es) % 128 == 0 && reinterpret_cast<uintptr_t>(dlogits) % 128 == 0;
    if (dtype == DART_F32 && nvec >= kGradWideVectors && !lines)
        launch(std::integral_constant<int, 2 * kGradThreads>{});
    else
        launch(std::integral_constant<int, kGradThreads>{});
    return launch_status();
}

dart_status_t dart_tis_grad(const void* logits, dart_dtype_t dtype, int64_t T, int64_t V,
                            int64_t ld, const int32_t* target, const float* logp,
                            const float* lse, const float* tok_coef, void* dlogits,
                            int64_t ld_out, hipStream_t stream) {
    return dart_tis_grad_ex(logits, dtype, T, V, ld, target, logp, lse, tok_coef, 1.f, 0u,
                            dlogits, ld_out, stream);
}

dart_status_t dart_tis_loss_fwd_bwd(const void* logits, dart_dtype_t dtype, int64_t T, int64_t V,
                                    int64_t ld, const int32_t* target, const float* logp,
                                    const float* lse, const float* logp_old,
                                    const float* logp_rollout, const float* adv,
                                    const int32_t* step_offsets, int64_t S,
                                    const uint8_t* step_mask, float eps_low, float eps_high,
                                    float C, void* dlogits, int64_t ld_out, double* loss,
                                    float* tok_coef, float* stats, void* workspace,
                                    size_t workspace_bytes, hipStream_t stream) {
    // validate both halves before enqueuing either
    if (!logits || !target || !lse || !dlogits) return DART_ERR_INVALID_ARG;
    if (bad_dtype(dtype) || V < 1 || ld < V || ld_out < V) return DART_ERR_INVALID_ARG;
    const size_t es = elem_size(dtype);
    if (reinterpret_cast<uintptr_t>(logits) % es || reinterpret_cast<uintptr_t>(dlogits) % es)
        return DART_ERR_INVALID_ARG;
    if (T >= 1 && bad_overlap(logits, ld, dlogits, ld_out, T, V, es)) return DART_ERR_INVALID_ARG;
    // with checks on, all device data is validated before either half enqueues
    if (T >= 1 && S >= 1 && S <= T) {
        const dart_status_t ck = dart_check::run(
            stream, {{dart_check::Item::Ids, target, T, V},
                     {dart_check::Item::Offsets, step_offsets, S, T},
                     {dart_check::Item::Mask, step_mask, S, 0}});
        if (ck != DART_OK) return ck;
    }
    dart_status_t st = dart_tis_loss_fwd(T, logp, logp_old, logp_rollout, adv, step_offsets, S,
                                         step_mask, eps_low, eps_high, C, loss, tok_coef, stats,
                                         workspace, workspace_bytes, stream);
    if (st != DART_OK) return st;
    return dart_tis_grad(logits, dtype, T, V, ld, target, logp, lse, tok_coef, dlogits, ld_out,
                         stream);
}


dart_status_t dart_tis_loss_fwd_bwd_noalloc(const void* logits, dart_dtype_t dtype, int64_t T,
                                            int64_t V, int64_t ld, const int32_t* target,
                                            const float* logp, const float* lse,
                                            const float* logp_old, const float* logp_rollout,
                                            const float* adv, const int32_t* step_offsets,
                                            int64_t S, const uint8_t* step_mask, float eps_low,
                                            float eps_high, float C, void* dlogits, int64_t ld_out,
                                            double* loss, float* tok_coef, float* stats,
                                            hipStream_t stream) {
    // host-side rules first: a bad argument is reported before any HIP call
    if (bad_fwd_bwd_args(logits, dtype, T, V, ld, target, logp, lse, logp_old, logp_rollout, adv,
                         step_offsets, S, step_mask, eps_low, eps_high, C, dlogits, ld_out, loss,
                         tok_coef))
        return DART_ERR_INVALID_ARG;
    // the workspace this T needs must fit the scratch array (always true for
    // T <= INT32_MAX: the many-workgroup launch is capped at kCoefMaxBlocks)
    if (dart_tis_loss_workspace_bytes(T) > kNoAllocScratchBytes) return DART_ERR_UNSUPPORTED;
    const int dev = stream_device(stream);
    if (dev < 0) return DART_ERR_HIP;
    void* ws = device_scratch(dev);
    if (!ws) return DART_ERR_HIP;
    // every argument rule of dart_tis_loss_fwd_bwd applies unchanged
    return dart_tis_loss_fwd_bwd(logits, dtype, T, V, ld, target, logp, lse, logp_old,
                                 logp_rollout, adv, step_offsets, S, step_mask, eps_low, eps_high,
                                 C, dlogits, ld_out, loss, tok_coef, stats, ws,
                                 kNoAllocScratchBytes, stream);
}

}  // extern "C"
