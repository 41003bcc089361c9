// libdart, LM-head part: the token statistics and the gradient of the
// policy-update hot path computed straight from the LM head's inputs, so that
// the [T, V] logits are never written to memory.
//
// Paper: DART, arXiv 2509.23866. The statistics are those of Sec. 4.3 (token
// entropy, the target's log-prob of Eq. 1) for logits z = h W^T, where h [T, d]
// are the final hidden states of the T action tokens and W [V, d] the LM-head
// weight of the policy (the 7B VLM of Sec. 5.1); the gradient is the chain
// rule of Eq. 2's loss through them. Both kernels apply an inverse sampling
// temperature s (1 in the paper, App. A.4) in their epilogues: the fp32 tile
// stays unscaled, and s enters the factor of the base-2 exponent (s log2 e)
// and the row maximum (s > 0), so that s = 1 changes no bit.
//
//   lmhead_stats_kernel   one 256 x 256 tile of z per workgroup (64 or 128 rows
//                         where T is small) on MFMA
//                         (v_mfma_f32_32x32x16_bf16, fp32 accumulation), K = d
//                         in slices of 64 loaded straight into two LDS buffers;
//                         the tile is reduced in the epilogue to one (max,
//                         normaliser, entropy) triple per row over its 256
//                         columns (the target column kept apart), written to a
//                         workspace.
//   lmhead_merge_kernel   one wave per row: merges the row's V / 256 triples in
//                         a fixed order, adds the target logit, writes logp, H
//                         and lse exactly as tok_stats_kernel defines them.
//   lmhead_dlogits_kernel the same tile, its epilogue writing
//                         dz = g (onehot - softmax) in bf16.
// The backward forms dz block by block (rows x vocabulary entries, the blocked
// entry point optionally over the rows with a non-zero coefficient only) and
// adds dh = dz W and dW = dz^T h per block in one launch of
// lmhead_bwd_gemms_kernel (the same MFMA tile, its operands stored with K as
// their row index read through LDS transpose loads).
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

#include "internal.h"
#include "dart.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

// Waits until at most N loads of this wave are outstanding (vmcnt), leaving
// the LDS and export counters alone.
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
    static_assert(N >= 0 && N < 64, "vmcnt");
    __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4) | (0xF << 8));
}

// A buffer resource over [base, base + bytes) (bytes capped at 2^32 - 1): raw
// loads past its end return zero. Dword 3 selects 32-bit data, untyped.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t tile_rsrc(const void* base, int64_t bytes) {
    const uint32_t n = bytes > 0xFFFFFFFFll ? 0xFFFFFFFFu : (uint32_t)bytes;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)n, 0x00020000);
}

// Bytes from a matrix's row to the end of the last of `rows` rows of K bf16: the
// padding after that one need not belong to the caller's allocation (the last
// columns of a wider matrix), so a K slice that runs past K must not read it.
__host__ __device__ constexpr int64_t rows_bytes(int64_t rows, int64_t ld, int64_t K) {
    return ((rows - 1) * ld + K) * 2;
}
static_assert(rows_bytes(1, 80, 72) == 72 * 2 && rows_bytes(3, 80, 72) == (2 * 80 + 72) * 2,
              "the last row's padding is left out");

__device__ __forceinline__ __attribute__((address_space(3))) void* lds_ptr(void* p) {
    return (__attribute__((address_space(3))) void*)p;
}

// Workgroup barrier of the LDS ring: the caller has waited for its own loads
// into LDS (vmcnt); lgkmcnt(0) retires its LDS reads; the empty asm
// statements keep the compiler from moving memory accesses across it. Unlike
// __syncthreads it carries no fence, which would wait for every load in flight.
[[maybe_unused]] __device__ __forceinline__ void lds_ring_barrier() {
    __builtin_amdgcn_s_waitcnt(0xF | (0x3 << 14) | (0x7 << 4));  // lgkmcnt(0)
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Orders a wave's LDS accesses before it against those after it, across its lanes
// (which the convergent barrier brings together): the hardware runs them in the
// program's order, so nothing is waited for.
[[maybe_unused]] __device__ __forceinline__ void lds_wave_order() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
    asm volatile("" ::: "memory");
}

// Tile configuration: BM tokens x BN vocabulary entries per workgroup, K in
// slices of 64 through an NS-buffer LDS ring filled by direct global->LDS
// loads (no staging registers), WM x WN waves each owning a (BM/WM) x (BN/WN)
// block of 32 x 32 MFMA tiles.
// A K slice of BK bf16 per tile row is BK/8 chunks of 16 B. Chunk c of row r
// sits in LDS slot c ^ swz(r). gfx950's LDS serves 16-byte-per-lane reads 16
// lanes at a time across 64 four-byte banks (16 bank quads); a row of CH
// chunks covers CH quads, so 16 / CH consecutive rows tile the banks once and
// the swizzle shifts each such run of rows: the 16 rows that one read cycle
// takes (same chunk c) land in 16 distinct quads. With the plain c ^ (r % 8)
// of a 32-bank LDS, the bank-conflict counter showed half of all LDS cycles
// in two-way conflicts.
template <int CH>
__device__ __forceinline__ int swz(int r) { return (r / (16 / CH)) % CH; }

// Columns of a row that the statistics reduce together, in every configuration.
constexpr int kStatsUnit = 64;

template <int BM_, int BN_, int WM_, int WN_, int NS_, int BK_ = 64>
struct Cfg {
    static constexpr int BM = BM_, BN = BN_, BK = BK_, WM = WM_, WN = WN_, NS = NS_;
    static_assert(NS == 2 || NS == 3, "buffers of the K loop");
    static constexpr int CH = BK / 8;          // 16-byte chunks per row and slice
    static constexpr int LROWS = 64 / CH;      // rows one load instruction fills
    static constexpr int KSTEPS = BK / 16;     // MFMA k-steps per slice
    static constexpr int THREADS = 64 * WM * WN, WAVES = WM * WN;
    static constexpr int TM = BM / WM / 32, TN = BN / WN / 32;  // MFMA tiles per wave
    // a wave's TM row blocks of 32 sit RS = WM * 32 rows apart, so that each
    // epilogue pass over EPI = RS rows takes one block from every wave
    static constexpr int RS = BM / TM;
    static constexpr int IA = BM / LROWS / WAVES, IB = BN / LROWS / WAVES;  // loads per slice
    // LDS rows of a result tile: 16 bytes beyond BN elements, so that
    // consecutive rows start one bank quad apart and the rows that the lanes of
    // one write cycle hold fall in distinct banks. A bf16 tile goes through LDS
    // whole, an fp32 one EPI rows at a time: one 32-row block of every wave
    static constexpr int CROW = BN + 4, CROW16 = BN + 8;
    static constexpr int EPI = RS;
    static_assert(BK == 32 || BK == 64, "slice depth");
    static_assert(BM % (32 * WM) == 0 && BN % (32 * WN) == 0, "tile shape");
    static_assert(IA * LROWS * WAVES == BM && IB * LROWS * WAVES == BN, "rows per wave");
    static_assert(THREADS % EPI == 0 || EPI % THREADS == 0, "epilogue rows");
    struct alignas(16) Smem {
        union {
            struct {
                // slice buffers: BK bf16 per row, chunk c of row r in slot c ^ swz(r)
                uint16_t a[NS][BM][BK];
                uint16_t b[NS][BN][BK];
            } in;
            float c[EPI][CROW];
            uint16_t c16[BM][CROW16];
            float4 red[BN / kStatsUnit][BM];  // per-row partial triples of the statistics
        };
    };
};
// Measured on MI355X at T = 4096, d = 3584, V = 152064 among 128/256-square
// tiles, 4 or 8 waves, 2-4 buffers, 32- or 64-wide slices and register-staged
// loads: 256 x 256 with 8 waves as 4 x 2 (64 x 128 per wave) and two 64-wide
// buffers is the fastest.
using LmCfg = Cfg<256, 256, 4, 2, 2>;
// Tiles of fewer rows, for few rows in all: a third buffer fits the LDS, so that
// two slices are in flight where W comes from HBM and little is multiplied per
// byte of it. Measured (d = 3584, V = 152064; statistics and dlogits, us): 64
// rows 213 and 204 with the 64-row tile (243 and 241 with two buffers), 279 and
// 270 with the 256-row one; 128 rows 231 and 220 with the 128-row tile (274 and
// 267 with two buffers), 285 and 281.
using LmCfg128 = Cfg<128, 256, 2, 4, 3>;
using LmCfg64 = Cfg<64, 256, 2, 4, 3>;
static_assert(sizeof(LmCfg::Smem) <= 160 * 1024 && sizeof(LmCfg128::Smem) <= 160 * 1024 &&
                  sizeof(LmCfg64::Smem) <= 160 * 1024,
              "LDS per workgroup");
constexpr int kMergeWaves = 4;
constexpr int kMergeBatch = 5;

struct Triple {
    float m, s, w;  // reference, sum of e^{z-m}, sum of e^{z-m} (z-m), natural units
};

// float -> bf16 bits, round to nearest even, a NaN kept quiet with its
// payload: the __bf16 conversion, which is gfx950's v_cvt_pk_bf16_f32 (two
// values per instruction; the same bits as the integer rounding
// u + 0x7FFF + ((u >> 16) & 1) for every one of the 2^32 fp32 inputs, checked
// on the GPU)
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint16_t bf16_bits(float f) {
    return __builtin_bit_cast(uint16_t, (__bf16)f);
}

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    const bf16x2_t v = {(__bf16)lo, (__bf16)hi};
    return __builtin_bit_cast(uint32_t, v);
}

// Exact merge of two partial triples; an empty triple has s == 0. Contracted by
// hand alone, so that every kernel it is inlined into rounds the same.
__device__ __forceinline__ Triple merge(const Triple& a, const Triple& b) {
#pragma clang fp contract(off)
    if (b.s == 0.f) return a;
    if (a.s == 0.f) return b;
    const float m = fmaxf(a.m, b.m);
    const float ca = expf(a.m - m), cb = expf(b.m - m);
    Triple r;
    r.m = m;
    r.s = fmaf(ca, a.s, cb * b.s);
    r.w = fmaf(ca, fmaf(a.m - m, a.s, a.w), cb * fmaf(b.m - m, b.s, b.w));
    return r;
}

// acc = this wave's part of the tile A[m0:m0+BM, :] B[n0:n0+BN, :]^T (A [M, K]
// and B [N, K] row-major bf16, rows 16-byte aligned, K % 8 == 0). Rows past M
// or N read as zero (their results are not used); K past the end is zeroed in
// LDS. Layout of acc[i][j]: value v of lane l is
// tile row (wave / WN) * 32 + i * RS + l%32, column
// (wave % WN) * BN/WN + j*32 + (v/4)*8 + (l/32)*4 + v%4: the MFMA takes B's rows
// as its first operand, so that a lane holds 16 TN columns of one row, four
// adjacent ones in consecutive registers. (With A's rows first a lane holds
// one column of 16 rows, and every epilogue had to turn the fp32 tile round in
// LDS, one value at a time. Measured at d = 3584, V = 152064, the same box:
// statistics 3450 -> 3378 us at T = 4096 and 950 -> 925 at 1000, the backward
// with bf16 gradients 10702 -> 10565 and 2953 -> 2856, dlogits 928 -> 917 at
// 1000, the fp32 gradients within 0.3%.) Ends on a barrier with no loads in
// flight, so the caller may reuse the LDS.
template <class C>
__device__ __forceinline__ void gemm_tile(const uint16_t* __restrict__ A, int64_t M, int64_t lda,
                                          const uint16_t* __restrict__ B, int64_t N, int64_t ldb,
                                          int64_t K, int64_t m0, int64_t n0,
                                          typename C::Smem& sm,
                                          f32x16 (&acc)[C::TM][C::TN]) {
#if defined(__HIP_DEVICE_COMPILE__)  // the gfx950 builtins below have no host form
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: addresses in SGPRs
    const int wr = (wave / C::WN) * 32, wc = (wave % C::WN) * (C::BN / C::WN);
#pragma unroll
    for (int i = 0; i < C::TM; ++i)
#pragma unroll
        for (int j = 0; j < C::TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    // One load instruction fills LROWS rows x CH slots (1 KB): lane l writes
    // slot l % CH of row r0 + l / CH, i.e. chunk (l % CH) ^ swz(row) of that
    // row. The loads are buffer loads into LDS: each operand's tile rows are a
    // buffer resource whose range ends at the matrix's last element, so rows
    // past M or N read as zero (their results are not used). A lane's byte
    // offset within its instruction's rows is the same for every instruction
    // and slice (the swizzle repeats every 16 rows, and the rows of one
    // instruction of every wave together are a multiple of that), so one VGPR
    // serves all of an operand's loads; the instruction's rows and the slice
    // enter as a scalar offset.
    constexpr int CH = C::CH, BK = C::BK;
    const int lrow = lane / CH, lslot = lane % CH;
    static_assert((C::WAVES * C::LROWS) % (16 / CH * CH) == 0, "swizzle period");
    const int r_lane = wave * C::LROWS + lrow;  // row of the lane in instruction 0
    const uint32_t voff_a = (uint32_t)((r_lane * lda + (lslot ^ swz<CH>(r_lane)) * 8) * 2);
    const uint32_t voff_b = (uint32_t)((r_lane * ldb + (lslot ^ swz<CH>(r_lane)) * 8) * 2);
    const uint32_t qstride_a = (uint32_t)(C::WAVES * C::LROWS * lda * 2);
    const uint32_t qstride_b = (uint32_t)(C::WAVES * C::LROWS * ldb * 2);
    const __amdgpu_buffer_rsrc_t rsrc_a = tile_rsrc(A + m0 * lda, rows_bytes(M - m0, lda, K));
    const __amdgpu_buffer_rsrc_t rsrc_b = tile_rsrc(B + n0 * ldb, rows_bytes(N - n0, ldb, K));
    // rows of instruction q of wave `wave + hh * HW`
    auto lds_a = [&](int buf, int q, int hh) {
        return &sm.in.a[buf][(q * C::WAVES + wave + hh * (C::WAVES / 2)) * C::LROWS][0];
    };
    auto lds_b = [&](int buf, int q, int hh) {
        return &sm.in.b[buf][(q * C::WAVES + wave + hh * (C::WAVES / 2)) * C::LROWS][0];
    };
    const int64_t nk = (K + BK - 1) / BK;
    // slice kt into buffer buf; a slice that ends past K reads chunks past K
    // (in the row padding, the next row or, at the end, as zero) that are
    // zeroed after landing
    // The first half of the waves (one per SIMD) issue every load of a
    // slice: their own rows and those of the wave HW above, with the same lane
    // offsets (the rows between them are a whole number of swizzle periods).
    // Issuing a slice's 64 loads holds each issuing wave for ~700 cycles; the
    // other wave of its SIMD multiplies meanwhile.
    constexpr int HW = C::WAVES / 2;
    static_assert((HW * C::LROWS) % 16 == 0, "swizzle period");
    const uint32_t hstride_a = (uint32_t)(HW * C::LROWS * lda * 2);
    const uint32_t hstride_b = (uint32_t)(HW * C::LROWS * ldb * 2);
    auto issue = [&](int64_t kt, int buf) {
        if (wave >= HW) return;
        const uint32_t kb = (uint32_t)(kt * BK * 2);
#pragma unroll
        for (int q = 0; q < C::IA; ++q)
#pragma unroll
            for (int hh = 0; hh < 2; ++hh)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_a, lds_ptr(lds_a(buf, q, hh)), 16,
                                                        voff_a, kb + q * qstride_a + hh * hstride_a,
                                                        0, 0);
#pragma unroll
        for (int q = 0; q < C::IB; ++q)
#pragma unroll
            for (int hh = 0; hh < 2; ++hh)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_b, lds_ptr(lds_b(buf, q, hh)), 16,
                                                        voff_b, kb + q * qstride_b + hh * hstride_b,
                                                        0, 0);
    };
    // a partial last slice: zero the chunks past K
    auto zero_tail = [&](int64_t kt, int buf) {
        const u32x4 z = {0u, 0u, 0u, 0u};
        for (int e = tid; e < (C::BM + C::BN) * CH; e += C::THREADS) {
            const int r = e / CH, c = e % CH;
            if (kt * BK + c * 8 < K) continue;
            if (r < C::BM)
                *reinterpret_cast<u32x4*>(&sm.in.a[buf][r][(c ^ swz<CH>(r)) * 8]) = z;
            else
                *reinterpret_cast<u32x4*>(
                    &sm.in.b[buf][r - C::BM][(c ^ swz<CH>(r - C::BM)) * 8]) = z;
        }
    };

    // MFMA operands: lane l reads row (l % 32) of each 32-row block, chunk
    // 2 ks + l / 32. The rows' swizzle depends only on l % 32 (blocks start at
    // multiples of 32), so one byte offset per k-step serves every block, the
    // block and the buffer entering as immediate offsets.
    // The B offsets include the B buffers' start (64 KB into the LDS) and are
    // kept opaque to the compiler, so that the buffer and the 32-column block
    // enter as the read's 16-bit immediate (below 64 KB); folded into the
    // immediate, they did not fit, and every B read cost an address add.
    uint32_t rda[C::KSTEPS], rdb[C::KSTEPS];
    const char* const lds0 = reinterpret_cast<const char*>(&sm);
    const uint32_t b_at = (uint32_t)(reinterpret_cast<const char*>(&sm.in.b[0][0][0]) - lds0);
#pragma unroll
    for (int ks = 0; ks < C::KSTEPS; ++ks) {
        const int c = ks * 2 + (lane >> 5), ra = wr + (lane & 31), rb = wc + (lane & 31);
        rda[ks] = (uint32_t)(ra * BK + (c ^ swz<CH>(ra)) * 8) * 2;
        rdb[ks] = b_at + (uint32_t)(rb * BK + (c ^ swz<CH>(rb)) * 8) * 2;
        asm volatile("" : "+v"(rdb[ks]));
    }
    bf16x8 af[2][C::TM], bfr[2][C::TN];
    auto read_step = [&](auto bufc, int ks, int set) {
        constexpr int buf = decltype(bufc)::value;
        const char* ba = reinterpret_cast<const char*>(&sm.in.a[buf][0][0]);
#pragma unroll
        for (int i = 0; i < C::TM; ++i)
            af[set][i] = __builtin_bit_cast(
                bf16x8, *reinterpret_cast<const u32x4*>(ba + rda[ks] + i * C::RS * BK * 2));
#pragma unroll
        for (int j = 0; j < C::TN; ++j)
            bfr[set][j] = __builtin_bit_cast(
                bf16x8, *reinterpret_cast<const u32x4*>(lds0 + rdb[ks] + buf * C::BN * BK * 2 +
                                                        j * 32 * BK * 2));
    };
    // the MFMAs of row blocks [i0, i1) of one k-step
    auto mfmas = [&](int set, int i0 = 0, int i1 = C::TM) {
#pragma unroll
        for (int i = 0; i < C::TM; ++i)
#pragma unroll
            for (int j = 0; j < C::TN; ++j)
                if (i >= i0 && i < i1)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[set][j], af[set][i],
                                                                        acc[i][j], 0, 0, 0);
    };
    // Every wave holds back the last k-step's MFMAs of its last row block
    // and issues them after the next slice's barrier (and its loads), while
    // the first operand reads of that slice are in flight.
    constexpr int LASTSET = (C::KSTEPS - 1) & 1;

    // NS LDS buffers: slices kt+1 .. kt+NS-1 load while slice kt is multiplied
    constexpr int LOADS = 2 * (C::IA + C::IB);  // of an issuing wave and slice
    auto slice = [&](auto bufc, int64_t kt) {
        constexpr int buf = decltype(bufc)::value;
        // slice kt has landed for this wave; the barrier makes it so for all,
        // and every wave has finished reading the buffer of slice kt-1
        if (C::NS == 2 || kt + C::NS - 2 >= nk)
            wait_vmcnt<0>();
        else
            wait_vmcnt<(C::NS - 2) * LOADS>();
        lds_ring_barrier();
        if ((K % BK) && kt == nk - 1) {
            zero_tail(kt, buf);
            lds_ring_barrier();
        }
        if (kt + C::NS - 1 < nk) issue(kt + C::NS - 1, (buf + C::NS - 1) % C::NS);
        // the operands of k-step ks+1 are read while the MFMAs of k-step ks issue
        read_step(bufc, 0, 0);
        __builtin_amdgcn_s_setprio(1);
        if (kt > 0) mfmas(LASTSET, C::TM - 1, C::TM);
#pragma unroll
        for (int ks = 0; ks < C::KSTEPS; ++ks) {
            const int cs = ks & 1;
            if (ks < C::KSTEPS - 1) read_step(bufc, ks + 1, cs ^ 1);
            mfmas(cs, 0, ks == C::KSTEPS - 1 ? C::TM - 1 : C::TM);
            if (ks < C::KSTEPS - 1) {
                // interleave: one LDS read, then a share of the MFMAs
#pragma unroll
                for (int g = 0; g < C::TM + C::TN; ++g) {
                    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x008, (C::TM * C::TN) / (C::TM + C::TN), 0);
                }
            }
        }
        __builtin_amdgcn_s_setprio(0);
    };
    // the loop body has no condition on the accumulators: the last slices that
    // do not fill a round of the buffers run after it (a conditional second
    // slice in the body made the compiler copy every accumulator at the join)
#pragma unroll
    for (int b = 0; b < C::NS - 1; ++b)
        if (b == 0 || b < nk) issue(b, b);
    int64_t kt = 0;
    for (; kt + C::NS - 1 < nk; kt += C::NS) {
        slice(std::integral_constant<int, 0>{}, kt);
        slice(std::integral_constant<int, 1>{}, kt + 1);
        if constexpr (C::NS > 2) slice(std::integral_constant<int, 2 % C::NS>{}, kt + 2);
    }
    if (kt < nk) slice(std::integral_constant<int, 0>{}, kt);
    if (C::NS > 2 && kt + 1 < nk) slice(std::integral_constant<int, 1>{}, kt + 1);
    mfmas(LASTSET, C::TM - 1, C::TM);
    __syncthreads();
#else
    (void)A, (void)M, (void)lda, (void)B, (void)N, (void)ldb, (void)K, (void)m0, (void)n0;
    (void)sm, (void)acc;
#endif
}

// NJ 32-column blocks (acc[0] is block j0) of the wave's row block i in the
// workgroup's result tile in LDS, rounded to bf16: four adjacent columns of a row
// leave a lane as one 8-byte write.
template <class C, int NJ>
__device__ __forceinline__ void blocks_to_lds_bf16(const f32x16* acc, int i, int j0,
                                                   typename C::Smem& sm) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wr = (wave / C::WN) * 32 + (lane & 31), wc = (wave % C::WN) * (C::BN / C::WN);
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int v = 0; v < 16; v += 4) {
            u32x2 pk;
            pk.x = pack_bf16x2(acc[j][v], acc[j][v + 1]);
            pk.y = pack_bf16x2(acc[j][v + 2], acc[j][v + 3]);
            *reinterpret_cast<u32x2*>(
                &sm.c16[wr + i * C::RS][wc + (j0 + j) * 32 + (v >> 2) * 8 + (lane >> 5) * 4]) = pk;
        }
}

// Logical tile of workgroup b: the hardware places workgroup b on XCD b % 8,
// so each XCD gets a contiguous run of logical tiles. Logical tiles come in
// groups of G token tiles x every vocabulary tile, token tile fastest within
// a group, so the ~32 tiles an XCD runs at once share G tiles of h and a few
// slices of W in its L2. (Token tile fastest over all of them made each XCD
// read a different h tile per workgroup: at T = 152569 that re-read the 1.09
// GB of h from HBM once per vocabulary slice, 15% slower than groups of 4.)
constexpr int64_t kTileGroup = 4;  // token tiles per group
__device__ __forceinline__ void tile_of_block(int64_t nmt, int64_t nvt, int64_t& mt, int64_t& vt) {
    const int64_t nb = nmt * nvt, q = nb / 8, rr = nb % 8;
    const int64_t b = blockIdx.x, x = b % 8, sl = b / 8;
    const int64_t lg = x * q + min(x, rr) + sl;
    constexpr int64_t G = kTileGroup;
    const int64_t g = lg / (G * nvt), first = g * G;
    const int64_t gm = nmt - first < G ? nmt - first : G;
    const int64_t in = lg - first * nvt;
    mt = first + in % gm;
    vt = in / gm;
}

// The configuration of a last row tile of at most 128 rows where the others have
// 256: the 128-row one, in the place the order gives it, among the tiles that read
// the same slice of W. Only with 3 or 4 row tiles, one group of the order: with 2
// it saves nothing, beyond 4 the last group's tiles are one XCD's, and the gain
// is lost waiting for the others. Measured at d = 3584, V = 152064 (statistics,
// us): 800 rows 945 -> 832, 600 rows 639 -> 616; put after all others, where they
// read W from HBM once more, 600 rows 655.
__host__ __device__ constexpr bool has_rest(int64_t nmt) { return nmt == 3 || nmt == 4; }
template <class C>
struct Rest {
    using type = typename std::conditional<C::BM == LmCfg::BM, LmCfg128, C>::type;
};
// f(configuration, LDS, first row, vocabulary tile) for this workgroup's tile of M
// rows x nvt vocabulary tiles, if it has one.
template <class C, class F>
__device__ __forceinline__ void with_row_tile(int64_t M, int64_t nvt, F&& f) {
    using R = typename Rest<C>::type;
    __shared__ union {
        typename C::Smem full;
        typename R::Smem rest;
    } sm;
    const int64_t nmt = (M + C::BM - 1) / C::BM;
    if ((int64_t)blockIdx.x >= nmt * nvt) return;
    int64_t mt, vt;
    tile_of_block(nmt, nvt, mt, vt);
    const int64_t m0 = mt * C::BM;
    if constexpr (R::BM < C::BM) {
        if (has_rest(nmt) && M - m0 <= R::BM) {
            f(R{}, sm.rest, m0, vt);
            return;
        }
    }
    f(C{}, sm.full, m0, vt);
}

// part[t * nvt + vt] receives the triple of row t over the tile's columns
// other than target[t]; the workgroup holding target[t] writes z_y[t].
template <class C>
__device__ __forceinline__ void lmhead_stats_tile(
    const uint16_t* __restrict__ h, int64_t T, int64_t ldh, const uint16_t* __restrict__ w,
    int64_t V, int64_t ldw, int64_t d, const int32_t* __restrict__ target, float scale,
    int64_t nvt, float4* __restrict__ part, float* __restrict__ z_y, typename C::Smem& sm,
    int64_t m0, int64_t vt) {
#pragma clang fp contract(off)  // the same roundings in every configuration
    const int64_t n0 = vt * C::BN;
    f32x16 acc[C::TM][C::TN];
    gemm_tile<C>(h, T, ldh, w, V, ldw, d, m0, n0, sm, acc);

    // The row's 256 columns are reduced in units of 64, in whatever configuration:
    // a lane's 32 columns of a unit (two 32-column blocks of its half-wave): their
    // maximum, then the sums in base-2 units against it, one partial sum per
    // block; merged with the lane that holds the unit's other columns; the four
    // units merged in column order through LDS. So a row's triple does not depend
    // on the tile height its call takes, or on the tile the row falls in: equal
    // rows have equal statistics, and a step recomputed in another batch the same.
    // (Reducing all of a wave's columns of a row at once, 64 or 128 by the
    // configuration, is 0.3 to 0.7% faster: 3373 against 3384 us at T = 4096, 913
    // against 922 at 1000, d = 3584, V = 152064.) The whole epilogue stays in
    // registers until the last merge.
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), half = lane >> 5;
    const int wr = (wave / C::WN) * 32 + (lane & 31), wc = (wave % C::WN) * (C::BN / C::WN);
    // the inverse temperature enters the base-2 exponent's factor (1 at scale
    // 1: the same bits)
    const float c2 = scale * 1.4426950408889634f;
    static_assert(C::TN % 2 == 0, "units of two 32-column blocks");
#pragma unroll
    for (int i = 0; i < C::TM; ++i) {
        const int64_t t = m0 + wr + i * C::RS;
        const int64_t y = t < T ? (int64_t)target[t] : -1;
#pragma unroll
        for (int u = 0; u < C::TN / 2; ++u) {
            const int64_t u0 = n0 + wc + u * kStatsUnit;
            // columns below vlim (counted from the unit's first) exist
            const int vlim = (int)max(min(V - u0, (int64_t)kStatsUnit), (int64_t)0);
            // the target's column within the unit's (-1: not here)
            const int64_t yrel = y - u0;
            const int y64 = yrel >= 0 && yrel < vlim ? (int)yrel : -1;
            // only the tile's last columns past V and a row's target column drop
            // out: the selects run only in lanes that hold such a column
            const bool masked = vlim < kStatsUnit || (y64 >= 0 && ((y64 >> 2) & 1) == half);
            if (masked) {
                float zy = 0.f;
                // opaque, so that the compiler does not take the comparisons of
                // every row block's columns together, and spill their masks
                int vl = vlim - half * 4, yl = y64 - half * 4;
                asm volatile("" : "+v"(vl), "+v"(yl));
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int col = j * 32 + (v >> 2) * 8 + (v & 3);
                        const float x = acc[i][2 * u + j][v];
                        const bool at_y = col == yl;
                        zy = at_y ? x : zy;
                        acc[i][2 * u + j][v] = col >= vl || at_y ? -INFINITY : x;
                    }
                if (y64 >= 0 && ((y64 >> 2) & 1) == half) z_y[t] = zy * scale;
            }
            float mx = -INFINITY;
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) mx = fmaxf(mx, acc[i][2 * u + j][v]);
            // scale > 0: the maximum of the scaled row is the scaled maximum
            Triple mine = {mx * scale, 0.f, 0.f};
            if (mx > -INFINITY) {
                // e = 2^xl with xl = (x - mx) scale log2(e); where a column was
                // dropped (-inf) xl is floored at -200, where 2^xl is already 0 in
                // fp32, so that it adds 0 (other columns are finite)
                const float ml = mx * c2;
                float s2[2], w2[2];
                auto sums = [&](auto floored) {
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        s2[j] = w2[j] = 0.f;
#pragma unroll
                        for (int v = 0; v < 16; ++v) {
                            float xl = fmaf(acc[i][2 * u + j][v], c2, -ml);
                            if constexpr (decltype(floored)::value) xl = fmaxf(xl, -200.f);
                            const float e = __builtin_amdgcn_exp2f(xl);
                            s2[j] += e;
                            w2[j] = fmaf(e, xl, w2[j]);
                        }
                    }
                };
                if (masked)
                    sums(std::true_type{});
                else
                    sums(std::false_type{});
                mine.s = s2[0] + s2[1];
                mine.w = (w2[0] + w2[1]) * 0.6931471805599453f;
            }
            Triple o;
            o.m = __shfl_xor(mine.m, 32);
            o.s = __shfl_xor(mine.s, 32);
            o.w = __shfl_xor(mine.w, 32);
            mine = half ? merge(o, mine) : merge(mine, o);
            if (half == 0)
                sm.red[wc / kStatsUnit + u][wr + i * C::RS] =
                    make_float4(mine.m, mine.s, mine.w, 0.f);
        }
    }
    lds_ring_barrier();
    for (int r = tid; r < C::BM && m0 + r < T; r += C::THREADS) {
        Triple x = {-INFINITY, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < C::BN / kStatsUnit; ++k) {
            const float4 q = sm.red[k][r];
            x = merge(x, Triple{q.x, q.y, q.z});
        }
        part[(m0 + r) * nvt + vt] = make_float4(x.m, x.s, x.w, 0.f);
    }
}

template <class C>
__global__ void __launch_bounds__(C::THREADS)
lmhead_stats_kernel(const uint16_t* __restrict__ h, int64_t T, int64_t ldh,
                    const uint16_t* __restrict__ w, int64_t V, int64_t ldw, int64_t d,
                    const int32_t* __restrict__ target, float scale, int64_t nvt,
                    float4* __restrict__ part, float* __restrict__ z_y) {
    with_row_tile<C>(T, nvt, [&](auto cfg, auto& sm, int64_t m0, int64_t vt) {
        lmhead_stats_tile<decltype(cfg)>(h, T, ldh, w, V, ldw, d, target, scale, nvt, part, z_y,
                                         sm, m0, vt);
    });
}

// dlogits = s g_t (onehot(y_t) - exp(s z - lse_t)) (s = scale, the inverse
// temperature; lse_t that of s z) for rows [0, M) of the block
// (h and out already offset to the block's first row) and the V vocabulary
// entries vbase .. vbase + V - 1 (w already offset to entry vbase), written in
// bf16 (nearest even) to out [M, ld_out]: the gradient pass of the logits
// path with the logits formed on the fly. The target element is
// s g_t * -expm1(logp_t), accurate when p_y -> 1.
template <class C>
__device__ __forceinline__ void lmhead_dlogits_tile(
    const uint16_t* __restrict__ h, int64_t M, int64_t ldh, const uint16_t* __restrict__ w,
    int64_t V, int64_t ldw, int64_t d, const int32_t* __restrict__ target,
    const float* __restrict__ lse, const float* __restrict__ logp, const float* __restrict__ coef,
    float scale, uint16_t* __restrict__ out, int64_t ld_out, int64_t vbase, typename C::Smem& sm,
    int64_t m0, int64_t vt) {
    const int64_t n0 = vt * C::BN;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), half = lane >> 5;
    const int wr = (wave / C::WN) * 32 + (lane & 31), wc = (wave % C::WN) * (C::BN / C::WN);
    f32x16 acc[C::TM][C::TN];
    gemm_tile<C>(h, M, ldh, w, V, ldw, d, m0, n0, sm, acc);

    // the inverse temperature enters the base-2 exponent's factor (1 at scale
    // 1: the same bits)
    const float c2 = scale * 1.4426950408889634f;
    // the constants of all of the lane's rows ahead of the first store, which a later
    // load would wait for
    float gs[C::TM], lses[C::TM];
    int32_t ys[C::TM];
#pragma unroll
    for (int i = 0; i < C::TM; ++i) {
        const int64_t t = min(m0 + wr + i * C::RS, M - 1);  // rows past M are not stored
        gs[i] = coef[t], lses[i] = lse[t], ys[i] = target[t];
    }
    // Row blocks of 32 rows x the wave's columns: turned into bf16 in registers, then
    // through the wave's own part of the LDS (its accesses run in order: no barrier), so
    // that a row's 256 bytes leave together while the next block is formed. With the
    // whole tile formed, a barrier, and then every store, the stores came in one burst
    // behind the exponentials, which a short K loop does not hide: at d = 512 1000 rows
    // of V = 32000 took 42.2 us, now 39.9, 4096 of 8000 43.9 and 42.7, at d = 3584 4096
    // of 152064 3439 and 3394. (128 bytes at a time are 1 to 3% better where they are
    // whole lines, but rows of 60328 elements took 343 us in place of 300.)
    constexpr int CPR = C::TN * 4, RPI = 64 / CPR;  // 16-byte chunks a row, rows a store
#pragma unroll
    for (int i = 0; i < C::TM; ++i) {
        // -g, -lse log2(e), the target's gradient g (-expm1(logp)) (accurate when
        // p_y -> 1), the target's column; g carries the inverse temperature (the
        // chain rule through scale z)
        const float g = gs[i] * scale;
        const float neg_g = -g, neg_lse = -lses[i] * 1.4426950408889634f;
        const int64_t yrel = (int64_t)ys[i] - vbase - n0 - wc;
        const int y32 = yrel >= 0 && yrel < C::BN / C::WN ? (int)yrel : -1;
#pragma unroll
        for (int j = 0; j < C::TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                acc[i][j][v] = neg_g * __builtin_amdgcn_exp2f(fmaf(acc[i][j][v], c2, neg_lse));
        if (y32 >= 0 && ((y32 >> 2) & 1) == half) {
            const float dy = g * -expm1f(logp[min(m0 + wr + i * C::RS, M - 1)]);
#pragma unroll
            for (int j = 0; j < C::TN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int col = j * 32 + (v >> 2) * 8 + (v & 3);
                    acc[i][j][v] = col == y32 - half * 4 ? dy : acc[i][j][v];
                }
        }
        blocks_to_lds_bf16<C, C::TN>(acc[i], i, 0, sm);
        lds_wave_order();
#pragma unroll
        for (int q = 0; q < 32 / RPI; ++q) {
            const int r = (wave / C::WN) * 32 + i * C::RS + q * RPI + lane / CPR;
            const int c = wc + lane % CPR * 8;
            const int64_t t = m0 + r, col = n0 + c;
            if (t >= M || col >= V) continue;
            const u32x4 pk = *reinterpret_cast<const u32x4*>(&sm.c16[r][c]);
            uint16_t* dst = out + t * ld_out + col;
            if (col + 8 <= V)
                __builtin_nontemporal_store(pk, reinterpret_cast<u32x4*>(dst));
            else
                for (int k = 0; k < 8 && col + k < V; ++k) dst[k] = sm.c16[r][c + k];
        }
    }
}

// With dyn_rows, the block holds only rows below *dyn_rows - dyn_base (the grid
// covers the most it can hold): the tiles are laid over the live rows' tiles,
// so that they spread over every XCD, and the workgroups past them (the last
// ones dispatched) have nothing to do.
template <class C>
__global__ void __launch_bounds__(C::THREADS)
lmhead_dlogits_kernel(const uint16_t* __restrict__ h, int64_t M, int64_t ldh,
                      const uint16_t* __restrict__ w, int64_t V, int64_t ldw, int64_t d,
                      const int32_t* __restrict__ target, const float* __restrict__ lse,
                      const float* __restrict__ logp, const float* __restrict__ coef,
                      float scale, uint16_t* __restrict__ out, int64_t ld_out, int64_t vbase,
                      int64_t nvt, const int32_t* __restrict__ dyn_rows, int64_t dyn_base) {
    if (dyn_rows) {
        const int64_t live = (int64_t)*dyn_rows - dyn_base;
        M = live < M ? (live > 0 ? live : 0) : M;
    }
    with_row_tile<C>(M, nvt, [&](auto cfg, auto& sm, int64_t m0, int64_t vt) {
        lmhead_dlogits_tile<decltype(cfg)>(h, M, ldh, w, V, ldw, d, target, lse, logp, coef, scale,
                                           out, ld_out, vbase, sm, m0, vt);
    });
}

// One wave per row: the row's nvt triples merged lane-strided in index order,
// then across lanes by a butterfly; the target logit is added last, as in
// tok_stats_kernel: lse = M + log S, H = log S - W / S, and logp from
// -log1p(s_rest / e_y) when the target dominates.
__global__ void __launch_bounds__(kMergeWaves * 64)
lmhead_merge_kernel(const float4* __restrict__ part, const float* __restrict__ z_y, int64_t T,
                    int64_t nvt, int64_t V, const int32_t* __restrict__ target,
                    float* __restrict__ logp, float* __restrict__ entropy,
                    float* __restrict__ lse) {
    const int lane = threadIdx.x & 63;
    const int64_t t = (int64_t)blockIdx.x * kMergeWaves + (threadIdx.x >> 6);
    if (t >= T) return;
    Triple acc = {-INFINITY, 0.f, 0.f};
    // a lane's next kMergeBatch triples are loaded together (an empty triple
    // past the last): one after the other, their latency was the kernel's time
    for (int64_t j0 = lane; j0 < nvt; j0 += 64 * kMergeBatch) {
        float4 p[kMergeBatch];
#pragma unroll
        for (int k = 0; k < kMergeBatch; ++k) {
            const int64_t j = j0 + 64 * k;
            p[k] = j < nvt ? part[t * nvt + j] : make_float4(-INFINITY, 0.f, 0.f, 0.f);
        }
#pragma unroll
        for (int k = 0; k < kMergeBatch; ++k) acc = merge(acc, Triple{p[k].x, p[k].y, p[k].z});
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        Triple o;
        o.m = __shfl_xor(acc.m, off);
        o.s = __shfl_xor(acc.s, off);
        o.w = __shfl_xor(acc.w, off);
        acc = merge(acc, o);
    }
    if (lane != 0) return;
    const int64_t y = target[t];
    const float zy = (y >= 0 && y < V) ? z_y[t] : __builtin_nanf("");
    const float M = acc.s > 0.f ? fmaxf(acc.m, zy) : zy;
    float sx = 0.f, wx = 0.f;
    if (acc.s > 0.f) {
        const float dx = acc.m - M;
        const float cx = expf(dx);
        sx = cx * acc.s;
        wx = cx * fmaf(dx, acc.s, acc.w);
    }
    const float xy = zy - M;
    const float ey = expf(xy);
    const float S = sx + ey;
    const float W = fmaf(ey, xy, wx);
    const float ln_s = logf(S);
    lse[t] = M + ln_s;
    entropy[t] = fmaxf(ln_s - W / S, 0.f);
    logp[t] = sx < ey ? -log1pf(sx / ey) : xy - ln_s;
}

// ---------------------------------------------------------------------------
// Backward GEMMs on the matrix cores: C[M, N] (+)= A B with B stored [K][N]
// (N contiguous), for dh = dz W (A = the dz block read along its rows, K
// contiguous; B = the block's rows of W) and dW = dz^T h (A = the dz block
// read down its columns, M contiguous; B = the block's rows of h). The tile,
// waves, K slices and LDS ring are those of the forward tile; what differs is
// how an operand stored with K as its row index reaches the MFMA.
//
// Such an operand's slice sits in LDS as BK rows of 256 elements (its k rows
// as they are stored), chunk c (8 elements, 16 bytes) of row k in slot
// c ^ (4 (k mod 4)). The MFMA wants, in lane l, 8 consecutive k of one column;
// ds_read_b64_tr_b16 transposes 4 x 16 blocks within each 16 lanes: lane l
// receives element l % 4 of the 8 bytes that lane 16 (l / 16) + 4 j + (l % 16) / 4
// loaded, for j = 0..3 (whatever addresses the lanes gave). So lane L of a
// group points at row k0 + L / 4, columns 4 (L % 4) .. + 3 of its group's 16
// columns, and receives column L at rows k0 .. k0 + 3; two such reads give the
// 8 k of one MFMA operand. In one read, the 32 lanes of a half-wave take 4
// rows x 32 columns; the swizzle puts the 4 rows' chunks in 16 distinct bank
// quads (gfx950: 64 banks of 4 bytes), so the reads do not conflict.
// ---------------------------------------------------------------------------

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4* lds_s16x4_ptr;

// Elements of one transposed operand row in LDS (the tile width).
constexpr int kTw = 256;
static_assert(LmCfg::BM == kTw && LmCfg::BN == kTw, "transposed rows are one tile wide");

// Slot of chunk c of row k of a transposed operand tile.
__device__ __forceinline__ int tr_slot(int c, int k) { return c ^ (4 * (k & 3)); }

// acc = this wave's part of C[m0:m0+BM, n0:n0+BN] = A B over k in [kbeg, K), kbeg
// a multiple of BK.
// A_KMAJ: A(m, k) = A[m lda + k], else A(m, k) = A[k lda + m]. B(k, n) =
// B[k ldb + n]. Rows and columns past M, N read zero or whatever lies there
// in the matrices (their results are not stored); k past K is zero in LDS
// (also inside a chunk that straddles K), so the stored row padding up to a
// multiple of 8 may hold anything. lda >= ceil8(K) (A_KMAJ) or ceil8(M),
// ldb >= ceil8(N); rows 16-byte aligned. Layout of acc as in gemm_tile. Ends
// on a barrier with no loads in flight.
template <class C, bool A_KMAJ>
__device__ __forceinline__ void gemm_tile_bwd(const uint16_t* __restrict__ A, int64_t lda,
                                              const uint16_t* __restrict__ B, int64_t ldb,
                                              int64_t M, int64_t N, int64_t kbeg, int64_t K,
                                              int64_t m0, int64_t n0, typename C::Smem& sm,
                                              f32x16 (&acc)[C::TM][C::TN]) {
#if defined(__HIP_DEVICE_COMPILE__)
    static_assert(C::BK == 64 && C::BM == kTw && C::BN == kTw, "backward tile");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = (wave / C::WN) * 32, wc = (wave % C::WN) * (C::BN / C::WN);
#pragma unroll
    for (int i = 0; i < C::TM; ++i)
#pragma unroll
        for (int j = 0; j < C::TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    constexpr int CH = C::CH, BK = C::BK;
    // transposed operands: one load instruction fills 2 rows of 32 chunks
    constexpr int TQ = BK / 2 / C::WAVES;  // load instructions per wave and slice
    static_assert(TQ * 2 * C::WAVES == BK, "transposed rows per wave");
    const int trow = lane >> 5, tslot = lane & 31;
    const int64_t nk = (K + BK - 1) / BK;

    // Buffer loads into LDS, as in gemm_tile: one per-lane offset VGPR per
    // operand, the instruction's rows and the slice as scalar offsets (or,
    // for a transposed operand, the slice in the resource base). A transposed
    // operand's resource ends at the last element of row K - 1 that exists
    // (columns < ceil8(len)), so k rows past K read as zero; chunks past len
    // within a row read the row padding or the next row (their results are
    // not stored).
    const int lrow = lane / CH, lslot = lane % CH;
    static_assert((C::WAVES * C::LROWS) % (16 / CH * CH) == 0, "swizzle period");
    static_assert(C::WAVES % 2 == 0, "transposed swizzle period");
    const int tr_k = wave * 2 + trow;  // transposed row of the lane in instruction 0
    const int tr_c = 8 * tr_slot(tslot, tr_k);
    uint32_t voff_a, qstride_a;
    if constexpr (A_KMAJ) {
        const int r_lane = wave * C::LROWS + lrow;
        voff_a = (uint32_t)((r_lane * lda + (lslot ^ swz<CH>(r_lane)) * 8) * 2);
        qstride_a = (uint32_t)(C::WAVES * C::LROWS * lda * 2);
    } else {
        voff_a = (uint32_t)((tr_k * lda + tr_c) * 2);
        qstride_a = (uint32_t)(C::WAVES * 2 * lda * 2);
    }
    const uint32_t voff_b = (uint32_t)((tr_k * ldb + tr_c) * 2);
    const uint32_t qstride_b = (uint32_t)(C::WAVES * 2 * ldb * 2);
    const __amdgpu_buffer_rsrc_t rsrc_ak = tile_rsrc(A + m0 * lda, (M - m0) * lda * 2);
    // resource of a transposed operand's slice kt: rows kt*BK .. K-1 from column t0
    auto tr_rsrc = [&](const uint16_t* X, int64_t ld, int64_t t0, int64_t len, int64_t kt) {
        const int64_t first = kt * BK * ld + t0;
        const int64_t end = (K - 1) * ld + (len + 7) / 8 * 8;
        return tile_rsrc(X + first, (end - first) * 2);
    };

    // instruction q of wave `wave + hh * HW`
    constexpr int HW = C::WAVES / 2;
    auto lds_a = [&](int buf, int q, int hh) {
        constexpr int per = A_KMAJ ? C::LROWS * BK : 2 * kTw;  // elements per instruction
        return &sm.in.a[buf][0][0] + (q * C::WAVES + wave + hh * HW) * per;
    };
    auto lds_b = [&](int buf, int q, int hh) {
        return &sm.in.b[buf][0][0] + (q * C::WAVES + wave + hh * HW) * 2 * kTw;
    };

    // As in gemm_tile, the first half of the waves issue every load, their
    // own rows and those of the wave HW above (HW * LROWS K-major rows or
    // 2 HW transposed rows further: whole swizzle periods, so the same lane
    // offsets)
    static_assert((HW * C::LROWS) % 16 == 0 && (2 * HW) % 4 == 0, "swizzle periods");
    const uint32_t hstride_ak = (uint32_t)(HW * C::LROWS * lda * 2);
    const uint32_t hstride_at = (uint32_t)(2 * HW * lda * 2);
    const uint32_t hstride_b = (uint32_t)(2 * HW * ldb * 2);
    auto issue = [&](int64_t kt, int buf) {
        if (wave >= HW) return;
        if constexpr (A_KMAJ) {
            const uint32_t kb = (uint32_t)(kt * BK * 2);
#pragma unroll
            for (int q = 0; q < C::IA; ++q)
#pragma unroll
                for (int hh = 0; hh < 2; ++hh)
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(
                        rsrc_ak, lds_ptr(lds_a(buf, q, hh)), 16, voff_a,
                        kb + q * qstride_a + hh * hstride_ak, 0, 0);
        } else {
            const __amdgpu_buffer_rsrc_t ra = tr_rsrc(A, lda, m0, M, kt);
#pragma unroll
            for (int q = 0; q < TQ; ++q)
#pragma unroll
                for (int hh = 0; hh < 2; ++hh)
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, lds_ptr(lds_a(buf, q, hh)), 16,
                                                            voff_a, q * qstride_a + hh * hstride_at,
                                                            0, 0);
        }
        const __amdgpu_buffer_rsrc_t rb = tr_rsrc(B, ldb, n0, N, kt);
#pragma unroll
        for (int q = 0; q < TQ; ++q)
#pragma unroll
            for (int hh = 0; hh < 2; ++hh)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, lds_ptr(lds_b(buf, q, hh)), 16, voff_b,
                                                        q * qstride_b + hh * hstride_b, 0, 0);
    };
    // the partial last slice of a K-major A: k >= K set to 0, also inside the
    // chunk that straddles K (transposed operands read zero rows there)
    auto zero_tail = [&](int64_t kt, int buf) {
        const int kv = (int)(K - kt * BK);  // valid k in this slice, 1 .. BK-1
        uint16_t* a = &sm.in.a[buf][0][0];
        for (int e = tid; e < BK * kTw; e += C::THREADS) {
            // [BM][BK] rows with swizzled chunks: element e is row e / BK,
            // slot (e % BK) / 8, holding chunk slot ^ swz(row)
            const int r = e / BK, sl = (e % BK) / 8;
            const int kk = ((sl ^ swz<CH>(r)) * 8) + (e % 8);
            if (kk >= kv) a[e] = 0;
        }
    };

    // MFMA operand offsets. A (K-major): as gemm_tile. Transposed: lane l
    // points at row ks*16 + 8 (l / 32) + 4 h + (l / 4) % 4 and columns
    // mb + 16 ((l / 16) % 2) + 4 (l % 4) of its 32-column block mb (a multiple
    // of 32, so the chunk is (mb / 8) | ((l / 16) % 2) * 2 | (l % 4) / 2).
    const int kq = (lane >> 2) & 3;
    const int tr_lane_row = 8 * (lane >> 5) + kq;
    const int tr_delta = 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
    auto tr_off = [&](int mb) -> uint32_t {
        const int slot = ((mb / 8) ^ (4 * kq)) | tr_delta;
        return (uint32_t)(tr_lane_row * kTw * 2 + slot * 16 + 8 * (lane & 1));
    };
    uint32_t rda[A_KMAJ ? C::KSTEPS : C::TM], rdb[C::TN];
    if constexpr (A_KMAJ) {
#pragma unroll
        for (int ks = 0; ks < C::KSTEPS; ++ks) {
            const int c = ks * 2 + (lane >> 5), ra = wr + (lane & 31);
            rda[ks] = (uint32_t)(ra * BK + (c ^ swz<CH>(ra)) * 8) * 2;
        }
    } else {
#pragma unroll
        for (int i = 0; i < C::TM; ++i) rda[i] = tr_off(wr + i * C::RS);
    }
    // B's offsets carry its buffers' start (64 KB into the LDS), opaque to the
    // compiler, so that the buffer, the k-step and the half enter as the
    // read's 16-bit immediate (as in gemm_tile)
    const char* const lds0 = reinterpret_cast<const char*>(&sm);
    const uint32_t b_at = (uint32_t)(reinterpret_cast<const char*>(&sm.in.b[0][0][0]) - lds0);
#pragma unroll
    for (int j = 0; j < C::TN; ++j) {
        rdb[j] = b_at + tr_off(wc + j * 32);
        asm volatile("" : "+v"(rdb[j]));
    }
    static_assert(C::NS == 2, "two buffers");
    static_assert((C::NS - 1) * C::BN * BK * 2 + (C::KSTEPS - 1) * 16 * kTw * 2 + 4 * kTw * 2 <
                      65536,
                  "B read immediates");

    auto tr_pair = [&](const char* base, uint32_t off, int ks) -> bf16x8 {
        const int k0 = ks * 16 * kTw * 2;
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (lds_s16x4_ptr)(base + off + k0));
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (lds_s16x4_ptr)(base + off + k0 + 4 * kTw * 2));
        typedef short s16x8 __attribute__((ext_vector_type(8)));
        const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        return __builtin_bit_cast(bf16x8, v);
    };
    bf16x8 af[2][C::TM], bfr[2][C::TN];
    auto read_step = [&](auto bufc, int ks, int set) {
        constexpr int buf = decltype(bufc)::value;
        const char* ba = reinterpret_cast<const char*>(&sm.in.a[buf][0][0]);
        const char* bb = lds0 + buf * C::BN * BK * 2;
#pragma unroll
        for (int i = 0; i < C::TM; ++i) {
            if constexpr (A_KMAJ)
                af[set][i] = __builtin_bit_cast(
                    bf16x8, *reinterpret_cast<const u32x4*>(ba + rda[ks] + i * C::RS * BK * 2));
            else
                af[set][i] = tr_pair(ba, rda[i], ks);
        }
#pragma unroll
        for (int j = 0; j < C::TN; ++j) bfr[set][j] = tr_pair(bb, rdb[j], ks);
    };
    auto mfmas = [&](int set) {
#pragma unroll
        for (int i = 0; i < C::TM; ++i)
#pragma unroll
            for (int j = 0; j < C::TN; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[set][j], af[set][i],
                                                                    acc[i][j], 0, 0, 0);
    };
    auto slice = [&](auto bufc, int64_t kt) {
        constexpr int buf = decltype(bufc)::value;
        wait_vmcnt<0>();
        lds_ring_barrier();
        if (A_KMAJ && (K % BK) && kt == nk - 1) {
            zero_tail(kt, buf);
            lds_ring_barrier();
        }
        if (kt + 1 < nk) issue(kt + 1, buf ^ 1);
        read_step(bufc, 0, 0);
        __builtin_amdgcn_s_setprio(1);
        constexpr int NREAD = (A_KMAJ ? C::TM : 2 * C::TM) + 2 * C::TN;
#pragma unroll
        for (int ks = 0; ks < C::KSTEPS; ++ks) {
            const int cs = ks & 1;
            if (ks < C::KSTEPS - 1) read_step(bufc, ks + 1, cs ^ 1);
            mfmas(cs);
            if (ks < C::KSTEPS - 1) {
#pragma unroll
                for (int g = 0; g < C::TM * C::TN; ++g) {
                    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                }
                __builtin_amdgcn_sched_group_barrier(0x100, NREAD - C::TM * C::TN, 0);
            }
        }
        __builtin_amdgcn_s_setprio(0);
    };
    int64_t kt = kbeg / BK;
    if (kt < nk) issue(kt, 0);
    for (; kt + 1 < nk; kt += 2) {
        slice(std::integral_constant<int, 0>{}, kt);
        slice(std::integral_constant<int, 1>{}, kt + 1);
    }
    if (kt < nk) slice(std::integral_constant<int, 0>{}, kt);
    __syncthreads();
#else
    (void)A, (void)lda, (void)B, (void)ldb, (void)M, (void)N, (void)kbeg, (void)K, (void)m0;
    (void)n0, (void)sm, (void)acc;
#endif
}

// One GEMM of the backward: C[M, N] (+)= A B with gemm_tile_bwd's operands,
// written to out [M, ldc] (fp32, or bf16 bits rounded to nearest even); vec:
// out 16-byte aligned and ldc a multiple of 16 bytes' worth of elements.
struct BwdGemm {
    const uint16_t* A;
    int64_t lda;
    const uint16_t* B;
    int64_t ldb;
    int64_t M, N, K;
    void* out;
    int64_t ldc;
    int vec;
    int64_t nmt, nnt;  // tiles
    // optional device row count: M (dyn_m) or K (dyn_k) is at most
    // *dyn - dyn_base (the grid covers the host values, the most there can be)
    const int32_t* dyn;
    int64_t dyn_base;
    bool dyn_m, dyn_k;
    // optional: row m of the result belongs at row map[m] of out
    const int32_t* map;
    // the sum over k in ksplit parts of kper (a multiple of BK), part i written
    // to out + i * part_stride elements
    int64_t ksplit, kper, part_stride;
};

// Output modes of a backward GEMM: fp32 written, fp32 added to, bf16 written.
enum BwdOut { kOutF32 = 0, kOutF32Acc = 1, kOutBf16 = 2 };

// Logical tile of the workgroup with index b among the nb workgroups of one
// GEMM whose first workgroup sits on XCD 0 (workgroup i of a launch runs on
// XCD i % 8): each XCD takes a contiguous run of logical tiles, column tile
// fastest, so the tiles that share a row block of A run together on one XCD
// and read it from that XCD's L2.
__device__ __forceinline__ void tile_of_block_nfast(int64_t b, int64_t nmt, int64_t nnt,
                                                    int64_t& mt, int64_t& nt) {
    const int64_t nb = nmt * nnt, q = nb / 8, rr = nb % 8;
    const int64_t x = b % 8, sl = b / 8;
    const int64_t lg = x * q + min(x, rr) + sl;
    nt = lg % nnt;
    mt = lg / nnt;
}

// Tile b of GEMM g: the MFMA tile, then the result through LDS.
template <class C, bool A_KMAJ, int OUT>
__device__ __forceinline__ void bwd_gemm_tile(const BwdGemm& g, int64_t b, typename C::Smem& sm) {
    using OutT = typename std::conditional<OUT == kOutBf16, uint16_t, float>::type;
    constexpr bool ACC = OUT == kOutF32Acc;
    int64_t M = g.M, K = g.K, nmt = g.nmt, kbeg = 0;
    const int64_t N = g.N;
    if (g.dyn) {
        const int64_t live = (int64_t)*g.dyn - g.dyn_base;
        const int64_t lim = live > 0 ? live : 0;
        if (g.dyn_k && lim < K) K = lim;
        // no rows of this block to add: nothing to do
        if (K == 0 && ACC) return;
        if (g.dyn_m && lim < M) {
            // the tiles laid over the live rows' tiles (spread over every XCD)
            M = lim;
            nmt = (M + C::BM - 1) / C::BM;
            if (b >= nmt * g.nnt * g.ksplit) return;
        }
    }
    int64_t mt, nt;
    tile_of_block_nfast(b, nmt * g.ksplit, g.nnt, mt, nt);
    OutT* out = static_cast<OutT*>(g.out);
    if (g.ksplit > 1) {  // row tiles of part 0, then of part 1, ...
        const int64_t part = mt / nmt;
        mt -= part * nmt;
        out += part * g.part_stride;
        kbeg = part * g.kper;
        K = kbeg + g.kper < K ? kbeg + g.kper : K;
        if (kbeg >= K && ACC) return;
    }
    const int64_t m0 = mt * C::BM, n0 = nt * C::BN;
    f32x16 acc[C::TM][C::TN];
    gemm_tile_bwd<C, A_KMAJ>(g.A, g.lda, g.B, g.ldb, M, N, kbeg, K, m0, n0, sm, acc);

    // Pieces of 32 rows x 64 columns through the wave's own part of the LDS, without
    // barriers, as in lmhead_dlogits_tile: a row's piece leaves as 16-byte vectors (vec),
    // else one element at a time.
    constexpr int EPC = 16 / sizeof(OutT), CPR = 64 / EPC, RPI = 64 / CPR;  // a chunk, a row,
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;             // a store
    const int wr = (wave / C::WN) * 32, wc = (wave % C::WN) * (C::BN / C::WN);
    const int rr = lane / CPR, cc = lane % CPR * EPC;
#pragma unroll
    for (int i = 0; i < C::TM; ++i)
#pragma unroll
        for (int u = 0; u < C::TN / 2; ++u) {
            const OutT* src;  // the lane's chunk of the piece's first RPI rows
            int ld;
            lds_wave_order();  // fp32 pieces of every i share their rows of the LDS
            if constexpr (OUT == kOutBf16) {
                blocks_to_lds_bf16<C, 2>(&acc[i][2 * u], i, 2 * u, sm);
                src = &sm.c16[wr + i * C::RS + rr][wc + u * 64 + cc];
                ld = C::CROW16;
            } else {
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int v = 0; v < 16; v += 4) {
                        const f32x16& t = acc[i][2 * u + j];
                        const f32x4 x = {t[v], t[v + 1], t[v + 2], t[v + 3]};
                        *reinterpret_cast<f32x4*>(
                            &sm.c[wr + (lane & 31)]
                                 [wc + u * 64 + j * 32 + (v >> 2) * 8 + (lane >> 5) * 4]) = x;
                    }
                src = &sm.c[wr + rr][wc + u * 64 + cc];
                ld = C::CROW;
            }
            lds_wave_order();
            const int64_t m = m0 + wr + i * C::RS + rr, n = n0 + wc + u * 64 + cc;
            // the lane's q-th row of the piece, which is below M
            auto dst = [&](int q) {
                const int64_t r = m + q * RPI;
                return out + (g.map ? (int64_t)g.map[r] : r) * g.ldc + n;
            };
            if (g.vec && n + EPC <= N) {
                typedef typename std::conditional<ACC, f32x4, u32x4>::type Vec;
                Vec x[32 / RPI];
#pragma unroll
                for (int q = 0; q < 32 / RPI; ++q)
                    if constexpr (ACC)
                        if (m + q * RPI < M) x[q] = *reinterpret_cast<const Vec*>(dst(q));
#pragma unroll
                for (int q = 0; q < 32 / RPI; ++q) {
                    const Vec y = *reinterpret_cast<const Vec*>(src + q * RPI * ld);
                    if (m + q * RPI >= M) continue;
                    if constexpr (ACC)
                        x[q] += y;
                    else
                        x[q] = y;
                    *reinterpret_cast<Vec*>(dst(q)) = x[q];
                }
            } else {
                for (int q = 0; q < 32 / RPI && m + q * RPI < M; ++q) {
                    OutT* o = dst(q);
                    for (int e = 0; e < EPC && n + e < N; ++e) {
                        const OutT y = src[q * RPI * ld + e];
                        o[e] = ACC ? o[e] + y : y;
                    }
                }
            }
        }
}

// The two GEMMs of one backward block in one launch: dh = dz W (dz read
// along its rows) on the first n_dh workgroups (a multiple of 8; those past
// dh's tiles return at once), dW = dz^T h (dz read down its columns) on the
// rest. dh has few tiles with a long sum (a block's rows x d) and dW many
// with a short one, so dW's tiles fill the compute units that dh leaves
// free, and both start from the dz block just written.
template <class C, int DH_OUT, int DW_OUT>
__global__ void __launch_bounds__(C::THREADS)
lmhead_bwd_gemms_kernel(BwdGemm dh, BwdGemm dw, int64_t n_dh) {
    __shared__ typename C::Smem sm;
    const int64_t b = blockIdx.x;
    if (b < n_dh) {
        if (b < dh.nmt * dh.nnt * dh.ksplit) bwd_gemm_tile<C, true, DH_OUT>(dh, b, sm);
    } else {
        bwd_gemm_tile<C, false, DW_OUT>(dw, b - n_dh, sm);
    }
}

int64_t vocab_tiles(int64_t V) { return (V + LmCfg::BN - 1) / LmCfg::BN; }

// Whether row t takes part in the compact problem. Its dlogits are zeros when
// its coefficient is 0: by the caller's word under the skip flag (lse null),
// else where lse is finite (an infinity or a NaN in the row would give NaNs).
__device__ __forceinline__ bool row_counts(const float* __restrict__ coef,
                                           const float* __restrict__ lse, int64_t t) {
    return coef[t] != 0.f || (lse && !(fabsf(lse[t]) < INFINITY));
}

// The rows that count, in increasing order: map[0 .. n) and count[0] = n. One
// workgroup walks the rows 1024 at a time; the position of each kept row is its
// wave's ballot prefix plus the earlier waves' counts.
constexpr int kCompactThreads = 1024;
__global__ void __launch_bounds__(kCompactThreads)
compact_rows_kernel(const float* __restrict__ coef, const float* __restrict__ lse, int64_t T,
                    int32_t* __restrict__ map, int32_t* __restrict__ count) {
    __shared__ int wave_n[kCompactThreads / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int64_t base = 0;
    for (int64_t t0 = 0; t0 < T; t0 += kCompactThreads) {
        const int64_t t = t0 + tid;
        const bool keep = t < T && row_counts(coef, lse, t);
        const uint64_t ballot = __ballot(keep);
        const int before = __popcll(ballot & ((uint64_t(1) << lane) - 1));
        if (lane == 0) wave_n[wave] = __popcll(ballot);
        __syncthreads();
        int off = 0, total = 0;
        for (int w = 0; w < kCompactThreads / 64; ++w) {
            off += w < wave ? wave_n[w] : 0;
            total += wave_n[w];
        }
        if (keep) map[base + off + before] = (int32_t)t;
        base += total;
        __syncthreads();
    }
    if (tid == 0) count[0] = (int32_t)base;
}

// An element of a gradient output: fp32, or bf16 bits rounded to nearest even.
__device__ __forceinline__ void put(float* p, float v) { *p = v; }
__device__ __forceinline__ void put(uint16_t* p, float v) { *p = bf16_bits(v); }

// Row i < count of the compact problem: hidden row map[i] and its per-row
// values; and row i of dh set to 0 where it does not count: one workgroup per row
// (grid-stride over the rows). lse_word: lse or null, as row_counts takes it.
template <class O>
__global__ void __launch_bounds__(128)
gather_rows_kernel(const int32_t* __restrict__ map, const int32_t* __restrict__ count, int64_t T,
                   const uint16_t* __restrict__ h, int64_t ld_h, int64_t d,
                   const int32_t* __restrict__ target, const float* __restrict__ lse,
                   const float* __restrict__ logp, const float* __restrict__ coef,
                   const float* __restrict__ lse_word, uint16_t* __restrict__ h_c,
                   int32_t* __restrict__ target_c, float* __restrict__ lse_c,
                   float* __restrict__ logp_c, float* __restrict__ coef_c, O* __restrict__ dh,
                   int64_t ld_dh) {
    const int64_t n = count[0];
    for (int64_t i = blockIdx.x; i < T; i += gridDim.x) {
        if (!row_counts(coef, lse_word, i))
            for (int64_t c = threadIdx.x; c < d; c += 128) put(dh + i * ld_dh + c, 0.f);
        if (i >= n) continue;
        const int64_t t = map[i];
        const u32x4* src = reinterpret_cast<const u32x4*>(h + t * ld_h);
        u32x4* dst = reinterpret_cast<u32x4*>(h_c + i * d);
        for (int64_t j = threadIdx.x; j < d / 8; j += 128) dst[j] = src[j];
        if (threadIdx.x == 0) {
            target_c[i] = target[t];
            lse_c[i] = lse[t];
            logp_c[i] = logp[t];
            coef_c[i] = coef[t];
        }
    }
}

// dst[r, c] = bf16(src[r, c]) for rows [0, rows), columns [0, cols).
__global__ void __launch_bounds__(256)
to_bf16_kernel(const float* __restrict__ src, int64_t ld_src, int64_t rows, int64_t cols,
               uint16_t* __restrict__ dst, int64_t ld_dst) {
    for (int64_t r = blockIdx.x; r < rows; r += gridDim.x)
        for (int64_t c = threadIdx.x; c < cols; c += 256)
            dst[r * ld_dst + c] = bf16_bits(src[r * ld_src + c]);
}

// The sum of the ksplit parts of dh (each [rows, d] fp32, part_stride elements
// apart) in part order, for rows [0, rows), with dyn_rows those below
// *dyn_rows - dyn_base; row r goes to row r of out, or (map, its first entry
// that of row 0) to row map[r]. Four columns a work-item at a time, grid-stride: all
// T rows at once (the compact rows of one sum) are more than a dispatch holds from
// T d = 2^34 on.
template <class O>
__global__ void __launch_bounds__(256)
sum_parts_kernel(const float* __restrict__ part, int64_t ksplit, int64_t part_stride, int64_t rows,
                 int64_t d, const int32_t* __restrict__ map, O* __restrict__ out, int64_t ld_out,
                 const int32_t* __restrict__ dyn_rows, int64_t dyn_base) {
    if (dyn_rows) {
        const int64_t live = (int64_t)*dyn_rows - dyn_base;
        rows = live < rows ? live : rows;
    }
    const int64_t step = (int64_t)gridDim.x * 256;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i * 4 < rows * d; i += step) {
        const f32x4* p = reinterpret_cast<const f32x4*>(part) + i;  // d % 8 == 0
        f32x4 x = p[0];
#pragma unroll 8
        for (int64_t k = 1; k < ksplit; ++k) x += p[k * (part_stride / 4)];
        const int64_t r = i * 4 / d;
        O* o = out + (map ? (int64_t)map[r] : r) * ld_out + (i * 4 - r * d);
#pragma unroll
        for (int q = 0; q < 4; ++q) put(o + q, x[q]);
    }
}

// Workgroups of the row kernels above: one per row (of the sum of parts: per 1024
// elements) up to this many.
constexpr int64_t kRowBlocks = 65536;

// The MFMA tile addresses its rows by 32-bit byte offsets from the tile's first
// row: (BM - 1) rows of ld elements must stay below 2^31 bytes.
constexpr int64_t kMaxLd = int64_t(1) << 22;

// Rows of the tile that forms rows x V logits fastest: 64, 128 or 256. One
// workgroup runs per compute unit, so a launch takes its tiles in rounds of
// kUnits, and a round of 256-, 128- or 64-row tiles takes 92, 54 or 45 us at
// d = 3584 (T = 1000, 1000 and 256): the tile with the least rounds x time. So
// 64 rows go as one 64-row tile, up to 128 and 129 - 256 as 128-row tiles at
// V = 152064, more as 256-row ones (the last one of up to 128 rows as in Rest),
// unless those would leave units idle (1000 rows of V = 8000).
// The times' ratios at d = 3584 serve every depth: of 99 sizes (d = 512, 1024 and 2048;
// V = 8000, 32000 and 152064; T from 16 to 2100) the choice is within 5% of the fastest
// of the three but for 600 rows of V = 32000 (58.1 against 54.4 us at d = 1024, 96.6
// against 88.3 at 2048, by the last tile's rule), and none takes longer than with
// 256-row tiles alone (statistics).
// A round of 128-row tiles of dlogits is worth 57 us up to d = 1024, where the two
// heights come within 5% of each other (129 to 256 rows of V = 152064): the taller tile
// reads W once and has fewer first slices to wait for. 130 rows 50.0 us in 128-row
// tiles and 45.8 in 256-row ones at d = 512, 87.0 and 83.0 at 1024; 170 and 181 at 2048.
constexpr int64_t kUnits = 256;
int tile_rows(int64_t rows, int64_t V, double t128 = 54) {
    const double nvt = (double)((V + LmCfg::BN - 1) / LmCfg::BN), t256 = 92, t64 = 45;
    auto rounds = [](double tiles) { return ceil(tiles / kUnits); };
    const int64_t nmt = (rows + 255) / 256, r = rows % 256;
    double least = rounds((double)nmt * nvt) * t256;
    // short tiles among the long ones take 71 us, and half a tile's wait at the end
    if (has_rest(nmt) && r > 0 && r <= 128)
        least = fmin(least, fmax(((double)(nmt - 1) * t256 + 71) * nvt / kUnits + 27, t256));
    int best = 256;
    const double c128 = rounds((double)((rows + 127) / 128) * nvt) * t128;
    const double c64 = rounds((double)((rows + 63) / 64) * nvt) * t64;
    if (c128 < least) best = 128, least = c128;
    if (c64 < least) best = 64;
    return best;
}

// Host-side argument rules shared by the LM-head entry points.
bool bad_lmhead_args(const void* hidden, int64_t T, int64_t d, int64_t ld_h, const void* weight,
                     int64_t V, int64_t ld_w) {
    if (!hidden || !weight) return true;
    if (T < 1 || V < 1 || d < 8 || T > 0x7FFFFFFFll || V > 0x7FFFFFFFll || d > 0x7FFFFFFFll)
        return true;
    if (d % 8 || ld_h < d || ld_w < d || ld_h % 8 || ld_w % 8) return true;
    return reinterpret_cast<uintptr_t>(hidden) % 16 || reinterpret_cast<uintptr_t>(weight) % 16;
}

// f(configuration of bm-row tiles) for rows x V logits. The launch's limits are checked
// with 256-row tiles, as ever; smaller ones are taken where they fit too.
template <class F>
void with_tile(int bm, int64_t rows, int64_t V, F&& f) {
    if (!grid_fits((rows + bm - 1) / bm * vocab_tiles(V), LmCfg::THREADS)) bm = 256;
    if (bm == 64)
        f(LmCfg64{});
    else if (bm == 128)
        f(LmCfg128{});
    else
        f(LmCfg{});
}

dart_status_t launch_dlogits(const uint16_t* hidden, int64_t rows, int64_t d, int64_t ld_h,
                             const uint16_t* weight, int64_t V, int64_t ld_w,
                             const int32_t* target, const float* lse, const float* logp,
                             const float* coef, float scale, uint16_t* out, int64_t ld_out,
                             int64_t vbase, hipStream_t stream, const int32_t* dyn_rows = nullptr,
                             int64_t dyn_base = 0) {
    const int64_t nmt = (rows + LmCfg::BM - 1) / LmCfg::BM, nvt = vocab_tiles(V);
    if (!grid_fits(nmt * nvt, LmCfg::THREADS) || ld_h > kMaxLd || ld_w > kMaxLd)
        return DART_ERR_UNSUPPORTED;
    with_tile(tile_rows(rows, V, d <= 1024 ? 57 : 54), rows, V, [&](auto cfg) {
        using C = decltype(cfg);
        const int64_t nm = (rows + C::BM - 1) / C::BM;
        hipLaunchKernelGGL(lmhead_dlogits_kernel<C>, dim3((unsigned)(nm * nvt)), dim3(C::THREADS),
                           0, stream, hidden, rows, ld_h, weight, V, ld_w, d, target, lse, logp,
                           coef, scale, out, ld_out, vbase, nvt, dyn_rows, dyn_base);
    });
    return hipGetLastError() == hipSuccess ? DART_OK : DART_ERR_HIP;
}

}  // namespace

extern "C" {

size_t dart_lmhead_stats_workspace_bytes(int64_t T, int64_t V) {
    if (T < 1 || V < 1 || T > 0x7FFFFFFFll || V > 0x7FFFFFFFll) return 0;
    return (size_t)T * (size_t)vocab_tiles(V) * sizeof(float4) + (size_t)T * sizeof(float);
}

dart_status_t dart_lmhead_tok_stats_ex(const void* hidden, int64_t T, int64_t d, int64_t ld_h,
                                       const void* weight, int64_t V, int64_t ld_w,
                                       const int32_t* target, float inv_temp, float* logp,
                                       float* entropy, float* lse, void* workspace,
                                       size_t workspace_bytes, hipStream_t stream) {
    if (bad_lmhead_args(hidden, T, d, ld_h, weight, V, ld_w)) return DART_ERR_INVALID_ARG;
    if (!(inv_temp > 0.f) || isinf(inv_temp)) return DART_ERR_INVALID_ARG;
    if (!target || !logp || !entropy || !lse || !workspace ||
        reinterpret_cast<uintptr_t>(workspace) % 16)
        return DART_ERR_INVALID_ARG;
    if (const dart_status_t ck = dart_check::run(
            stream, {{dart_check::Item::Ids, target, T, V}}); ck != DART_OK)
        return ck;

    if (workspace_bytes < dart_lmhead_stats_workspace_bytes(T, V)) return DART_ERR_INVALID_ARG;
    const int64_t nmt = (T + LmCfg::BM - 1) / LmCfg::BM, nvt = vocab_tiles(V);
    if (!grid_fits(nmt * nvt, LmCfg::THREADS) ||
        !grid_fits((T + kMergeWaves - 1) / kMergeWaves, kMergeWaves * 64) || ld_h > kMaxLd ||
        ld_w > kMaxLd)
        return DART_ERR_UNSUPPORTED;
    float4* part = static_cast<float4*>(workspace);
    float* z_y = reinterpret_cast<float*>(part + T * nvt);
    with_tile(tile_rows(T, V), T, V, [&](auto cfg) {
        using C = decltype(cfg);
        const int64_t nm = (T + C::BM - 1) / C::BM;
        hipLaunchKernelGGL(lmhead_stats_kernel<C>, dim3((unsigned)(nm * nvt)), dim3(C::THREADS), 0,
                           stream, static_cast<const uint16_t*>(hidden), T, ld_h,
                           static_cast<const uint16_t*>(weight), V, ld_w, d, target, inv_temp, nvt,
                           part, z_y);
    });
    hipLaunchKernelGGL(lmhead_merge_kernel, dim3((unsigned)((T + kMergeWaves - 1) / kMergeWaves)),
                       dim3(kMergeWaves * 64), 0, stream, part, z_y, T, nvt, V, target, logp,
                       entropy, lse);
    return hipGetLastError() == hipSuccess ? DART_OK : DART_ERR_HIP;
}

dart_status_t dart_lmhead_tok_stats(const void* hidden, int64_t T, int64_t d, int64_t ld_h,
                                    const void* weight, int64_t V, int64_t ld_w,
                                    const int32_t* target, float* logp, float* entropy,
                                    float* lse, void* workspace, size_t workspace_bytes,
                                    hipStream_t stream) {
    return dart_lmhead_tok_stats_ex(hidden, T, d, ld_h, weight, V, ld_w, target, 1.f, logp,
                                    entropy, lse, workspace, workspace_bytes, stream);
}

dart_status_t dart_lmhead_dlogits_ex(const void* hidden, int64_t T, int64_t d, int64_t ld_h,
                                     const void* weight, int64_t V, int64_t ld_w,
                                     const int32_t* target, const float* lse, const float* logp,
                                     const float* tok_coef, float inv_temp, void* dlogits,
                                     int64_t ld_out, hipStream_t stream) {
    if (bad_lmhead_args(hidden, T, d, ld_h, weight, V, ld_w)) return DART_ERR_INVALID_ARG;
    if (!(inv_temp > 0.f) || isinf(inv_temp)) return DART_ERR_INVALID_ARG;
    if (!target || !lse || !logp || !tok_coef || !dlogits || ld_out < V || ld_out % 8 ||
        reinterpret_cast<uintptr_t>(dlogits) % 16)
        return DART_ERR_INVALID_ARG;
    if (const dart_status_t ck = dart_check::run(
            stream, {{dart_check::Item::Ids, target, T, V}}); ck != DART_OK)
        return ck;

    return launch_dlogits(static_cast<const uint16_t*>(hidden), T, d, ld_h,
                          static_cast<const uint16_t*>(weight), V, ld_w, target, lse, logp,
                          tok_coef, inv_temp, static_cast<uint16_t*>(dlogits), ld_out, 0, stream);
}

dart_status_t dart_lmhead_dlogits(const void* hidden, int64_t T, int64_t d, int64_t ld_h,
                                  const void* weight, int64_t V, int64_t ld_w,
                                  const int32_t* target, const float* lse, const float* logp,
                                  const float* tok_coef, void* dlogits, int64_t ld_out,
                                  hipStream_t stream) {
    return dart_lmhead_dlogits_ex(hidden, T, d, ld_h, weight, V, ld_w, target, lse, logp, tok_coef,
                                  1.f, dlogits, ld_out, stream);
}

size_t dart_lmhead_backward_workspace_bytes(int64_t chunk_rows, int64_t V) {
    if (chunk_rows < 1 || V < 1 || chunk_rows > 0x7FFFFFFFll || V > 0x7FFFFFFFll) return 0;
    return (size_t)chunk_rows * (size_t)((V + 7) / 8 * 8) * 2;
}

}  // extern "C"

namespace {

constexpr uint32_t kBackwardFlags = DART_LMHEAD_SKIP_ZERO_ROWS | DART_LMHEAD_BF16_GRADS;

int64_t ceil8(int64_t x) { return (x + 7) / 8 * 8; }
size_t align256(size_t x) { return (x + 255) / 256 * 256; }

// How a backward call runs and where its parts sit in the workspace (byte
// offsets, each part 256-byte aligned; total is the end of the last part).
struct BackwardPlan {
    bool bf16, skip;
    int64_t rows, cols;  // block of rows x vocabulary entries, at most T x V
    bool acc_w;          // dW summed over row blocks into bf16: through fp32
    bool acc_h;          // dh summed over vocabulary blocks into bf16: through fp32
    size_t dz, accw, acch, h_c, dh_c, target_c, lse_c, logp_c, coef_c, map, count, total;
    // beyond total, used where the caller's workspace reaches split_total: dh's
    // sum over the vocabulary in ksplit parts (1: none), and room to leave out
    // rows with zero dlogits without being told to (compact)
    int64_t ksplit;
    bool compact;
    size_t parts, split_total;
};

// Whether a call that is not told to skip zero rows leaves them out all the
// same, as the gradient pass on logits does: where that is worth the kernels
// around it (finding the rows and copying them: 7 us at T = 1000, 20 at 2500, d = 3584,
// against the share of zero rows of a backward that takes at least 0.5 ms) and the
// compact rows fit 128 MiB. Few rows are bound by W and dW, not by their number.
// Measured at d = 3584, V = 152064, bf16 gradients: with 20% zero rows 2738 -> 2568
// us at T = 1000 and 10107 -> 8629 at 4096, with 50% 2668 -> 1658 and 9830 -> 5626;
// with none 2801 -> 2808 and 10475 -> 10490, at T = 2500 1425 -> 1442 (V = 32000) and
// 979 -> 990 (V = 20000). Below the line, at T = 1500, V = 14000, d = 1776 (3.7e10),
// leaving none out costs 3%.
bool leaves_zero_rows_out(int64_t T, int64_t d, int64_t V) {
    return T >= 256 && (double)T * (double)V * (double)d >= 1e11 &&
           (double)T * (double)(6 * d + 20) <= double(128 << 20);
}

// Parts of a block's dh sum. dh has rows / 256 x d / 256 tiles, each a sum over
// the block's whole vocabulary, and one launch holds them and dW's tiles, the
// same work in many short sums: while dh's tiles fill less than half of the
// compute units the launch waits for them (at 1000 rows, d = 3584, V = 152064:
// 56 tiles of 2376 slices, 3.62 ms; in 2, 4 or 9 parts 2.10, 1.95 or 2.02 ms, adding
// them up 7, 17 or 37 us more). So that at least half
// and at most all of the units have a part, none shorter than kMinPartSlices.
constexpr int64_t kMinPartSlices = 32;
int64_t dh_parts(int64_t rows, int64_t d, int64_t cols) {
    const int64_t tiles =
        ((rows + LmCfg::BM - 1) / LmCfg::BM) * ((d + LmCfg::BN - 1) / LmCfg::BN);
    const int64_t by_units = kUnits / tiles, by_k = cols / (LmCfg::BK * kMinPartSlices);
    const int64_t n = by_units < by_k ? by_units : by_k;
    return n > 1 ? n : 1;
}

// total = 0 when the sizes do not fit the address arithmetic.
BackwardPlan plan_backward(int64_t T, int64_t d, int64_t V, int64_t chunk_rows,
                           int64_t chunk_cols, uint32_t flags) {
    BackwardPlan P = {};
    P.bf16 = flags & DART_LMHEAD_BF16_GRADS;
    P.skip = flags & DART_LMHEAD_SKIP_ZERO_ROWS;
    P.rows = chunk_rows < T ? chunk_rows : T;
    P.cols = chunk_cols < V ? chunk_cols : V;
    // with rows skipped, dh is summed in the compact fp32 rows
    P.acc_w = P.bf16 && P.rows < T;
    P.acc_h = P.bf16 && P.cols < V && !P.skip;
    const double big = double(int64_t(1) << 60);
    if ((double)P.rows * (double)ceil8(P.cols) * 2 > big || (double)V * (double)d * 4 > big ||
        (double)T * (double)d * 6 > big)
        return P;
    size_t end = 0;
    auto take = [&](size_t bytes) {
        const size_t at = align256(end);
        end = at + bytes;
        return at;
    };
    P.dz = take((size_t)P.rows * (size_t)ceil8(P.cols) * 2);
    if (P.acc_w) P.accw = take((size_t)V * (size_t)d * 4);
    if (P.acc_h) P.acch = take((size_t)T * (size_t)d * 4);
    auto take_rows = [&] {
        P.h_c = take((size_t)T * (size_t)d * 2);
        P.dh_c = take((size_t)T * (size_t)d * 4);
        P.target_c = take((size_t)T * 4);
        P.lse_c = take((size_t)T * 4);
        P.logp_c = take((size_t)T * 4);
        P.coef_c = take((size_t)T * 4);
        P.map = take((size_t)T * 4);
        P.count = take(4);
    };
    if (P.skip) take_rows();
    P.total = end;
    P.ksplit = dh_parts(P.rows, d, P.cols);
    P.compact = !P.skip && leaves_zero_rows_out(T, d, V);
    if (P.compact) take_rows();
    if (P.ksplit > 1) P.parts = take((size_t)P.ksplit * (size_t)P.rows * (size_t)d * 4);
    P.split_total = end;
    return P;
}

// A gradient output: row-major, fp32 or bf16.
struct Grad {
    void* p;
    int64_t ld;
    bool bf16;
    void* row(int64_t r) const {
        return static_cast<char*>(p) + r * ld * (bf16 ? 2 : 4);
    }
};

// The GEMM description of one backward output (out.p at the block's first
// row); mode: kOutF32, kOutF32Acc or kOutBf16.
BwdGemm make_bwd_gemm(const uint16_t* A, int64_t lda, const uint16_t* B, int64_t ldb, int64_t M,
                      int64_t N, int64_t K, const Grad& out) {
    BwdGemm g;
    g.A = A, g.lda = lda, g.B = B, g.ldb = ldb, g.M = M, g.N = N, g.K = K;
    g.out = out.p, g.ldc = out.ld;
    const size_t esz = out.bf16 ? 2 : 4;
    g.vec = reinterpret_cast<uintptr_t>(out.p) % 16 == 0 && (out.ld * esz) % 16 == 0;
    g.nmt = (M + LmCfg::BM - 1) / LmCfg::BM;
    g.nnt = (N + LmCfg::BN - 1) / LmCfg::BN;
    g.dyn = nullptr, g.dyn_base = 0, g.dyn_m = g.dyn_k = false;
    g.map = nullptr, g.ksplit = 1, g.kper = K, g.part_stride = 0;
    return g;
}

int out_mode(const Grad& out, bool accumulate) {
    return out.bf16 ? kOutBf16 : accumulate ? kOutF32Acc : kOutF32;
}

template <int DH, int DW>
void launch_bwd_gemms_t(const BwdGemm& dh, const BwdGemm& dw, int64_t n_dh, int64_t blocks,
                        hipStream_t stream) {
    hipLaunchKernelGGL((lmhead_bwd_gemms_kernel<LmCfg, DH, DW>), dim3((unsigned)blocks),
                       dim3(LmCfg::THREADS), 0, stream, dh, dw, n_dh);
}

template <int DH>
void launch_bwd_gemms_dw(int dw_mode, const BwdGemm& dh, const BwdGemm& dw, int64_t n_dh,
                         int64_t blocks, hipStream_t stream) {
    if (dw_mode == kOutF32) launch_bwd_gemms_t<DH, kOutF32>(dh, dw, n_dh, blocks, stream);
    else if (dw_mode == kOutF32Acc) launch_bwd_gemms_t<DH, kOutF32Acc>(dh, dw, n_dh, blocks, stream);
    else launch_bwd_gemms_t<DH, kOutBf16>(dh, dw, n_dh, blocks, stream);
}

// One block's dh[rows, d] (+)= dz[rows, cols] W[cols, d] and
// dW[cols, d] (+)= dz[rows, cols]^T h[rows, d], in one launch. A bf16 output
// is never added to (sums over blocks go through fp32). With ksplit > 1 dh_out is
// ksplit fp32 matrices part_stride elements apart, which each get their part of
// the sum. With dh_map row i of dh goes to row dh_map[i] of dh_out. With dyn_rows,
// the block's rows are at most *dyn_rows - dyn_base (read on the device).
dart_status_t launch_bwd_gemms(const uint16_t* dz, int64_t ld_dz, int64_t rows, int64_t cols,
                               const uint16_t* w, int64_t ld_w, const uint16_t* h, int64_t ld_h,
                               int64_t d, const Grad& dh_out, bool dh_acc, int64_t ksplit,
                               int64_t part_stride, const Grad& dw_out, bool dw_acc,
                               hipStream_t stream, const int32_t* dh_map, const int32_t* dyn_rows,
                               int64_t dyn_base) {
    if ((dh_out.bf16 && dh_acc) || (dw_out.bf16 && dw_acc)) return DART_ERR_INVALID_ARG;
    if (ld_dz > kMaxLd || ld_w > kMaxLd || ld_h > kMaxLd || dh_out.ld > kMaxLd ||
        dw_out.ld > kMaxLd)
        return DART_ERR_UNSUPPORTED;
    BwdGemm dh = make_bwd_gemm(dz, ld_dz, w, ld_w, rows, d, cols, dh_out);
    BwdGemm dw = make_bwd_gemm(dz, ld_dz, h, ld_h, cols, d, rows, dw_out);
    // the block's rows are dh's M and dW's K
    dh.dyn = dw.dyn = dyn_rows;
    dh.dyn_base = dw.dyn_base = dyn_base;
    dh.dyn_m = dw.dyn_k = dyn_rows != nullptr;
    dh.map = dh_map;
    if (ksplit > 1) {
        const int64_t nk = (cols + LmCfg::BK - 1) / LmCfg::BK;
        dh.ksplit = ksplit, dh.kper = (nk + ksplit - 1) / ksplit * LmCfg::BK;
        dh.part_stride = part_stride;
    }
    const int64_t n_dh = (dh.nmt * dh.nnt * ksplit + 7) / 8 * 8;
    const int64_t blocks = n_dh + dw.nmt * dw.nnt;
    if (!grid_fits(blocks, LmCfg::THREADS)) return DART_ERR_UNSUPPORTED;
    const int dhm = out_mode(dh_out, dh_acc), dwm = out_mode(dw_out, dw_acc);
    if (dhm == kOutF32) launch_bwd_gemms_dw<kOutF32>(dwm, dh, dw, n_dh, blocks, stream);
    else if (dhm == kOutF32Acc) launch_bwd_gemms_dw<kOutF32Acc>(dwm, dh, dw, n_dh, blocks, stream);
    else launch_bwd_gemms_dw<kOutBf16>(dwm, dh, dw, n_dh, blocks, stream);
    return hipGetLastError() == hipSuccess ? DART_OK : DART_ERR_HIP;
}

void launch_to_bf16(const float* src, int64_t rows, int64_t cols, const Grad& dst,
                    hipStream_t stream) {
    const unsigned blocks = (unsigned)(rows < kRowBlocks ? rows : kRowBlocks);
    hipLaunchKernelGGL(to_bf16_kernel, dim3(blocks), dim3(256), 0, stream, src, cols, rows, cols,
                       static_cast<uint16_t*>(dst.p), dst.ld);
}

// The gradient pass over rows [0, T) of h in blocks of rows x vocabulary
// entries: per block, its dlogits into dz (bf16), then the block's share of
// dh (summed over the vocabulary blocks of its rows) and of dW (summed over
// the row blocks of its entries). A sum goes into its fp32 output directly,
// or, for a bf16 output that more than one block adds to, into acc_h ([T, d])
// or acc_w ([V, d]) and is rounded to bf16 once at the end; an output that
// one block writes is that GEMM's fp32 result rounded once. With dyn_rows, T
// is the most rows there can be and only the first *dyn_rows are formed (the
// count is read on the device: blocks past it have nothing to do, and the
// first row block writes dW even when it holds no rows). With parts (ksplit > 1),
// a row block's dh is summed there, [ksplit][R, d], and added up once its last
// vocabulary block is in. With map (and dyn_rows), the rows are compact ones and
// row i of dh belongs at row map[i]: the GEMM puts it there, unless its sum needs
// acc_h ([T, d]) or the parts, from where it is put there at the end. (With every sum
// in acc_h first, 2500 rows of V = 20000, d = 3584, none of them zero, took 1012 us
// with bf16 gradients and 1052 with fp32 ones, now 990 and 1022; 999 and 1006 where
// the rows are not looked at.)
dart_status_t backward_core(const uint16_t* h, int64_t T, int64_t d,
                            int64_t ld_h, const uint16_t* w, int64_t V, int64_t ld_w,
                            const int32_t* target, const float* lse, const float* logp,
                            const float* coef, float scale, const Grad& dh, const Grad& dw,
                            int64_t R,
                            int64_t C, uint16_t* dz, float* acc_h, float* acc_w, float* parts,
                            int64_t ksplit, hipStream_t stream, const int32_t* map = nullptr,
                            const int32_t* dyn_rows = nullptr) {
    if (R > T) R = T;
    if (C > V) C = V;
    const int64_t ld_dz = ceil8(C);
    const bool via_h = !parts && dh.bf16 && C < V, via_w = dw.bf16 && R < T;
    const bool put = map && !parts && !via_h;
    auto sum_parts = [&](const float* p, int64_t n, int64_t stride, int64_t r0, int64_t rows) {
        const int64_t blocks = (rows * d / 4 + 255) / 256;
        const dim3 grid((unsigned)(blocks < kRowBlocks ? blocks : kRowBlocks));
        const int32_t* m = map ? map + r0 : nullptr;
        void* out = map ? dh.p : dh.row(r0);
        if (dh.bf16)
            hipLaunchKernelGGL(sum_parts_kernel<uint16_t>, grid, dim3(256), 0, stream, p, n, stride,
                               rows, d, m, static_cast<uint16_t*>(out), dh.ld, dyn_rows, r0);
        else
            hipLaunchKernelGGL(sum_parts_kernel<float>, grid, dim3(256), 0, stream, p, n, stride,
                               rows, d, m, static_cast<float*>(out), dh.ld, dyn_rows, r0);
    };
    const Grad sum_h = via_h ? Grad{acc_h, d, false} : dh;
    const Grad sum_w = via_w ? Grad{acc_w, d, false} : dw;
    for (int64_t r0 = 0; r0 < T; r0 += R) {
        const int64_t rows = T - r0 < R ? T - r0 : R;
        const uint16_t* hr = h + r0 * ld_h;
        for (int64_t c0 = 0; c0 < V; c0 += C) {
            const int64_t cols = V - c0 < C ? V - c0 : C;
            const uint16_t* wc = w + c0 * ld_w;
            const dart_status_t st =
                launch_dlogits(hr, rows, d, ld_h, wc, cols, ld_w, target + r0, lse + r0,
                               logp + r0, coef + r0, scale, dz, ld_dz, c0, stream, dyn_rows, r0);
            if (st != DART_OK) return st;
            const dart_status_t sg = launch_bwd_gemms(
                dz, ld_dz, rows, cols, wc, ld_w, hr, ld_h, d,
                parts ? Grad{parts, d, false}
                      : Grad{put ? sum_h.p : sum_h.row(r0), sum_h.ld, sum_h.bf16},
                c0 > 0, parts ? ksplit : 1, R * d, Grad{sum_w.row(c0), sum_w.ld, sum_w.bf16},
                r0 > 0, stream, put ? map + r0 : nullptr, dyn_rows, r0);
            if (sg != DART_OK) return sg;
        }
        if (parts) sum_parts(parts, ksplit, R * d, r0, rows);
    }
    if (via_h && map)
        sum_parts(acc_h, 1, 0, 0, T);
    else if (via_h)
        launch_to_bf16(acc_h, T, d, dh, stream);
    if (via_w) launch_to_bf16(acc_w, V, d, dw, stream);
    return hipGetLastError() == hipSuccess ? DART_OK : DART_ERR_HIP;
}

}  // namespace

extern "C" {

size_t dart_lmhead_backward_ex_workspace_bytes(int64_t T, int64_t d, int64_t V,
                                               int64_t chunk_rows, int64_t chunk_cols,
                                               uint32_t flags) {
    if (T < 1 || d < 1 || V < 1 || chunk_rows < 1 || chunk_cols < 1 || T > 0x7FFFFFFFll ||
        d > 0x7FFFFFFFll || V > 0x7FFFFFFFll || (flags & ~kBackwardFlags))
        return 0;
    return plan_backward(T, d, V, chunk_rows, chunk_cols, flags).total;
}

size_t dart_lmhead_backward_split_workspace_bytes(int64_t T, int64_t d, int64_t V,
                                                  int64_t chunk_rows, int64_t chunk_cols,
                                                  uint32_t flags) {
    if (dart_lmhead_backward_ex_workspace_bytes(T, d, V, chunk_rows, chunk_cols, flags) == 0)
        return 0;
    return plan_backward(T, d, V, chunk_rows, chunk_cols, flags).split_total;
}

dart_status_t dart_lmhead_backward_ex(const void* hidden, int64_t T, int64_t d, int64_t ld_h,
                                      const void* weight, int64_t V, int64_t ld_w,
                                      const int32_t* target, const float* lse, const float* logp,
                                      const float* tok_coef, float inv_temp, void* dhidden,
                                      int64_t ld_dh, void* dweight, int64_t ld_dw,
                                      int64_t chunk_rows, int64_t chunk_cols, uint32_t flags,
                                      void* workspace, size_t workspace_bytes,
                                      hipStream_t stream) {
    if (bad_lmhead_args(hidden, T, d, ld_h, weight, V, ld_w)) return DART_ERR_INVALID_ARG;
    if (!(inv_temp > 0.f) || isinf(inv_temp)) return DART_ERR_INVALID_ARG;
    if (!target || !lse || !logp || !tok_coef || !dhidden || !dweight || !workspace)
        return DART_ERR_INVALID_ARG;
    if (ld_dh < d || ld_dw < d || chunk_rows < 1 || chunk_cols < 1 ||
        (flags & ~kBackwardFlags) || reinterpret_cast<uintptr_t>(workspace) % 16)
        return DART_ERR_INVALID_ARG;
    // the MFMA tiles address rows by 32-bit offsets from a tile's first row
    if (ld_h > kMaxLd || ld_w > kMaxLd || ld_dh > kMaxLd || ld_dw > kMaxLd)
        return DART_ERR_UNSUPPORTED;
    const BackwardPlan P = plan_backward(T, d, V, chunk_rows, chunk_cols, flags);
    if (P.total == 0) return DART_ERR_UNSUPPORTED;
    if (workspace_bytes < P.total) return DART_ERR_INVALID_ARG;
    if (const dart_status_t ck = dart_check::run(
            stream, {{dart_check::Item::Ids, target, T, V}}); ck != DART_OK)
        return ck;

    const uint16_t* h = static_cast<const uint16_t*>(hidden);
    const uint16_t* w = static_cast<const uint16_t*>(weight);
    char* ws = static_cast<char*>(workspace);
    uint16_t* dz = reinterpret_cast<uint16_t*>(ws + P.dz);
    float* acc_w = P.acc_w ? reinterpret_cast<float*>(ws + P.accw) : nullptr;
    float* acc_h = P.acc_h ? reinterpret_cast<float*>(ws + P.acch) : nullptr;
    const bool split = P.ksplit > 1 && workspace_bytes >= P.split_total;
    float* parts = split ? reinterpret_cast<float*>(ws + P.parts) : nullptr;
    const Grad dh{dhidden, ld_dh, P.bf16}, dw{dweight, ld_dw, P.bf16};
    if (!P.skip && !(P.compact && workspace_bytes >= P.split_total))
        return backward_core(h, T, d, ld_h, w, V, ld_w, target, lse, logp, tok_coef, inv_temp, dh,
                             dw, P.rows, P.cols, dz, acc_h, acc_w, parts, P.ksplit, stream);

    // rows with a zero coefficient have dz = 0: they add nothing to dW and
    // their rows of dh are 0, so the GEMMs run over the other rows only
    int32_t* map = reinterpret_cast<int32_t*>(ws + P.map);
    int32_t* count = reinterpret_cast<int32_t*>(ws + P.count);
    uint16_t* h_c = reinterpret_cast<uint16_t*>(ws + P.h_c);
    float* dh_c = reinterpret_cast<float*>(ws + P.dh_c);
    int32_t* target_c = reinterpret_cast<int32_t*>(ws + P.target_c);
    float* lse_c = reinterpret_cast<float*>(ws + P.lse_c);
    float* logp_c = reinterpret_cast<float*>(ws + P.logp_c);
    float* coef_c = reinterpret_cast<float*>(ws + P.coef_c);
    const float* lse_word = P.skip ? nullptr : lse;
    hipLaunchKernelGGL(compact_rows_kernel, dim3(1), dim3(kCompactThreads), 0, stream, tok_coef,
                       lse_word, T, map, count);
    const dim3 row_blocks((unsigned)(T < kRowBlocks ? T : kRowBlocks));
    if (P.bf16)
        hipLaunchKernelGGL(gather_rows_kernel<uint16_t>, row_blocks, dim3(128), 0, stream, map,
                           count, T, h, ld_h, d, target, lse, logp, tok_coef, lse_word, h_c,
                           target_c, lse_c, logp_c, coef_c, static_cast<uint16_t*>(dhidden), ld_dh);
    else
        hipLaunchKernelGGL(gather_rows_kernel<float>, row_blocks, dim3(128), 0, stream, map, count,
                           T, h, ld_h, d, target, lse, logp, tok_coef, lse_word, h_c, target_c,
                           lse_c, logp_c, coef_c, static_cast<float*>(dhidden), ld_dh);
    if (hipGetLastError() != hipSuccess) return DART_ERR_HIP;
    // the kernels read the kept-row count on the device: T rows at most
    return backward_core(h_c, T, d, d, w, V, ld_w, target_c, lse_c, logp_c, coef_c, inv_temp, dh,
                         dw, P.rows, P.cols, dz, dh_c, acc_w, parts, P.ksplit, stream, map, count);
}

dart_status_t dart_lmhead_backward(const void* hidden, int64_t T, int64_t d, int64_t ld_h,
                                   const void* weight, int64_t V, int64_t ld_w,
                                   const int32_t* target, const float* lse, const float* logp,
                                   const float* tok_coef, float* dhidden, int64_t ld_dh,
                                   float* dweight, int64_t ld_dw, int64_t chunk_rows,
                                   void* workspace, size_t workspace_bytes, hipStream_t stream) {
    return dart_lmhead_backward_ex(hidden, T, d, ld_h, weight, V, ld_w, target, lse, logp,
                                   tok_coef, 1.f, dhidden, ld_dh, dweight, ld_dw, chunk_rows, V,
                                   0u, workspace, workspace_bytes, stream);
}

}  // extern "C"
