// bf16 packed linear operator on 256 x 256 tiles (tokens x features): y = x w^T + bias +
// residual for long reductions over enough of them.
//  - What bounds it: power, then the loop's waits.  With random operands and two waves
//    per SIMD this card sustains 1830 TFLOP/s of v_mfma_f32_16x16x32_bf16 and 1290 to 1400
//    of the 32x32x16 form (no memory traffic at all; 2230 and 1640 with constant
//    operands), so every byte moved from L2 or LDS and the MFMA form itself cost rate.  A
//    256 x 256 tile moves 4 bytes per 512 products from L2 into LDS, a 128 x 256 tile 6.
//  - Eight waves of 128 tokens x 64 features, one workgroup per CU; both operands staged 64
//    k deep (128-byte rows, whole lines per copy request) in two stages of 64 KB.  The
//    next 32-k group's fragments are read while a group's MFMAs run; before a step's last
//    group the next stage is waited for, and the copies two steps ahead go out between
//    that group's MFMAs.
//  - One workgroup per CU leaves a tile's prologue and epilogue exposed, and a partial last
//    round idle: its tiles run as four 128 x 128 quarters each (gemm_small_tile).
// Against the 128 x 256 tiles (two workgroups per CU, 32x32x16 MFMAs): 35475 x 4096 x 1024
// 281 -> 255 us, 20000 x 3072 x 768 83.3 -> 79.1, 8192^3 884 -> 829; but 35475 x 1024 x 4096
// 270 -> 294, where sixteen steps do not pay for the exposed epilogue.
#include <algorithm>

#include "gemm_small_tile.h"

namespace rag {
namespace {

struct BigCfg {
    static constexpr int TM = 256, TN = 256, WM = 2, WN = 4, kThreads = 512;
    static constexpr int FM = TM / WM / 16, FN = TN / WN / 16;  // 16-wide blocks of a wave: 8 x 4
    static constexpr int kStageElems = (TM + TN) * 64;
    static constexpr int kCopies = (TM + TN) / 8 / 8;           // 1 KB copies per wave and stage
    static constexpr int kLds = 2 * kStageElems * 2;            // also the epilogue's 128 fp32 rows
};
using BigTail = SmallCfg<128, 128, 2, 4, 1, 1, 3>;  // a quarter of a last-round tile
static_assert(BigTail::kThreads == BigCfg::kThreads && BigTail::kLds <= BigCfg::kLds, "quarters");

// Workgroup barrier for LDS traffic with a wait the compiler's own wait insertion sees, so
// that it adds none of its own for reads that have landed.
__device__ __forceinline__ void wait_lds() { __builtin_amdgcn_s_waitcnt(0xc07f); }  // lgkmcnt(0) only
__device__ __forceinline__ void barrier_lds_seen() {
    asm volatile("" ::: "memory");
    wait_lds();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

__device__ __forceinline__ void gemm_big_tile(const uint16_t* __restrict__ x, int ldx, const uint16_t* __restrict__ w,
                                              const uint16_t* __restrict__ bias, const uint16_t* residual, int ldr,
                                              uint16_t* y, int ldy, int T, int K, int N, int m0, int n0, uint16_t* sm) {
    using C = BigCfg;
    constexpr int TM = C::TM, TN = C::TN, FM = C::FM, FN = C::FN, NC = C::kCopies;
    // the epilogue's arguments are loaded here: a scalar load pending at the loop's head
    // would turn every LDS wait in the loop into a full one (they share a counter)
    asm volatile("" ::"s"(bias), "s"(residual), "s"(y), "s"(ldr), "s"(ldy), "s"(N));
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
    const int l16 = lane % 16, q4 = lane / 16;
    const int wm = wave / C::WN, wn = wave % C::WN;
    const int nk = K / 64;
    const __amdgpu_buffer_rsrc_t rx = make_rsrc(x + (int64_t)m0 * ldx, (uint32_t)min(T - m0, TM) * ldx * 2u);
    const __amdgpu_buffer_rsrc_t rw = make_rsrc(w + (int64_t)n0 * K, (uint32_t)min(N - n0, TN) * K * 2u);
    // copy c of this wave fills block id = wave * NC + c of a stage (x rows, then w rows; 8
    // rows of 128 bytes, lane l slot l, physical chunk l % 8 holding logical l % 8 ^ swz2(row))
    int voff[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const int b = wave * NC + c, row = (b < TM / 8 ? b : b - TM / 8) * 8 + lane / 8;
        voff[c] = row * (b < TM / 8 ? ldx : K) * 2 + ((lane % 8) ^ swz2(row)) * 16;
    }
    auto issue_one = [&](int step, uint16_t* st, int c) {
        const int b = wave * NC + c, past = step < nk ? 0 : kPastEnd;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(b < TM / 8 ? rx : rw, (lds_void_t*)(st + b * 512), 16, voff[c] | past,
                                                 step * 128, 0, 0);
    };
    floatx4 acc[FN][FM];
#pragma unroll
    for (int i = 0; i < FN; ++i)
#pragma unroll
        for (int j = 0; j < FM; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    bf16x8 a[2][FN], b[2][FM];
    auto read = [&](const uint16_t* st, int g) {  // 32-k group g of a landed stage into slot g
        const uint16_t* const wb = st + TM * 64;
        const int ch = g * 4 + q4;
#pragma unroll
        for (int i = 0; i < FN; ++i) {
            const int r = wn * (TN / C::WN) + i * 16 + l16;
            a[g][i] = as_bf16x8(*reinterpret_cast<const u32x4*>(wb + r * 64 + ((ch ^ swz2(r)) * 8)));
        }
#pragma unroll
        for (int j = 0; j < FM; ++j) {
            const int r = wm * (TM / C::WM) + j * 16 + l16;
            b[g][j] = as_bf16x8(*reinterpret_cast<const u32x4*>(st + r * 64 + ((ch ^ swz2(r)) * 8)));
        }
    };
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int c = 0; c < NC; ++c) issue_one(s, sm + s * C::kStageElems, c);
    wait_vm<NC>();
    barrier_lds_seen();
    uint16_t* st = sm;
    read(st, 0);
    wait_lds();
    auto step = [&](int k, auto last) {
        constexpr bool kLast = decltype(last)::value;
        uint16_t* const next = st == sm ? sm + C::kStageElems : sm;
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            if (g == 0) {
                read(st, 1);
            } else if constexpr (!kLast) {
                __builtin_amdgcn_sched_barrier(0);  // group 0's MFMAs go out before the wait
                wait_vm<0>();
                barrier_lds_seen();
                read(next, 0);
            }
            __builtin_amdgcn_sched_barrier(0);  // else the reads sink below the MFMAs meant to hide them
            __builtin_amdgcn_s_setprio(1);  // the SIMD's other wave reads or waits meanwhile
#pragma unroll
            for (int i = 0; i < FN; ++i)
#pragma unroll
                for (int j = 0; j < FM; ++j) {
                    acc[i][j] = mfma16x16x32(a[g][i], b[g][j], acc[i][j]);
                    if constexpr (!kLast) {
#pragma unroll
                        for (int c = 0; c < NC; ++c)
                            if (g == 1 && c * FM * FN / NC == i * FM + j) issue_one(k + 2, st, c);
                    }
                }
            __builtin_amdgcn_s_setprio(0);
        }
        st = next;
    };
    int k = 0;
    for (; k + 1 < nk; ++k) step(k, std::false_type{});
    step(k, std::true_type{});
    wait_vm<0>();  // the copies past the reduction have landed: LDS is free

    // Epilogue in two slices of 128 rows (half of each wave's tokens): fp32 sums through LDS
    // (row r's 16-byte chunk c at c ^ (r & 15)), then whole 512-byte rows: 32 threads per
    // row, bias and residual applied, the sum rounded once.
    constexpr int kSliceRows = 128, kRowStep = C::kThreads / 32, kIt = kSliceRows / kRowStep;
    const int ch = threadIdx.x % 32, r0 = threadIdx.x / 32, n = n0 + ch * 8;
    // token of row r0 + t * kRowStep of slice s: rows kHalf wm .. of a slice are wave row wm's
    // tokens kHalf s ..
    constexpr int kHalf = kSliceRows / C::WM;
    auto token = [&](int s, int t) {
        const int r = r0 + t * kRowStep;
        return m0 + (r / kHalf) * (2 * kHalf) + s * kHalf + r % kHalf;
    };
    u32x2 bb[2] = {u32x2{0u, 0u}, u32x2{0u, 0u}};
    if (bias) {
#pragma unroll
        for (int hb = 0; hb < 2; ++hb) bb[hb] = *reinterpret_cast<const u32x2*>(bias + min(n, N - 8) + 4 * hb);
    }
    float* const ep = reinterpret_cast<float*>(sm);
    auto slot = [&](int row, int c) { return row * TN + ((c ^ (row & 15)) * 4); };
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        u32x4 res[kIt];
        if (residual) {  // (the slice's rows at once; tokens and features clamped into range)
#pragma unroll
            for (int t = 0; t < kIt; ++t)
                res[t] = *reinterpret_cast<const u32x4*>(residual + (int64_t)min(token(s, t), T - 1) * ldr + min(n, N - 8));
        }
        barrier_lds_seen();
#pragma unroll
        for (int jj = 0; jj < FM / 2; ++jj)
#pragma unroll
            for (int i = 0; i < FN; ++i)
                // acc[i][j][e]: token j*16 + l16, feature i*16 + 4 q4 + e of the wave's sub-tile
                *reinterpret_cast<floatx4*>(ep + slot((wm * (FM / 2) + jj) * 16 + l16, (wn * (TN / C::WN) + i * 16 + 4 * q4) >> 2)) =
                    acc[i][(FM / 2) * s + jj];
        barrier_lds_seen();
        float bv[8];
#pragma unroll
        for (int hb = 0; hb < 2; ++hb) {
            bv[4 * hb] = lo_bf16(bb[hb][0]);
            bv[4 * hb + 1] = hi_bf16(bb[hb][0]);
            bv[4 * hb + 2] = lo_bf16(bb[hb][1]);
            bv[4 * hb + 3] = hi_bf16(bb[hb][1]);
        }
#pragma unroll
        for (int t = 0; t < kIt; ++t) {
            const int m = token(s, t);
            if (m >= T || n >= N) continue;
            float v[8];
#pragma unroll
            for (int hc = 0; hc < 2; ++hc) {
                const floatx4 o = *reinterpret_cast<const floatx4*>(ep + slot(r0 + t * kRowStep, 2 * ch + hc));
#pragma unroll
                for (int e = 0; e < 4; ++e) v[4 * hc + e] = o[e] + bv[4 * hc + e];
            }
            if (residual) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    v[2 * e] += lo_bf16(res[t][e]);
                    v[2 * e + 1] += hi_bf16(res[t][e]);
                }
            }
            *reinterpret_cast<u32x4*>(y + (int64_t)m * ldy + n) = u32x4{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]),
                                                                        pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7])};
        }
    }
}

// Workgroups [0, n_full) run whole tiles in the grouped XCD-aware order, then four per tile
// of the last round run its quarters; workgroups from n_gemm on (if any) build a
// batch's plan.
__global__ __launch_bounds__(BigCfg::kThreads) __attribute__((amdgpu_waves_per_eu(2)))
void k_gemm_big(const uint16_t* __restrict__ x, int ldx, const uint16_t* __restrict__ w,
                const uint16_t* __restrict__ bias, const uint16_t* residual, int ldr, uint16_t* y, int ldy, int T, int K,
                int N, int tiles_m, int tiles_n, int n_full, int n_gemm, PlanFillArgs pf) {
    extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
    if ((int)blockIdx.x >= n_gemm) {
        plan_fused_body(pf, blockIdx.x - n_gemm, *reinterpret_cast<PlanSmem*>(smem));
        return;
    }
    int tm, tn;
    if ((int)blockIdx.x < n_full) {
        tile_coords(blockIdx.x, n_full, tiles_m, tiles_n, tm, tn);
        gemm_big_tile(x, ldx, w, bias, residual, ldr, y, ldy, T, K, N, tm * 256, tn * 256, smem);
    } else {
        const int u = blockIdx.x - n_full;
        group_walk(n_full + u / 4, tiles_m, tiles_n, tm, tn);
        const int m0 = tm * 256 + (u & 1) * 128, n0 = tn * 256 + ((u >> 1) & 1) * 128;
        if (m0 >= T || n0 >= N) return;  // a quarter past the last token or feature
        gemm_small_tile<BigTail, 0>(x, ldx, w, bias, residual, ldr, y, ldy, T, K, N, m0, n0, smem);
    }
}

}  // namespace

// Whole tiles where a launch has nearly a round of them or more; else its last, partial round,
// which may be all of it, runs as quarters.
static int64_t big_whole_tiles(int64_t tiles, int64_t cus) {
    const int64_t rest = tiles % cus;
    return 4 * rest > 3 * cus ? tiles : tiles - rest;  // nearly full: quarters would take as long
}

// Long reductions only (sixteen 64-k steps barely pay for the exposed epilogue: of 162
// timed shapes, T = 2236 to 35475, those with K >= 1536 ran 1-12% faster than on the other
// tiles and nearly all shorter ones slower), without an activation.
//  - A second round of whole tiles, or part of one, only where the 128 x 256 tiles, which
//    pad the tokens less, need one too (2580 x 2048 x 6144: 66.5 us, 59.1 on 504 of them).
//  - A launch of quarters alone not where 64 x 128 tiles make one round (100 x 4096 x 12288
//    28.7 us, 23.3 on those; 32 x 4096 x 16384 34.9 and 21.5; but 2236 x 4096 x 1024 28.0, and
//    30.9 on 128 x 128 tiles), nor with a nearly empty second round (0.95-1.01x
//    there), which empty quarters cause too: they go to the XCDs in turn with the others, and
//    33 full ones on one XCD take two rounds (2580 x 6144 x 1536, 252 of 264 full: 84 us, 52
//    on 128 x 128 tiles).  In more than one round without a residual, whose epilogue the other
//    tiles are slow at, it takes K >= 2048 (2442 x 1536 x 4608: 42.1 us, 39.5 on the others).
bool gemm_big_wins(int64_t T, int64_t K, int64_t N, int act, bool residual, int64_t cus) {
    if (act != 0 || K < 1536) return false;
    const int64_t tiles = ((T + 255) / 256) * ((N + 255) / 256), halves = ((T + 127) / 128) * ((N + 255) / 256);
    if (big_whole_tiles(tiles, cus) > 0) return tiles <= cus || halves > 2 * cus;
    if (((T + 63) / 64) * ((N + 127) / 128) <= cus) return false;
    const int64_t full = ((T + 127) / 128) * ((N + 127) / 128);  // of 4 * tiles quarters
    return 4 * tiles <= cus || (10 * full >= 13 * cus && (residual || K >= 2048));
}

hipError_t launch_gemm_big(const LinearArgs& a, const PlanView* plan, hipStream_t s) {
    static bool attr_set = false;  // benign race: every thread sets the same value
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm_big),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, BigCfg::kLds);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const int cus = device_cu_count();
    const int tiles_m = (a.T + 255) / 256, tiles_n = (a.N + 255) / 256, tiles = tiles_m * tiles_n;
    const int n_full = (int)big_whole_tiles(tiles, cus);
    const int n_gemm = n_full + 4 * (tiles - n_full);
    const PlanFillArgs pf = plan ? plan_fill_args(*plan) : PlanFillArgs{};
    hipLaunchKernelGGL(k_gemm_big, dim3(n_gemm + (plan ? plan->batch : 0)), dim3(BigCfg::kThreads), BigCfg::kLds, s, a.x,
                       a.ldx, a.w, a.bias, a.residual, a.ldr, a.y, a.ldy, a.T, a.K, a.N, tiles_m, tiles_n, n_full,
                       n_gemm, pf);
    return hipGetLastError();
}

}  // namespace rag
