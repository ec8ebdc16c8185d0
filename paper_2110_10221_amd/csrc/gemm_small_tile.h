// The tile body of the small-launch bf16 GEMM (gemm_small.hip), which the 256 x 256 GEMM
// (gemm_big.hip) also runs on the tiles of its last, partial round.
#pragma once

#include <type_traits>

#include "gemm_common.h"
#include "plan_device.h"

namespace rag {
namespace {

// TM x TN tile, WM x WN sub-tiles of WK waves each, SB blocks of 64 k per stage, ST
// stages.
template <int TM_, int TN_, int WM_, int WN_, int WK_, int SB_, int ST_>
struct SmallCfg {
    static constexpr int TM = TM_, TN = TN_, WM = WM_, WN = WN_, WK = WK_, SB = SB_, ST = ST_;
    static constexpr int kWaves = WM * WN * WK, kThreads = kWave * kWaves;
    static constexpr int FM = TM / WM / 32, FN = TN / WN / 32;  // 32-wide blocks of a wave
    static constexpr int kBlockElems = (TM + TN) * 64, kStageElems = SB * kBlockElems;
    static constexpr int G = 4 * SB / WK;                       // 16-k groups per wave and stage
    static constexpr int kSumBytes = TM * TN * 4 * WK;          // the epilogue's fp32 tile, per k share
    static constexpr int kLds = ST * kStageElems * 2 > kSumBytes ? ST * kStageElems * 2 : kSumBytes;
    static constexpr int kStageCopies = (TM + TN) / 8 * SB;     // 1 KB wave copies per stage
    static constexpr int kCopies = kStageCopies / kWaves;
    static_assert(kStageCopies % kWaves == 0 && G % 2 == 0 && kLds <= 160 * 1024, "configuration");
    static_assert(kThreads == kFusedBatch || kThreads == kFusedMaxThreads, "the plan body's workgroup sizes");
    static_assert(sizeof(PlanSmem) <= kLds, "the plan's LDS fits the GEMM's");
};

constexpr int kPastEnd = 0x7ffffff0;  // a byte offset past every descriptor: reads as zero

template <class C, int ACT>
__device__ __forceinline__ void gemm_small_tile(const uint16_t* __restrict__ x, int ldx, const uint16_t* __restrict__ w,
                                                const uint16_t* __restrict__ bias, const uint16_t* residual, int ldr,
                                                uint16_t* y, int ldy, int T, int K, int N, int m0, int n0,
                                                uint16_t* sm) {
    constexpr int TM = C::TM, TN = C::TN, FM = C::FM, FN = C::FN, ST = C::ST, G = C::G, NC = C::kCopies;
    constexpr int kRowBlocks = (TM + TN) / 8;  // 8-row copy blocks of a 64-k block: x rows, then w rows
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
    const int l32 = lane % 32, h2 = lane / 32;
    const int wk = wave % C::WK, wm = wave / C::WK / C::WN, wn = wave / C::WK % C::WN;
    const int nk = (K + 64 * C::SB - 1) / (64 * C::SB);
    const __amdgpu_buffer_rsrc_t rx = make_rsrc(x + (int64_t)m0 * ldx, (uint32_t)min(T - m0, TM) * ldx * 2u);
    const __amdgpu_buffer_rsrc_t rw = make_rsrc(w + (int64_t)n0 * K, (uint32_t)min(N - n0, TN) * K * 2u);
    // copy c of this wave fills block id = wave * NC + c of a stage (8 rows of 128 bytes,
    // lane l slot l: row l / 8, physical chunk l % 8, logical chunk XORed with swz2(row))
    int voff[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const int id = wave * NC + c, sb = id / kRowBlocks, b = id % kRowBlocks;
        const int row = (b < TM / 8 ? b : b - TM / 8) * 8 + lane / 8;
        voff[c] = row * (b < TM / 8 ? ldx : K) * 2 + ((lane % 8) ^ swz2(row)) * 16 + sb * 128;
    }
    auto issue_one = [&](int step, uint16_t* st, int c) {
        const int id = wave * NC + c, sb = id / kRowBlocks, b = id % kRowBlocks;
        const int past = (step * C::SB + sb) * 64 < K ? 0 : kPastEnd;  // K is a multiple of 64
        __builtin_amdgcn_raw_ptr_buffer_load_lds(b < TM / 8 ? rx : rw, (lds_void_t*)(st + id * 512), 16,
                                                 voff[c] | past, step * C::SB * 128, 0, 0);
    };
    floatx16 acc[FN][FM];
#pragma unroll
    for (int i = 0; i < FN; ++i)
#pragma unroll
        for (int j = 0; j < FM; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    bf16x8 a[2][FN], b[2][FM];
    // operands of the wave's g-th 16-k group of a landed stage
    auto read = [&](int slot, const uint16_t* st, int g) {
        const int q = g * C::WK + wk, ch = (q & 3) * 2 + h2;
        const uint16_t* const xb = st + (q >> 2) * C::kBlockElems;
        const uint16_t* const wb = xb + TM * 64;
#pragma unroll
        for (int j = 0; j < FM; ++j) {
            const int r = wm * (TM / C::WM) + j * 32 + l32;
            b[slot][j] = as_bf16x8(*reinterpret_cast<const u32x4*>(xb + r * 64 + ((ch ^ swz2(r)) * 8)));
        }
#pragma unroll
        for (int i = 0; i < FN; ++i) {
            const int r = wn * (TN / C::WN) + i * 32 + l32;
            a[slot][i] = as_bf16x8(*reinterpret_cast<const u32x4*>(wb + r * 64 + ((ch ^ swz2(r)) * 8)));
        }
    };
#pragma unroll
    for (int s = 0; s < ST; ++s)
#pragma unroll
        for (int c = 0; c < NC; ++c) issue_one(s, sm + s * C::kStageElems, c);
    wait_vm<(ST - 1) * NC>();
    barrier_lds();
    uint16_t* st = sm;
    read(0, st, 0);
    // Step k's operands sit in stage k % ST; before its last group the next step's copies
    // are waited for and its first group read, and the copies of step k + ST go out
    // between the MFMAs into the stage every wave has now read.
    auto step = [&](int k, auto last) {
        constexpr bool kLast = decltype(last)::value;
        uint16_t* const next = st + C::kStageElems == sm + ST * C::kStageElems ? sm : st + C::kStageElems;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            if (g + 1 < G) {
                read((g + 1) % 2, st, g + 1);
            } else if constexpr (!kLast) {
                wait_vm<(ST - 2) * NC>();
                barrier_lds();
                read(0, next, 0);
            }
            __builtin_amdgcn_sched_barrier(0);  // else the reads sink below the MFMAs meant to hide them
#pragma unroll
            for (int i = 0; i < FN; ++i)
#pragma unroll
                for (int j = 0; j < FM; ++j) {
                    acc[i][j] = mfma32x32x16(a[g % 2][i], b[g % 2][j], acc[i][j]);
                    if constexpr (!kLast) {
#pragma unroll
                        for (int c = 0; c < NC; ++c)
                            if (g + 1 == G && c * FM * FN / NC == i * FM + j) issue_one(k + ST, st, c);
                    }
                }
        }
        st = next;
    };
    int k = 0;
    for (; k + 1 < nk; ++k) step(k, std::false_type{});
    step(k, std::true_type{});
    wait_vm<0>();  // the copies past the reduction have landed: LDS is free

    // Epilogue: the fp32 sums go through LDS (row r's 16-byte chunk c at c ^ (r & 15), one
    // tile per k share), then each thread finishes 8 features of a row at a time.  Bias
    // and residual are loaded first (indexes clamped into range), their latency passing
    // under the staging.
    constexpr int kChunks = TN / 8, kRowStep = C::kThreads / kChunks, kIt = (TM + kRowStep - 1) / kRowStep;
    constexpr int kSwz = TN / 4 < 16 ? TN / 4 - 1 : 15;
    const int ch = threadIdx.x % kChunks, r0 = threadIdx.x / kChunks, n = n0 + ch * 8;
    u32x4 res[kIt];
    u32x2 bb[2] = {u32x2{0u, 0u}, u32x2{0u, 0u}};
    if (bias) {
#pragma unroll
        for (int hb = 0; hb < 2; ++hb) bb[hb] = *reinterpret_cast<const u32x2*>(bias + min(n, N - 8) + 4 * hb);
    }
    if (residual) {
#pragma unroll
        for (int t = 0; t < kIt; ++t)
            res[t] = *reinterpret_cast<const u32x4*>(residual + (int64_t)min(m0 + r0 + t * kRowStep, T - 1) * ldr +
                                                     min(n, N - 8));
    }
    barrier_lds();
    float* const ep = reinterpret_cast<float*>(sm);
    auto slot = [&](int row, int c) { return row * TN + ((c ^ (row & kSwz)) * 4); };
#pragma unroll
    for (int i = 0; i < FN; ++i)
#pragma unroll
        for (int j = 0; j < FM; ++j)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                // acc[i][j][4 g + e]: token j*32 + l32, feature i*32 + 8 g + 4 h2 + e of the sub-tile
                const int row = wm * (TM / C::WM) + j * 32 + l32, c = (wn * (TN / C::WN) + i * 32 + 8 * g + 4 * h2) >> 2;
                *reinterpret_cast<floatx4*>(ep + wk * TM * TN + slot(row, c)) =
                    floatx4{acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
            }
    barrier_lds();
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
        const int row = r0 + t * kRowStep, m = m0 + row;
        if (row >= TM || m >= T || n >= N) break;  // later rows are past the end too
        float v[8];
#pragma unroll
        for (int hc = 0; hc < 2; ++hc) {
            floatx4 s = *reinterpret_cast<const floatx4*>(ep + slot(row, 2 * ch + hc));
#pragma unroll
            for (int q = 1; q < C::WK; ++q)
                s += *reinterpret_cast<const floatx4*>(ep + q * TM * TN + slot(row, 2 * ch + hc));
#pragma unroll
            for (int e = 0; e < 4; ++e) v[4 * hc + e] = activate_bf16<ACT>(s[e] + bv[4 * hc + e]);
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

}  // namespace
}  // namespace rag
