// fp32 contractions on the matrix cores: the packed linear operator, the
// variable-sized batched GEMM and the triangular product in fp32 (Sections 5.1 and
// 7.1), all on one tile body of v_mfma_f32_32x32x2f32 (fp32 products and fp32
// accumulation; 256 FLOP per CU and cycle, 157 TFLOP/s).
//  - Operands go global -> LDS with bounds-checked buffer loads, 32 k per stage,
//    kStages stages.  Rows past the operand's last one and k past the reduction
//    read as zeros, so no size needs padding.  WIDE copies move 16 bytes per lane
//    (16-byte aligned rows); the others 4 bytes per lane into the same LDS layout,
//    for rows that start at any element (odd leading dimensions, packed problems of
//    odd sizes).  An fp32 MFMA step is slow enough to pay for four times the copy
//    instructions.
//  - K-contiguous operands: 128-byte LDS rows whose 16-byte chunks are XOR-swizzled
//    by row.  In MFMA step s of an 8-k group a lane supplies k = 4 (lane / 32) + s
//    (the same k order for both operands), so one 16-byte LDS read feeds four MFMAs.
//  - A lane ends with one output feature of 16 tokens per 32 x 32 block, so each
//    register is stored as 32 consecutive floats of two rows (whole 128-byte lines at
//    any alignment; the transposed form, 16 bytes per lane in 32 rows, kept the address
//    unit busy 32 cycles per store instruction).
#include <algorithm>
#include <type_traits>

#include "gemm_common.h"

namespace rag {
namespace {

constexpr int kF32K = 32;  // k per LDS stage

// Tile TM tokens x TN features, four waves: WM x WN sub-tiles, each shared by WK waves
// that take every WK-th 8-k group of a stage and add their sums at the end.
template <int TM_, int TN_, int WM_, int WN_, int WK_, int ST_>
struct F32Cfg {
    static constexpr int TM = TM_, TN = TN_, WM = WM_, WN = WN_, WK = WK_, kStages = ST_;
    static constexpr int kFM = TM / WM / 32, kFN = TN / WN / 32;  // 32-wide blocks of a wave
    static constexpr int kStageFloats = (TM + TN) * kF32K;
    static constexpr int kReduceFloats = WK > 1 ? TM * TN * WK : 0;
    static constexpr int kLdsBytes =
        4 * (kStages * kStageFloats > kReduceFloats ? kStages * kStageFloats : kReduceFloats);
    static_assert(WM * WN * WK == 4 && kFM >= 1 && kFN >= 1, "four waves");
    static_assert(TM % 32 == 0 && TN % 32 == 0 && (WK == 1 || WK == 2 || WK == 4), "tile shape");
    static_assert(ST_ >= 2 && ST_ <= 4 && kLdsBytes <= 160 * 1024, "stages");
};

// One wave copy: BYTES (16 or 4) per lane, lane l landing at dst + l * BYTES.
template <int BYTES>
__device__ __forceinline__ void copy_lds(__amdgpu_buffer_rsrc_t r, float* dst, int off) {
    if constexpr (BYTES == 16) __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void_t*)dst, 16, off, 0, 0, 0);
    else __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void_t*)dst, 4, off, 0, 0, 0);
}

constexpr int kF32Out = 0x7ffffff0;  // a byte offset past every descriptor: reads as zero

// One tile at (m0, n0) of y = act(x w^T + bias) + residual, x [T, K] (ldx), w [N, K]
// (ldw), any K >= 0; called by the whole workgroup (256 threads), sm holds C::kLdsBytes.
//   W_KN  w is instead [K][N] (ldw): y = x w.
//   TRI   x is lower triangular: x[i][k] counts only for k <= i (entries past the
//         diagonal are dropped after they are read, so NaN there is harmless).  Zero times
//         an infinity in w is not zero: a non-finite row k of w reaches the rows of y in
//         its 64-row block, but none above (tiles of 128 rows drop w rows there too).
// Valid rows of x and w must lie within 2^31 bytes of the tile's first (the caller
// checks); y may have any stride.
template <class C, int ACT, bool WIDE, bool W_KN, bool TRI>
__device__ __forceinline__ void gemm_tile_f32(const float* __restrict__ x, int ldx, const float* __restrict__ w,
                                              int ldw, const float* __restrict__ bias, const float* residual,
                                              int ldr, float* y, int ldy, int T, int K, int N, int m0, int n0,
                                              float* sm) {
    constexpr int TM = C::TM, TN = C::TN, FM = C::kFM, FN = C::kFN, ST = C::kStages;
    constexpr int kPer = WIDE ? 256 : 64;  // floats one wave copy moves
    constexpr int kXB = TM * kF32K / kPer / 4, kWB = TN * kF32K / kPer / 4;  // copies per wave and step
    constexpr int kCopies = kXB + kWB;
    static_assert((ST - 1) * kCopies < 64, "the wait counter holds 63 loads");
    static_assert(!W_KN || TN >= 64, "the [K][N] swizzle moves columns by 32");
    static_assert(!TRI || (W_KN && (TM == 64 || TM / C::WM == 64)), "64-row blocks of a triangular operand");
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
    const int l32 = lane % 32, h2 = lane / 32;
    const int wk = wave % C::WK, wm = wave / C::WK / C::WN, wn = wave / C::WK % C::WN;
    const int nk = (K + kF32K - 1) / kF32K;
    const int rows_x = min(T - m0, TM);
    const __amdgpu_buffer_rsrc_t rx =
        make_rsrc(x + (int64_t)m0 * ldx, K > 0 ? (uint32_t)((rows_x - 1) * ldx + K) * 4u : 0u);
    __amdgpu_buffer_rsrc_t rw;
    if constexpr (!W_KN)
        rw = make_rsrc(w + (int64_t)n0 * ldw, K > 0 ? (uint32_t)((min(N - n0, TN) - 1) * ldw + K) * 4u : 0u);

    // copies of `step` into `st`.  K-contiguous rows: float f = blk * kPer + ... of the
    // stage is row f / 32, physical 16-byte chunk f % 32 / 4, which holds the logical
    // chunk XORed with swz2(row).
    auto issue_one = [&](int step, float* st, int c) {
        auto rows_copy = [&](const __amdgpu_buffer_rsrc_t& r, int ld, float* dst, int blk) {
            int row, kl;  // the lane's row and first k
            if constexpr (WIDE) {
                row = blk * 8 + lane / 8;
                kl = ((lane % 8) ^ swz2(row)) * 4;
            } else {
                row = blk * 2 + h2;
                kl = ((((l32 >> 2)) ^ swz2(row)) << 2) + (l32 & 3);
            }
            const int k = step * kF32K + kl;
            // k < K: whole chunks when WIDE.  (The offset of a row past the last may wrap back
            // into the range at strides of millions; what it reads there is never used.)
            const int off = k < K ? (int)(((uint32_t)row * (uint32_t)ld + (uint32_t)k) * 4u) : kF32Out;
            copy_lds<WIDE ? 16 : 4>(r, dst + blk * kPer, off);
        };
        if (c < kXB) {
            rows_copy(rx, ldx, st, wave * kXB + c);
            return;
        }
        float* const wst = st + TM * kF32K;
        const int blk = wave * kWB + c - kXB;
        if constexpr (W_KN) {
            // stage row k holds TN columns, column c at c ^ (32 if k & 4), so the two half
            // waves of an operand read (k and k + 4) meet different banks
            const int k0 = step * kF32K;
            const __amdgpu_buffer_rsrc_t rk =
                make_rsrc(w + (int64_t)k0 * ldw + n0,
                          k0 < K ? (uint32_t)((min(K - k0, kF32K) - 1) * ldw + min(N - n0, TN)) * 4u : 0u);
            const int f = blk * kPer + lane * (WIDE ? 4 : 1);
            const int row = f / TN, col = (f % TN) ^ ((row & 4) << 3);
            copy_lds<WIDE ? 16 : 4>(rk, wst + blk * kPer, (row * ldw + col) * 4);
        } else {
            rows_copy(rw, ldw, wst, blk);
        }
    };

    floatx16 acc[FM][FN];
#pragma unroll
    for (int j = 0; j < FM; ++j)
#pragma unroll
        for (int i = 0; i < FN; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[j][i][r] = 0.f;

    // operands of the wave's g-th 8-k group of a landed stage; EDGE drops x entries past
    // the diagonal
    auto read = [&](floatx4 (&a)[FM], floatx4 (&b)[FN], const float* st, int step, int g, auto edge) {
        const int gq = g * C::WK + wk;
        const float* const wst = st + TM * kF32K;
#pragma unroll
        for (int j = 0; j < FM; ++j) {
            const int r = wm * (TM / C::WM) + j * 32 + l32;
            a[j] = *reinterpret_cast<const floatx4*>(st + r * kF32K + (((gq * 2 + h2) ^ swz2(r)) * 4));
            if constexpr (decltype(edge)::value) {
                const int over = step * kF32K + gq * 8 + 4 * h2 - (m0 + r);  // k - i of element 0
#pragma unroll
                for (int e = 0; e < 4; ++e) a[j][e] = over + e > 0 ? 0.f : a[j][e];
            }
        }
#pragma unroll
        for (int i = 0; i < FN; ++i) {
            const int c = wn * (TN / C::WN) + i * 32 + l32;
            if constexpr (W_KN) {
#pragma unroll
                for (int e = 0; e < 4; ++e) b[i][e] = wst[(gq * 8 + 4 * h2 + e) * TN + (c ^ (h2 << 5))];
                if constexpr (decltype(edge)::value && TM > 64) {
                    const bool past = step * kF32K >= m0 + (wm + 1) * 64;  // the wave's last row
#pragma unroll
                    for (int e = 0; e < 4; ++e) b[i][e] = past ? 0.f : b[i][e];
                }
            } else {
                b[i] = *reinterpret_cast<const floatx4*>(wst + c * kF32K + (((gq * 2 + h2) ^ swz2(c)) * 4));
            }
        }
    };

    // Step k's operands sit in stage k % ST.  The next group's operands are read while
    // this group's MFMAs run; before the step's last group the next step's copies are
    // waited for, its first group is read, and the copies of step k + ST go out between
    // the MFMAs into the stage every wave has now read.  No branch sits between a read
    // and its use (the compiler would wait for the newest reads where paths meet):
    // the last step is its own code, and copies past it are issued all the same (every
    // lane out of range, zeros into a stage nobody reads).
    constexpr int kGroups = 4 / C::WK;
    const int kfree = TRI ? min(m0 / kF32K, nk) : nk;  // TRI: steps wholly at or below the diagonal
    if (nk > 0) {
#pragma unroll
        for (int s = 0; s < ST; ++s)
#pragma unroll
            for (int c = 0; c < kCopies; ++c) issue_one(s, sm + s * C::kStageFloats, c);
        wait_vm<(ST - 1) * kCopies>();
        barrier_lds();
        float* st = sm;
        floatx4 a[2][FM], b[2][FN];
        if (TRI && kfree == 0) read(a[0], b[0], st, 0, 0, std::true_type{});
        else read(a[0], b[0], st, 0, 0, std::false_type{});
        // `edge`: this step is masked; `edge_next`: the next one is
        auto step = [&](int k, auto edge, auto edge_next, auto last) {
            constexpr bool kLast = decltype(last)::value;
            float* const next = st + C::kStageFloats == sm + ST * C::kStageFloats ? sm : st + C::kStageFloats;
#pragma unroll
            for (int g = 0; g < kGroups; ++g) {
                // group g's operands are in a[g & 1] (kGroups is even, or 1 with a copy)
                const int cur = g & 1, nxt = kGroups == 1 ? 1 : cur ^ 1;
                if (g + 1 < kGroups) {
                    read(a[nxt], b[nxt], st, k, g + 1, edge);
                } else if constexpr (!kLast) {
                    wait_vm<(ST - 2) * kCopies>();
                    barrier_lds();
                    read(a[nxt], b[nxt], next, k + 1, 0, edge_next);
                }
                __builtin_amdgcn_sched_barrier(0);  // else the reads sink below the MFMAs meant to hide them
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int j = 0; j < FM; ++j)
#pragma unroll
                        for (int i = 0; i < FN; ++i) {
                            acc[j][i] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[cur][j][e], b[cur][i][e], acc[j][i], 0, 0, 0);
                            if constexpr (!kLast) {
                                constexpr int kM = 4 * FM * FN;
                                const int q = (e * FM + j) * FN + i;
#pragma unroll
                                for (int c = 0; c < kCopies; ++c)
                                    if (g + 1 == kGroups && c * kM / kCopies == q) {
                                        issue_one(k + ST, st, c);
                                        if constexpr (!WIDE) __builtin_amdgcn_sched_barrier(0);  // keep them apart
                                    }
                            }
                        }
                if constexpr (kGroups == 1 && !kLast) {
#pragma unroll
                    for (int j = 0; j < FM; ++j) a[0][j] = a[1][j];
#pragma unroll
                    for (int i = 0; i < FN; ++i) b[0][i] = b[1][i];
                }
            }
            st = next;
        };
        constexpr std::false_type no{};
        constexpr std::true_type yes{};
        int k = 0;
        if constexpr (TRI) {
            for (; k + 1 < kfree && k + 1 < nk; ++k) step(k, no, no, no);
            if (k + 1 < nk && k < kfree) step(k++, no, yes, no);
            for (; k + 1 < nk; ++k) step(k, yes, yes, no);
            step(k, yes, yes, yes);  // a no-op mask where the last step lies below the diagonal
        } else {
            for (; k + 1 < nk; ++k) step(k, no, no, no);
            step(k, no, no, yes);
        }
        wait_vm<0>();  // no copy may still be on its way into LDS when the workgroup ends
    }

    // acc[j][i][4 g + e]: token wm*(TM/WM) + j*32 + 8 g + 4 h2 + e, feature
    // wn*(TN/WN) + i*32 + l32: each register is stored as 32 consecutive floats of a row.
    if constexpr (C::WK > 1) {
        // the waves of a sub-tile add their sums: every wave stages all its groups, and
        // wave wk finishes the groups g = wk, wk + WK, ...
        barrier_lds();
        float* const red = sm + (wm * C::WN + wn) * C::WK * FN * FM * 1024;
#pragma unroll
        for (int j = 0; j < FM; ++j)
#pragma unroll
            for (int i = 0; i < FN; ++i)
#pragma unroll
                for (int g = 0; g < 4; ++g)
                    *reinterpret_cast<floatx4*>(red + ((((wk * FM + j) * FN + i) * 4 + g) * 64 + lane) * 4) =
                        floatx4{acc[j][i][4 * g], acc[j][i][4 * g + 1], acc[j][i][4 * g + 2], acc[j][i][4 * g + 3]};
        barrier_lds();
#pragma unroll
        for (int j = 0; j < FM; ++j)
#pragma unroll
            for (int i = 0; i < FN; ++i)
#pragma unroll
                for (int gg = 0; gg < 4 / C::WK; ++gg) {
                    floatx4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int q = 0; q < C::WK; ++q)
                        s += *reinterpret_cast<const floatx4*>(
                            red + ((((q * FM + j) * FN + i) * 4 + gg * C::WK + wk) * 64 + lane) * 4);
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[j][i][4 * gg + e] = s[e];
                }
    }
    // Stores through a descriptor that ends with the tile's last valid row (rows past it
    // are dropped; features past N get an offset past the end), so no store is branched
    // around.  A row past the last is dropped only if its 32-bit offset has not wrapped back
    // into the descriptor, so every row of the tile, not only the valid ones, must lie
    // within 2^31 bytes of the first; the rows of a wider stride are stored through 64-bit
    // addresses instead.
    constexpr int kRegs = 16 / C::WK;  // accumulator registers this wave stores per block
    const int cols = min(N - n0, TN);
    const bool near = ((int64_t)(TM - 1) * ldy + cols) * 4 < kF32Out;
    float* const yt = y + (int64_t)m0 * ldy + n0;
    const __amdgpu_buffer_rsrc_t ry = make_rsrc(yt, near ? (uint32_t)((rows_x - 1) * ldy + cols) * 4u : 0u);
#pragma unroll
    for (int i = 0; i < FN; ++i) {
        const int nl = wn * (TN / C::WN) + i * 32 + l32;
        const float bv = bias ? bias[min(n0 + nl, N - 1)] : 0.f;
#pragma unroll
        for (int j = 0; j < FM; ++j) {
            const int mb = wm * (TM / C::WM) + j * 32 + 4 * h2;
            // tile row of register r: its group is (r / 4) * WK + wk
            auto row = [&](int r) { return mb + 8 * ((r / 4) * C::WK + wk) + r % 4; };
            // the block's residuals are loaded before the first is used (rows clamped)
            float o[kRegs], rv[kRegs];
            if (residual) {
#pragma unroll
                for (int r = 0; r < kRegs; ++r)
                    rv[r] = residual[(int64_t)(m0 + min(row(r), rows_x - 1)) * ldr + min(n0 + nl, N - 1)];
            }
#pragma unroll
            for (int r = 0; r < kRegs; ++r) {
                o[r] = activate<ACT>(acc[j][i][r] + bv);
                if (residual) o[r] += rv[r];
            }
            if (near) {
#pragma unroll
                for (int r = 0; r < kRegs; ++r)
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(o[r]), ry,
                                                          nl < cols ? (row(r) * ldy + nl) * 4 : kF32Out, 0, 0);
            } else {
#pragma unroll
                for (int r = 0; r < kRegs; ++r)
                    if (row(r) < rows_x && nl < cols) yt[(int64_t)row(r) * ldy + nl] = o[r];
            }
        }
    }
}

// 128 x 128 (four waves of 64 x 64), 64 x 64 (four of 32 x 32), and 32 x 32 whose four
// waves share the tile's k.
using F32Big = F32Cfg<128, 128, 2, 2, 1, 2>;
using F32Mid = F32Cfg<64, 64, 2, 2, 1, 2>;
using F32Tiny = F32Cfg<32, 32, 1, 1, 4, 4>;

// Workgroups [0, n_full) run tiles of C in the grouped XCD-aware order; the tiles of a
// last, partial round (n_full on) run as four quarters each, one per workgroup, of CS
// (half of C's sides), so that round takes about a quarter of a tile's time.
template <class C, class CS, int ACT, bool WIDE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
void k_gemm_f32(const float* __restrict__ x, int ldx, const float* __restrict__ w, const float* __restrict__ bias,
                const float* residual, int ldr, float* y, int ldy, int T, int K, int N, int tiles_m, int tiles_n,
                int n_full) {
    static_assert(C::TM == 2 * CS::TM && C::TN == 2 * CS::TN, "quarters");
    extern __shared__ __attribute__((aligned(16))) float fsm[];
    int tm, tn;
    if ((int)blockIdx.x < n_full) {
        tile_coords(blockIdx.x, n_full, tiles_m, tiles_n, tm, tn);
        gemm_tile_f32<C, ACT, WIDE, false, false>(x, ldx, w, K, bias, residual, ldr, y, ldy, T, K, N, tm * C::TM,
                                                  tn * C::TN, fsm);
    } else {
        const int u = blockIdx.x - n_full;
        group_walk(n_full + u / 4, tiles_m, tiles_n, tm, tn);
        const int m0 = tm * C::TM + (u & 1) * CS::TM, n0 = tn * C::TN + ((u >> 1) & 1) * CS::TN;
        if (m0 >= T || n0 >= N) return;  // a quarter past the last token or feature
        gemm_tile_f32<CS, ACT, WIDE, false, false>(x, ldx, w, K, bias, residual, ldr, y, ldy, T, K, N, m0, n0, fsm);
    }
}

// Operands whose rows the tile body's 32-bit byte offsets cannot reach (leading
// dimensions past 2^23): 64 x 64 tiles of plain FMA with 64-bit addressing.
// [K][N] and triangular operands (TRI) as in the tile body above.
template <int ACT, bool TRI>
__global__ __launch_bounds__(256) void k_gemm_f32_far(const float* __restrict__ x, int64_t ldx,
                                                      const float* __restrict__ w, int64_t ldw,
                                                      const float* __restrict__ bias, const float* residual,
                                                      int64_t ldr, float* y, int64_t ldy, int T, int K, int N) {
    __shared__ float xs[16][64 + 1], ws[16][64 + 1];
    const int tx = threadIdx.x % 16, ty = threadIdx.x / 16;
    const int m0 = (TRI ? (int)(gridDim.x - 1 - blockIdx.x) : (int)blockIdx.x) * 64, n0 = blockIdx.y * 64;
    const int k_end = TRI ? min(m0 + 64, K) : K;
    float acc[4][4] = {};
    for (int k0 = 0; k0 < k_end; k0 += 16) {
        __syncthreads();
        for (int e = threadIdx.x; e < 64 * 16; e += 256) {
            const int r = e / 16, c = e % 16, k = k0 + c;
            xs[c][r] = (m0 + r < T && k < K && (!TRI || k <= m0 + r)) ? x[(m0 + r) * ldx + k] : 0.f;
            if constexpr (TRI) {
                const int kr = k0 + e / 64, n = n0 + e % 64;
                ws[e / 64][e % 64] = (kr < K && n < N) ? w[kr * ldw + n] : 0.f;
            } else {
                ws[c][r] = (n0 + r < N && k < K) ? w[(n0 + r) * ldw + k] : 0.f;
            }
        }
        __syncthreads();
#pragma unroll
        for (int c = 0; c < 16; ++c)
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[u][v] = fmaf(xs[c][ty * 4 + u], ws[c][tx + 16 * v], acc[u][v]);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int m = m0 + ty * 4 + u;
        if (m >= T) continue;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int n = n0 + tx + 16 * v;
            if (n >= N) continue;
            float o = activate<ACT>(acc[u][v] + (bias ? bias[n] : 0.f));
            if (residual) o += residual[m * ldr + n];
            y[m * ldy + n] = o;
        }
    }
}

// Largest byte offset of `rows` rows of leading dimension ld fits the tile body's offsets.
bool f32_reach(int64_t rows, int64_t ld, int64_t width) { return ((rows - 1) * ld + width) * 4 < kF32Out; }

bool al16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

template <class C, class CS, int ACT, bool WIDE>
hipError_t launch_f32(const float* x, int ldx, const float* w, const float* bias, const float* residual, int ldr,
                      float* y, int ldy, int T, int K, int N, bool split_tail, hipStream_t s) {
    constexpr int kLds = C::kLdsBytes > CS::kLdsBytes ? C::kLdsBytes : CS::kLdsBytes;
    static bool attr_set = false;  // benign race: every thread sets the same value
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm_f32<C, CS, ACT, WIDE>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const int tiles_m = (T + C::TM - 1) / C::TM, tiles_n = (N + C::TN - 1) / C::TN, tiles = tiles_m * tiles_n;
    const int n_full = split_tail ? tiles / device_cu_count() * device_cu_count() : tiles;
    hipLaunchKernelGGL((k_gemm_f32<C, CS, ACT, WIDE>), dim3(n_full + 4 * (tiles - n_full)), dim3(256), kLds, s, x, ldx,
                       w, bias, residual, ldr, y, ldy, T, K, N, tiles_m, tiles_n, n_full);
    return hipGetLastError();
}

template <int ACT, bool WIDE>
hipError_t launch_f32_tiles(const float* x, int ldx, const float* w, const float* bias, const float* residual, int ldr,
                            float* y, int ldy, int T, int K, int N, hipStream_t s) {
    const bool reach = f32_reach(std::min(T, 128), ldx, K) && f32_reach(std::min(N, 128), K, K);
    const int form = linear_form_f32(T, N, reach, device_cu_count());
    const bool split = (form & 1) != 0;
    if (form & 128)
        return launch_f32<F32Big, F32Mid, ACT, WIDE>(x, ldx, w, bias, residual, ldr, y, ldy, T, K, N, split, s);
    return launch_f32<F32Mid, F32Tiny, ACT, WIDE>(x, ldx, w, bias, residual, ldr, y, ldy, T, K, N, split, s);
}

template <int ACT>
hipError_t launch_linear_act(const float* x, int ldx, const float* w, const float* bias, const float* residual, int ldr,
                             float* y, int ldy, int T, int K, int N, hipStream_t s) {
    if (!f32_reach(std::min(T, 64), ldx, K) || !f32_reach(std::min(N, 64), K, K)) {
        hipLaunchKernelGGL((k_gemm_f32_far<ACT, false>), dim3((T + 63) / 64, (N + 63) / 64), dim3(256), 0, s, x, ldx, w,
                           K, bias, residual, ldr, y, ldy, T, K, N);
        return hipGetLastError();
    }
    if (K % 4 == 0 && ldx % 4 == 0 && al16(x) && al16(w))
        return launch_f32_tiles<ACT, true>(x, ldx, w, bias, residual, ldr, y, ldy, T, K, N, s);
    return launch_f32_tiles<ACT, false>(x, ldx, w, bias, residual, ldr, y, ldy, T, K, N, s);
}

// ---------------------------------------------------------------------------
// Variable-sized batched GEMM: one workgroup per C-sized part of a list entry's 128 x 256
// tile (LOOP: several, see vgemm_grid); parts past the problem's edge end at once.  The
// entries go to the XCDs round-robin, an entry's parts to one: these tiles wait for the matrix
// cores, not for their operands, and any unevenness shows (369 entries of sizes 512..1408: 182
// us, 205 in runs of two, 213 of four); from 1600 entries on, where it averages out, runs of
// four (2279 to 7259 entries: at most 3% between one and 16).
// ---------------------------------------------------------------------------
template <class C>
constexpr int kPerCu = C::kLdsBytes > 160 * 1024 / 3 ? 2 : 3;  // workgroups per CU of vgemm and trmm

template <class C, bool LOOP>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(kPerCu<C>, kPerCu<C>)))
void k_vgemm_f32(VgemmArgs va, const float* __restrict__ a, const float* __restrict__ b, float* c, int run) {
    constexpr int kPm = kVgemmTileM / C::TM, kParts = kPm * (kVgemmTileN / C::TN);
    extern __shared__ __attribute__((aligned(16))) float fsm[];
    if (!vgemm_ok(va, false)) return;
    const int n = uni(va.status[1]), runs = run * kParts;
    // (a batch that fits in memory has under 2^23 entries)
    for (int p = blockIdx.x; p - 8 * runs < n * kParts; p += gridDim.x) {  // (position p holds parts past p - 8 runs)
        const int part = dealt_to_xcds(p, runs), e = part / kParts, sub = part % kParts;
        if (e < n) {
            const VgemmTile t = vgemm_tile(va, e);
            const int m0 = t.m0 + sub % kPm * C::TM, n0 = t.n0 + sub / kPm * C::TN;
            if (m0 < t.m && n0 < t.n) {
                if (LOOP) barrier_lds();  // the previous part is done with LDS
                const float *ap = a + t.a_off, *bp = b + t.b_off;
                const bool wide =
                    (t.k & 3) == 0 && ((reinterpret_cast<uintptr_t>(ap) | reinterpret_cast<uintptr_t>(bp)) & 15) == 0;
                if (wide)
                    gemm_tile_f32<C, 0, true, false, false>(ap, t.k, bp, t.k, nullptr, nullptr, 0, c + t.c_off, t.n,
                                                            t.m, t.k, t.n, m0, n0, fsm);
                else
                    gemm_tile_f32<C, 0, false, false, false>(ap, t.k, bp, t.k, nullptr, nullptr, 0, c + t.c_off, t.n,
                                                             t.m, t.k, t.n, m0, n0, fsm);
            }
        }
        if (!LOOP) return;
    }
}

template <class C>
hipError_t launch_vgemm_tiles(const VgemmArgs& va, int64_t tile_cap, const float* a, const float* b, float* c,
                              hipStream_t s) {
    static bool attr_set = false;  // benign race: every thread sets the same value
    if (!attr_set) {
        for (auto* f : {&k_vgemm_f32<C, false>, &k_vgemm_f32<C, true>}) {
            hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(f),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, C::kLdsBytes);
            if (e != hipSuccess) return e;
        }
        attr_set = true;
    }
    const int run = tile_cap < 1600 ? 1 : 4;
    const VgemmGrid g = vgemm_grid(tile_cap, (kVgemmTileM / C::TM) * (kVgemmTileN / C::TN), run, device_cu_count());
    auto* f = g.loop ? &k_vgemm_f32<C, true> : &k_vgemm_f32<C, false>;
    hipLaunchKernelGGL(f, dim3(g.blocks), dim3(256), C::kLdsBytes, s, va, a, b, c, run);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Triangular product: tiles heaviest row first, dealt to the XCDs by column panels; the
// reduction of a tile stops at its last row.
// ---------------------------------------------------------------------------
// (At most three workgroups per CU: enough to hide each other's waits, few enough that the
// heaviest rows' tiles run first and the light ones fill in.  2500 x 1500, 960 tiles: 89
// us, 94 at two, 95.5 with all of them resident at once; the vgemm above 135, 145, 139.
// The LDS of 128 x 128 tiles allows two; registers for three would only spill.)
template <class C, bool WIDE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(kPerCu<C>, kPerCu<C>)))
void k_trmm_f32(const float* __restrict__ l, int ldl, const float* __restrict__ b, int ldb, float* c, int ldc, int n,
                int m, int tiles_m, int tiles_n) {
    extern __shared__ __attribute__((aligned(16))) float fsm[];
    int tm, tn;
    if (!trmm_tile_coords(blockIdx.x, tiles_m, tiles_n, max(1, tiles_n / 8), tm, tn)) return;
    const int m0 = tm * C::TM;
    gemm_tile_f32<C, 0, WIDE, true, true>(l, ldl, b, ldb, nullptr, nullptr, 0, c, ldc, n, min(m0 + C::TM, n), m, m0,
                                          tn * C::TN, fsm);
}

template <class C, bool WIDE>
hipError_t launch_trmm_tiles(const float* l, int ldl, const float* b, int ldb, float* c, int ldc, int n, int m,
                             hipStream_t s) {
    static bool attr_set = false;  // benign race: every thread sets the same value
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_trmm_f32<C, WIDE>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, C::kLdsBytes);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const int tiles_m = (n + C::TM - 1) / C::TM, tiles_n = (m + C::TN - 1) / C::TN;
    const int q = 8 * std::max(1, tiles_n / 8);  // the grid covers whole rounds of chunks
    const int per_xcd = (tiles_m * tiles_n + q - 1) / q * q / 8;
    hipLaunchKernelGGL((k_trmm_f32<C, WIDE>), dim3(8 * per_xcd), dim3(256), C::kLdsBytes, s, l, ldl, b, ldb, c, ldc, n,
                       m, tiles_m, tiles_n);
    return hipGetLastError();
}

}  // namespace

// Tiles and whether their last round runs as quarters: whichever gives the busiest CU
// the least work, in units of one 64 x 64 tile and rounds of one tile per CU.  A
// 128 x 128 tile re-reads its operands half as often (weight 4 against 4.2 for
// four 64 x 64) and a 32 x 32 quarter twice as often (0.31 against 0.25).  128 x 128 tiles
// that would all run as quarters are 64 x 64 tiles with registers and LDS for more (3000 x 1024
// x 1024: 56.7 us, 54.1 as those; 710 x 128 x 4076 13.5, 12.0).
int linear_form_f32(int64_t T, int64_t N, bool reach128, int64_t cus) {
    auto cost = [&](int64_t side, double tile, double quarter, bool& split, bool& whole) {
        const int64_t tiles = ((T + side - 1) / side) * ((N + side - 1) / side);
        const int64_t full = tiles / cus, rest = tiles % cus;
        const double q = ((4 * rest + cus - 1) / cus) * quarter;
        split = rest && q < tile;
        whole = full > 0 || !split;
        return full * tile + (rest ? (split ? q : tile) : 0.0);
    };
    bool split_big, split_mid, whole_big, whole_mid;
    const double big = cost(128, 4.0, 1.05, split_big, whole_big), mid = cost(64, 1.05, 0.31, split_mid, whole_mid);
    return reach128 && whole_big && big <= mid ? 128 + split_big : 64 + split_mid;
}

hipError_t launch_linear_f32(const float* x, int ldx, const float* w, const float* bias, const float* residual, int ldr,
                             int act, float* y, int ldy, int T, int K, int N, hipStream_t s) {
    if (act == 1) return launch_linear_act<1>(x, ldx, w, bias, residual, ldr, y, ldy, T, K, N, s);
    if (act == 2) return launch_linear_act<2>(x, ldx, w, bias, residual, ldr, y, ldy, T, K, N, s);
    return launch_linear_act<0>(x, ldx, w, bias, residual, ldr, y, ldy, T, K, N, s);
}

hipError_t launch_vgemm_f32(const VgemmArgs& va, int64_t tile_cap, const float* a, const float* b, float* c,
                            hipStream_t s) {
    if (tile_cap >= 16 * (int64_t)va.batch && tile_cap >= 2 * (int64_t)device_cu_count())
        return launch_vgemm_tiles<F32Big>(va, tile_cap, a, b, c, s);
    return launch_vgemm_tiles<F32Mid>(va, tile_cap, a, b, c, s);
}

hipError_t launch_trmm_f32(const float* l, int ldl, const float* b, int ldb, float* c, int ldc, int n, int m,
                           hipStream_t s) {
    if (!f32_reach(std::min(n, 64), ldl, n) || !f32_reach(kF32K, ldb, m)) {
        hipLaunchKernelGGL((k_gemm_f32_far<0, true>), dim3((n + 63) / 64, (m + 63) / 64), dim3(256), 0, s, l, ldl, b,
                           ldb, nullptr, nullptr, 0, c, ldc, n, n, m);
        return hipGetLastError();
    }
    const bool wide = n % 4 == 0 && m % 4 == 0 && ldl % 4 == 0 && ldb % 4 == 0 && al16(l) && al16(b);
    const int64_t big = (int64_t)((n + 127) / 128) * ((m + 127) / 128);
    if (big >= 4 * (int64_t)device_cu_count() && f32_reach(std::min(n, 128), ldl, n))
        return wide ? launch_trmm_tiles<F32Big, true>(l, ldl, b, ldb, c, ldc, n, m, s)
                    : launch_trmm_tiles<F32Big, false>(l, ldl, b, ldb, c, ldc, n, m, s);
    return wide ? launch_trmm_tiles<F32Mid, true>(l, ldl, b, ldb, c, ldc, n, m, s)
                : launch_trmm_tiles<F32Mid, false>(l, ldl, b, ldb, c, ldc, n, m, s);
}

}  // namespace rag
