// bf16 packed linear operator for launches whose 128 x 256 tiles would leave the GPU
// short of work: small token counts, or few output features with a long reduction.
// The same product as gemm.hip, y = act(x w^T + bias) + residual, on smaller tiles:
//   32 x 32, 64 x 64, 64 x 128, 128 x 128 (tokens x features), and 128 x 256 where all
//   of them run at once
//  - What bounds it: a CU copies at most 64 bytes per cycle from L2 into LDS, and a
//    T1 x T2 tile needs 2 (T1 + T2) bytes per k, so a 64 x 64 tile takes at least 1.7
//    ns per k (2.4 GHz; 2.3 measured at 777 x 4096 x 1024) where its MFMAs take 0.8;
//    larger tiles need fewer bytes per product but leave CUs idle.  The launch picks
//    the tile whose busiest CU finishes first (small_gemm_choice below).
//  - Both operands are staged 64 k deep, one 128-byte row per token or feature, so
//    every copy request is a whole line (64-byte rows: 21 against 35 TB/s from L2),
//    3 or 4 stages ahead: a small launch reads mostly from the Infinity Cache, whose
//    latency the ring covers (two stages: 23 against 15 us at 2236 x 2048 x 512 with
//    128 x 128 tiles).
//  - The waves of a tile split its features, and on the smaller tiles also the k of
//    each stage (WK): a wave then reads each operand fragment for more MFMAs, and
//    the partial fp32 sums meet in LDS before bias, activation and residual, in
//    wave order, rounded once.
//  - Fragments of the next 16-k group are read while this group's MFMAs run, and no
//    branch sits between a read and its use (where paths meet, the compiler would
//    wait for the newest reads): the last step is its own code, copies past the
//    reduction are issued out of range (zeros into a stage nobody reads).
// Measured against the 128 x 256 tiles (and their eight-wave, 64-token form, which
// these replace), us per call: 2236 x 512 x 1536 9.9 -> 8.0, x 512 x 512 10.0 -> 6.0,
// 2236 x 2048 x 512 22.3 -> 12.3; 777 x 4096 x 1024 38.9 -> 15.4; 400 x 3072 x 768
// 31.4 -> 9.7; 100 x 512 x 512 10.0 -> 5.0; over 224 shapes (33 to 20000 tokens, the
// projections of layers of d 256 to 1024) 1.46x in the geometric mean.
#include <algorithm>

#include "gemm_small_tile.h"

namespace rag {
namespace {

// One tile per workgroup in the grouped XCD-aware order; workgroups from n_gemm on (if
// any) build a batch's plan.
template <class C, int ACT>
__global__ __launch_bounds__(C::kThreads) __attribute__((amdgpu_waves_per_eu(C::kWaves / 4)))
void k_gemm_small(const uint16_t* __restrict__ x, int ldx, const uint16_t* __restrict__ w,
                  const uint16_t* __restrict__ bias, const uint16_t* residual, int ldr, uint16_t* y, int ldy, int T,
                  int K, int N, int tiles_m, int tiles_n, int n_gemm, PlanFillArgs pf) {
    extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
    if ((int)blockIdx.x >= n_gemm) {
        plan_fused_body(pf, blockIdx.x - n_gemm, *reinterpret_cast<PlanSmem*>(smem));
        return;
    }
    int tm, tn;
    tile_coords(blockIdx.x, n_gemm, tiles_m, tiles_n, tm, tn);
    gemm_small_tile<C, ACT>(x, ldx, w, bias, residual, ldr, y, ldy, T, K, N, tm * C::TM, tn * C::TN, smem);
}

using Small32 = SmallCfg<32, 32, 1, 1, 4, 2, 4>;
using Small64 = SmallCfg<64, 64, 1, 2, 2, 1, 4>;
using Small128w = SmallCfg<64, 128, 1, 4, 2, 1, 3>;
using Small128 = SmallCfg<128, 128, 2, 4, 1, 1, 3>;
using Small256w = SmallCfg<128, 256, 2, 4, 1, 1, 3>;

template <class C, int ACT>
hipError_t launch_small(const LinearArgs& a, const PlanView* plan, hipStream_t s) {
    static bool attr_set = false;  // benign race: every thread sets the same value
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm_small<C, ACT>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, C::kLds);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    const int tiles_m = (a.T + C::TM - 1) / C::TM, tiles_n = (a.N + C::TN - 1) / C::TN, n_gemm = tiles_m * tiles_n;
    const PlanFillArgs pf = plan ? plan_fill_args(*plan) : PlanFillArgs{};
    hipLaunchKernelGGL((k_gemm_small<C, ACT>), dim3(n_gemm + (plan ? plan->batch : 0)), dim3(C::kThreads), C::kLds, s,
                       a.x, a.ldx, a.w, a.bias, a.residual, a.ldr, a.y, a.ldy, a.T, a.K, a.N, tiles_m, tiles_n, n_gemm,
                       pf);
    return hipGetLastError();
}

template <int ACT>
hipError_t launch_small_act(int which, const LinearArgs& a, const PlanView* plan, hipStream_t s) {
    switch (which) {
        case 1: return launch_small<Small32, ACT>(a, plan, s);
        case 2: return launch_small<Small64, ACT>(a, plan, s);
        case 3: return launch_small<Small128w, ACT>(a, plan, s);
        case 5: return launch_small<Small256w, ACT>(a, plan, s);
        default: return launch_small<Small128, ACT>(a, plan, s);
    }
}

}  // namespace

// Estimated us of a launch on tiles of tm x tn: a start, plus per round of one tile per
// CU its reduction (us per 1024 k) and its prologue and epilogue.  The constants are
// least-squares fits (6 to 12% rms) to calls timed at 224 shapes: T = 33 to 20000, K x
// N of the projections of layers with d = 256 to 1024.
// One range apart: with more 128 x 128 tiles than CUs but no more of 128 x 256, the
// latter all run at once in eight waves of 64 x 64, a CU each, with three 64-k stages.
// Their fit grows with the share of CUs at work (the clock falls), and against the other
// forms long reductions gain (best of them -> this, 10076 x 2048 x 512 30.8 -> 26.7 us,
// 7000 x 4096 x 1024 60.5 -> 55.8, 10076 x 3072 x 768 49.5 -> 45.4, 1500 x 1024 x 4096 18.4
// -> 17.2), short ones do not (14000 x 512 x 512 12.0 -> 12.4): one workgroup per CU hides
// neither its first loads nor its epilogue.  Nor where two rounds of 64 x 128 are all there
// is to do (1310 x 1024 x 3072 12.5 -> 16.1), which the estimates show.
static int small_gemm_choice(int64_t T, int64_t K, int64_t N, bool residual, int64_t cus) {
    struct Form {
        int64_t tm, tn;
        double start, per_k, tile;
    };
    static constexpr Form kForms[] = {{32, 32, 3.1, 1.07, 0.8}, {64, 64, 2.9, 2.5, 0.94}, {64, 128, 2.1, 4.0, 1.7},
                                      {128, 128, 0.0, 5.85, 4.4}};
    const int64_t n128 = (T + 127) / 128 * ((N + 127) / 128), n256 = (T + 127) / 128 * ((N + 255) / 256);
    double best = 0.0;
    int which = 0;
    for (int i = 0; i < 4; ++i) {
        const Form& f = kForms[i];
        // 128 x 128 tiles in three rounds or more: timed, they never win, though the estimate
        // says so (4000 x 1024 x 3072: 34.5 us, 30.7 on 128 x 256 tiles)
        if (i == 3 && n128 > 2 * cus) continue;
        // nor in two where 128 x 256 tiles need one
        if (i == 3 && n128 > cus && n256 <= cus && K >= 1024 && 5.6 + (7.0 + 7.2 * n256 / cus) * 1e-3 * K < best)
            return kFormWide;
        const int64_t rounds = ((T + f.tm - 1) / f.tm * ((N + f.tn - 1) / f.tn) + cus - 1) / cus;
        const double c = f.start + rounds * (f.per_k * 1e-3 * K + f.tile);
        if (which == 0 || c < best) {
            best = c;
            which = i + 1;
        }
    }
    // the 128 x 256 tiles (last round as halves): with at most one 64-token half per CU they
    // always lose; otherwise the smaller tiles must win by a tenth, the fits' error.  Where a
    // single round gives some CUs one tile and some two, it takes between 1.5 and 2 times one
    // tile's time (4000 x 768 x 2304, 288 tiles: 23.4 us, 25.0 on 64 x 128 tiles, which two
    // full rounds' estimate let win), but nearly 2 with a residual, whose epilogue is longer
    // (13000 x 768 x 768, 306 tiles: 26.6 us, 24.8 on 64 x 128 tiles)
    const int64_t tiles_n = (N + 255) / 256, tiles = (T + 127) / 128 * tiles_n;
    if ((T + 63) / 64 * tiles_n <= cus) return which;
    const int64_t last = tiles - (tiles - 1) / (2 * cus) * (2 * cus);
    const double before = (double)((tiles - last) / cus);
    const double rounds = last <= cus               ? before + 0.5 * ((2 * last + cus - 1) / cus)
                          : before > 0 || residual ? before + 2.0
                                                   : 1.0 + 0.5 * last / cus;
    return best < 0.9 * (4.7 + rounds * (12.9e-3 * K + 2.7)) ? which : 0;
}

// The workgroups of a plan that rides along (plan_batch) ask for as much LDS as the tiles. On
// the forms with one workgroup per CU they wait for the CUs the tiles leave free, or for the
// tiles: a layer of 40 sequences, T = 2454, d = 1024, took 119.1 us (113.1 with its plan built
// before) and 114.5 on 128 x 256 tiles, two per CU; d = 512 64.3 (58.3) and 59.4, with 128
// sequences 67.2 and 60.4.  (Past K = 1024 these forms gain more than the 6 to 12 us.)
static bool plan_waits(int form, int64_t T, int64_t K, int64_t N, int64_t plan_batch, int64_t cus) {
    if ((form != 4 && form != kFormWide) || K > 1024) return false;
    const int64_t tiles = (T + 127) / 128 * (form == kFormWide ? (N + 255) / 256 : (N + 127) / 128);
    return plan_batch > (cus - tiles % cus) % cus;
}

int linear_form_bf16(int64_t T, int64_t K, int64_t N, int act, bool residual, int64_t plan_batch, int64_t cus) {
    int form = small_gemm_choice(T, K, N, residual, cus);
    if (form != kFormWide && gemm_big_wins(T, K, N, act, residual, cus)) form = kFormBig;
    return plan_waits(form, T, K, N, plan_batch, cus) ? 0 : form;
}

hipError_t launch_gemm_small(int form, int act, const LinearArgs& a, const PlanView* plan, hipStream_t s) {
    if (act == 1) return launch_small_act<1>(form, a, plan, s);
    if (act == 2) return launch_small_act<2>(form, a, plan, s);
    return launch_small_act<0>(form, a, plan, s);
}

}  // namespace rag
