// Pieces the matrix kernels share: buffer descriptors and direct global -> LDS
// copies, barriers that do not drain them, the tile orders, and the entry checks
// of the variable-sized batched GEMM.
#pragma once

#include "device_common.h"
#include "launch.h"

namespace rag {

constexpr int kGroupM = 8;  // token tiles per group in the tile order

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00020000);
}

// Workgroup barrier that waits for LDS traffic but not for the copies still in
// flight (a __syncthreads() fence would drain them all): the caller has already
// waited for the copies it needs.
__device__ __forceinline__ void barrier_lds() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

template <int N>
__device__ __forceinline__ void wait_vm() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// 128-byte LDS rows (eight 16-byte chunks) whose chunk index is XOR-swizzled with
// bits 1-3 of the row: the fragment reads of 16 consecutive rows (two rows per
// 256-byte bank line) hit 16 distinct bank groups.
__device__ __forceinline__ int swz2(int row) { return (row >> 1) & 7; }

// Output tile of a linear workgroup id.  Workgroups are dealt to the 8 XCDs
// round-robin, so the id is first remapped to give each XCD a contiguous range.
// That range is walked in groups of kGroupM token tiles, token tile fastest, so
// the tiles an XCD runs at once share both x rows and w rows in its L2 (groups of
// 2 to 16 measured alike on the layer's GEMMs except FF1, slower below 8).
__device__ __forceinline__ void group_walk(int t, int tiles_m, int tiles_n, int& tm, int& tn) {
    const int gsz = kGroupM * tiles_n, first = (t / gsz) * kGroupM;
    const int gm = min(tiles_m - first, kGroupM);
    tm = first + (t % gsz) % gm;
    tn = (t % gsz) / gm;
}

__device__ __forceinline__ void tile_coords(int bid, int nblocks, int tiles_m, int tiles_n, int& tm, int& tn) {
    const int per = nblocks / 8, rem = nblocks % 8;
    const int xcd = bid % 8, idx = bid / 8;
    const int t = xcd < rem ? xcd * (per + 1) + idx : rem * (per + 1) + (xcd - rem) * per + idx;
    group_walk(t, tiles_m, tiles_n, tm, tn);
}

// Triangular product tiles: listed heaviest row first, columns ascending, and dealt
// to the XCDs in chunks of `chunk` consecutive columns (workgroups go to the XCDs
// round-robin).  With chunk = tiles_n / 8 each XCD owns the same column panels
// of B in every row (so B is fetched into one L2, not eight) and gets the same
// share of every row, hence the same total work.
__device__ __forceinline__ bool trmm_tile_coords(int bid, int tiles_m, int tiles_n, int chunk, int& tm, int& tn) {
    const int xcd = bid % 8, idx = bid / 8;
    const int t = ((idx / chunk) * 8 + xcd) * chunk + idx % chunk;
    if (t >= tiles_m * tiles_n) return false;
    tm = tiles_m - 1 - t / tiles_n;
    tn = t % tiles_n;
    return true;
}

// List position of work position p when runs of `run` consecutive list positions go to one
// XCD (workgroups, and so positions taken with a stride that is a multiple of 8, go to the
// XCDs round-robin), the runs round-robin; a permutation of [0, n) for any n that is a
// multiple of 8 * run.
__device__ __forceinline__ int dealt_to_xcds(int p, int run) {
    const int xcd = p % 8, idx = p / 8;
    return ((idx / run) * 8 + xcd) * run + idx % run;
}

// ---------------------------------------------------------------------------
// Variable-sized batched GEMM: the plan's tile list (problems largest first), one
// entry per kVgemmTileM x kVgemmTileN output tile.
// ---------------------------------------------------------------------------
struct VgemmArgs {
    const int32_t* dims;
    const int64_t* a_off;
    const int64_t* b_off;
    const int64_t* c_off;
    const int4* items;
    int32_t* status;
    int batch;
    int64_t a_cap, b_cap, c_cap;
};

// The tile of one list entry: problem sizes, output rows [m0, m0 + 128) and
// columns [n0, n0 + 256) of C_p = A_p B_p^T.
struct VgemmTile {
    int m, n, k, m0, n0;
    int64_t a_off, b_off, c_off;
};

__device__ __forceinline__ VgemmTile vgemm_tile(const VgemmArgs& va, int e) {
    const int4 it = va.items[e];
    const int p = uni(it.x);
    VgemmTile t;
    t.m = uni(va.dims[3 * p]);
    t.n = uni(va.dims[3 * p + 1]);
    t.k = uni(va.dims[3 * p + 2]);
    t.m0 = uni(it.y) * kVgemmTileM;
    t.n0 = uni(it.z) * kVgemmTileN;
    t.a_off = uni64(va.a_off[p]);
    t.b_off = uni64(va.b_off[p]);
    t.c_off = uni64(va.c_off[p]);
    return t;
}

// False if the plan reports a data error or this call cannot run on it; one
// thread then records why and every workgroup returns.
__device__ __forceinline__ bool vgemm_ok(const VgemmArgs& va, bool bf16) {
    if (va.status[0] != 0) return false;
    int bad = 0;
    if (va.a_off[va.batch] > va.a_cap || va.b_off[va.batch] > va.b_cap || va.c_off[va.batch] > va.c_cap)
        bad |= kVgemmOperandCap;
    if (bf16 && va.status[2] != 0) bad |= kVgemmBf16Shape;
    if (bad) {
        if (blockIdx.x == 0 && threadIdx.x == 0) atomicOr(va.status, bad);
        return false;
    }
    return true;
}

// One bf16 packed linear call.
struct LinearArgs {
    const uint16_t* x;
    int ldx;
    const uint16_t* w;
    const uint16_t* bias;
    const uint16_t* residual;
    int ldr;
    uint16_t* y;
    int ldy, T, K, N;
};

// The tile form a bf16 packed linear call runs, by its sizes and the sequences of the plan it
// carries (0 without one): 0 the 128 x 256 tiles
// (gemm.hip), 1 .. 4 smaller tiles for small launches and 5 128 x 256 in one round
// (gemm_small.hip), 6 256 x 256 for long reductions (gemm_big.hip).
constexpr int kFormWide = 5, kFormBig = 6;
int linear_form_bf16(int64_t T, int64_t K, int64_t N, int act, bool residual, int64_t plan_batch, int64_t cus);
hipError_t launch_gemm_small(int form, int act, const LinearArgs& a, const PlanView* plan, hipStream_t s);
bool gemm_big_wins(int64_t T, int64_t K, int64_t N, int act, bool residual, int64_t cus);
hipError_t launch_gemm_big(const LinearArgs& a, const PlanView* plan, hipStream_t s);  // no activation

// Grid of a vgemm launch over `entries` list entries at most, `parts` workgroups each, dealt
// in runs of `run` entries.  The list's length is known on the device only, and a plan's
// capacity may be many times that (100,000 idle workgroups of 80 KB LDS take 70 us to come and
// go): past kVgemmPerCu entries per CU the workgroups loop over the positions instead.
constexpr int64_t kVgemmPerCu = 32;
struct VgemmGrid {
    int blocks;  // a multiple of 8
    bool loop;
};
inline VgemmGrid vgemm_grid(int64_t entries, int64_t parts, int64_t run, int64_t cus) {
    const int64_t all = (entries + 8 * run - 1) / (8 * run) * (8 * run) * parts, most = kVgemmPerCu * cus * parts / 8 * 8;
    return all <= most ? VgemmGrid{(int)all, false} : VgemmGrid{(int)most, true};
}

// The tiles of an fp32 packed linear call: 128 (128 x 128; only if 32-bit offsets reach 128
// rows of x and w: leading dimensions below 2^22) or 64 (64 x 64), plus one if the last round
// of tiles runs as quarters.
int linear_form_f32(int64_t T, int64_t N, bool reach128, int64_t cus);
// fp32 launchers (gemm_f32.hip), called by the launchers that take both types.
hipError_t launch_linear_f32(const float* x, int ldx, const float* w, const float* bias, const float* residual, int ldr,
                             int act, float* y, int ldy, int T, int K, int N, hipStream_t s);
hipError_t launch_vgemm_f32(const VgemmArgs& va, int64_t tile_cap, const float* a, const float* b, float* c,
                            hipStream_t s);
hipError_t launch_trmm_f32(const float* l, int ldl, const float* b, int ldb, float* c, int ldc, int n, int m,
                           hipStream_t s);

}  // namespace rag
