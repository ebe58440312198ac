// FP32 GEMM for gfx950 (the "f32_simt" variant): C = alpha * A * B + beta * C,
// row-major, any shape and leading dimension, every product and sum an FP32 FMA.
//
// Two launch forms share the tile code of f32_tile.h:
//   - one problem: a tile per workgroup, tiles renumbered so each XCD works
//     on a contiguous, L2-friendly block of C;
//   - a group of problems of uneven shapes: one persistent launch over eight
//     tile lists, one per XCD, with a counter each (common.h, TileQueues).  A
//     workgroup claims its next tile ahead of the stores of the current one
//     (64 x 64 tiles: at its start), and from the other lists once its own is
//     empty.  Lists hold whole problems where they can, balanced by work, in
//     decreasing order of K, so the longest tiles go first and the tail is
//     short.  The autotuner picks the tile shape per group from kGroupedConfigs.
#include <cmath>
#include <type_traits>

#include "common.h"
#include "kernels.h"
#include "f32_tile.h"

namespace cmp {
namespace {

using CfgL = F32Cfg<128, 256, 16, 32, 2>;
using CfgD = F32Cfg<128, 128, 32, 32, 2>;
using CfgM = F32Cfg<64, 64, 16, 32, 4>;
using CfgS = F32Cfg<32, 32, 64, 16, 2>;

template <typename Cfg, int WAVES>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(WAVES))) void gemm_f32_kernel(
    F32Problem p, bool vec, int tiles_m, int tiles_n) {
    __shared__ __attribute__((aligned(256))) float smem[Cfg::SMEM_FLOATS];
    int tm, tn;
    grouped_tile(xcd_remap(blockIdx.x, tiles_m * tiles_n), tiles_m, tiles_n, 8, tm, tn);
    f32_tile<Cfg>(p, (int64_t)tm * Cfg::BM, (int64_t)tn * Cfg::BN, vec, smem, [] {});
}

// Persistent grouped kernel over the tile lists of `q` (common.h): each
// workgroup works through tiles.  A list holds its pieces in decreasing order of
// K, so the longest tiles go first.  The next tile is claimed where the stores of
// one begin, but where a 64 x 64 tile begins, whose few stores do not cover the
// answer (512 problems up to 512: 111 us, claimed late 118); 128 x 128 tiles are
// long enough that an entry claimed early would wait for one while other
// workgroups idle (124 us, claimed late 114).
// Workgroups per CU a configuration is built for: the LDS of its ring (160 KiB
// a CU) and the accumulators allow no more.  A tile's fixed costs (first copies
// from HBM, the stores of C) hide under the other workgroups of the CU.
template <typename Cfg>
constexpr int grouped_waves() {
    constexpr int lds = 160 * 1024 / (Cfg::SMEM_FLOATS * 4 + 256);
    constexpr int regs = Cfg::MI * Cfg::NJ <= 2 ? 4 : Cfg::MI * Cfg::NJ <= 4 ? 3 : 2;
    return lds < regs ? lds : regs;
}

template <typename Cfg>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(grouped_waves<Cfg>())))
void gemm_f32_grouped_kernel(const GroupedDesc* __restrict__ desc, int count, TileQueues q,
                             unsigned* __restrict__ counters) {
    __shared__ __attribute__((aligned(256))) float smem[Cfg::SMEM_FLOATS];
    __shared__ int slot;
    typedef const __attribute__((address_space(1))) GroupedDesc* gdesc;
    const gdesc dg = (gdesc)desc;
    TileClaims claims(q, counters);
    constexpr bool EARLY = Cfg::MI * Cfg::NJ == 1;
    for (int tile = claims.first(&slot); tile >= 0; tile = claims.next(&slot)) {
        if (EARLY) claims.prefetch();
        const int lo = wave_find_last(count, tile, [&](int i) { return dg[i].tile_start; });
        const int tiles_n = dg[lo].tiles_n;
        const int local = tile - dg[lo].tile_start + dg[lo].tile_first;
        const int tm = local / tiles_n, tn = local - (local / tiles_n) * tiles_n;
        const F32Problem p{dg[lo].M, dg[lo].N, dg[lo].K, dg[lo].lda, dg[lo].ldb, dg[lo].ldc,
                            dg[lo].alpha, dg[lo].beta, dg[lo].A, dg[lo].B, dg[lo].C};
        f32_tile<Cfg>(p, (int64_t)tm * Cfg::BM, (int64_t)tn * Cfg::BN, dg[lo].vec != 0, smem,
                      [&]() __attribute__((always_inline)) {
                          if (!EARLY) claims.prefetch();
                      });
        // claims.next starts with a barrier: the ring is free for the next tile
    }
    claims.finish();
}

__global__ void scale_c_kernel(int64_t M, int64_t N, float beta, float* __restrict__ C,
                               int64_t ldc) {
    const int64_t total = M * N;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
         e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = e / N, j = e - i * N;
        float* p = C + i * ldc + j;
        *p = (beta == 0.f) ? 0.f : beta * *p;
    }
}

template <typename Cfg>
hipError_t launch_grouped_cfg(const GroupedDesc* desc, int count, const TileQueues& q, int grid,
                              unsigned* counters, hipStream_t stream) {
    hipLaunchKernelGGL(gemm_f32_grouped_kernel<Cfg>, dim3(grid), dim3(256), 0, stream, desc, count, q, counters);
    return hipGetLastError();
}

}  // namespace

const GroupedConfig kGroupedConfigs[kNumGroupedConfigs] = {
    {64, 64, 16}, {64, 64, 32}, {64, 128, 16}, {128, 64, 16},
    {128, 128, 16}, {128, 128, 32}, {256, 128, 16}, {128, 256, 16},
    {64, 64, 64}, {64, 128, 64},
};

hipError_t launch_gemm_f32_grouped(int config, const GroupedDesc* desc, int count, const TileQueues& q,
                                   int grid, unsigned* counters, hipStream_t stream) {
    if (q.start[kXcds] <= 0) return hipSuccess;
    if (grid < 1 || grid > q.start[kXcds] || !counters || count < 1) return hipErrorInvalidValue;
    switch (config) {
        case 0: return launch_grouped_cfg<F32Cfg<64, 64, 16, 32, 4>>(desc, count, q, grid, counters, stream);
        case 1: return launch_grouped_cfg<F32Cfg<64, 64, 32, 32, 3>>(desc, count, q, grid, counters, stream);
        case 2: return launch_grouped_cfg<F32Cfg<64, 128, 16, 32, 3>>(desc, count, q, grid, counters, stream);
        case 3: return launch_grouped_cfg<F32Cfg<128, 64, 16, 32, 3>>(desc, count, q, grid, counters, stream);
        case 4: return launch_grouped_cfg<F32Cfg<128, 128, 16, 32, 3>>(desc, count, q, grid, counters, stream);
        case 5: return launch_grouped_cfg<F32Cfg<128, 128, 32, 32, 2>>(desc, count, q, grid, counters, stream);
        case 6: return launch_grouped_cfg<F32Cfg<256, 128, 16, 32, 2>>(desc, count, q, grid, counters, stream);
        case 7: return launch_grouped_cfg<F32Cfg<128, 256, 16, 32, 2>>(desc, count, q, grid, counters, stream);
        case 8: return launch_grouped_cfg<F32Cfg<64, 64, 64, 32, 2>>(desc, count, q, grid, counters, stream);
        case 9: return launch_grouped_cfg<F32Cfg<64, 128, 64, 32, 2>>(desc, count, q, grid, counters, stream);
        default: return hipErrorInvalidValue;
    }
}

int grouped_blocks_per_cu(int config) {
    int nb = 0;
    hipError_t e = hipErrorInvalidValue;
    switch (config) {
        case 0: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, gemm_f32_grouped_kernel<F32Cfg<64, 64, 16, 32, 4>>, 256, 0); break;
        case 1: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, gemm_f32_grouped_kernel<F32Cfg<64, 64, 32, 32, 3>>, 256, 0); break;
        case 2: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, gemm_f32_grouped_kernel<F32Cfg<64, 128, 16, 32, 3>>, 256, 0); break;
        case 3: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, gemm_f32_grouped_kernel<F32Cfg<128, 64, 16, 32, 3>>, 256, 0); break;
        case 4: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, gemm_f32_grouped_kernel<F32Cfg<128, 128, 16, 32, 3>>, 256, 0); break;
        case 5: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, gemm_f32_grouped_kernel<F32Cfg<128, 128, 32, 32, 2>>, 256, 0); break;
        case 6: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, gemm_f32_grouped_kernel<F32Cfg<256, 128, 16, 32, 2>>, 256, 0); break;
        case 7: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, gemm_f32_grouped_kernel<F32Cfg<128, 256, 16, 32, 2>>, 256, 0); break;
        case 8: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, gemm_f32_grouped_kernel<F32Cfg<64, 64, 64, 32, 2>>, 256, 0); break;
        case 9: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, gemm_f32_grouped_kernel<F32Cfg<64, 128, 64, 32, 2>>, 256, 0); break;
        default: break;
    }
    return (e == hipSuccess && nb > 0) ? nb : 1;
}

template <typename Cfg, int WAVES>
hipError_t launch_f32(const F32Problem& p, bool vec, hipStream_t stream) {
    const int64_t tm = (p.M + Cfg::BM - 1) / Cfg::BM, tn = (p.N + Cfg::BN - 1) / Cfg::BN;
    if (!launch_fits(tm * tn, 256)) return hipErrorInvalidValue;
    hipLaunchKernelGGL((gemm_f32_kernel<Cfg, WAVES>), dim3((unsigned)(tm * tn)), dim3(256), 0, stream, p, vec, (int)tm,
                       (int)tn);
    return hipGetLastError();
}

hipError_t launch_gemm_f32_simt(int64_t M, int64_t N, int64_t K, float alpha, const float* A,
                                int64_t lda, const float* B, int64_t ldb, float beta, float* C,
                                int64_t ldc, hipStream_t stream) {
    if (M <= 0 || N <= 0) return hipSuccess;
    const bool vec = (lda % 4 == 0) && (ldb % 4 == 0) &&
                     ((reinterpret_cast<uintptr_t>(A) & 15) == 0) &&
                     ((reinterpret_cast<uintptr_t>(B) & 15) == 0);
    const F32Problem p{M, N, K, lda, ldb, ldc, alpha, beta, A, B, C};
    // The tile with the least expected time.  The CU with the most tiles, n =
    // ceil(tiles / 256) of them, takes (n + c) * BM * BN / rate (per K): `rate`
    // is what the tile reaches with many tiles on each CU and c the cost of
    // filling and draining the pipeline in tiles, both fitted to these
    // measurements (TFLOP/s, one launch, 5 us of it the launch itself):
    //               512^3  1024^3  2048^3  4096^3  8192^3  2000x3000x2500
    //   128 x 256                     67     143     148       88
    //   128 x 128                    124     143     146       95
    //    64 x  64       17      75   118     129     134      112
    //    32 x  32       29      74
    auto cost = [&](int bm, int bn, double c, double rate) {
        const int64_t tiles = ((M + bm - 1) / bm) * ((N + bn - 1) / bn);
        return launch_fits(tiles, 256) ? ((double)((tiles + 255) / 256) + c) * bm * bn / rate : INFINITY;
    };
    const double l = cost(128, 256, 0.1, 150), d = cost(128, 128, 0.19, 148), m = cost(64, 64, 0.35, 130),
                 q = cost(32, 32, 0.5, 98);
    if (q <= l && q <= d && q <= m) return launch_f32<CfgS, 4>(p, vec, stream);
    if (m <= l && m <= d) return launch_f32<CfgM, 4>(p, vec, stream);
    if (d <= l) return launch_f32<CfgD, 2>(p, vec, stream);
    return launch_f32<CfgL, 2>(p, vec, stream);
}

hipError_t launch_scale_c(int64_t M, int64_t N, float beta, float* C, int64_t ldc,
                          hipStream_t stream) {
    const int64_t total = M * N;
    if (total == 0) return hipSuccess;
    int64_t blocks = (total + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(scale_c_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, M, N, beta,
                       C, ldc);
    return hipGetLastError();
}

}  // namespace cmp
