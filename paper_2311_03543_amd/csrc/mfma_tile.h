// Pieces that the MFMA GEMM kernels share: the LDS slab layout, the stage
// barrier of their copy pipelines, and the end of a tile whose K range was
// divided among groups of waves.
#pragma once

#include <hip/hip_runtime.h>
#include <atomic>
#include <cstdint>
#include <type_traits>

namespace cmp {

typedef float floatx16 __attribute__((ext_vector_type(16)));

// Byte offset of 16-byte chunk c of slab row r (the panel swizzle).  gfx950's
// LDS serves a 16-byte-per-lane read 16 lanes at a time over 64 banks (256
// bytes = 4 slab rows); the 16 rows one lane group of a fragment read touches
// then occupy (r % 4, c ^ (r / 4) % 4): 16 distinct bank quads, no conflicts.
__device__ __forceinline__ int slab_off(int r, int c) { return r * 64 + ((c ^ ((r >> 2) & 3)) << 4); }

// s_waitcnt immediate: vmcnt <= vm (0..63), lgkmcnt <= lgkm (0..15), expcnt free.
constexpr int waitcnt_imm(int vm, int lgkm) {
    return (vm & 15) | ((vm >> 4) << 14) | (7 << 4) | (lgkm << 8);
}

// Stage barrier: this wave's LDS reads done, at most VM of its copies still
// in flight (copies complete in issue order), then the workgroup barrier:
// afterwards every wave's copies of the awaited stage have landed and every
// wave's reads of the slot about to be refilled are complete.  The empty asm
// statements keep the compiler from moving memory accesses across.
template <int VM>
__device__ __forceinline__ void stage_barrier() {
    static_assert(VM >= 0 && VM <= 63, "vmcnt range");
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(waitcnt_imm(VM, 0));
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// The main loops pin their instruction order explicitly: each MFMA is
// followed by the memory instructions that ride under it, and a
// sched_barrier after each group keeps the scheduler from clustering them.
__device__ __forceinline__ void sched_pin() { __builtin_amdgcn_sched_barrier(0); }

// f(integral_constant<int, I>) for I = B .. E - 1, unrolled at compile time.
template <int B, int E, class F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (B < E) {
        f(std::integral_constant<int, B>{});
        static_for<B + 1, E>(f);
    }
}

// The sums of KG groups of THREADS lanes, each with its run of K, added in the
// order of the runs.  Group g finishes registers r of [16 g / KG, 16 (g + 1) / KG)
// of every block.  `lds` (KG * MI * NJ * 64 * THREADS bytes, THREADS = lanes of a
// group) is free: every wave is past its last read and copy.
template <int KG, int THREADS, int MI, int NJ>
__device__ __forceinline__ void sum_groups(const floatx16 (&acc)[MI][NJ], float (&out)[MI][NJ][16 / KG], uint8_t* lds,
                                           int group, int t) {
    static_assert(KG == 1 || KG == 2 || KG == 4, "a group finishes whole quads of registers");
    typedef float quad __attribute__((ext_vector_type(4)));
    if constexpr (KG == 1) {
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) out[i][j][r] = acc[i][j][r];
    } else {
        quad* x = reinterpret_cast<quad*>(lds);    // [group][block][quad][thread]
        constexpr int QG = 4 / KG;                 // quads of a block that one group finishes
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    x[((group * MI * NJ + i * NJ + j) * 4 + v) * THREADS + t] =
                        quad{acc[i][j][4 * v], acc[i][j][4 * v + 1], acc[i][j][4 * v + 2], acc[i][j][4 * v + 3]};
        __syncthreads();
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
#pragma unroll
                for (int v = 0; v < QG; ++v) {
                    quad sum = x[((i * NJ + j) * 4 + group * QG + v) * THREADS + t];
#pragma unroll
                    for (int g = 1; g < KG; ++g) sum += x[((g * MI * NJ + i * NJ + j) * 4 + group * QG + v) * THREADS + t];
#pragma unroll
                    for (int e = 0; e < 4; ++e) out[i][j][4 * v + e] = sum[e];
                }
    }
}

// C = alpha * out + beta * C for a wave's blocks.  Lane l of a 32 x 32 block
// holds column l % 32, rows 8 (r / 4) + 4 (l / 32) + r % 4; `corner` is the
// address of register 0 of block (0, 0), blocks are RS rows and CS columns
// apart, and `rl` rows and `cl` columns from the corner on lie inside C.
template <bool FULL, int RS, int CS, int RG, int MI, int NJ>
__device__ __forceinline__ void store_blocks(const float (&out)[MI][NJ][RG], __attribute__((address_space(1))) float* corner,
                                             int64_t ldc, int rl, int cl, float alpha, float beta) {
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            if (!FULL && CS * j >= cl) continue;
            __attribute__((address_space(1))) float* c = corner + (RS * i * ldc + CS * j);
            float old[RG];
            if (beta != 0.f) {                     // all loads in flight before the first use
#pragma unroll
                for (int r = 0; r < RG; ++r) {
                    const int dr = (r >> 2) * 8 + (r & 3);
                    old[r] = FULL || RS * i + dr < rl ? c[dr * ldc] : 0.f;
                }
            }
#pragma unroll
            for (int r = 0; r < RG; ++r) {
                const int dr = (r >> 2) * 8 + (r & 3);
                if (FULL || RS * i + dr < rl) {
                    float v = alpha * out[i][j][r];
                    if (beta != 0.f) v = __builtin_fmaf(beta, old[r], v);
                    c[dr * ldc] = v;
                }
            }
        }
}

// The kernels use more than the default 64 KiB of dynamic LDS; the limit is a
// per-device function attribute, set once on each device the library runs on.
template <class Kernel>
hipError_t allow_lds(Kernel kernel, std::atomic<uint64_t>& done, size_t bytes) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = dev < 64 ? (uint64_t)1 << dev : 0;
    if (bit && (done.load(std::memory_order_relaxed) & bit)) return hipSuccess;
    e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e == hipSuccess) done.fetch_or(bit, std::memory_order_relaxed);
    return e;
}

}  // namespace cmp
