// bf16 and bf16x3 GEMM straight from the FP32 operands, for shapes whose
// operand images (prepass.hip) would cost more than they save: one launch
// instead of a pre-pass and the image kernel (and its split-K reduction).
//
// A group of 4 waves (2 x 2) computes a BM x BN tile over a run of K, in stages
// of 32.  Each thread loads its share of the next stages from global memory (PF
// register sets in flight), rounds it to bf16 or splits it into hi and lo, and
// writes it to LDS in the slab layout of the image kernels (64-byte rows of K,
// 16-byte chunks swizzled, conflict-free); the waves read their fragments from
// there.  A value is converted once per workgroup: converting the fragments as
// they leave LDS, once per wave that multiplies them, measured 103 us against
// 71 on 2048^3 (bf16x3).  A stage is a serial chain (read, convert, MFMAs on one
// or four accumulators, barrier) that leaves one wave per SIMD idle half its
// time, so KG groups of 4 waves share a workgroup, each with its run of K, and
// add their sums in LDS (bf16x3, 1024^3: 21.6 / 18.4 / 17.6 us for KG = 1 / 2 /
// 4).  One-term bf16 is bound by the tiles' traffic out of L2 (15 - 17 TB/s) and
// gains from more groups only where a CU has a single 128 x 128 tile.
//
// The arithmetic is the image kernels': the same hi and lo, the same products
// hi.hi + hi.lo + lo.hi per 16 k into FP32 accumulators; only the runs of K
// whose sums are added at the end differ, and their order is fixed.
#include <cmath>
#include <type_traits>

#include "common.h"
#include "kernels.h"
#include "mfma_tile.h"

namespace cmp {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef f32x4 f32x4_word __attribute__((aligned(4)));   // 16-byte load at 4-byte alignment
typedef const __attribute__((address_space(1))) char* gcbyte;
typedef const __attribute__((address_space(1))) float* gcfloat;
typedef const __attribute__((address_space(1))) f32x4_word* gcf32x4;
typedef __attribute__((address_space(1))) float* gfloat;

struct DirectProblem {
    int64_t M, N, K, lda, ldb, ldc;
    float alpha, beta;
    const float* A;
    const float* B;
    float* C;
    float* partial;   // != nullptr: slice y writes raw sums to partial + y M N (pitch N)
    int64_t slice;    // K values per slice (a multiple of 32)
};

template <int BM_, int BN_, int NT_, int KG_>
struct DirectCfg {
    static constexpr int BM = BM_, BN = BN_, NT = NT_, KG = KG_;
    static constexpr int PF = 2;                                 // stages in flight in registers (3 or 4: no faster, or spills)
    static constexpr int BK = 32, NL = NT == 3 ? 2 : 1;          // levels: hi, lo
    static constexpr int MI = BM / 64, NJ = BN / 64;             // 32 x 32 blocks per wave
    static constexpr int UA = BM / 32, UB = BN / 64;             // units per thread and stage: 4 values of A, 8 of B
    static constexpr int SLAB_A = BM * 64, SLAB_B = BN * 64;     // bytes of one level
    static constexpr int STAGE = NL * (SLAB_A + SLAB_B);
    static constexpr int U = PF;                                 // stages per unrolled pass: register sets and LDS halves
    static_assert(BM % 64 == 0 && BN % 64 == 0 && (NT == 1 || NT == 3), "tile");
    static_assert(KG == 1 || KG == 2 || KG == 4, "each group finishes its share of the accumulators");
    // LDS: each group's two stages; after the main loop the groups' accumulators
    static constexpr int ACC = MI * NJ * 16 * 256 * 4;           // bytes of one group's accumulators
    static constexpr int SMEM = KG * (2 * STAGE > ACC || KG == 1 ? 2 * STAGE : ACC);
};

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t pk_bf16(float a, float b) {   // v_cvt_pk_bf16_f32: nearest even
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}

// 2 W values -> W words of hi (and of lo = RNE(x - hi)).  lo is 0 for
// non-finite x, the only values whose x - hi is NaN: the fast form leaves them
// wrong and `sum` NaN (one test then stands for all values of a stage), SAFE
// tests each.
template <int W, int NL, bool SAFE>
__device__ __forceinline__ void split_words(const float (&x)[2 * W], uint32_t (&o)[NL][W], float& sum) {
#pragma unroll
    for (int v = 0; v < W; ++v) {
        const uint32_t h = pk_bf16(x[2 * v], x[2 * v + 1]);
        o[0][v] = h;
        if constexpr (NL == 2) {
            float l0 = x[2 * v] - __builtin_bit_cast(float, h << 16);
            float l1 = x[2 * v + 1] - __builtin_bit_cast(float, h & 0xffff0000u);
            if (SAFE && !__builtin_isfinite(x[2 * v])) l0 = 0.f;
            if (SAFE && !__builtin_isfinite(x[2 * v + 1])) l1 = 0.f;
            if (!SAFE) sum += l0 + l1;
            o[NL - 1][v] = pk_bf16(l0, l1);
        }
    }
}

template <typename Cfg, int WAVES>
__global__ __launch_bounds__(256 * Cfg::KG) __attribute__((amdgpu_waves_per_eu(WAVES)))
void gemm_direct_kernel(DirectProblem p, int tiles_m, int tiles_n) {
    constexpr int BM = Cfg::BM, BN = Cfg::BN, NT = Cfg::NT, NL = Cfg::NL, PF = Cfg::PF, U = Cfg::U;
    constexpr int MI = Cfg::MI, NJ = Cfg::NJ, UA = Cfg::UA, UB = Cfg::UB, KG = Cfg::KG;
    __shared__ __attribute__((aligned(256))) uint8_t lds[Cfg::SMEM];   // stage: A levels, then B levels
    int tm, tn;
    grouped_tile(xcd_remap(blockIdx.x, tiles_m * tiles_n), tiles_m, tiles_n, 8, tm, tn);
    const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;
    const int t = threadIdx.x & 255, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int group = KG == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
    uint8_t* smem = lds + group * 2 * Cfg::STAGE;
    const int wm = wave >> 1, wn = wave & 1;
    const int rows = (int)(p.M - m0 < BM ? p.M - m0 : BM), cols = (int)(p.N - n0 < BN ? p.N - n0 : BN);
    // K values of this workgroup (slice blockIdx.y), then of this group: the
    // stages are dealt out in runs that differ by one stage at most
    const int64_t slice0 = (int64_t)blockIdx.y * p.slice;
    const int64_t Ks = p.K - slice0 < p.slice ? p.K - slice0 : p.slice;
    const int all = (int)((Ks + 31) / 32), first = all * group / KG;
    const int nst = all * (group + 1) / KG - first, most = (all + KG - 1) / KG;
    const int64_t kbase = slice0 + (int64_t)first * 32;
    const int64_t K = slice0 + Ks - kbase < (int64_t)nst * 32 ? slice0 + Ks - kbase : (int64_t)nst * 32;
    const int whole = (int)(K / 32), steady = all / KG - (Ks % 32 ? 1 : 0);   // stages that are whole in every group

    // This thread's units: four k of a row of A (eight threads per row, so a wave
    // reads eight whole 128-byte rows); a k octet of a column of B (a wave reads 64
    // consecutive columns).  Uniform bases plus 32-bit byte offsets (the host
    // checks that they fit).
    const gcfloat abase = (gcfloat)p.A + m0 * p.lda + kbase, bbase = (gcfloat)p.B + kbase * p.ldb + n0;
    uint32_t oa[UA], ob[UB][8];
    int la[UA], lb[UB];                            // LDS byte offsets of the units' chunks
#pragma unroll
    for (int q = 0; q < UA; ++q) {
        const int u = t + 256 * q, r = u >> 3, c = u & 7;
        oa[q] = ((uint32_t)(r < rows ? r : rows - 1) * (uint32_t)p.lda + 4 * c) * 4u;
        la[q] = slab_off(r, c >> 1) + 8 * (c & 1);
    }
#pragma unroll
    for (int q = 0; q < UB; ++q) {
        const int u = t + 256 * q, n = u % BN, c = u / BN;
#pragma unroll
        for (int e = 0; e < 8; ++e)
            ob[q][e] = ((uint32_t)(8 * c + e) * (uint32_t)p.ldb + (n < cols ? n : cols - 1)) * 4u;
        lb[q] = NL * Cfg::SLAB_A + slab_off(n, c);
    }
    float ga[PF][UA][4], gb[PF][UB][8];            // raw values of the stages in flight
    auto load = [&](int s, int set) __attribute__((always_inline)) {              // a whole stage
        const gcfloat a = abase + (int64_t)s * 32, b = bbase + (int64_t)s * 32 * p.ldb;
#pragma unroll
        for (int q = 0; q < UA; ++q) {
            asm volatile("" : "+v"(oa[q]));        // keep it a 32-bit offset
            const f32x4 v = *(gcf32x4)((gcbyte)a + oa[q]);
#pragma unroll
            for (int e = 0; e < 4; ++e) ga[set][q][e] = v[e];
        }
#pragma unroll
        for (int q = 0; q < UB; ++q) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                asm volatile("" : "+v"(ob[q][e]));
                gb[set][q][e] = *(gcfloat)((gcbyte)b + ob[q][e]);
            }
        }
    };
    auto load_tail = [&](int s, int set) __attribute__((always_inline)) {         // the last stage: zero past K, addresses kept inside
        const int left = (int)(K - (int64_t)s * 32);
        const gcfloat a = abase + (int64_t)s * 32, b = bbase + (int64_t)s * 32 * p.ldb;
#pragma unroll
        for (int q = 0; q < UA; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int c = ((t + 256 * q) & 7) * 4;
                const bool in = c + e < left;
                const float v = *(gcfloat)((gcbyte)a + (in ? oa[q] + 4 * e : oa[q] - 4 * c));
                ga[set][q][e] = in ? v : 0.f;
            }
#pragma unroll
        for (int q = 0; q < UB; ++q)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int c = (t + 256 * q) / BN * 8;
                const bool in = c + e < left;
                const float v = *(gcfloat)((gcbyte)b + (in ? ob[q][e] : ob[q][0] - (uint32_t)c * (uint32_t)p.ldb * 4u));
                gb[set][q][e] = in ? v : 0.f;
            }
    };
    auto fetch = [&](int s, int set) __attribute__((always_inline)) {
        if (s < whole) load(s, set);
        else if (s < nst) load_tail(s, set);
    };
    float sum = 0.f;                               // NaN once a stage held a non-finite value
    auto convert = [&](int half, int set, auto safe_tag) __attribute__((always_inline)) {   // a stage's values to an LDS half
        constexpr bool SAFE = decltype(safe_tag)::value;
        uint8_t* st = smem + half * Cfg::STAGE;
        if (!SAFE) sum = 0.f;
#pragma unroll
        for (int q = 0; q < UA; ++q) {
            uint32_t o[NL][2];
            split_words<2, NL, SAFE>(ga[set][q], o, sum);
#pragma unroll
            for (int l = 0; l < NL; ++l) *reinterpret_cast<u32x2*>(st + l * Cfg::SLAB_A + la[q]) = u32x2{o[l][0], o[l][1]};
        }
#pragma unroll
        for (int q = 0; q < UB; ++q) {
            uint32_t o[NL][4];
            split_words<4, NL, SAFE>(gb[set][q], o, sum);
#pragma unroll
            for (int l = 0; l < NL; ++l)
                *reinterpret_cast<u32x4*>(st + l * Cfg::SLAB_B + lb[q]) = u32x4{o[l][0], o[l][1], o[l][2], o[l][3]};
        }
    };
    auto redo_if_needed = [&](int half, int set) __attribute__((always_inline)) {
        if (NL == 2 && __builtin_expect(__builtin_isnan(sum), 0)) convert(half, set, std::true_type{});
    };

    floatx16 acc[MI][NJ];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    // block (2 i + wm, 2 j + wn) of the tile; lane l feeds row l % 32, chunk 2 ks + l / 32
    const int fr = lane & 31, fk = lane >> 5;
    int fa[2], fb[2];                              // per k step: byte offset of this lane's chunk in block row 0
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        fa[ks] = slab_off(wm * 32 + fr, 2 * ks + fk);
        fb[ks] = NL * Cfg::SLAB_A + slab_off(wn * 32 + fr, 2 * ks + fk);
    }
    struct Frag {
        bf16x8 a[NL][MI], b[NL][NJ];
    };
    auto read = [&](Frag& f, int half, int ks) __attribute__((always_inline)) {
        const uint8_t* st = smem + half * Cfg::STAGE;
#pragma unroll
        for (int l = 0; l < NL; ++l) {
#pragma unroll
            for (int i = 0; i < MI; ++i)
                f.a[l][i] = *reinterpret_cast<const bf16x8*>(st + l * Cfg::SLAB_A + fa[ks] + i * 64 * 64);
#pragma unroll
            for (int j = 0; j < NJ; ++j)
                f.b[l][j] = *reinterpret_cast<const bf16x8*>(st + l * Cfg::SLAB_B + fb[ks] + j * 64 * 64);
        }
    };
    auto mfmas = [&](const Frag& f) __attribute__((always_inline)) {              // hi.hi, hi.lo, lo.hi
#pragma unroll
        for (int u = 0; u < NT; ++u)
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[u == 2 ? NL - 1 : 0][i],
                                                                        f.b[u == 1 ? NL - 1 : 0][j], acc[i][j], 0, 0, 0);
    };

    // Stage s: its bf16 slabs are in LDS half s % 2; the registers hold stages
    // s + 1 .. s + PF (set = stage % PF).  While stage s is multiplied, stage
    // s + 1 is converted into the other half and stage s + 1 + PF loaded in its
    // place; the group barriers spread the conversion between the MFMAs.
    auto work = [&](int u) __attribute__((always_inline)) {
        Frag f[2];
        read(f[0], u & 1, 0);
        read(f[1], u & 1, 1);
        convert((u + 1) & 1, (u + 1) % PF, std::false_type{});
        mfmas(f[0]);
        mfmas(f[1]);
        constexpr int NM = 2 * NT * MI * NJ;
        constexpr int VALU = (UA / 2 + UB) * (NL == 2 ? 36 : 4) / NM;   // VALU instructions of the conversion per MFMA
        __builtin_amdgcn_sched_group_barrier(0x100, 2 * NL * (MI + NJ), 0);
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            __builtin_amdgcn_sched_group_barrier(0x002, VALU + 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        }
        redo_if_needed((u + 1) & 1, (u + 1) % PF);
    };
#pragma unroll
    for (int s = 0; s < PF; ++s) fetch(s, s);
    if (nst > 0) {
        convert(0, 0, std::false_type{});
        redo_if_needed(0, 0);
    }
    fetch(PF, 0);
    __syncthreads();
    int s = 0;
    for (; s + U + PF < steady; s += U) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            work(u);
            load(s + u + 1 + PF, (u + 1) % PF);
            __syncthreads();
        }
    }
    for (; s < most; s += U) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (s + u < nst) {                     // (past the end the converted values are stale and not read)
                work(u);
                fetch(s + u + 1 + PF, (u + 1) % PF);
            }
            __syncthreads();
        }
    }

    float out[MI][NJ][16 / KG];
    sum_groups<KG, 256>(acc, out, lds, group, t);

    const bool part = p.partial != nullptr;
    const int64_t ldc = part ? p.N : p.ldc;
    const float alpha = part ? 1.f : p.alpha, beta = part ? 0.f : p.beta;
    const int r0 = wm * 32 + 4 * fk + group * (32 / KG), c0 = wn * 32 + fr;
    const gfloat corner = (part ? (gfloat)p.partial + (int64_t)blockIdx.y * p.M * p.N : (gfloat)p.C) + (m0 + r0) * ldc + n0 + c0;
    if (rows == BM && cols == BN) store_blocks<true, 64, 64>(out, corner, ldc, 0, 0, alpha, beta);
    else store_blocks<false, 64, 64>(out, corner, ldc, rows - r0, cols - c0, alpha, beta);
}

template <typename Cfg, int WAVES>
hipError_t launch_direct(const DirectProblem& p, int slices, hipStream_t stream) {
    const int64_t tm = (p.M + Cfg::BM - 1) / Cfg::BM, tn = (p.N + Cfg::BN - 1) / Cfg::BN;
    if (!launch_fits(tm * tn, 256 * Cfg::KG)) return hipErrorInvalidValue;
    hipLaunchKernelGGL((gemm_direct_kernel<Cfg, WAVES>), dim3((unsigned)(tm * tn), (unsigned)slices), dim3(256 * Cfg::KG),
                       0, stream, p, (int)tm, (int)tn);
    return hipGetLastError();
}

}  // namespace

// K values per slice: whole stages.
static int64_t direct_slice(int64_t K, int slices) { return ((K + slices - 1) / slices + 31) / 32 * 32; }

// Expected times (us) of the direct form and of the image form, fitted to
// measurements on MI355X (bf16 / bf16x3, image form measured first, one call):
//   256^3 18.6 -> 7.1 / 22 -> 9.0       512^3 21 -> 8.8 / 24.6 -> 11.2
//   1024^3 31 -> 13 / 36 -> 17.6        2048^3 54 -> 38 / 84 -> 63
//   4096^3 144 -> 250 / 324 -> 460 (the image form stays)
//   300 x 4000 x 8191, bf16, called from a host program 94 -> 78
// The CU with the most tiles, n of them, takes n (fixed + t K) for 128 x 128
// tiles, which follow each other on a CU, and (n + c) t K for 64 x 64 tiles,
// four of which share it.
DirectPlan direct_plan(int64_t M, int64_t N, int64_t K, int64_t lda, int64_t ldb, int nterms, int image_splits,
                       size_t ws_bytes) {
    DirectPlan best;
    // 32-bit byte offsets inside a tile
    if (M <= 0 || N <= 0 || K <= 0 || lda >= (1ll << 23) || ldb >= (1ll << 25)) return best;
    const bool x3 = nterms == 3;
    const double mn = (double)M * (double)N, bytes_per_us = 5e6, launch = 2.5;
    const auto reduce = [&](double s) { return s > 1 ? launch + (s + 1) * mn * 4 / bytes_per_us : 0.0; };
    const double tiles256 = (double)(((M + 255) / 256) * ((N + 255) / 256));
    const double blocks = (double)((K + 31) / 32), rounds = ceil(tiles256 * image_splits / 256);
    const double image = launch + (double)(M + N) * (double)K * (x3 ? 8 : 6) / bytes_per_us +
                         rounds * ceil(blocks / image_splits) * (x3 ? kStepNsBf16x3 : kStepNsBf16) * 1e-3 + 11 +
                         reduce(image_splits);
    double least = image;
    for (int big = 0; big < 2; ++big) {
        const int64_t b = big ? 128 : 64;
        const int64_t count = ((M + b - 1) / b) * ((N + b - 1) / b);
        const double tiles = (double)count;
        if (!launch_fits(count, x3 ? 512 : 256)) continue;   // (more groups over K run only where tiles are few)
        for (int s = 1; s <= 16 && (s == 1 || (s * 256 <= K && (double)s * mn * 4 <= (double)ws_bytes)); ++s) {
            const int64_t slice = direct_slice(K, s);
            if (slice * (s - 1) >= K) continue;    // every slice non-empty
            const double n = ceil(tiles * s / 256), k = (double)slice;
            const double us = reduce(s) + (big ? (x3 ? 1.5 + n * (4 + 0.0275 * k) : 1.5 + n * (3 + 0.0148 * k))
                                               : (x3 ? 4 + (n + 0.64) * 0.0081 * k : 4 + (n + 0.87) * 0.0047 * k));
            if (us < least) {
                least = us;
                best = {big ? (n > 1 && !x3 ? 127 : 128) : x3 && tiles * s <= 256 ? 63 : 64, s};
            }
        }
    }
    return best;
}

hipError_t launch_gemm_bf16_direct(const DirectPlan& plan, int64_t M, int64_t N, int64_t K, int nterms, float alpha,
                                   const float* A, int64_t lda, const float* B, int64_t ldb, float beta, float* C,
                                   int64_t ldc, float* partial, hipStream_t stream) {
    if (plan.tile == 0 || plan.slices < 1 || (plan.slices > 1 && !partial) || M <= 0 || N <= 0 || K <= 0)
        return hipErrorInvalidValue;
    const int64_t slice = direct_slice(K, plan.slices);
    if (slice * (plan.slices - 1) >= K) return hipErrorInvalidValue;   // every slice non-empty
    const DirectProblem p{M, N, K, lda, ldb, ldc, alpha, beta, A, B, C, plan.slices > 1 ? partial : nullptr, slice};
    if (nterms == 3) {
        if (plan.tile == 128) return launch_direct<DirectCfg<128, 128, 3, 2>, 2>(p, plan.slices, stream);
        if (plan.tile == 64) return launch_direct<DirectCfg<64, 64, 3, 2>, 4>(p, plan.slices, stream);
        return launch_direct<DirectCfg<64, 64, 3, 4>, 4>(p, plan.slices, stream);
    }
    // several tiles per CU: 300 x 4000 x 8192 in 5 slices 52 us with one group (two
    // workgroups share a CU), 56 with two; one tile: 2048^3 41.7 and 38.1
    if (plan.tile == 127) return launch_direct<DirectCfg<128, 128, 1, 1>, 2>(p, plan.slices, stream);
    if (plan.tile == 128) return launch_direct<DirectCfg<128, 128, 1, 2>, 2>(p, plan.slices, stream);
    return launch_direct<DirectCfg<64, 64, 1, 1>, 4>(p, plan.slices, stream);
}

}  // namespace cmp
