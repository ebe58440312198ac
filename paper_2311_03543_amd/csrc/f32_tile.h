// FP32 GEMM tile on the FP32 matrix instructions, shared by the single-problem
// kernel and the grouped (batched) kernel: one workgroup of 4 waves (2 x 2)
// computes a BM x BN tile of C = alpha * A * B + beta * C, walking K in stages
// of BK.
//
// Arithmetic: v_mfma_f32_32x32x2 and v_mfma_f32_16x16x4 add their 2 or 4
// products one after the other, in increasing k, each with one rounding (FMA),
// subnormals kept: 2.6 M random, subnormal, infinite and NaN cases agreed bit
// for bit with a chain of fmaf.  Every output entry is therefore the chain of
// FP32 FMAs over k in increasing order, whatever the tile shape, so all
// configurations give bit-identical C.
//
// Rate: both instructions do 256 flop per cycle and CU, as the vector ALUs do
// on paper, but an operand value is read once for 16 or 32 products.  The
// vector form needed 230 registers of outer product per lane and stayed at
// 88-92 TFLOP/s; the matrix form leaves the vector ALU, the LDS and most of
// the registers free, so loads and fragment reads hide under it.  Registers
// only, 32x32x2 runs 143 / 153 / 155 TFLOP/s with 1 / 2 / 4 waves per SIMD and
// 16x16x4 runs 122 / 134 / 139; 16x16x4 takes half as long for twice the k, so
// a chain over K is four times shorter.
//
// Staging: NS ring slots in LDS, filled by global_load_lds with NS - 1 stages
// in flight (no registers held).  The lanes of a copy choose their global
// address freely, so the bank swizzle costs nothing:
//   A  BM rows of BK floats; the 16-byte chunk c of row r sits at position
//      c ^ ((r / RPB) % CPR), RPB rows filling the 64 banks once;
//   B  BK rows of BN floats; the chunk of a row is moved by a constant of
//      k % 4 so that the k values one MFMA reads lie in different banks.
// Aligned operands are copied 16 bytes a lane, others and the last, partial
// stage 4 bytes a lane; k >= K reads a zero word instead, -0 for A and +0 for
// B, whose product -0 leaves every sum as it is (+0 would turn a sum of -0 into
// +0, so that C depended on the stage depth); rows and columns past the edge
// repeat the last one (their products are never stored).
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>
#include <type_traits>

namespace cmp {

struct F32Problem {
    int64_t M, N, K, lda, ldb, ldc;
    float alpha, beta;
    const float* A;
    const float* B;
    float* C;
};

// Global-address-space views of the operand pointers: pointers that arrive
// through memory (the grouped descriptors) are generic to the compiler and
// would otherwise turn every access into a FLAT instruction.
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef const __attribute__((address_space(1))) float* gcfloat;
typedef __attribute__((address_space(1))) float* gfloat;

// MF_: the MFMA block (32: 32x32x2, 16: 16x16x4).  A wave owns MI x NJ blocks,
// block row i at (2 i + wave row) * MF: edge tiles then leave every wave
// about the same share of the blocks that lie inside C.
template <int BM_, int BN_, int BK_, int MF_, int NS_>
struct F32Cfg {
    static constexpr int BM = BM_, BN = BN_, BK = BK_, MF = MF_, NS = NS_;
    static constexpr int THREADS = 256;
    static constexpr int MI = BM / 2 / MF, NJ = BN / 2 / MF;   // blocks per wave
    static constexpr int KS = MF == 32 ? 2 : 4;                // k per MFMA
    static constexpr int CPR = BK / 4, CPB = BN / 4;           // chunks per row of A, of B
    static constexpr int RPB = 64 / BK;                        // rows of A per 64 banks
    // chunks of k per step of the main loop: at least 4 MFMAs, an even number of steps per stage
    static constexpr int CH = MF == 16 ? (MI * NJ >= 4 ? 1 : MI * NJ == 2 ? 2 : 4) : (MI * NJ >= 2 ? 1 : 2);
    static_assert((CPR / CH) % 2 == 0 && CPR % CH == 0, "two fragment buffers");
    static constexpr int QA = BM * BK / 4 / THREADS, QB = BK * BN / 4 / THREADS;   // 16-byte copies per lane
    static constexpr int ASZ = BM * BK, STAGE = ASZ + BK * BN;  // floats
    static constexpr int SMEM_FLOATS = NS * STAGE;
    static_assert(MF == 32 || MF == 16, "MFMA block");
    static_assert(MI >= 1 && NJ >= 1 && QA >= 1 && QB >= 1, "tile too small for 4 waves");
    static_assert(BM % (2 * MF) == 0 && BN % (2 * MF) == 0, "whole blocks per wave");
    static_assert(BK == 16 || BK == 32 || BK == 64, "rows of A fill the banks evenly");
    static_assert((MF / RPB) % CPR == 0, "the A swizzle is the same in every block row");
    static_assert(NS >= 2 && (NS - 2) * 4 * (QA + QB) <= 63, "vmcnt range");
    // chunk displacement of B row k (see above)
    __host__ __device__ static constexpr int swz_b(int k) {
        return MF == 32 ? (k & 1) * 8 : (BN >= 64 ? (k & 3) * 4 : ((k >> 1) & 1) * 4);
    }
    static_assert(BN >= (MF == 32 ? 64 : 32), "B rows hold the displaced chunks");
};

// The zero words of A and of B for the copies past the end of K.
static __device__ float f32_tile_zero[2] = {-0.f, 0.f};

template <int VM>
__device__ __forceinline__ void f32_stage_wait() {
    static_assert(VM >= 0 && VM <= 63, "vmcnt range");
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt((VM & 15) | ((VM >> 4) << 14) | (7 << 4) | (15 << 8));
    asm volatile("" ::: "memory");
}
__device__ __forceinline__ void f32_stage_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(15 | (3 << 14) | (7 << 4));   // lgkmcnt(0): own LDS reads done
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// The whole tile at (m0, n0): main loop and epilogue.  `smem` holds
// Cfg::SMEM_FLOATS floats, 256-byte aligned; it may be reused after a
// workgroup barrier.  vec: A and B allow 16-byte loads (16-byte aligned, lda
// and ldb multiples of 4).  alpha == 0 or K == 0 never reads A or B.
// before_stores() runs once between the two.
template <typename Cfg, class Hook>
__device__ __forceinline__ void f32_tile(const F32Problem& p, int64_t m0, int64_t n0, bool vec, float* smem,
                                         Hook&& before_stores) {
    constexpr int BK = Cfg::BK, BN = Cfg::BN, MF = Cfg::MF, NS = Cfg::NS, MI = Cfg::MI, NJ = Cfg::NJ;
    constexpr int QA = Cfg::QA, QB = Cfg::QB, CPR = Cfg::CPR, CPB = Cfg::CPB, CH = Cfg::CH;
    typedef const __attribute__((address_space(1))) void* gptr;
    typedef const __attribute__((address_space(1))) char* gcbyte;
    typedef __attribute__((address_space(3))) void* lptr;
    using Acc = std::conditional_t<MF == 32, f32x16, f32x4>;
    constexpr int AR = MF == 32 ? 16 : 4;          // accumulators per lane and block
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = wave >> 1, wn = wave & 1;

    Acc acc[MI][NJ];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int r = 0; r < AR; ++r) acc[i][j][r] = 0.f;

    const int rows = (int)(p.M - m0 < Cfg::BM ? p.M - m0 : Cfg::BM);
    const int cols = (int)(p.N - n0 < BN ? p.N - n0 : BN);
    const int64_t K = p.alpha == 0.f ? 0 : p.K;
    const int nst = (int)((K + BK - 1) / BK);
    const int whole = (int)(K / BK);               // stages without a K tail
    // 16-byte copies of B need whole chunks of every row
    const bool x4 = vec && (n0 + BN <= p.N || (p.N & 3) == 0);

    // Copy sources of whole stages: a uniform base that moves with k, and per
    // lane a constant byte offset.  16-byte form: copy q of a stage moves chunk
    // q * 256 + t of the slot; 4-byte form: word q * 256 + t (four times the
    // copies).  Leading dimensions whose offsets pass 32 bits (`far`) take the
    // per-lane addresses of the tail for every stage.
    const bool far = (int64_t)Cfg::BM * p.lda >= (1ll << 30) || (int64_t)BK * p.ldb >= (1ll << 30);
    const gcfloat a_base = (gcfloat)p.A + m0 * p.lda, b_base = (gcfloat)p.B + n0;
    uint32_t oa[4 * QA], ob[4 * QB];
    auto offsets = [&](auto x4_tag) {
        constexpr int UNIT = decltype(x4_tag)::value ? 4 : 1;
#pragma unroll
        for (int q = 0; q < 4 / UNIT * QA; ++q) {
            const int w = (q * 256 + t) * UNIT;    // word of the slot's A region
            const int r = w / BK, c = ((w / 4) % CPR) ^ ((r / Cfg::RPB) % CPR);
            const int row = r < rows ? r : rows - 1;
            oa[q] = ((uint32_t)row * (uint32_t)p.lda + 4 * c + w % 4) * 4u;
        }
#pragma unroll
        for (int q = 0; q < 4 / UNIT * QB; ++q) {
            const int w = (q * 256 + t) * UNIT;
            const int k = w / BN, c = ((w / 4) % CPB) ^ Cfg::swz_b(k);
            const int col = 4 * c + w % 4, last = cols - UNIT;
            ob[q] = ((uint32_t)k * (uint32_t)p.ldb + (col < last ? col : last)) * 4u;
        }
    };
    // copy m of stage s (whole): the QA (4 QA) copies of A, then those of B
    auto copy = [&](int s, int slot, int m, auto x4_tag) {
        constexpr int UNIT = decltype(x4_tag)::value ? 4 : 1, NA = 4 / UNIT * QA;
        float* dst = smem + slot * Cfg::STAGE + wave * 64 * UNIT;
        const int64_t k0 = (int64_t)s * BK;
        asm volatile("" : "+v"(m < NA ? oa[m < NA ? m : 0] : ob[m < NA ? 0 : m - NA]));   // keep it a 32-bit offset
        const gptr src = m < NA ? (gptr)((gcbyte)(a_base + k0) + oa[m < NA ? m : 0])
                                : (gptr)((gcbyte)(b_base + k0 * p.ldb) + ob[m < NA ? 0 : m - NA]);
        const lptr to = (lptr)(m < NA ? dst + m * 256 * UNIT : dst + Cfg::ASZ + (m - NA) * 256 * UNIT);
        if constexpr (UNIT == 4) __builtin_amdgcn_global_load_lds(src, to, 16, 0, 0);
        else __builtin_amdgcn_global_load_lds(src, to, 4, 0, 0);
    };
    // any stage: word by word with per-lane addresses, a zero word where k >= K
    auto copy_tail = [&](int s) {
        float* word = smem + (s % NS) * Cfg::STAGE + wave * 64;
        const int64_t k0 = (int64_t)s * BK;
        const int left = (int)(K - k0 < BK ? K - k0 : BK);
        const gcfloat zero_a = (gcfloat)f32_tile_zero, zero_b = zero_a + 1;
#pragma unroll 4
        for (int q = 0; q < 4 * QA; ++q) {
            const int w = q * 256 + t, r = w / BK;
            const int k = 4 * (((w / 4) % CPR) ^ ((r / Cfg::RPB) % CPR)) + w % 4;
            const gcfloat src = k < left ? a_base + (r < rows ? r : rows - 1) * p.lda + k0 + k : zero_a;
            __builtin_amdgcn_global_load_lds((gptr)src, (lptr)(word + q * 256), 4, 0, 0);
        }
#pragma unroll 4
        for (int q = 0; q < 4 * QB; ++q) {
            const int w = q * 256 + t, k = w / BN;
            const int col = 4 * (((w / 4) % CPB) ^ Cfg::swz_b(k)) + w % 4;
            const gcfloat src = k < left ? b_base + (k0 + k) * p.ldb + (col < cols ? col : cols - 1) : zero_b;
            __builtin_amdgcn_global_load_lds((gptr)src, (lptr)(word + Cfg::ASZ + q * 256), 4, 0, 0);
        }
    };

    // Fragments: lane l holds row (A) or column (B) l % MF of a block, k value
    // KS s + l / MF of MFMA s.
    const int fr = lane % MF, fk = lane / MF;
    const int a_lane = (wm * MF + fr) * BK + 4 * ((fr / Cfg::RPB) % CPR) + fk;
    const int b_lane = Cfg::ASZ + fk * BN + ((wn * MF + fr) ^ (4 * Cfg::swz_b(fk)));
    // fragments of one step: CH chunks, k values 4 CH c .. 4 CH c + 4 CH - 1 of a stage
    struct Frag {
        float a[4 * CH / Cfg::KS][MI], b[4 * CH / Cfg::KS][NJ];
    };
    auto read = [&](Frag& f, const float* slot, int c) {
#pragma unroll
        for (int u = 0; u < 4 * CH / Cfg::KS; ++u) {
            const int k = 4 * CH * c + u * Cfg::KS;
            const float* as = slot + (a_lane ^ (k & ~3)) + (k & 3);
#pragma unroll
            for (int i = 0; i < MI; ++i) f.a[u][i] = as[2 * i * MF * BK];
#pragma unroll
            for (int j = 0; j < NJ; ++j) f.b[u][j] = slot[(b_lane ^ (2 * j * MF)) + k * BN];
        }
    };
    constexpr int NM = 4 * CH / Cfg::KS * MI * NJ;      // MFMAs per step and wave
    auto mfma = [&](const Frag& f, int q, auto full_tag) {
        const int u = q / (MI * NJ), i = q / NJ % MI, j = q % NJ;
        if (!decltype(full_tag)::value && ((2 * i + wm) * MF >= rows || (2 * j + wn) * MF >= cols)) return;
        if constexpr (MF == 32)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(f.a[u][i], f.b[u][j], acc[i][j], 0, 0, 0);
        else
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(f.a[u][i], f.b[u][j], acc[i][j], 0, 0, 0);
    };
    auto pin = []() { __builtin_amdgcn_sched_barrier(0); };
    // Main loop.  Stage s: the copies of stage s + NS - 1 go out one by one
    // under its MFMAs, into the slot that the barrier at the end of stage s - 1
    // freed; a step's fragments are read under the MFMAs of the step before.
    // The steady loop runs while stage s + NS - 1 is a whole one, without a
    // branch but its own; the rest has at most the K tail left to copy.
    constexpr int STEPS = CPR / CH, PRE = NM / 2;  // PRE: MFMAs of the last step ahead of the stage barrier
    constexpr int NC4 = QA + QB, NC1 = 4 * NC4;    // copies per whole stage, 16-byte and 4-byte form
    Frag f[2];
    int s = 0, cur = 0, put = NS - 1;              // stage; slots of stage s and of stage s + NS - 1
    auto stage = [&](auto steady_tag, auto full_tag, auto x4_tag) {
        constexpr bool STEADY = decltype(steady_tag)::value;
        constexpr int NC = decltype(x4_tag)::value ? NC4 : NC1;
        // PER copies after every GAP-th MFMA: all of them ahead of the stage barrier, whose wait counts them
        constexpr int ROOM = (STEPS - 1) * NM + PRE;
        constexpr int PER = (NC + ROOM - 1) / ROOM, GAP = ROOM / ((NC + PER - 1) / PER);
        static_assert(GAP >= 1 && ((NC + PER - 1) / PER - 1) * GAP < ROOM, "copies precede the barrier");
        const float* slot = smem + cur * Cfg::STAGE;
        cur = cur + 1 == NS ? 0 : cur + 1;
        if (!STEADY && s + NS - 1 < nst) copy_tail(s + NS - 1);
#pragma unroll
        for (int c = 0; c < STEPS; ++c) {
            const Frag& g = f[c & 1];
            const int pre = c + 1 < STEPS ? 1 : PRE;
#pragma unroll
            for (int q = 0; q < NM; ++q) {
                if (q == pre) {
                    pin();
                    if (c + 1 < STEPS) {
                        read(f[(c + 1) & 1], slot, c + 1);
                    } else if (STEADY || s + 1 < nst) {
                        // stage s + 1 has landed (s + 2 .. s + NS - 1 may stay in flight)
                        // and every wave has read all of stage s
                        if (STEADY) f32_stage_wait<(NS - 2) * NC>();
                        else if (s + NS <= nst && x4) f32_stage_wait<(NS - 2) * NC4>();
                        else if (s + NS <= nst) f32_stage_wait<(NS - 2) * NC1>();
                        else f32_stage_wait<0>();
                        f32_stage_barrier();
                        read(f[0], smem + cur * Cfg::STAGE, 0);
                    }
                    pin();
                }
                mfma(g, q, full_tag);
                if (STEADY) {
                    const int at = c * NM + q;
#pragma unroll
                    for (int m = 0; m < PER; ++m)
                        if (at % GAP == 0 && at / GAP * PER + m < NC) copy(s + NS - 1, put, at / GAP * PER + m, x4_tag);
                    pin();
                }
            }
            pin();
        }
        put = put + 1 == NS ? 0 : put + 1;
    };
    auto steady = [&](auto full_tag, auto x4_tag) {
        for (; s + NS - 1 < whole; ++s) stage(std::true_type{}, full_tag, x4_tag);
    };
    // edge tiles skip the blocks outside C (a wave-uniform branch per MFMA)
    const bool full = MI * NJ == 1 || (rows == Cfg::BM && cols == BN);
    if (nst > 0) {
        if (x4) offsets(std::true_type{});
        else offsets(std::false_type{});
        for (int i = 0; i < NS - 1 && i < nst; ++i) {
            if (i >= whole || far) {
                copy_tail(i);
            } else if (x4) {
#pragma unroll
                for (int m = 0; m < NC4; ++m) copy(i, i, m, std::true_type{});
            } else {
#pragma unroll
                for (int m = 0; m < NC1; ++m) copy(i, i, m, std::false_type{});
            }
        }
        if (nst < NS - 1) f32_stage_wait<0>();
        else if (x4) f32_stage_wait<(NS - 2) * NC4>();
        else f32_stage_wait<(NS - 2) * NC1>();
        f32_stage_barrier();
        read(f[0], smem, 0);
        pin();
        if (!far) {
            if (x4) full ? steady(std::true_type{}, std::true_type{}) : steady(std::false_type{}, std::true_type{});
            else full ? steady(std::true_type{}, std::false_type{}) : steady(std::false_type{}, std::false_type{});
        }
        for (; s < nst; ++s)
            stage(std::false_type{}, std::integral_constant<bool, MI * NJ == 1>{}, std::true_type{});
    }

    before_stores();
    // Epilogue: C = alpha * acc + beta * C (C not read when beta == 0).  Lane l
    // holds column l % MF; rows 8 (r / 4) + 4 (l / 32) + r % 4 of a 32 x 32
    // block, 4 (l / 16) + r of a 16 x 16 one.  A block's old values are all
    // loaded before the first is used; interior tiles check no bounds.
    const int64_t ldc = p.ldc;
    const gfloat corner = (gfloat)p.C + (m0 + wm * MF + 4 * fk) * ldc + n0 + wn * MF + fr;
    auto finish = [&](auto full_tag, auto beta_tag) {
        constexpr bool FULL = decltype(full_tag)::value, BETA = decltype(beta_tag)::value;
        const int rl = rows - (wm * MF + 4 * fk), cl = cols - (wn * MF + fr);   // rows and columns from `corner` on
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                if (!FULL && 2 * j * MF >= cl) continue;
                const gfloat c = corner + (2 * i * MF * ldc + 2 * j * MF);
                float old[AR];
                if (BETA) {
#pragma unroll
                    for (int r = 0; r < AR; ++r) {
                        const int dr = (r >> 2) * 8 + (r & 3);
                        old[r] = FULL || 2 * i * MF + dr < rl ? c[dr * ldc] : 0.f;
                    }
                }
#pragma unroll
                for (int r = 0; r < AR; ++r) {
                    const int dr = (r >> 2) * 8 + (r & 3);
                    if (FULL || 2 * i * MF + dr < rl) {
                        float v = p.alpha * acc[i][j][r];
                        if (BETA) v = __builtin_fmaf(p.beta, old[r], v);
                        c[dr * ldc] = v;
                    }
                }
            }
    };
    const bool whole_tile = rows == Cfg::BM && cols == BN;
    if (p.beta != 0.f) whole_tile ? finish(std::true_type{}, std::true_type{}) : finish(std::false_type{}, std::true_type{});
    else whole_tile ? finish(std::true_type{}, std::false_type{}) : finish(std::false_type{}, std::false_type{});
}

}  // namespace cmp
