// The fp8 product with refinement over smaller tiles than the 256 x 256 ones of
// gemm_mfma.hip, for shapes that leave CUs idle there: the same operand images,
// products and order of MFMAs per accumulator, so a tile whose K range is not
// divided gives the same bits.
//
// A group of W = WM x WN waves computes a BM x BN tile over a run of K blocks
// (64 bytes of K each), KG groups share the workgroup and add their sums in
// LDS.  A stage is one K block of the four images [Aq | Bq | Ar | Br], copied
// by global_load_lds into a ring of NS slots (a tile's rows of a panel block are
// contiguous); a wave's fragments are read one stage ahead of their MFMAs, one or
// two reads and a copy under each MFMA (left to the scheduler, which put every
// copy first and waited for the scale bytes mid-stage: 256 x 128 tiles 4 - 9 %
// slower on zeros).  Small tiles are bound by the latency of their few stages,
// large ones by power: 3000 x 2500 x 4100 takes 90 us on zeros, 108 on random
// codes.
#include <atomic>
#include <cmath>
#include <type_traits>

#include "common.h"
#include "kernels.h"
#include "mfma_tile.h"

namespace cmp {
namespace {

typedef int intx8 __attribute__((ext_vector_type(8)));
typedef int intx4 __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(1))) uint8_t* gbytes;
typedef const __attribute__((address_space(1))) void* gptr_t;
typedef __attribute__((address_space(3))) void* lptr_t;
typedef __attribute__((address_space(1))) float* gfloat;

struct Fp8Problem {
    int64_t M, N, ldc;
    float alpha, beta;
    const uint8_t* img[4];     // Aq, Bq, Ar, Br panel images
    const uint8_t* scale[4];   // E8M0 bytes of their 128 x 128 tiles
    float* C;
    float* partial;            // != nullptr: slice y writes raw sums to partial + y M N (pitch N)
    int nkb, kb_split;         // K blocks in all, and per slice
};

template <int BM_, int BN_, int WM_, int WN_, int KG_, int NS_>
struct Fp8Cfg {
    static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, KG = KG_, NS = NS_;
    static constexpr int W = WM * WN, THREADS = 64 * W;          // waves and lanes of a group
    static constexpr int MI = BM / 32 / WM, NJ = BN / 32 / WN;   // 32 x 32 blocks per wave
    static constexpr int SA = BM * 64, SB = BN * 64, STAGE = 2 * (SA + SB);
    static constexpr int COPIES = STAGE / 1024 / W;              // 1 KiB copies per wave and stage
    static constexpr int PER = (SA > SB ? SA : SB) / 1024 / W;   // of them, for one image
    static constexpr int ACC = MI * NJ * 64 * THREADS;           // bytes of one group's accumulators
    static constexpr int SMEM = KG * (NS * STAGE > ACC || KG == 1 ? NS * STAGE : ACC);
    static_assert(256 % BM == 0 && 256 % BN == 0, "a tile lies in one panel");
    static_assert(128 % (32 * MI) == 0 && 128 % (32 * NJ) == 0, "a wave's rows and columns have one scale each");
    static_assert(SA / 1024 % W == 0 && SB / 1024 % W == 0, "whole copies per wave and image");
    static_assert(NS >= 2 && (NS - 1) * COPIES <= 63, "vmcnt range");
    static_assert(SMEM <= 160 * 1024, "LDS");
};

template <typename Cfg>
__global__ __launch_bounds__(Cfg::THREADS * Cfg::KG) __attribute__((amdgpu_waves_per_eu(Cfg::W * Cfg::KG / 4)))
void gemm_fp8r_tile_kernel(Fp8Problem p, int tiles_m, int tiles_n) {
    constexpr int BM = Cfg::BM, BN = Cfg::BN, W = Cfg::W, MI = Cfg::MI, NJ = Cfg::NJ, KG = Cfg::KG, NS = Cfg::NS;
    constexpr int COPIES = Cfg::COPIES, SA = Cfg::SA, SB = Cfg::SB, STAGE = Cfg::STAGE;
    extern __shared__ __attribute__((aligned(256))) uint8_t lds[];
    int tm, tn;
    grouped_tile(xcd_remap(blockIdx.x, tiles_m * tiles_n), tiles_m, tiles_n, 8, tm, tn);
    const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;
    const int t = threadIdx.x % Cfg::THREADS, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int group = KG == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / Cfg::THREADS);
    const int wm = wave / Cfg::WN, wn = wave % Cfg::WN;
    uint8_t* ring = lds + group * NS * STAGE;
    // K blocks of this workgroup (slice blockIdx.y), then of this group
    const int kb0 = (int)blockIdx.y * p.kb_split;
    const int all = p.nkb - kb0 < p.kb_split ? p.nkb - kb0 : p.kb_split;
    const int first = kb0 + all * group / KG, nst = kb0 + all * (group + 1) / KG - first;
    const int most = (all + KG - 1) / KG;

    // Sources of the copies: a tile's rows of image X start at src[X] in each panel block
    const int64_t panel = (int64_t)p.nkb * kPanelBlock;
    gbytes src[4];
#pragma unroll
    for (int x = 0; x < 4; ++x) {
        const int64_t r0 = x & 1 ? n0 : m0;
        src[x] = (gbytes)p.img[x] + (r0 / kPanelRows) * panel + (r0 % kPanelRows) * 64 + wave * 1024;
    }
    uint32_t from[Cfg::PER];                       // byte offsets of copy q of an image
#pragma unroll
    for (int q = 0; q < Cfg::PER; ++q) from[q] = lane * 16 + q * W * 1024;
    int ld_s = 0, ld_slot = 0;                     // the copies' stage (past the last: the last again) and slot
    int64_t ld_off = 0;
    uint8_t* ld_dst = nullptr;
    auto prepare = [&]() __attribute__((always_inline)) {
        const int kb = first + (ld_s < nst ? ld_s : nst - 1);
        ld_off = (int64_t)(kb < 0 ? 0 : kb) * kPanelBlock;
        ld_dst = ring + ld_slot * STAGE + wave * 1024;
        ++ld_s;
        ld_slot = ld_slot + 1 == NS ? 0 : ld_slot + 1;
    };
    auto copy = [&](auto n_tag) __attribute__((always_inline)) {  // copy n of the prepared stage
        constexpr int n = decltype(n_tag)::value, NA = SA / 1024 / W, NB = SB / 1024 / W;
        constexpr int level = n / (NA + NB), m = n % (NA + NB), x = 2 * level + (m >= NA), q = m >= NA ? m - NA : m;
        constexpr int at = level * (SA + SB) + (m >= NA ? SA : 0) + q * W * 1024;
        asm volatile("" : "+v"(from[q]));          // a uniform base plus a 32-bit offset
        __builtin_amdgcn_global_load_lds((gptr_t)(src[x] + ld_off + from[q]), (lptr_t)(ld_dst + at), 16, 0, 0);
    };

    // Scales: bytes of this wave's 128-row tiles of A and B, one per 128 k; the
    // words are loaded a stage before they are unpacked
    const int nkt = p.nkb / 2;
    const int64_t sa0 = (m0 + wm * 32 * MI) / 128 * nkt, sb0 = (n0 + wn * 32 * NJ) / 128 * nkt;
    typedef const __attribute__((address_space(4))) uint32_t* cword;
    uint32_t word[4];
    int shift_a = 0, shift_b = 0, sc_s = 0;
    auto load_words = [&]() __attribute__((always_inline)) {
        const int kb = first + (sc_s < nst ? sc_s : nst - 1), kt = (kb < 0 ? 0 : kb) >> 1;
        const int64_t ia = sa0 + kt, ib = sb0 + kt;
#pragma unroll
        for (int x = 0; x < 4; ++x) word[x] = *(cword)(p.scale[x] + ((x & 1 ? ib : ia) & ~(int64_t)3));
        shift_a = (int)(ia & 3) * 8;
        shift_b = (int)(ib & 3) * 8;
        ++sc_s;
    };
    struct Frag {
        intx4 a[2][MI][2], b[2][NJ][2];           // [level][block][half of a lane's 32 bytes]
        int sa[2], sb[2];
    };
    auto unpack = [&](Frag& f) __attribute__((always_inline)) {
#pragma unroll
        for (int l = 0; l < 2; ++l) {
            f.sa[l] = (int)(word[2 * l] >> shift_a & 0xffu);
            f.sb[l] = (int)(word[2 * l + 1] >> shift_b & 0xffu);
        }
    };
    // lane l feeds row l % 32 of a block, bytes 32 (l / 32) .. + 31 of the K block
    const int fr = lane & 31, fc = (lane >> 5) * 2;
    int fa[2], fb[2];                             // byte offsets of a lane's halves in block 0
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        fa[h] = slab_off(wm * 32 * MI + fr, fc + h);
        fb[h] = SA + slab_off(wn * 32 * NJ + fr, fc + h);
    }
    const uint8_t* rd = ring;                     // the slot being read
    int rd_slot = 0;
    constexpr int NR = 4 * (MI + NJ), NM = 4 * MI * NJ;
    auto read = [&](Frag& f, auto n_tag) __attribute__((always_inline)) {        // fragment read n of a stage
        constexpr int n = decltype(n_tag)::value, level = n / (NR / 2), m = n % (NR / 2);
        constexpr int h = m & 1, blk = m / 2;
        const uint8_t* st = rd + level * (SA + SB);
        if constexpr (blk < MI) f.a[level][blk][h] = *reinterpret_cast<const intx4*>(st + fa[h] + blk * 2048);
        else f.b[level][blk - MI][h] = *reinterpret_cast<const intx4*>(st + fb[h] + (blk - MI) * 2048);
    };
    auto next_slot = [&]() __attribute__((always_inline)) {
        rd_slot = rd_slot + 1 == NS ? 0 : rd_slot + 1;
        rd = ring + rd_slot * STAGE;
    };
    floatx16 acc[MI][NJ];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    auto mfma = [&](const Frag& f, auto n_tag) __attribute__((always_inline)) {  // q.q, q.r, r.q, r.r
        constexpr int n = decltype(n_tag)::value, u = n / (MI * NJ), i = n / NJ % MI, j = n % NJ, la = u >> 1, lb = u & 1;
        const intx8 av = __builtin_shufflevector(f.a[la][i][0], f.a[la][i][1], 0, 1, 2, 3, 4, 5, 6, 7);
        const intx8 bv = __builtin_shufflevector(f.b[lb][j][0], f.b[lb][j][1], 0, 1, 2, 3, 4, 5, 6, 7);
        acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(av, bv, acc[i][j], 0, 0, 0, f.sa[la], 0, f.sb[lb]);
    };

    Frag f[2];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        prepare();
        static_for<0, COPIES>(copy);
    }
    load_words();
    unpack(f[0]);
    load_words();
    stage_barrier<(NS - 1) * COPIES>();
    static_for<0, NR>([&](auto n) { read(f[0], n); });
    // Stage s: stage s + 1 has landed (NS - 2 younger ones may be in flight) and
    // slot s % NS has been read by every wave; under the MFMAs of stage s its slot
    // is refilled and the fragments of stage s + 1 are read
    auto step = [&](const Frag& now, Frag& then) __attribute__((always_inline)) {
        stage_barrier<(NS - 2) * COPIES>();
        prepare();
        next_slot();
        unpack(then);
        load_words();
        sched_pin();
        static_for<0, NM>([&](auto n_tag) __attribute__((always_inline)) {
            constexpr int n = decltype(n_tag)::value;
            mfma(now, n_tag);
            static_for<n * NR / NM, (n + 1) * NR / NM>([&](auto r) { read(then, r); });
            static_for<n * COPIES / NM, (n + 1) * COPIES / NM>(copy);
            sched_pin();
        });
    };
    int s = 1;
    for (; s + 2 <= most; s += 2) {
        step(f[0], f[1]);
        step(f[1], f[0]);
    }
    if (s < most) {
        step(f[0], f[1]);
        if (nst == most) static_for<0, NM>([&](auto n) { mfma(f[1], n); });
    } else if (nst == most) {
        static_for<0, NM>([&](auto n) { mfma(f[0], n); });
    }
    __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 0));                // the trailing copies and reads
    if (KG > 1) __syncthreads();
    float out[MI][NJ][16 / KG];
    sum_groups<KG, Cfg::THREADS>(acc, out, lds, group, t);

    const bool part = p.partial != nullptr;
    const int64_t ldc = part ? p.N : p.ldc;
    const float alpha = part ? 1.f : p.alpha, beta = part ? 0.f : p.beta;
    const int r0 = wm * 32 * MI + 4 * (lane >> 5) + group * (32 / KG), c0 = wn * 32 * NJ + fr;
    const gfloat corner = (part ? (gfloat)p.partial + (int64_t)blockIdx.y * p.M * p.N : (gfloat)p.C) + (m0 + r0) * ldc + n0 + c0;
    const int64_t rl = p.M - m0 - r0, cl = p.N - n0 - c0;
    if (p.M - m0 >= BM && p.N - n0 >= BN) store_blocks<true, 32, 32>(out, corner, ldc, 0, 0, alpha, beta);
    else store_blocks<false, 32, 32>(out, corner, ldc, rl < BM ? (int)rl : BM, cl < BN ? (int)cl : BN, alpha, beta);
}

template <typename Cfg>
hipError_t launch_tiles(const Fp8Problem& p, int slices, hipStream_t stream) {
    const int64_t tm = (p.M + Cfg::BM - 1) / Cfg::BM, tn = (p.N + Cfg::BN - 1) / Cfg::BN;
    if (!launch_fits(tm * tn, Cfg::THREADS * Cfg::KG)) return hipErrorInvalidValue;
    static std::atomic<uint64_t> ready{0};
    if (hipError_t e = allow_lds(gemm_fp8r_tile_kernel<Cfg>, ready, Cfg::SMEM)) return e;
    hipLaunchKernelGGL(gemm_fp8r_tile_kernel<Cfg>, dim3((unsigned)(tm * tn), (unsigned)slices),
                       dim3(Cfg::THREADS * Cfg::KG), Cfg::SMEM, stream, p, (int)tm, (int)tn);
    return hipGetLastError();
}

int slice_blocks(int nkb, int slices) { return (nkb + slices - 1) / slices; }

}  // namespace

// Expected times (us), fitted to measurements on MI355X (normal operands; 256 x
// 256 tiles with their split-K reduction first):
//   256^3 23 -> 6.3     512^3 24 -> 7.4          700 x 900 x 1300 34 -> 11.5
//   1024^3 30 -> 10.6   1536^3 38 -> 21          2048^3 54 -> 36
//   2000^2 x 200 48 -> 12.3                      300 x 4000 x 8191 67 -> 55
//   3000 x 2500 x 4100 120 -> 98                 6000^3 690 -> 640
//   4096^3 172 -> 181, 8192^3 1340 -> 1450 (the 256 x 256 tiles stay: their
//   traffic is least and their rounds are full)
// 64 x 64 tiles pay off up to 2048^3 or so; five of their workgroups share a CU,
// so only half of a started round counts, and with more than two per CU dividing
// a workgroup's K range stops paying (2048^3: 39.6 us with two groups, 37.4 with
// one; 700 x 900 x 1300: 11.5 and 13.9).  128 x 128 tiles measured between the
// other two (2048^3 38.5, 4096^3 210) and are left out.
Fp8rPlan fp8r_plan(int64_t M, int64_t N, int64_t Kp, int image_splits) {
    const int nkb = (int)(Kp / kPanelRowBytes);
    const double mn = (double)M * (double)N, bytes_per_us = 5e6;
    const auto reduce = [&](int s) { return s > 1 ? 2.5 + (s + 1) * mn * 4 / bytes_per_us : 0.0; };
    const auto tiles = [&](int bm, int bn) { return (double)((M + bm - 1) / bm) * (double)((N + bn - 1) / bn); };
    Fp8rPlan best;
    double least = 15 + ceil(tiles(256, 256) * image_splits / 256) *
                            (double)slice_blocks(nkb, image_splits) * kStepNsFp8r * 1e-3 + reduce(image_splits);
    const auto offer = [&](int tile, int s, double us) {
        if (us < least && (tile == 256 ? launch_fits((int64_t)tiles(256, 128), 512) : launch_fits((int64_t)tiles(64, 64), 256)))
            least = us, best = {tile, s};
    };
    for (int s = 1; s <= image_splits; ++s) {
        const double kb = slice_blocks(nkb, s);
        if (kb * (s - 1) >= nkb) continue;         // every slice non-empty
        const double n64 = tiles(64, 64) * s / 256;
        offer(n64 > 2 ? 63 : 64, s, 5 + (n64 <= 1 ? 1 : (n64 + ceil(n64)) / 2) * (0.24 * kb + 0.9) + reduce(s));
        offer(256, s, 5 + ceil(tiles(256, 128) * s / 256) * (1.31 * kb + 6) + reduce(s));
    }
    return best;
}

hipError_t launch_gemm_fp8r_tiles(const Fp8rPlan& plan, int64_t M, int64_t N, int64_t Kp, float alpha, const uint8_t* Aq,
                                  const uint8_t* Ar, const uint8_t* Asq, const uint8_t* Asr, const uint8_t* Bq,
                                  const uint8_t* Br, const uint8_t* Bsq, const uint8_t* Bsr, float beta, float* C,
                                  int64_t ldc, float* partial, hipStream_t stream) {
    if (Kp % kFp8TileK || Kp <= 0 || M <= 0 || N <= 0 || plan.slices < 1 || (plan.slices > 1 && !partial))
        return hipErrorInvalidValue;
    const int nkb = (int)(Kp / kPanelRowBytes), kbs = slice_blocks(nkb, plan.slices);
    if ((int64_t)(plan.slices - 1) * kbs >= nkb) return hipErrorInvalidValue;   // every slice non-empty
    const Fp8Problem p{M, N, ldc, alpha, beta, {Aq, Bq, Ar, Br}, {Asq, Bsq, Asr, Bsr}, C,
                       plan.slices > 1 ? partial : nullptr, nkb, kbs};
    switch (plan.tile) {
        case 256: return launch_tiles<Fp8Cfg<256, 128, 4, 2, 1, 3>>(p, plan.slices, stream);
        case 64: return launch_tiles<Fp8Cfg<64, 64, 2, 2, 2, 2>>(p, plan.slices, stream);
        case 63: return launch_tiles<Fp8Cfg<64, 64, 2, 2, 1, 2>>(p, plan.slices, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace cmp
