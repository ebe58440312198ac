// The MX FP6 product over 64 x 64 and 128 x 128 tiles, for shapes that leave CUs
// idle with the 256 x 256 ones of gemm_mfma.hip: the same images, products and
// order of MFMAs per accumulator, so a tile whose K range is not divided gives
// the same bits.
//
// A group of 4 waves (2 x 2) computes a tile over a run of K blocks (64 values),
// KG groups share the workgroup and add their sums in LDS.  A stage is one K
// block: the codes [Ah | Bh | Al | Bl], wave w copying image w's rows (contiguous
// in a panel block), and the scale bytes, 256 bytes a wave.  A ring of NS slots;
// fragments are read one stage ahead of their MFMAs.
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
typedef int intx2 __attribute__((ext_vector_type(2)));
typedef const __attribute__((address_space(1))) uint8_t* gbytes;
typedef const __attribute__((address_space(1))) void* gptr_t;
typedef __attribute__((address_space(3))) void* lptr_t;
typedef __attribute__((address_space(1))) float* gfloat;

struct Fp6Problem {
    int64_t M, N, ldc;
    float alpha, beta;
    const uint8_t* img[4];     // Ah, Bh, Al, Bl code images
    const uint8_t* scale[2];   // scale blocks of A, B
    float* C;
    float* partial;            // != nullptr: slice y writes raw sums to partial + y M N (pitch N)
    int nkb, kb_split;         // K blocks in all, and per slice
};

template <int B_, int KG_, int NS_>
struct Fp6Cfg {
    static constexpr int B = B_, KG = KG_, NS = NS_;             // tile rows and columns
    static constexpr int MI = B / 64;                            // 32 x 32 blocks of a wave, each way
    static constexpr int IMG = B * kMx6RowBytes;                 // bytes of one image's rows
    static constexpr int STAGE = 4 * IMG + 1024;                 // codes, then 4 x 256 bytes of scales
    static constexpr int PIECES = B * 8 / 256;                   // 256-byte pieces of A's and B's scales
    static constexpr int COPIES = IMG / 1024 + 1;                // per wave and stage
    static constexpr int ACC = MI * MI * 64 * 256;               // bytes of one group's accumulators
    static constexpr int SMEM = KG * (NS * STAGE > ACC || KG == 1 ? NS * STAGE : ACC);
    static_assert(B == 64 || B == 128, "tile");
    static_assert(NS >= 2 && (NS - 1) * COPIES <= 63, "vmcnt range");
};

template <typename Cfg>
__global__ __launch_bounds__(256 * Cfg::KG) __attribute__((amdgpu_waves_per_eu(Cfg::KG)))
void gemm_fp6x3_tile_kernel(Fp6Problem p, int tiles_m, int tiles_n) {
    constexpr int B = Cfg::B, MI = Cfg::MI, KG = Cfg::KG, NS = Cfg::NS, IMG = Cfg::IMG, STAGE = Cfg::STAGE;
    constexpr int COPIES = Cfg::COPIES;
    extern __shared__ __attribute__((aligned(256))) uint8_t lds[];
    int tm, tn;
    grouped_tile(xcd_remap(blockIdx.x, tiles_m * tiles_n), tiles_m, tiles_n, 8, tm, tn);
    const int64_t m0 = (int64_t)tm * B, n0 = (int64_t)tn * B;
    const int t = threadIdx.x & 255, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int group = KG == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
    const int wm = wave >> 1, wn = wave & 1;
    uint8_t* ring = lds + group * NS * STAGE;
    // K blocks of this workgroup (slice blockIdx.y), then of this group
    const int kb0 = (int)blockIdx.y * p.kb_split;
    const int all = p.nkb - kb0 < p.kb_split ? p.nkb - kb0 : p.kb_split;
    const int first = kb0 + all * group / KG, nst = kb0 + all * (group + 1) / KG - first;
    const int most = (all + KG - 1) / KG;

    // This wave's sources: image `wave` (even: A's rows), and a piece of the scales
    const int64_t r0 = wave & 1 ? n0 : m0;
    const gbytes codes = (gbytes)p.img[wave] + r0 / kPanelRows * p.nkb * kMx6Block + r0 % kPanelRows * kMx6RowBytes;
    const int piece = wave % Cfg::PIECES, side = piece / (Cfg::PIECES / 2);
    const int64_t s0 = side ? n0 : m0;
    const gbytes scales = (gbytes)p.scale[side] + s0 / kPanelRows * p.nkb * kMx6ScaleBlock + s0 % kPanelRows * 4 +
                          piece % (Cfg::PIECES / 2) * 256;
    uint32_t from[COPIES];                         // byte offsets of the copies
#pragma unroll
    for (int q = 0; q < COPIES; ++q) from[q] = q == COPIES - 1 ? lane * 4 : lane * 16 + q * 1024;
    int ld_s = 0, ld_slot = 0;                     // the copies' stage (past the last: the last again) and slot
    int ld_kb = 0;
    uint8_t* ld_dst = nullptr;
    auto prepare = [&]() __attribute__((always_inline)) {
        const int kb = first + (ld_s < nst ? ld_s : nst - 1);
        ld_kb = kb < 0 ? 0 : kb;
        ld_dst = ring + ld_slot * STAGE;
        ++ld_s;
        ld_slot = ld_slot + 1 == NS ? 0 : ld_slot + 1;
    };
    auto copy = [&](auto n_tag) __attribute__((always_inline)) {
        constexpr int n = decltype(n_tag)::value;
        asm volatile("" : "+v"(from[n]));          // a uniform base plus a 32-bit offset
        if constexpr (n == COPIES - 1)
            __builtin_amdgcn_global_load_lds((gptr_t)(scales + (int64_t)ld_kb * kMx6ScaleBlock + from[n]),
                                             (lptr_t)(ld_dst + 4 * IMG + wave * 256), 4, 0, 0);
        else
            __builtin_amdgcn_global_load_lds((gptr_t)(codes + (int64_t)ld_kb * kMx6Block + from[n]),
                                             (lptr_t)(ld_dst + wave * IMG + n * 1024), 16, 0, 0);
    };

    // fragments of two stages, [buffer][image or side][block]: a lane's code bytes
    // 0-15 and 16-23, and the scales of both levels
    intx4 c4[2][4][MI];
    intx2 c2[2][4][MI];
    int sc[2][2][MI];
    // lane l feeds row l % 32 of a block, K half l / 32
    const int row[2] = {wm * 32 * MI + (lane & 31), wn * 32 * MI + (lane & 31)}, half = lane >> 5;
    const uint8_t* rd = ring;                      // the slot being read
    int rd_slot = 0;
    constexpr int NR = 10 * MI, NM = 3 * MI * MI;
    auto read = [&](auto buf_tag, auto n_tag) __attribute__((always_inline)) {   // fragment read n of a stage
        constexpr int f = decltype(buf_tag)::value, n = decltype(n_tag)::value;
        if constexpr (n < 2 * MI) {
            constexpr int sd = n / MI, b = n % MI;
            sc[f][sd][b] = *reinterpret_cast<const uint16_t*>(rd + 4 * IMG + sd * (Cfg::PIECES / 2) * 256 +
                                                            4 * (row[sd] + 32 * b) + 2 * half);
        } else {
            constexpr int x = (n - 2 * MI) / (2 * MI), b = (n - 2 * MI) / 2 % MI;
            const uint8_t* at = rd + x * IMG + (row[x & 1] + 32 * b) * kMx6RowBytes;
            if constexpr (n % 2 == 0) c4[f][x][b] = *reinterpret_cast<const intx4*>(at + 16 * half);
            else c2[f][x][b] = *reinterpret_cast<const intx2*>(at + 32 + 8 * half);
        }
    };
    auto next_slot = [&]() __attribute__((always_inline)) {
        rd_slot = rd_slot + 1 == NS ? 0 : rd_slot + 1;
        rd = ring + rd_slot * STAGE;
    };
    floatx16 acc[MI][MI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < MI; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    auto mfma = [&](auto buf_tag, auto n_tag) __attribute__((always_inline)) {   // h.h, h.l, l.h
        constexpr int f = decltype(buf_tag)::value, n = decltype(n_tag)::value;
        constexpr int u = n / (MI * MI), i = n / MI % MI, j = n % MI, xa = u == 2 ? 2 : 0, xb = u == 1 ? 3 : 1;
        const intx8 av = __builtin_shufflevector(
            c4[f][xa][i], __builtin_shufflevector(c2[f][xa][i], c2[f][xa][i], 0, 1, 0, 1), 0, 1, 2, 3, 4, 5, 6, 7);
        const intx8 bv = __builtin_shufflevector(
            c4[f][xb][j], __builtin_shufflevector(c2[f][xb][j], c2[f][xb][j], 0, 1, 0, 1), 0, 1, 2, 3, 4, 5, 6, 7);
        // operand format 2 = FP6 E2M3 for both (dwords 0-5 used); scale byte 0 high, 1 low level
        acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(av, bv, acc[i][j], 2, 2, u == 2 ? 1 : 0, sc[f][0][i],
                                                                    u == 1 ? 1 : 0, sc[f][1][j]);
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;

#pragma unroll
    for (int s = 0; s < NS; ++s) {
        prepare();
        static_for<0, COPIES>(copy);
    }
    stage_barrier<(NS - 1) * COPIES>();
    static_for<0, NR>([&](auto n) __attribute__((always_inline)) { read(I0{}, n); });
    // Stage s: stage s + 1 has landed (NS - 2 younger ones may be in flight) and
    // slot s % NS has been read by every wave; under the MFMAs of stage s its slot
    // is refilled and the fragments of stage s + 1 are read
    auto step = [&](auto now, auto then) __attribute__((always_inline)) {
        stage_barrier<(NS - 2) * COPIES>();
        prepare();
        next_slot();
        sched_pin();
        static_for<0, NM>([&](auto n_tag) __attribute__((always_inline)) {
            constexpr int n = decltype(n_tag)::value;
            mfma(now, n_tag);
            static_for<n * NR / NM, (n + 1) * NR / NM>([&](auto r) __attribute__((always_inline)) { read(then, r); });
            static_for<n * COPIES / NM, (n + 1) * COPIES / NM>(copy);
            sched_pin();
        });
    };
    int s = 1;
    for (; s + 2 <= most; s += 2) {
        step(I0{}, I1{});
        step(I1{}, I0{});
    }
    if (s < most) {
        step(I0{}, I1{});
        if (nst == most) static_for<0, NM>([&](auto n) __attribute__((always_inline)) { mfma(I1{}, n); });
    } else if (nst == most) {
        static_for<0, NM>([&](auto n) __attribute__((always_inline)) { mfma(I0{}, n); });
    }
    __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 0));                // the trailing copies and reads
    if (KG > 1) __syncthreads();
    float out[MI][MI][16 / KG];
    sum_groups<KG, 256>(acc, out, lds, group, t);

    const bool part = p.partial != nullptr;
    const int64_t ldc = part ? p.N : p.ldc;
    const float alpha = part ? 1.f : p.alpha, beta = part ? 0.f : p.beta;
    const int rr = wm * 32 * MI + 4 * half + group * (32 / KG), cc = row[1];
    const gfloat corner = (part ? (gfloat)p.partial + (int64_t)blockIdx.y * p.M * p.N : (gfloat)p.C) + (m0 + rr) * ldc + n0 + cc;
    const int64_t rl = p.M - m0 - rr, cl = p.N - n0 - cc;
    if (p.M - m0 >= B && p.N - n0 >= B) store_blocks<true, 32, 32>(out, corner, ldc, 0, 0, alpha, beta);
    else store_blocks<false, 32, 32>(out, corner, ldc, rl < B ? (int)rl : B, cl < B ? (int)cl : B, alpha, beta);
}

template <typename Cfg>
hipError_t launch_tiles(const Fp6Problem& p, int slices, hipStream_t stream) {
    const int64_t tm = (p.M + Cfg::B - 1) / Cfg::B, tn = (p.N + Cfg::B - 1) / Cfg::B;
    if (!launch_fits(tm * tn, 256 * Cfg::KG)) return hipErrorInvalidValue;
    static std::atomic<uint64_t> ready{0};
    if (hipError_t e = allow_lds(gemm_fp6x3_tile_kernel<Cfg>, ready, Cfg::SMEM)) return e;
    hipLaunchKernelGGL(gemm_fp6x3_tile_kernel<Cfg>, dim3((unsigned)(tm * tn), (unsigned)slices), dim3(256 * Cfg::KG),
                       Cfg::SMEM, stream, p, (int)tm, (int)tn);
    return hipGetLastError();
}

int slice_blocks(int nkb, int slices) { return (nkb + slices - 1) / slices; }

}  // namespace

// Expected times (us), fitted to measurements on MI355X with random codes (256 x
// 256 tiles with their split-K reduction first):
//   256^3 18.3 -> 6.2    512^2 x 1000 17.3 -> 7.8    700 x 900 x 1300 27 -> 9.8
//   1024^3 25 -> 9.1     1536^3 30 -> 15.4           2048^3 43.5 -> 23.6
//   300 x 4000 x 8191 51 -> 41                       2000^2 x 200 44 -> 12
//   3000 x 2500 x 4100 86.5 -> 69
//   4096^3 119 -> 123 (the 256 x 256 tiles stay)
// Few stages: latency bounds small tiles; four or five workgroups of 64 x 64
// tiles share a CU, so only half of a started round counts, and K is divided
// between two groups of waves only while there is one (128 x 100 x 2000: 9.8 us,
// undivided 11.5; 2048^3 29.9 and 28.5).  128 x 128 tiles end together, so their
// stores are not hidden (2000^2 x 200: 17.4 us, 64 x 64 tiles 12); their third ring
// slot saves a wait for HBM (300 x 4000 x 8191: 81 -> 49 us).  The 256 x 256 tiles'
// 1.25 us per K block is the fit over these shapes (kStepNsFp6x3 is 8192^3).
Fp6x3Plan fp6x3_plan(int64_t M, int64_t N, int64_t Kp, int image_splits) {
    const int nkb = (int)(Kp / 64);
    const double mn = (double)M * (double)N, bytes_per_us = 5e6;
    const auto reduce = [&](int s) { return s > 1 ? 2.5 + (s + 1) * mn * 4 / bytes_per_us : 0.0; };
    const auto tiles = [&](int b) { return (double)((M + b - 1) / b) * (double)((N + b - 1) / b); };
    Fp6x3Plan best;
    double least = 15 + ceil(tiles(256) * image_splits / 256) * (double)slice_blocks(nkb, image_splits) * 1.25 +
                   reduce(image_splits);
    const auto offer = [&](int tile, int s, double us) {
        if (us < least && launch_fits((int64_t)tiles(tile == 128 ? 128 : 64), 256)) least = us, best = {tile, s};
    };
    for (int s = 1; s <= image_splits; ++s) {
        const double kb = slice_blocks(nkb, s);
        if (kb * (s - 1) >= nkb) continue;         // every slice non-empty
        const double n64 = tiles(64) * s / 256;
        offer(n64 > 1 ? 63 : 64, s, 4.5 + (n64 <= 1 ? 1 : (n64 + ceil(n64)) / 2) * (0.17 * kb + 0.9) + reduce(s));
        offer(128, s, 5 + ceil(tiles(128) * s / 256) * 0.31 * kb + mn * s / 380e3 + reduce(s));
    }
    return best;
}

hipError_t launch_gemm_fp6x3_tiles(const Fp6x3Plan& plan, int64_t M, int64_t N, int64_t Kp, float alpha,
                                   const uint8_t* Ah, const uint8_t* Al, const uint8_t* As, const uint8_t* Bh,
                                   const uint8_t* Bl, const uint8_t* Bs, float beta, float* C, int64_t ldc,
                                   float* partial, hipStream_t stream) {
    if (Kp % 64 || Kp <= 0 || M <= 0 || N <= 0 || plan.slices < 1 || (plan.slices > 1 && !partial))
        return hipErrorInvalidValue;
    const int nkb = (int)(Kp / 64), kbs = slice_blocks(nkb, plan.slices);
    if ((int64_t)(plan.slices - 1) * kbs >= nkb) return hipErrorInvalidValue;   // every slice non-empty
    const Fp6Problem p{M, N, ldc, alpha, beta, {Ah, Bh, Al, Bl}, {As, Bs}, C, plan.slices > 1 ? partial : nullptr,
                       nkb, kbs};
    switch (plan.tile) {
        case 128: return launch_tiles<Fp6Cfg<128, 1, 3>>(p, plan.slices, stream);
        case 64: return launch_tiles<Fp6Cfg<64, 2, 3>>(p, plan.slices, stream);
        case 63: return launch_tiles<Fp6Cfg<64, 1, 3>>(p, plan.slices, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace cmp
