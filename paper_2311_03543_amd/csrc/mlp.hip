// The learned selector's network on the GPU: 4 -> 64 (ReLU) -> 64 (ReLU) -> 4,
// MSE loss over all outputs, full-batch Adam.  Parameters are packed layer by
// layer as [W (out x in, row-major), b (out)] (4740 floats).
//
// Training works on 32 rows per workgroup of 16 waves.  The 64 x 64 products
// (layer 2 forward, its backward product and its weight gradient) run on
// v_mfma_f32_16x16x4, which adds its products one by one in increasing k with
// one rounding each, so every value is the chain of FP32 FMAs that one lane
// per hidden unit would form.  A weight's gradient is the sum, in this order,
// of four chains over the rows 4 m + w (w = 0..3) of each workgroup, then of
// the workgroups; a second kernel sums the workgroup partials and applies
// Adam.  Every order is fixed, so results are deterministic.
// Inference keeps one wave per sample, lane j owning hidden unit j.
#include "common.h"
#include "kernels.h"

namespace cmp {
namespace {

constexpr int H = 64;
constexpr int OFF_W1 = 0, OFF_B1 = OFF_W1 + H * 4, OFF_W2 = OFF_B1 + H, OFF_B2 = OFF_W2 + H * H,
              OFF_W3 = OFF_B2 + H, OFF_B3 = OFF_W3 + 4 * H, NPAR = OFF_B3 + 4;
static_assert(NPAR == kMlpParams, "parameter packing");
constexpr int GRAD_THREADS = 1024;
constexpr int ROWS_PER_WG = 32;
constexpr int MAX_WG = (kMlpMaxRows + ROWS_PER_WG - 1) / ROWS_PER_WG;
constexpr int ADAM_THREADS = 64;
// LDS row pitch of the 64-wide operands: 4 banks more than a whole turn, so
// 16 rows x 4 consecutive values touch all 64 banks once.
constexpr int HP = H + 4;

struct SParams {
    float w1[H * 4], b1[H], w2t[H * H], b2[H], w3[4 * H], b3[4];
};

__device__ __forceinline__ void load_params(SParams& s, const float* __restrict__ p) {
    for (int i = threadIdx.x; i < NPAR; i += blockDim.x) {
        const float v = p[i];
        if (i < OFF_B1) s.w1[i - OFF_W1] = v;
        else if (i < OFF_W2) s.b1[i - OFF_B1] = v;
        else if (i < OFF_B2) {
            const int q = i - OFF_W2;
            s.w2t[(q % H) * H + q / H] = v;
        } else if (i < OFF_W3) s.b2[i - OFF_B2] = v;
        else if (i < OFF_B3) s.w3[i - OFF_W3] = v;
        else s.b3[i - OFF_B3] = v;
    }
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

__device__ __forceinline__ float bcast(float v, int lane) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}

// Forward pass of one sample (lane j: hidden unit j); every lane returns all 4 outputs.
struct Fwd {
    float z1, h1, z2, h2, y[4];
};
__device__ __forceinline__ Fwd forward(const SParams& s, const float x[4], int j) {
    Fwd f;
    f.z1 = s.b1[j];
#pragma unroll
    for (int c = 0; c < 4; ++c) f.z1 = __builtin_fmaf(s.w1[j * 4 + c], x[c], f.z1);
    f.h1 = fmaxf(f.z1, 0.f);
    f.z2 = s.b2[j];
#pragma unroll 16
    for (int i = 0; i < H; ++i) f.z2 = __builtin_fmaf(s.w2t[i * H + j], bcast(f.h1, i), f.z2);
    f.h2 = fmaxf(f.z2, 0.f);
#pragma unroll
    for (int o = 0; o < 4; ++o) f.y[o] = s.b3[o] + wave_sum(s.w3[o * H + j] * f.h2);
    return f;
}

typedef float floatx4 __attribute__((ext_vector_type(4)));

// 16 x 16 block of init + X W over k = 0 .. 63 in order: X[row][k] at
// x + row * HP + k, W[k][col] at w + k * wk + col * wc (block origin included).
__device__ __forceinline__ floatx4 mlp_block(const float* x, const float* w, int wk, int wc, float init, int lane) {
    const int r = lane & 15, q = lane >> 4;
    floatx4 acc = {init, init, init, init};
#pragma unroll
    for (int s = 0; s < H / 4; ++s)
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x[r * HP + 4 * s + q], w[(4 * s + q) * wk + r * wc], acc, 0, 0, 0);
    return acc;                                  // element i: row 4 q + i, column r
}

// Partial gradient of the summed squared error (scaled by 2 / (4 n)) over this
// workgroup's 32 rows; writes part[wg * (NPAR + 1) + p] and the summed squared
// error.  Bound by latency: 16 waves share each of its phases (a serial pass
// per row and wave, four waves, took 33 us a step on 2000 rows; this takes 9).
__global__ __launch_bounds__(GRAD_THREADS) void mlp_grad_kernel(int n, const float* __restrict__ X,
                                                                const float* __restrict__ Y,
                                                                const float* __restrict__ params,
                                                                float* __restrict__ part) {
    __shared__ float w1[H * 4], b1[H], w2[H * HP], b2[H], w3[4 * H], b3[4];
    __shared__ float xs[ROWS_PER_WG][4], h1[ROWS_PER_WG * HP], z2[ROWS_PER_WG * HP], h2[ROWS_PER_WG * HP];
    __shared__ float dz1[ROWS_PER_WG * HP], dz2[ROWS_PER_WG * HP], dys[2][ROWS_PER_WG][4], ds[ROWS_PER_WG][4], factor[2];
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    constexpr int PL = (NPAR + GRAD_THREADS - 1) / GRAD_THREADS;   // every load in flight before the first store
    float pv[PL];
#pragma unroll
    for (int l = 0; l < PL; ++l) {
        const int i = t + l * GRAD_THREADS;
        pv[l] = params[i < NPAR ? i : NPAR - 1];
    }
    const int r0 = blockIdx.x * ROWS_PER_WG;
    const int rows = min(n - r0, ROWS_PER_WG);   // absent rows are zero in every array that feeds a gradient
    if (t < 4 * ROWS_PER_WG) xs[t >> 2][t & 3] = t < 4 * rows ? X[4 * r0 + t] : 0.f;
    const float yv = lane < 4 && r0 + wave < n ? Y[4 * (r0 + wave) + lane] : 0.f;
    const float yw = lane < 4 && r0 + wave + 16 < n ? Y[4 * (r0 + wave + 16) + lane] : 0.f;
#pragma unroll
    for (int l = 0; l < PL; ++l) {
        const int i = t + l * GRAD_THREADS;
        if (i < OFF_B1) w1[i - OFF_W1] = pv[l];
        else if (i < OFF_W2) b1[i - OFF_B1] = pv[l];
        else if (i < OFF_B2) w2[(i - OFF_W2) / H * HP + (i - OFF_W2) % H] = pv[l];
        else if (i < OFF_W3) b2[i - OFF_B2] = pv[l];
        else if (i < OFF_B3) w3[i - OFF_W3] = pv[l];
        else if (i < NPAR) b3[i - OFF_B3] = pv[l];
    }
    const float scale = 2.f / (4.f * (float)n);
    if (t < 2) factor[t] = t ? scale : 1.f;
    __syncthreads();
    // layer 1: lane = unit, rows wave and wave + 16
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int r = wave + 16 * h;
        float z = b1[lane];
#pragma unroll
        for (int c = 0; c < 4; ++c) z = __builtin_fmaf(w1[lane * 4 + c], xs[r][c], z);
        h1[r * HP + lane] = r < rows ? fmaxf(z, 0.f) : 0.f;
    }
    __syncthreads();
    // layer 2: 2 x 4 blocks of 16 rows x 16 units
    if (wave < 8) {
        const int rb = (wave >> 2) * 16, ub = (wave & 3) * 16;
        const floatx4 z = mlp_block(h1 + rb * HP, w2 + ub * HP, 1, HP, b2[ub + (lane & 15)], lane);
#pragma unroll
        for (int i = 0; i < 4; ++i) z2[(rb + 4 * (lane >> 4) + i) * HP + ub + (lane & 15)] = z[i];
    }
    __syncthreads();
    // outputs, their error, and layer 2's deltas: lane = unit, rows wave and wave + 16.
    // The first step of the sum over units is one FMA, so units 0-31 and 32-63 hold
    // outputs that may differ in the last bit; each uses its own (b3 and the loss: unit 0's).
    {
        float zz[2], hh[2], y[2][4];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            zz[h] = z2[(wave + 16 * h) * HP + lane];
            hh[h] = fmaxf(zz[h], 0.f);
#pragma unroll
            for (int o = 0; o < 4; ++o) {
                const float w = w3[o * H + lane];
                y[h][o] = __builtin_fmaf(w, hh[h], __shfl_xor(w * hh[h], 32));
            }
        }
#pragma unroll
        for (int off = 16; off > 0; off >>= 1)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int o = 0; o < 4; ++o) y[h][o] += __shfl_xor(y[h][o], off);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int r = wave + 16 * h;
            const bool in = r < rows;
            float dh2 = 0.f;
#pragma unroll
            for (int o = 0; o < 4; ++o) {
                const float d = (b3[o] + y[h][o]) - bcast(h ? yw : yv, o);
                const float dy = scale * d;
                dh2 = __builtin_fmaf(w3[o * H + lane], dy, dh2);
                if ((lane & 31) == 0) dys[lane >> 5][r][o] = in ? dy : 0.f;
                if (lane == 0) ds[r][o] = in ? d : 0.f;
            }
            h2[r * HP + lane] = in ? hh[h] : 0.f;
            dz2[r * HP + lane] = in && zz[h] > 0.f ? dh2 : 0.f;
        }
    }
    __syncthreads();
    float* dst = part + (size_t)blockIdx.x * (NPAR + 1);
    const int lr = lane & 15, lq = lane >> 4;
    // layer 1's deltas (8 waves): dh1 = dz2 W2, then dz1 where unit 1 was active (h1 > 0)
    if (wave < 8) {
        const int rb = (wave >> 2) * 16, ub = (wave & 3) * 16;
        const floatx4 d = mlp_block(dz2 + rb * HP, w2 + ub, HP, 1, 0.f, lane);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int at = (rb + 4 * lq + i) * HP + ub + lr;
            dz1[at] = h1[at] > 0.f ? d[i] : 0.f;
        }
    }
    // layer 2's weight gradient: block (jb, ib) of units x inputs per wave, four chains over 8 rows
    {
        const int jb = (wave >> 2) * 16, ib = (wave & 3) * 16;
        floatx4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            floatx4 g = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const int r = w + 4 * (4 * s + lq);
                g = __builtin_amdgcn_mfma_f32_16x16x4f32(dz2[r * HP + jb + lr], h1[r * HP + ib + lr], g, 0, 0, 0);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) sum[i] += g[i];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) dst[OFF_W2 + (jb + 4 * lq + i) * H + ib + lr] = sum[i];
    }
    __syncthreads();
    // the other gradients, one entry per lane: four chains over 8 rows each of
    // u * v, v = 1 or the error's scale where an entry has no second factor.
    // Entries: W1 (256), b1 (64), b2 (64), W3 (256), b3 (4); the squared error
    // on the first lane of the next wave.
    constexpr int E_B1 = 4 * H, E_B2 = E_B1 + H, E_W3 = E_B2 + H, E_B3 = E_W3 + 4 * H, E_END = E_B3 + 4;
    constexpr int E_SQ = (E_END + 63) / 64 * 64;
    static_assert(E_SQ < GRAD_THREADS, "one entry per lane");
    if (t < E_END) {
        const float *u = &ds[0][t & 3], *v = &factor[1];   // b3
        int up = 4, vp = 0, out = OFF_B3 + t - E_B3;
        if (t < E_B1) u = dz1 + (t >> 2), up = HP, v = &xs[0][t & 3], vp = 4, out = OFF_W1 + t;
        else if (t < E_B2) u = dz1 + (t - E_B1), up = HP, v = factor, out = OFF_B1 + t - E_B1;
        else if (t < E_W3) u = dz2 + (t - E_B2), up = HP, v = factor, out = OFF_B2 + t - E_B2;
        else if (t < E_B3) u = h2 + (t & 63), up = HP, v = &dys[(t >> 5) & 1][0][(t - E_W3) >> 6], vp = 4, out = OFF_W3 + t - E_W3;
        float a[ROWS_PER_WG], b[ROWS_PER_WG], sum = 0.f;
#pragma unroll
        for (int r = 0; r < ROWS_PER_WG; ++r) a[r] = u[r * up], b[r] = v[r * vp];
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            float g = 0.f;
#pragma unroll
            for (int m = 0; m < 8; ++m) g = __builtin_fmaf(a[w + 4 * m], b[w + 4 * m], g);
            sum += g;
        }
        dst[out] = sum;
    } else if (t == E_SQ) {
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            float g = 0.f;
#pragma unroll
            for (int m = 0; m < 8; ++m)
#pragma unroll
                for (int o = 0; o < 4; ++o) g = __builtin_fmaf(ds[w + 4 * m][o], ds[w + 4 * m][o], g);
            sum += g;
        }
        dst[NPAR] = sum;
    }
}

// Adam's bias corrections 1 - 0.9^t and 1 - 0.999^t of steps t0 + 1 .. t0 + steps.
__global__ void mlp_bias_kernel(int t0, int steps, double* __restrict__ bias) {
    for (int s = blockIdx.x * blockDim.x + threadIdx.x; s < steps; s += gridDim.x * blockDim.x) {
        bias[2 * s] = 1.0 - pow(0.9, (double)(t0 + s + 1));
        bias[2 * s + 1] = 1.0 - pow(0.999, (double)(t0 + s + 1));
    }
}

// Sum the workgroup partials (fixed order) and apply an Adam step with the
// bias corrections bias[0], bias[1], or only write the gradient when grad_out
// is set.  One wave per workgroup, one parameter per lane, 64 records in
// flight: bound by the latency of reading what other XCDs just wrote.  As one
// workgroup for all parameters this took 88 us a step on 2000 rows, now 4.5
// (8 to 10 with 16 or 32 records in flight).
__global__ __launch_bounds__(ADAM_THREADS) void mlp_adam_kernel(int nwg, int n, const float* __restrict__ part,
                                                                float* __restrict__ params, float* __restrict__ m,
                                                                float* __restrict__ v,
                                                                const double* __restrict__ bias, float lr,
                                                                float* __restrict__ loss_out,
                                                                float* __restrict__ grad_out) {
    const int p = blockIdx.x * ADAM_THREADS + threadIdx.x;
    if (p > NPAR) return;
    const bool update = p < NPAR && !grad_out;
    const double bc1 = update ? bias[0] : 1.0, bc2 = update ? bias[1] : 1.0;
    const float m0 = update ? m[p] : 0.f, v0 = update ? v[p] : 0.f, p0 = update ? params[p] : 0.f;
    float g = 0.f;
    for (int w0 = 0; w0 < nwg; w0 += 64) {       // 64 records in flight
        float x[64];
#pragma unroll
        for (int w = 0; w < 64; ++w) x[w] = w0 + w < nwg ? part[(size_t)(w0 + w) * (NPAR + 1) + p] : 0.f;
#pragma unroll
        for (int w = 0; w < 64; ++w) g += x[w];   // + 0 past the end: g is never -0
    }
    if (p == NPAR) {
        if (loss_out) *loss_out = g / (4.f * (float)n);
        return;
    }
    if (grad_out) {
        grad_out[p] = g;
        return;
    }
    const float mm = __builtin_fmaf(0.1f, g, 0.9f * m0);
    const float vv = __builtin_fmaf(g, 0.001f * g, 0.999f * v0);
    m[p] = mm;
    v[p] = vv;
    const float mh = (float)((double)mm / bc1);
    const float vh = (float)((double)vv / bc2);
    params[p] = p0 - lr * mh / (sqrtf(vh) + 1e-8f);
}

__global__ void fill_zero(float* __restrict__ p, int count) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < count; i += gridDim.x * blockDim.x) p[i] = 0.f;
}

// Batched inference: one wave per sample, four samples per workgroup pass.
__global__ __launch_bounds__(256) void mlp_infer_kernel(int n, const float* __restrict__ X,
                                                        const float* __restrict__ params,
                                                        float* __restrict__ Y) {
    __shared__ SParams s;
    load_params(s, params);
    __syncthreads();
    const int j = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int r = blockIdx.x * 4 + wave; r < n; r += gridDim.x * 4) {
        float x[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) x[c] = X[4 * r + c];
        const Fwd f = forward(s, x, j);
        if (j < 4) Y[4 * r + j] = j == 0 ? f.y[0] : j == 1 ? f.y[1] : j == 2 ? f.y[2] : f.y[3];
    }
}

}  // namespace

static_assert(MAX_WG * (NPAR + 1) <= kMlpPartFloats, "partial-gradient buffer");

hipError_t launch_mlp_train(int n, const float* X, const float* Y, float* params, float* m,
                            float* v, float* part, int steps, int t0, float lr, double* bias, float* loss_trace,
                            float* grad_out, hipStream_t stream) {
    if (n < 1 || n > kMlpMaxRows) return hipErrorInvalidValue;
    const int nwg = (n + ROWS_PER_WG - 1) / ROWS_PER_WG;
    const dim3 adam((NPAR + 1 + ADAM_THREADS - 1) / ADAM_THREADS);
    if (grad_out) {
        hipLaunchKernelGGL(mlp_grad_kernel, dim3(nwg), dim3(GRAD_THREADS), 0, stream, n, X, Y, params, part);
        hipLaunchKernelGGL(mlp_adam_kernel, adam, dim3(ADAM_THREADS), 0, stream, nwg, n, part, params, m, v,
                           nullptr, 0.f, loss_trace, grad_out);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(fill_zero, dim3(10), dim3(512), 0, stream, m, NPAR);
    hipLaunchKernelGGL(fill_zero, dim3(10), dim3(512), 0, stream, v, NPAR);
    if (steps > 0) {
        if (!bias) return hipErrorInvalidValue;
        hipLaunchKernelGGL(mlp_bias_kernel, dim3(steps < 65536 ? (steps + 255) / 256 : 256), dim3(256), 0, stream, t0,
                           steps, bias);
    }
    for (int s = 0; s < steps; ++s) {
        hipLaunchKernelGGL(mlp_grad_kernel, dim3(nwg), dim3(GRAD_THREADS), 0, stream, n, X, Y, params, part);
        hipLaunchKernelGGL(mlp_adam_kernel, adam, dim3(ADAM_THREADS), 0, stream, nwg, n, part, params, m, v,
                           bias + 2 * (size_t)s, lr, loss_trace ? loss_trace + s : nullptr, nullptr);
    }
    return hipGetLastError();
}

hipError_t launch_mlp_infer(int n, const float* X, const float* params, float* Y,
                            hipStream_t stream) {
    if (n <= 0) return hipSuccess;
    int b = (n + 3) / 4;
    if (b > 1024) b = 1024;
    hipLaunchKernelGGL(mlp_infer_kernel, dim3(b), dim3(256), 0, stream, n, X, params, Y);
    return hipGetLastError();
}

}  // namespace cmp
