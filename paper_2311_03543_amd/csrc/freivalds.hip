// FP64 residual probe of a finished product (verify mode).  With a probe
// vector x of +-1 entries, y = B x, z = alpha A y + beta C0 x and w = C x;
// since E||E x||^2 = ||E||_F^2 for Rademacher x, ||w - z|| / ||z|| estimates
// the relative Frobenius error of C without forming A B.  Each matrix is read
// once (HBM-bound), all arithmetic in FP64; the sums over rows are added in a
// fixed order, so a probe repeats bit for bit.
#include "common.h"
#include "kernels.h"

namespace cmp {
namespace {

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

// s[r] += sum_k X[row_r][k] v[k] over this lane's share of k = 0 .. n - 1, for
// the R rows at p[r].  vec: rows allow 16-byte loads.  The next values of all
// rows are in flight while the previous ones are multiplied (unroll).
template <int R>
__device__ __forceinline__ void dot_rows(const float* const (&p)[R], bool vec, int64_t n,
                                         const double* __restrict__ v, int lane, double (&s)[R]) {
    int64_t k = 0;
    if (vec) {
        const int64_t n4 = n & ~(int64_t)3;
#pragma unroll 4
        for (k = 4 * lane; k < n4; k += 256) {
            float4 x[R];
#pragma unroll
            for (int r = 0; r < R; ++r) x[r] = *reinterpret_cast<const float4*>(p[r] + k);
            const double2 a = *reinterpret_cast<const double2*>(v + k), b = *reinterpret_cast<const double2*>(v + k + 2);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                s[r] += (double)x[r].x * a.x;
                s[r] += (double)x[r].y * a.y;
                s[r] += (double)x[r].z * b.x;
                s[r] += (double)x[r].w * b.y;
            }
        }
        k = n4;
    }
#pragma unroll 4
    for (k += lane; k < n; k += 64) {
        float x[R];
#pragma unroll
        for (int r = 0; r < R; ++r) x[r] = p[r][k];
        const double a = v[k];
#pragma unroll
        for (int r = 0; r < R; ++r) s[r] += (double)x[r] * a;
    }
}

// y[k] = sum_j B[k][j] x[j], R rows k per wave.
template <int R>
__global__ __launch_bounds__(256) void bx_kernel(int64_t K, int64_t N, const float* __restrict__ B,
                                                 int64_t ldb, bool vec, const double* __restrict__ x,
                                                 double* __restrict__ y) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (int64_t k = ((int64_t)blockIdx.x * 4 + wave) * R; k < K; k += (int64_t)gridDim.x * 4 * R) {
        const float* p[R];
        double s[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            p[r] = B + (k + r < K ? k + r : K - 1) * ldb;
            s[r] = 0.0;
        }
        dot_rows<R>(p, vec, N, x, lane, s);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            s[r] = wave_sum(s[r]);
            if (lane == 0 && k + r < K) y[k + r] = s[r];
        }
    }
}

// R rows i of C per wave: part[2 b], part[2 b + 1] = the sums of (w_i - z_i)^2
// and z_i^2 over the rows of workgroup b.  (One atomic add per row and sum on
// one address kept 3000 rows of 4100 at 102 us; the partials take 14.6.)
template <int R>
__global__ __launch_bounds__(256) void rows_kernel(int64_t M, int64_t N, int64_t K, float alpha,
                                                   const float* __restrict__ A, int64_t lda, bool va,
                                                   float beta, const float* __restrict__ C0,
                                                   int64_t ldc0, bool v0, const float* __restrict__ C,
                                                   int64_t ldc, bool vc, const double* __restrict__ x,
                                                   const double* __restrict__ y,
                                                   double* __restrict__ part) {
    __shared__ double sums[4][2];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    double dd = 0.0, zz = 0.0;
    for (int64_t i = ((int64_t)blockIdx.x * 4 + wave) * R; i < M; i += (int64_t)gridDim.x * 4 * R) {
        const float* p[R];
        double za[R], w[R], c0[R];
        int64_t row[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            row[r] = i + r < M ? i + r : M - 1;
            za[r] = w[r] = c0[r] = 0.0;
        }
        if (alpha != 0.f) {
#pragma unroll
            for (int r = 0; r < R; ++r) p[r] = A + row[r] * lda;
            dot_rows<R>(p, va, K, y, lane, za);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) p[r] = C + row[r] * ldc;
        dot_rows<R>(p, vc, N, x, lane, w);
        if (beta != 0.f) {
#pragma unroll
            for (int r = 0; r < R; ++r) p[r] = C0 + row[r] * ldc0;
            dot_rows<R>(p, v0, N, x, lane, c0);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const double z = (double)alpha * wave_sum(za[r]) + (double)beta * wave_sum(c0[r]);
            const double d = wave_sum(w[r]) - z;
            if (i + r < M) {
                dd += d * d;
                zz += z * z;
            }
        }
    }
    if (lane == 0) {
        sums[wave][0] = dd;
        sums[wave][1] = zz;
    }
    __syncthreads();
    if (threadIdx.x < 2)
        part[2 * (int64_t)blockIdx.x + threadIdx.x] = ((sums[0][threadIdx.x] + sums[1][threadIdx.x]) +
                                                       sums[2][threadIdx.x]) + sums[3][threadIdx.x];
}

// out[0], out[1] = the sums of the `blocks` (<= kFreivaldsBlocks) partial pairs.
__global__ __launch_bounds__(256) void probe_sum_kernel(int blocks, const double* __restrict__ part,
                                                        double* __restrict__ out) {
    __shared__ double sums[4][2];
    const int t = threadIdx.x;
    double dd = 0.0, zz = 0.0;
    for (int b = t; b < blocks; b += 256) {
        dd += part[2 * b];
        zz += part[2 * b + 1];
    }
    dd = wave_sum(dd);
    zz = wave_sum(zz);
    if ((t & 63) == 0) {
        sums[t >> 6][0] = dd;
        sums[t >> 6][1] = zz;
    }
    __syncthreads();
    if (t < 2) out[t] = ((sums[0][t] + sums[1][t]) + sums[2][t]) + sums[3][t];
}

__device__ __forceinline__ uint64_t splitmix64_at(uint64_t seed, uint64_t j) {
    uint64_t z = seed + (j + 1) * 0x9e3779b97f4a7c15ull;
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    return z ^ (z >> 31);
}

__global__ void rademacher_kernel(int64_t n, uint64_t seed, double* __restrict__ x) {
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < n;
         j += (int64_t)gridDim.x * blockDim.x)
        x[j] = (splitmix64_at(seed, (uint64_t)j) >> 63) ? -1.0 : 1.0;
}

unsigned rows_grid(int64_t rows, int per_wave) {
    int64_t b = (rows + 4 * per_wave - 1) / (4 * per_wave);
    if (b > kFreivaldsBlocks) b = kFreivaldsBlocks;
    return (unsigned)(b < 1 ? 1 : b);
}
bool rows_vec(const float* x, int64_t ld) { return ld % 4 == 0 && (reinterpret_cast<uintptr_t>(x) & 15) == 0; }
// Rows per wave: 4 share each probe value they load (a double per float of the
// matrix), 1 keeps every CU busy on matrices with few rows.
constexpr int64_t kManyRows = 8192;

}  // namespace

hipError_t launch_freivalds(int64_t M, int64_t N, int64_t K, float alpha, const float* A,
                            int64_t lda, const float* B, int64_t ldb, float beta, const float* C0,
                            int64_t ldc0, const float* C, int64_t ldc, const double* x, double* ws,
                            double* part, double* out, hipStream_t stream) {
    double* y = ws;
    if (alpha != 0.f && K > 0) {
        const bool vb = rows_vec(B, ldb);
        if (K >= kManyRows)
            hipLaunchKernelGGL(bx_kernel<4>, dim3(rows_grid(K, 4)), dim3(256), 0, stream, K, N, B, ldb, vb, x, y);
        else
            hipLaunchKernelGGL(bx_kernel<1>, dim3(rows_grid(K, 1)), dim3(256), 0, stream, K, N, B, ldb, vb, x, y);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const bool va = rows_vec(A, lda), v0 = rows_vec(C0, ldc0), vc = rows_vec(C, ldc);
    const int per_wave = M >= kManyRows ? 4 : 1;
    const unsigned blocks = rows_grid(M, per_wave);
    if (per_wave == 4)
        hipLaunchKernelGGL(rows_kernel<4>, dim3(blocks), dim3(256), 0, stream, M, N, K, alpha, A, lda, va, beta, C0,
                           ldc0, v0, C, ldc, vc, x, y, part);
    else
        hipLaunchKernelGGL(rows_kernel<1>, dim3(blocks), dim3(256), 0, stream, M, N, K, alpha, A, lda, va, beta, C0,
                           ldc0, v0, C, ldc, vc, x, y, part);
    hipLaunchKernelGGL(probe_sum_kernel, dim3(1), dim3(256), 0, stream, (int)blocks, part, out);
    return hipGetLastError();
}

hipError_t launch_rademacher(int64_t n, uint64_t seed, double* x, hipStream_t stream) {
    int64_t b = (n + 255) / 256;
    if (b > 4096) b = 4096;
    hipLaunchKernelGGL(rademacher_kernel, dim3((unsigned)(b < 1 ? 1 : b)), dim3(256), 0, stream, n,
                       seed, x);
    return hipGetLastError();
}

}  // namespace cmp
