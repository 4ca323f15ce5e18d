// Learned start vector for the inner CG loop: a 3-layer perceptron
//   y = W3^T silu(W2^T silu(W1^T x + b1) + b2) + b3
// mapping a column's descriptor (the 48 nearest atoms of atom(j): scaled
// distance and direction, plus the orbital type of j) to the coefficients of
// s_j = S^-1 e_j on the orbitals of the 12 atoms nearest to atom(j).
//
// Inference: one fused kernel, BF16 operands on the matrix cores
// (v_mfma_f32_16x16x16bf16_1k) with FP32 accumulation; the 16 rows of a
// workgroup stay in LDS between layers.  Training: FP32 products
// on the matrix cores and element-wise kernels (forward, MSE, backward, Adam).
#include <math.h>

#include <algorithm>

#include "ma_internal.h"

namespace ma {

namespace {

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ unsigned short to_bf16(float x)
{
    // round to nearest even
    unsigned u = __float_as_uint(x);
    if ((u & 0x7f800000u) == 0x7f800000u) return (unsigned short)(u >> 16);   // inf / nan
    u += 0x7fffu + ((u >> 16) & 1u);
    return (unsigned short)(u >> 16);
}

__device__ __forceinline__ float silu(float z) { return z / (1.0f + expf(-z)); }

__device__ __forceinline__ float silu_grad(float z)
{
    const float s = 1.0f / (1.0f + expf(-z));
    return s * (1.0f + z * (1.0f - s));
}

// ---------------------------------------------------------------------------
// descriptors
// ---------------------------------------------------------------------------
__global__ void k_features(const int32_t *cols, int ncols, int o, const float *geo, int nf_geo,
                           int nf, float *feat)
{
    const int64_t total = (int64_t)ncols * nf;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total;
         e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t c = e / nf;
        const int f = (int)(e - c * nf);
        const int j = cols[c], A = j / o, r = j - A * o;
        feat[e] = f < nf_geo ? geo[(int64_t)A * nf_geo + f] : (f - nf_geo == r ? 1.0f : 0.0f);
    }
}

// ---------------------------------------------------------------------------
// fused BF16 inference
// ---------------------------------------------------------------------------
// One layer for the 16 rows of the workgroup: out[16 x n_out] =
// act(in[16 x k_pad] W + b), `in` and `out` bf16 rows in LDS (row strides in
// elements, a multiple of four), W given transposed (n_out_pad x k_pad, bf16);
// wavefront w takes the 16-column output tiles w, w + 4, ...
template <bool ACT, bool OUT_F32>
__device__ void mlp_layer(const unsigned short *in, int in_stride, int k_pad,
                          const unsigned short *__restrict__ Wt, const float *__restrict__ bias,
                          int n_out, unsigned short *out, int out_stride, float *outf,
                          int64_t outf_stride, int rows_valid)
{
    const int lane = threadIdx.x & 63;
    const int r16 = lane & 15, kq = lane >> 4;
    const int ntile = (n_out + 15) >> 4;
    for (int t = threadIdx.x >> 6; t < ntile; t += 4) {
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        const int ncol = t * 16 + r16;                       // B column of this lane
        const bf16x4 *wrow = reinterpret_cast<const bf16x4 *>(Wt + (int64_t)ncol * k_pad) + kq;
        const bf16x4 *arow = reinterpret_cast<const bf16x4 *>(in + r16 * in_stride) + kq;
#pragma unroll 4
        for (int k0 = 0; k0 < k_pad / 4; k0 += 4)
            acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(arow[k0], wrow[k0], acc, 0, 0, 0);
        // lane holds D[4*kq + jj][r16]
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
            const int row = 4 * kq + jj, col = t * 16 + r16;
            if (col < n_out) {
                float v = acc[jj] + bias[col];
                if (ACT) v = silu(v);
                if (OUT_F32) {
                    if (row < rows_valid) outf[row * outf_stride + col] = v;
                } else {
                    out[row * out_stride + col] = to_bf16(v);
                }
            }
        }
    }
}

constexpr int kRowPad = 8;   // elements between LDS rows, so that 16 rows do not share banks

// 16 rows per workgroup of 256 threads, the output columns spread over its
// wavefronts: a batch of 6,912 rows is 432 workgroups (with 16 rows per
// wavefront it was 108 on 256 compute units: 133 us, now 42).
__global__ void __launch_bounds__(256) k_mlp_infer(const float *X, int64_t n, int nf, int nf_pad,
                                                   int nh, int no, const unsigned short *W1t,
                                                   const float *b1, const unsigned short *W2t,
                                                   const float *b2, const unsigned short *W3t,
                                                   const float *b3, float *Y)
{
    extern __shared__ __attribute__((aligned(16))) unsigned short lds[];
    const int stride_a = (nf_pad > nh ? nf_pad : nh) + kRowPad, stride_b = nh + kRowPad;
    unsigned short *bufA = lds;                     // x, then h2
    unsigned short *bufB = lds + 16 * stride_a;     // h1
    for (int64_t r0 = (int64_t)blockIdx.x * 16; r0 < n; r0 += (int64_t)gridDim.x * 16) {
        const int valid = (int)((n - r0) < 16 ? (n - r0) : 16);
        for (int e = threadIdx.x; e < 16 * nf_pad; e += 256) {
            const int rr = e / nf_pad, f = e - rr * nf_pad;
            const float v = (rr < valid && f < nf) ? X[(r0 + rr) * nf + f] : 0.0f;
            bufA[rr * stride_a + f] = to_bf16(v);
        }
        __syncthreads();
        mlp_layer<true, false>(bufA, stride_a, nf_pad, W1t, b1, nh, bufB, stride_b, nullptr, 0, 16);
        __syncthreads();
        mlp_layer<true, false>(bufB, stride_b, nh, W2t, b2, nh, bufA, stride_a, nullptr, 0, 16);
        __syncthreads();
        mlp_layer<false, true>(bufA, stride_a, nh, W3t, b3, no, nullptr, 0, Y + r0 * no, no, valid);
        __syncthreads();
    }
}

// Transposed BF16 copy of an (rows x cols) FP32 matrix into (cols_pad x rows_pad).
__global__ void k_to_bf16_t(const float *W, int rows, int cols, int rows_pad, int cols_pad,
                            unsigned short *Wt)
{
    const int64_t total = (int64_t)cols_pad * rows_pad;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total;
         e += (int64_t)gridDim.x * blockDim.x) {
        const int c = (int)(e / rows_pad), r = (int)(e - (int64_t)c * rows_pad);
        Wt[e] = (r < rows && c < cols) ? to_bf16(W[(int64_t)r * cols + c]) : (unsigned short)0;
    }
}

// ---------------------------------------------------------------------------
// FP32 training kernels
// ---------------------------------------------------------------------------
// C[M x N] (row-major, ldc) = beta*C + A B (+ bias) with A(i,k) = A[i*sa0 + k*sa1],
// B(k,j) = B[k*sb0 + j*sb1]; rows of A optionally gathered through `gather`.
// If Z != nullptr, Z receives the pre-activation and C = silu(Z); if Zg !=
// nullptr, C is multiplied by silu'(Zg).
__device__ __forceinline__ void gemm_store(float r, int64_t at, int j, const float *bias, float beta,
                                           float *C, float *Z, const float *Zg)
{
    r += bias ? bias[j] : 0.f;
    if (beta != 0.f) r += beta * C[at];
    if (Z) {
        Z[at] = r;
        r = silu(r);
    }
    if (Zg) r *= silu_grad(Zg[at]);
    C[at] = r;
}

// One 16 x 16 tile of C per workgroup on v_mfma_f32_16x16x4f32 (FP32 products and
// sums), K split over the four wavefronts in runs of 16 and their sums added in
// LDS.  The products of a training step are small (1,024 x 256 x 256 and
// 256 x 256 x 1,024): what bounds them is the number of workgroups and the chain
// along K, not the operand traffic, which L2 serves.  The 64 x 64 tiles below put
// 16 to 64 workgroups on 256 compute units there: 99 us a product on average, 14
// here.
__global__ void __launch_bounds__(256) k_gemm(int M, int N, int K, const float *A, int64_t sa0,
                                              int64_t sa1, const int32_t *gather, const float *B,
                                              int64_t sb0, int64_t sb1, const float *bias,
                                              float beta, float *C, int64_t ldc, float *Z,
                                              const float *Zg)
{
    __shared__ float part[4][16][17];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int r16 = lane & 15, kq = lane >> 4;
    const int i0 = blockIdx.y * 16, j0 = blockIdx.x * 16;
    // rows and columns past the edge repeat the last one; their sums are not stored
    const int ia = min(i0 + r16, M - 1), jb = min(j0 + r16, N - 1);
    const float *Ap = A + (int64_t)(gather ? gather[ia] : ia) * sa0;
    const float *Bp = B + (int64_t)jb * sb1;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
    for (int k0 = 16 * w; k0 < K; k0 += 64) {
        float a[4], b[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int k = k0 + 4 * kq + e;
            const bool in = k < K;
            const float av = Ap[(in ? k : 0) * sa1], bv = Bp[(in ? k : 0) * sb0];
            a[e] = in ? av : 0.f;
            b[e] = in ? bv : 0.f;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[e], acc, 0, 0, 0);
    }
    // lane holds D[4 * kq + jj][r16]
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) part[w][4 * kq + jj][r16] = acc[jj];
    __syncthreads();
    const int u = threadIdx.x >> 4, v = threadIdx.x & 15;
    const int i = i0 + u, j = j0 + v;
    if (i < M && j < N)
        gemm_store(((part[0][u][v] + part[1][u][v]) + part[2][u][v]) + part[3][u][v], i * ldc + j, j, bias,
                   beta, C, Z, Zg);
}

// The same by 64 x 64 tiles staged in LDS, 4 x 4 values per thread: each operand is
// read once per 64 rows instead of once per 16.  For products of so many tiles that
// the operand traffic bounds them (the rule is launch_gemm's).
constexpr int TB = 64, TK = 16;
__global__ void __launch_bounds__(256) k_gemm_tile(int M, int N, int K, const float *A, int64_t sa0,
                                                   int64_t sa1, const int32_t *gather, const float *B,
                                                   int64_t sb0, int64_t sb1, const float *bias,
                                                   float beta, float *C, int64_t ldc, float *Z,
                                                   const float *Zg)
{
    __shared__ float sA[TK][TB + 1], sB[TK][TB + 1];
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    const int i0 = blockIdx.y * TB, j0 = blockIdx.x * TB;
    float acc[4][4] = {};
    for (int k0 = 0; k0 < K; k0 += TK) {
        for (int e = threadIdx.x; e < TK * TB; e += 256) {
            const int kk = e / TB, ii = e - kk * TB;
            const int i = i0 + ii, k = k0 + kk;
            float v = 0.f;
            if (i < M && k < K) {
                const int64_t ri = gather ? gather[i] : i;
                v = A[ri * sa0 + k * sa1];
            }
            sA[kk][ii] = v;
            const int j = j0 + ii;
            sB[kk][ii] = (j < N && k < K) ? B[k * sb0 + j * sb1] : 0.f;
        }
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < TK; ++kk) {
            float a[4], b[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                a[u] = sA[kk][ty * 4 + u];
                b[u] = sB[kk][tx * 4 + u];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[u][v] += a[u] * b[v];
        }
        __syncthreads();
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int i = i0 + ty * 4 + u, j = j0 + tx * 4 + v;
            if (i < M && j < N) gemm_store(acc[u][v], i * ldc + j, j, bias, beta, C, Z, Zg);
        }
}

// dY = 2 (Y - T) / (n * no); partial sums of (Y - T)^2 per block.
__global__ void __launch_bounds__(256) k_mse(const float *Y, const float *T, const int32_t *gather,
                                             int64_t n, int no, float *dY, double *partial)
{
    __shared__ double red[4];
    double s = 0.0;
    const int64_t total = n * no;
    const float scale = 2.0f / (float)total;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total;
         e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = e / no;
        const int c = (int)(e - i * no);
        const int64_t ri = gather ? gather[i] : i;
        const float d = Y[e] - T[ri * no + c];
        dY[e] = scale * d;
        s += (double)d * d;
    }
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) partial[blockIdx.x] = ((red[0] + red[1]) + red[2]) + red[3];
}

// db[j] = sum_i G[i, j]: 16 columns per workgroup, thread (group, column) takes
// rows group, group + 16, ...; the groups are added in order (1,024 x 256: one
// thread per column walked 1,024 rows in 168 us, now 5)
__global__ void __launch_bounds__(256) k_colsum(const float *G, int64_t n, int m, float *db)
{
    __shared__ float part[16][17];
    const int v = threadIdx.x & 15, u = threadIdx.x >> 4;
    const int j = blockIdx.x * 16 + v;
    float s = 0.f;
    if (j < m) {
#pragma unroll 8
        for (int64_t i = u; i < n; i += 16) s += G[i * m + j];
    }
    part[u][v] = s;
    __syncthreads();
    if (u == 0 && j < m) {
        s = 0.f;
#pragma unroll
        for (int k = 0; k < 16; ++k) s += part[k][v];
        db[j] = s;
    }
}

// (bad: a row index of the batch was outside its table, no update)
__global__ void k_adam(float *p, const float *g, float *m, float *v, int64_t count, float lr,
                       float b1, float b2, float eps, float c1, float c2, const int *bad)
{
    if (bad && *bad) return;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < count;
         e += (int64_t)gridDim.x * blockDim.x) {
        const float gg = g[e];
        const float mm = b1 * m[e] + (1.f - b1) * gg;
        const float vv = b2 * v[e] + (1.f - b2) * gg * gg;
        m[e] = mm;
        v[e] = vv;
        p[e] -= lr * (mm / c1) / (sqrtf(vv / c2) + eps);
    }
}

// out row i = in row idx[i]; an index outside [0, rows) writes zeros and
// sets *bad
__global__ void k_gather_rows(const float *in, const int32_t *idx, int64_t n, int m, int64_t rows,
                              float *out, int *bad)
{
    const int64_t total = n * m;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total;
         e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = e / m;
        const int64_t r = idx[i];
        const bool ok = r >= 0 && r < rows;
        if (!ok && e == i * m) atomicOr(bad, 1);
        out[e] = ok ? in[r * m + (e - i * m)] : 0.0f;
    }
}

inline int grid_for(int64_t n, int block) { return (int)std::min<int64_t>(4096, (n + block - 1) / block); }

}  // namespace

hipError_t launch_features(const int32_t *cols, int ncols, int o, const float *geo, int nf_geo,
                           int nf, float *feat, hipStream_t st)
{
    hipLaunchKernelGGL(k_features, dim3(grid_for((int64_t)ncols * nf, 256)), dim3(256), 0, st, cols,
                       ncols, o, geo, nf_geo, nf, feat);
    return hipGetLastError();
}

hipError_t launch_gather_rows(const float *in, const int32_t *idx, int64_t n, int m, int64_t rows,
                              float *out, int *bad, hipStream_t st)
{
    hipLaunchKernelGGL(k_gather_rows, dim3(grid_for(n * m, 256)), dim3(256), 0, st, in, idx, n, m,
                       rows, out, bad);
    return hipGetLastError();
}

hipError_t launch_to_bf16_t(const float *W, int rows, int cols, int rows_pad, int cols_pad,
                            unsigned short *Wt, hipStream_t st)
{
    hipLaunchKernelGGL(k_to_bf16_t, dim3(grid_for((int64_t)rows_pad * cols_pad, 256)), dim3(256), 0,
                       st, W, rows, cols, rows_pad, cols_pad, Wt);
    return hipGetLastError();
}

size_t mlp_infer_smem(int nf_pad, int nh)
{
    const int stride_a = nf_pad > nh ? nf_pad : nh;
    return sizeof(unsigned short) * (size_t)16 * (stride_a + nh + 2 * kRowPad);
}

hipError_t launch_mlp_infer(const float *X, int64_t n, int nf, int nf_pad, int nh, int no,
                            const unsigned short *W1t, const float *b1, const unsigned short *W2t,
                            const float *b2, const unsigned short *W3t, const float *b3, float *Y,
                            hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    const size_t smem = mlp_infer_smem(nf_pad, nh);
    hipError_t e = hipFuncSetAttribute((const void *)k_mlp_infer,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return e;
    const int grid = (int)std::min<int64_t>(8192, (n + 15) / 16);
    hipLaunchKernelGGL(k_mlp_infer, dim3(grid), dim3(256), smem, st, X, n, nf, nf_pad, nh, no, W1t,
                       b1, W2t, b2, W3t, b3, Y);
    return hipGetLastError();
}

hipError_t launch_gemm(int M, int N, int K, const float *A, int64_t sa0, int64_t sa1,
                       const int32_t *gather, const float *B, int64_t sb0, int64_t sb1,
                       const float *bias, float beta, float *C, int64_t ldc, float *Z,
                       const float *Zg, hipStream_t st)
{
    // The 64 x 64 tiles once there are 640 of them (2.5 per compute unit).  Forward
    // pass in FP32 (196 -> 256 -> 256 -> 48) of 10,240, 16,384, 65,536 and 300,000
    // rows: 177, 208, 526 and 2,109 us; 16 x 16 tiles throughout 177, 253, 929 and
    // 4,149, 64 x 64 throughout 214, 234, 524 and 2,105.
    const bool large = (int64_t)((M + TB - 1) / TB) * ((N + TB - 1) / TB) >= 640;
    const int tile = large ? TB : 16;
    // at most 65,535 row tiles per launch
    for (int64_t i0 = 0; i0 < M; i0 += 16 * 65535) {
        const int rows = (int)std::min<int64_t>(M - i0, 16 * 65535);
        dim3 grid((N + tile - 1) / tile, (rows + tile - 1) / tile);
        hipLaunchKernelGGL(large ? k_gemm_tile : k_gemm, grid, dim3(256), 0, st, rows, N, K,
                           gather ? A : A + i0 * sa0, sa0, sa1, gather ? gather + i0 : nullptr, B, sb0,
                           sb1, bias, beta, C + i0 * ldc, ldc, Z ? Z + i0 * ldc : nullptr,
                           Zg ? Zg + i0 * ldc : nullptr);
    }
    return hipGetLastError();
}

hipError_t launch_mse(const float *Y, const float *T, const int32_t *gather, int64_t n, int no,
                      float *dY, double *partial, int nblocks, hipStream_t st)
{
    hipLaunchKernelGGL(k_mse, dim3(nblocks), dim3(256), 0, st, Y, T, gather, n, no, dY, partial);
    return hipGetLastError();
}

hipError_t launch_colsum(const float *G, int64_t n, int m, float *db, hipStream_t st)
{
    hipLaunchKernelGGL(k_colsum, dim3((m + 15) / 16), dim3(256), 0, st, G, n, m, db);
    return hipGetLastError();
}

hipError_t launch_adam(float *p, const float *g, float *m, float *v, int64_t count, float lr,
                       float b1, float b2, float eps, int step, const int *bad, hipStream_t st)
{
    const float c1 = 1.f - powf(b1, (float)step), c2 = 1.f - powf(b2, (float)step);
    hipLaunchKernelGGL(k_adam, dim3(grid_for(count, 256)), dim3(256), 0, st, p, g, m, v, count, lr,
                       b1, b2, eps, c1, c2, bad);
    return hipGetLastError();
}

}  // namespace ma
