// Kernels of the learned initial density (an extension: the paper's SCF starts
// from a conventional guess).  A small multilayer perceptron maps features of
// an atom pair to that pair's density block in the pair's bond frame; the
// blocks are rotated to the molecular frame and scattered into D, which the
// SCF step then purifies.  The same library trains the network: forward,
// backward, a masked squared-error loss and Adam are the kernels below.
//
// Everything here is FP32 except the scatter (FP64 rotation and output).
#include <hip/hip_runtime.h>

#include <math.h>
#include <stdint.h>

#include <algorithm>

#include "fk_guess.h"

namespace {

// C[M][N] = op(A)[M][K] op(B)[K][N], row-major, FP32 products and sums on the
// matrix cores (v_mfma_f32_16x16x4_f32).
//   TA = 0: A[m][k] at A[m * lda + k];  TA = 1: A stored [K][M], A[k * lda + m]
//   TB = 0: B[k][n] at B[k * ldb + n];  TB = 1: B stored [N][K], B[n * ldb + k]
// Epilogues: EPI_BIAS adds bias (and writes SiLU(C) to A_out when that is not
// null), EPI_SILU multiplies by SiLU'(Z), EPI_SUM writes C and, from the
// workgroups of the first 16 rows, the column sums of B to bsum (the bias
// gradient beside a weight gradient).
//
// A training step's products are small (2048 x 256 x 256) and chained, so what
// counts is the time of one tile and how many run at once, not operand reuse: a
// workgroup computes 16 x 32 outputs, operands coming from L1/L2 straight into
// registers.  The forward layers (of few rows; many stage slabs, k_layer_tall)
// give each tile to one wave, which multiplies k by k: the matrix instruction
// adds its four products one after the other, so an output is the same chain of
// FMAs as in a scalar loop (equal bit for bit); its operands are read value by
// value in that order.  The backward products split K over NW waves (4 for the
// input gradient, 16 for the weight gradient; every NW-th 16-deep slice; the lane
// group g takes k = 4 g + j in step j, so that the input gradient, whose operands
// both lie along k, reads four consecutive k with one load) and add the waves'
// parts in LDS in a fixed order: 16 waves turn a weight gradient's sum over 2048
// rows, which had 16 workgroups of 64 x 64 outputs, into 128 workgroups of 8
// slices per wave.  Forward, loss and backward at 2048 rows: 1.54 ms with vector
// FMAs in 64 x 64 tiles, 0.13 ms with these (0.10 with the forward split as well,
// whose sums round differently).
constexpr int EPI_BIAS = 0, EPI_SILU = 1, EPI_SUM = 2;
typedef float f4 __attribute__((ext_vector_type(4)));

// four consecutive k (k0 .. k0 + 3) of row r of a matrix stored [rows][K]; zero outside
template <bool VEC>
__device__ __forceinline__ f4 load_k4(const float *__restrict X, int ld, int r, int rows, int k0, int K)
{
    f4 v = {0.0f, 0.0f, 0.0f, 0.0f};
    if (r >= rows) return v;
    const float *p = X + (size_t)r * ld + k0;
    if (VEC) {  // ld and K are multiples of 4 and X is 16-byte aligned
        if (k0 < K) v = *(const f4 *)p;
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (k0 + j < K) v[j] = p[j];
    }
    return v;
}
// the same of column c of a matrix stored [K][cols]
__device__ __forceinline__ f4 load_k4t(const float *__restrict X, int ld, int c, int cols, int k0, int K)
{
    f4 v = {0.0f, 0.0f, 0.0f, 0.0f};
    if (c >= cols) return v;
    const float *p = X + (size_t)k0 * ld + c;
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if (k0 + j < K) v[j] = p[(size_t)j * ld];
    return v;
}

// k = k0 + 4 s + g for s = 0 .. 3: the order in which one wave multiplies k by k
__device__ __forceinline__ f4 load_ordered(const float *__restrict X, size_t at, size_t step, bool in, int k, int K)
{
    f4 v = {0.0f, 0.0f, 0.0f, 0.0f};
    if (!in) return v;
#pragma unroll
    for (int s = 0; s < 4; ++s)
        if (k + 4 * s < K) v[s] = X[at + (size_t)(4 * s) * step];
    return v;
}

template <int TA, int TB, int EPI, int NW, bool VEC>
__global__ void __launch_bounds__(64 * NW) k_mm(const float *__restrict A, int lda, const float *__restrict B, int ldb,
                                                float *__restrict C, float *__restrict A_out,
                                                const float *__restrict aux, float *__restrict bsum, int M, int N,
                                                int K)
{
    static_assert(NW > 1 || (!TA && !TB), "one wave per tile: plain operands");
    __shared__ f4 part[NW][2][64];
    __shared__ float bpart[NW][2][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i = lane & 15, g = lane >> 4;
    const int m0 = blockIdx.y * 16, n0 = blockIdx.x * 32;
    f4 acc[2] = {{0.0f, 0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f, 0.0f}};
    float bs[2] = {0.0f, 0.0f};
    auto loadA = [&](int k0) {
        if constexpr (NW == 1) return load_ordered(A, (size_t)(m0 + i) * lda + k0 + g, 1, m0 + i < M, k0 + g, K);
        return TA ? load_k4t(A, lda, m0 + i, M, k0 + 4 * g, K) : load_k4<VEC>(A, lda, m0 + i, M, k0 + 4 * g, K);
    };
    auto loadB = [&](int k0, int h) {
        if constexpr (NW == 1) return load_ordered(B, (size_t)(k0 + g) * ldb + n0 + 16 * h + i, ldb, n0 + 16 * h + i < N, k0 + g, K);
        return TB ? load_k4<VEC>(B, ldb, n0 + 16 * h + i, N, k0 + 4 * g, K)
                  : load_k4t(B, ldb, n0 + 16 * h + i, N, k0 + 4 * g, K);
    };
    // the next slice's operands are in flight while this one's are multiplied
    int k0 = 16 * wave;
    f4 a = {}, b0 = {}, b1 = {};
    if (k0 < K) { a = loadA(k0); b0 = loadB(k0, 0); b1 = loadB(k0, 1); }
    while (k0 < K) {
        const int kn = k0 + 16 * NW;
        f4 an = {}, c0 = {}, c1 = {};
        if (kn < K) { an = loadA(kn); c0 = loadB(kn, 0); c1 = loadB(kn, 1); }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[j], b0[j], acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[j], b1[j], acc[1], 0, 0, 0);
        }
        if (EPI == EPI_SUM) {
            bs[0] += (b0[0] + b0[1]) + (b0[2] + b0[3]);
            bs[1] += (b1[0] + b1[1]) + (b1[2] + b1[3]);
        }
        a = an; b0 = c0; b1 = c1; k0 = kn;
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        part[wave][h][lane] = acc[h];
        if (EPI == EPI_SUM) bpart[wave][h][lane] = bs[h];
    }
    __syncthreads();
    // the 2 x 64 lanes' quarters of the tile: column n0 + 16 h + (l & 15), rows m0 + 4 (l >> 4) + r
    for (int x = threadIdx.x; x < 128; x += 64 * NW) {
        const int h = x >> 6, l = x & 63;
        f4 v = part[0][h][l];
        for (int w = 1; w < NW; ++w) v += part[w][h][l];
        const int n = n0 + 16 * h + (l & 15);
        if (n >= N) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = m0 + 4 * (l >> 4) + r;
            if (m >= M) continue;
            const size_t o = (size_t)m * N + n;
            float c = v[r];
            if (EPI == EPI_BIAS) {
                c += aux[n];
                if (A_out) A_out[o] = c / (1.0f + expf(-c));
            } else if (EPI == EPI_SILU) {
                // SiLU'(z) = s (1 + z (1 - s)), s = 1 / (1 + exp(-z))
                const float z = aux[o], sg = 1.0f / (1.0f + expf(-z));
                c *= sg * (1.0f + z * (1.0f - sg));
            }
            C[o] = c;
        }
        if (EPI == EPI_SUM && blockIdx.y == 0 && l < 16) {
            float t = 0.0f;
            for (int w = 0; w < NW; ++w)
                t += (bpart[w][h][l] + bpart[w][h][l + 16]) + (bpart[w][h][l + 32] + bpart[w][h][l + 48]);
            bsum[n] = t;
        }
    }
}

// The forward layer for many rows: a workgroup stages 16-deep slabs of 64 rows
// of X and 64 columns of W in LDS (the next slab's values on their way in
// registers meanwhile), and each of its four waves multiplies 16 rows by 64
// columns, k by k as above: the same bits.  Straight from L1/L2 a wave reads X
// four bytes of a row at a time and once per 32 columns, which bounds many rows:
// the guess network's forward pass at 60000 rows took 0.72 ms with waves alone
// (0.52 with vector FMAs on 64 x 64 tiles) and takes 0.31 with slabs, 67 TFLOP/s;
// one 1024 x 1024 layer of 16384 rows 1.04, 0.65 and 0.39 ms.
constexpr int TM = 64, TK = 16;
constexpr int SA = 20, SB = 80;  // row strides in LDS: a wave's reads touch every bank once
__global__ void __launch_bounds__(256) k_layer_tall(const float *__restrict X, const float *__restrict W,
                                                    const float *__restrict bias, float *__restrict out,
                                                    float *__restrict act, int M, int N, int K)
{
    __shared__ float As[TM * SA], Bs[TK * SB];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, i = lane & 15, g = lane >> 4;
    const int row0 = blockIdx.y * TM, n0 = blockIdx.x * TM;
    // this thread's elements of a slab: X at rows tx >> 4 + 16 r, W at k tx >> 6 + 4 r
    const int am = threadIdx.x >> 4, ak = threadIdx.x & 15, bk = threadIdx.x >> 6, bn = threadIdx.x & 63;
    float va[4], vb[4];
    auto load = [&](int k0) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = row0 + am + 16 * r;
            const int ka = k0 + ak, kb = k0 + bk + 4 * r;
            va[r] = m < M && ka < K ? X[(size_t)m * K + ka] : 0.0f;
            vb[r] = kb < K && n0 + bn < N ? W[(size_t)kb * N + n0 + bn] : 0.0f;
        }
    };
    f4 acc[4] = {};
    load(0);
    for (int k0 = 0; k0 < K; k0 += TK) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            As[(am + 16 * r) * SA + ak] = va[r];
            Bs[(bk + 4 * r) * SB + bn] = vb[r];
        }
        __syncthreads();
        if (k0 + TK < K) load(k0 + TK);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const float a = As[(16 * wave + i) * SA + 4 * s + g];
#pragma unroll
            for (int c = 0; c < 4; ++c)
                acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, Bs[(4 * s + g) * SB + 16 * c + i], acc[c], 0, 0, 0);
        }
        __syncthreads();
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int n = n0 + 16 * c + i;
        if (n >= N) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = row0 + 16 * wave + 4 * g + r;
            if (m >= M) continue;
            const float v = acc[c][r] + bias[n];
            out[(size_t)m * N + n] = v;
            if (act) act[(size_t)m * N + n] = v / (1.0f + expf(-v));
        }
    }
}

// Masked squared error over the (width x width) blocks of each row: entry
// (i, j) of row r counts if i < shape_r >> 8 and j < shape_r & 255.
// dY = 2 (Y - T) mask / count; per-workgroup partial sums of the squares.
constexpr int LB = 256;
__global__ void __launch_bounds__(LB) k_block_mse(const float *__restrict Y, const float *__restrict T,
                                                  const int *__restrict shape, int rows, int width, double inv_count,
                                                  float *__restrict dY, double *__restrict part)
{
    __shared__ double red[LB];
    const int m = width * width;
    const long long total = (long long)rows * m;
    double s = 0.0;
    for (long long e = (long long)blockIdx.x * LB + threadIdx.x; e < total; e += (long long)gridDim.x * LB) {
        const int r = (int)(e / m), k = (int)(e % m);
        const int i = k / width, j = k % width;
        const int sh = shape[r];
        float g = 0.0f;
        if (i < (sh >> 8) && j < (sh & 255)) {
            const double d = (double)Y[e] - (double)T[e];
            s += d * d;
            g = (float)(2.0 * d * inv_count);
        }
        dY[e] = g;
    }
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = LB / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

__global__ void __launch_bounds__(64) k_sum_parts(const double *__restrict part, int n, double scale, double *out)
{
    __shared__ double red[64];
    double s = 0.0;
    for (int i = threadIdx.x; i < n; i += 64) s += part[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = 32; w > 0; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = red[0] * scale;
}

// Adam (Kingma and Ba) with bias corrections c1 = 1 / (1 - b1^t), c2 = 1 / (1 - b2^t)
__global__ void __launch_bounds__(256) k_adam(float *__restrict W, const float *__restrict g, float *__restrict m1,
                                              float *__restrict m2, long long n, float lr, float b1, float b2,
                                              float eps, float c1, float c2)
{
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float a = b1 * m1[i] + (1.0f - b1) * gi;
    const float v = b2 * m2[i] + (1.0f - b2) * gi * gi;
    m1[i] = a;
    m2[i] = v;
    W[i] -= lr * (a * c1) / (sqrtf(v * c2) + eps);
}

// One workgroup per atom pair: L = T_1^T B T_2 with B the predicted
// bond-frame block (rows: functions of the pair's first atom) and T_k the
// block-diagonal rotation of atom k's Cartesian components, written to D at
// (first, second) and its transpose; an on-site block is symmetrised.
__global__ void __launch_bounds__(256) k_guess_scatter(const float *__restrict Y, const FkGuessPair *__restrict pairs,
                                                       const double *__restrict rot, int n, double *__restrict D)
{
    constexpr int W = FK_GUESS_NB;
    __shared__ double B[W][W + 1];
    __shared__ double H[W][W + 1];
    const FkGuessPair p = pairs[blockIdx.x];
    const double *T1 = rot + (size_t)blockIdx.x * 2 * W * W;
    const double *T2 = T1 + W * W;
    const int t = threadIdx.x;
    const int i = t / W, j = t % W;
    const bool act = t < W * W;
    if (act) B[i][j] = (i < p.n1 && j < p.n2) ? (double)Y[(size_t)blockIdx.x * W * W + t] : 0.0;
    __syncthreads();
    // H = B T_2
    if (act) {
        double v = 0.0;
        if (i < p.n1 && j < p.n2)
            for (int k = 0; k < p.n2; ++k) v += B[i][k] * T2[k * W + j];
        H[i][j] = v;
    }
    __syncthreads();
    // L = T_1^T H (kept in B)
    double v = 0.0;
    if (act && i < p.n1 && j < p.n2)
        for (int k = 0; k < p.n1; ++k) v += T1[k * W + i] * H[k][j];
    __syncthreads();
    if (act) B[i][j] = v;
    __syncthreads();
    if (!act || i >= p.n1 || j >= p.n2) return;
    if (p.a1 == p.a2) {
        D[(size_t)(p.f1 + i) * n + p.f2 + j] = 0.5 * (B[i][j] + B[j][i]);
    } else {
        D[(size_t)(p.f1 + i) * n + p.f2 + j] = B[i][j];
        D[(size_t)(p.f2 + j) * n + p.f1 + i] = B[i][j];
    }
}

__global__ void __launch_bounds__(256) k_fill(double *__restrict p, long long n)
{
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = 0.0;
}

int ok() { return hipGetLastError() == hipSuccess ? 0 : -3; }

unsigned nblk(long long n) { return (unsigned)((n + 255) / 256); }

// Rows per launch of the products whose rows are a call's: at 16 to a tile half
// of what a grid's y may count (65535).  Rows on z as well would cost a call of
// few rows 0.3 us per kernel, which then has to find out whether its tile exists.
constexpr long long MAX_ROWS = 1 << 19;

template <int TA, int TB, int EPI, int NW>
int mm(const float *A, int lda, const float *B, int ldb, float *C, float *A_out, const float *aux, float *bsum, int M,
       int N, int K, void *stream)
{
    if (M <= 0 || N <= 0) return 0;
    const dim3 grid((N + 31) / 32, (M + 15) / 16);
    // both operands read along k (the input gradient): four values with one load
    // where every row starts aligned
    constexpr bool along_k = !TA && TB;
    if (along_k && K % 4 == 0 && lda % 4 == 0 && ldb % 4 == 0 && (uintptr_t)A % 16 == 0 && (uintptr_t)B % 16 == 0)
        hipLaunchKernelGGL((k_mm<TA, TB, EPI, NW, along_k>), grid, dim3(64 * NW), 0, (hipStream_t)stream, A, lda, B, ldb, C,
                           A_out, aux, bsum, M, N, K);
    else
        hipLaunchKernelGGL((k_mm<TA, TB, EPI, NW, false>), grid, dim3(64 * NW), 0, (hipStream_t)stream, A, lda, B, ldb, C,
                           A_out, aux, bsum, M, N, K);
    return ok();
}

}  // namespace

extern "C" {

// out[M][N] = X[M][K] W[K][N] + bias; act (if not null) its SiLU
int fk_guess_layer(const float *X, const float *W, const float *bias, float *out, float *act, int M, int N, int K,
                   void *stream)
{
    // Slabs from 128 tiles of 64 x 64 outputs on, half a tile per CU; below, sixteen-row
    // waves fill more of the chip.  256 x 256 layer, waves and slabs: 1000 rows (64 tiles)
    // 14.0 and 15.6 us, 1500 (96) 14.6 and 15.7, 2048 (128) 16.8 and 15.9, 4096 27.3 and
    // 16.5; 1024 x 1024: 100 rows (32) 40.6 and 47.4, 500 (128) 51.0 and 47.0.
    const int ct = (N + TM - 1) / TM;
    for (long long r = 0; r < M; r += MAX_ROWS) {
        const int rows = (int)std::min(MAX_ROWS, M - r), rt = (rows + TM - 1) / TM;
        const float *x = X + r * K;
        float *y = out + r * N, *a = act ? act + r * N : nullptr;
        if (rt * ct >= 128)
            hipLaunchKernelGGL(k_layer_tall, dim3(ct, rt), dim3(256), 0, (hipStream_t)stream, x, W, bias, y, a, rows, N, K);
        else if (mm<0, 0, EPI_BIAS, 1>(x, K, W, N, y, a, bias, nullptr, rows, N, K, stream))
            return -3;
    }
    return ok();
}

// out[M][N] = (G[M][K] W^T) SiLU'(Z), W stored [N][K]
int fk_guess_layer_back(const float *G, const float *W, const float *Z, float *out, int M, int N, int K, void *stream)
{
    for (long long r = 0; r < M; r += MAX_ROWS)
        if (mm<0, 1, EPI_SILU, 4>(G + r * K, K, W, K, out + r * N, nullptr, Z + r * N, nullptr,
                                  (int)std::min(MAX_ROWS, M - r), N, K, stream))
            return -3;
    return 0;
}

// gW[M][N] = X^T G and gb[N] = column sums of G, X stored [rows][M], G [rows][N]
int fk_guess_layer_grad(const float *X, const float *G, float *gW, float *gb, int M, int N, int rows, void *stream)
{
    return mm<1, 0, EPI_SUM, 16>(X, M, G, N, gW, nullptr, nullptr, gb, M, N, rows, stream);
}

int fk_guess_mse_parts() { return 480; }

int fk_guess_block_mse(const float *Y, const float *T, const int *shape, int rows, int width, double count, float *dY,
                       double *part, double *loss, void *stream)
{
    if (rows <= 0) return 0;
    const long long total = (long long)rows * width * width;
    const int g = (int)std::min<long long>(fk_guess_mse_parts(), (total + LB - 1) / LB);
    hipLaunchKernelGGL(k_block_mse, dim3(g), dim3(LB), 0, (hipStream_t)stream, Y, T, shape, rows, width,
                       1.0 / count, dY, part);
    if (ok()) return -3;
    hipLaunchKernelGGL(k_sum_parts, dim3(1), dim3(64), 0, (hipStream_t)stream, part, g, 1.0 / count, loss);
    return ok();
}

int fk_guess_adam(float *W, const float *g, float *m1, float *m2, long long n, float lr, float b1, float b2, float eps,
                  float c1, float c2, void *stream)
{
    if (n <= 0) return 0;
    hipLaunchKernelGGL(k_adam, dim3(nblk(n)), dim3(256), 0, (hipStream_t)stream, W, g, m1, m2, n, lr, b1, b2, eps, c1,
                       c2);
    return ok();
}

int fk_guess_scatter(const float *Y, const FkGuessPair *pairs, const double *rot, int npair, int n, double *D,
                     void *stream)
{
    const long long nn = (long long)n * n;
    if (nn <= 0) return 0;
    hipLaunchKernelGGL(k_fill, dim3(nblk(nn)), dim3(256), 0, (hipStream_t)stream, D, nn);
    if (ok()) return -3;
    if (npair <= 0) return 0;
    hipLaunchKernelGGL(k_guess_scatter, dim3(npair), dim3(256), 0, (hipStream_t)stream, Y, pairs, rot, n, D);
    return ok();
}

}  // extern "C"
