// Element-wise kernels on the r x r cores and the small fp64 factorizations used by the
// subspace refresh (Cholesky + triangular inverse for the thin QR, one-sided Jacobi SVD).
#include "small.h"

#include "device_lds.h"

namespace tsr {

// ------------------------------------------------------------------ Adam on the core
// m <- b1 m + (1-b1) c ; v <- b2 v + (1-b2) c^2 ; d = (m/c1) / (sqrt(v/c2) + eps)
__global__ __launch_bounds__(256) void adam_kernel(const CoreBlock* table, const CoreBlock single,
                                                   const AdamScalars s) {
    const CoreBlock* b = table ? table + blockIdx.y : &single;
    const float* C = b->C;
    float* __restrict__ M = b->M;
    float* __restrict__ Vm = b->Vm;
    float* D = b->D;
    const long long n = b->count;
    const float omb1 = 1.0f - s.beta1, omb2 = 1.0f - s.beta2;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x) {
        const float g = C[i];
        const float m = s.beta1 * M[i] + omb1 * g;
        const float v = s.beta2 * Vm[i] + omb2 * (g * g);
        M[i] = m;
        Vm[i] = v;
        D[i] = (m * s.inv_c1) / (sqrtf(v * s.inv_c2) + s.eps);
    }
}

hipError_t launch_adam(const CoreBlock* table_dev, const CoreBlock* single, int blocks, long long max_count,
                       const AdamScalars& s, hipStream_t stream) {
    if (blocks <= 0 || max_count <= 0) return hipSuccess;
    long long bx = (max_count + 255) / 256;
    if (bx > 2048) bx = 2048;
    CoreBlock sb{};
    if (single) sb = *single;
    hipLaunchKernelGGL(adam_kernel, dim3((unsigned)bx, blocks), dim3(256), 0, stream, table_dev, sb, s);
    return hipGetLastError();
}

// 32 x 32 patch per workgroup (256 threads = 32 x 8): coalesced reads and writes of the fp32
// arrays, LDS transpose for the bf16 D^T.
__global__ __launch_bounds__(256) void adam_t_kernel(const AdamTBlock* table, const AdamScalars s) {
    const AdamTBlock b = table[blockIdx.z];
    const int r = b.r;
    const int row0 = blockIdx.y * 32, col0 = blockIdx.x * 32;
    if (row0 >= r || col0 >= r) return;
    __shared__ unsigned short tile[32][34];
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    const float omb1 = 1.0f - s.beta1, omb2 = 1.0f - s.beta2;
    for (int i = ty; i < 32; i += 8) {
        const int row = row0 + i, col = col0 + tx;
        float d = 0.0f;
        if (row < r && col < r) {
            const long long idx = (long long)row * r + col;
            const float g = b.C[idx];
            const float m = s.beta1 * b.M[idx] + omb1 * g;
            const float v = s.beta2 * b.Vm[idx] + omb2 * (g * g);
            b.M[idx] = m;
            b.Vm[idx] = v;
            d = (m * s.inv_c1) / (sqrtf(v * s.inv_c2) + s.eps);
            b.D[idx] = d;
        }
        __bf16 h = (__bf16)d;
        tile[i][tx] = __builtin_bit_cast(unsigned short, h);
        if (b.Db && row < r && col < r) ((unsigned short*)b.Db)[(long long)row * b.ldt + col] = tile[i][tx];
    }
    __syncthreads();
    unsigned short* DT = (unsigned short*)b.DTb;
    unsigned short* DF = (unsigned short*)b.DTf;
    const int ksteps = r / 16;
    for (int i = ty; i < 32; i += 8) {
        const int trow = col0 + i, tcol = row0 + tx;     // D^T[col][row]
        if (trow < r && tcol < r) {
            if (DF) DF[(((long long)(trow / 32) * ksteps + tcol / 16) * 64 + ((tcol % 16) / 8) * 32 + trow % 32) * 8 + tcol % 8] = tile[tx][i];
            else DT[(long long)trow * b.ldt + tcol] = tile[tx][i];
        }
    }
}

hipError_t launch_adam_t(const AdamTBlock* table_dev, int blocks, int max_r, const AdamScalars& s,
                         hipStream_t stream) {
    if (blocks <= 0 || max_r <= 0) return hipSuccess;
    const int g = (max_r + 31) / 32;
    hipLaunchKernelGGL(adam_t_kernel, dim3(g, g, blocks), dim3(256), 0, stream, table_dev, s);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void sgd_kernel(const float* C, float* M, float* D, long long n, float beta) {
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x) {
        const float m = beta * M[i] + (1.0f - beta) * C[i];
        M[i] = m;
        D[i] = m;
    }
}

hipError_t launch_sgd(const float* C, float* M, float* D, long long count, float beta, hipStream_t stream) {
    if (count <= 0) return hipSuccess;
    long long bx = (count + 255) / 256;
    if (bx > 4096) bx = 4096;
    hipLaunchKernelGGL(sgd_kernel, dim3((unsigned)bx), dim3(256), 0, stream, C, M, D, count, beta);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void average_kernel(const float* Cs, int K, long long n, float* out) {
    const float inv = 1.0f / (float)K;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x) {
        float s = 0.0f;
        for (int w = 0; w < K; ++w) s += Cs[(long long)w * n + i];
        out[i] = s * inv;
    }
}

hipError_t launch_average(const float* Cs, int K, long long count, float* out, hipStream_t stream) {
    if (count <= 0) return hipSuccess;
    long long bx = (count + 255) / 256;
    if (bx > 4096) bx = 4096;
    hipLaunchKernelGGL(average_kernel, dim3((unsigned)bx), dim3(256), 0, stream, Cs, K, count, out);
    return hipGetLastError();
}

// ------------------------------------------------------------------ helpers of the exact-SVD refresh
// out (k x k fp32) = identity
__global__ __launch_bounds__(256) void identity_kernel(float* out, int k) {
    const long long n = (long long)k * k;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x)
        out[i] = (i / k == i % k) ? 1.0f : 0.0f;
}

hipError_t launch_identity(float* out, int k, hipStream_t stream) {
    if (k <= 0) return hipSuccess;
    long long bx = ((long long)k * k + 255) / 256;
    if (bx > 4096) bx = 4096;
    hipLaunchKernelGGL(identity_kernel, dim3((unsigned)bx), dim3(256), 0, stream, out, k);
    return hipGetLastError();
}

// The gradient as a tall contiguous fp32 matrix: out = G (rows x cols -> rows x cols) or, with
// transpose, out = G^T (cols x rows), through a 32 x 33 LDS tile so that both sides are coalesced.
template <bool BF16>
__global__ __launch_bounds__(256) void tall_copy_kernel(const void* G, long long ldg, int rows, int cols, int transpose,
                                                        float* out) {
    __shared__ float tile[32][33];
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    const int r0 = blockIdx.y * 32, c0 = blockIdx.x * 32;
    for (int i = ty; i < 32; i += 8) {
        const int r = r0 + i, c = c0 + tx;
        float v = 0.0f;
        if (r < rows && c < cols) {
            if constexpr (BF16) v = __uint_as_float(((unsigned)((const unsigned short*)G)[(long long)r * ldg + c]) << 16);
            else v = ((const float*)G)[(long long)r * ldg + c];
        }
        tile[i][tx] = v;
    }
    __syncthreads();
    for (int i = ty; i < 32; i += 8) {
        if (transpose) {
            const int c = c0 + i, r = r0 + tx;             // out[c][r]
            if (c < cols && r < rows) out[(long long)c * rows + r] = tile[tx][i];
        } else {
            const int r = r0 + i, c = c0 + tx;
            if (r < rows && c < cols) out[(long long)r * cols + c] = tile[i][tx];
        }
    }
}

hipError_t launch_tall_copy(const void* G, int g_bf16, long long ldg, int rows, int cols, int transpose, float* out,
                            hipStream_t stream) {
    if (rows <= 0 || cols <= 0) return hipSuccess;
    dim3 grid((cols + 31) / 32, (rows + 31) / 32);
    if (g_bf16) hipLaunchKernelGGL(tall_copy_kernel<true>, grid, dim3(256), 0, stream, G, ldg, rows, cols, transpose, out);
    else hipLaunchKernelGGL(tall_copy_kernel<false>, grid, dim3(256), 0, stream, G, ldg, rows, cols, transpose, out);
    return hipGetLastError();
}

// ------------------------------------------------------------------ stream calibration
typedef __attribute__((ext_vector_type(4))) float f32x4_s;
__global__ __launch_bounds__(256) void stream_kernel(f32x4_s* dst, const f32x4_s* src, long long n4, float scale) {
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n4;
         i += (long long)gridDim.x * blockDim.x) {
        f32x4_s v = src[i];
        dst[i] = v * scale;
    }
}

hipError_t launch_stream(float* dst, const float* src, long long count, float scale, hipStream_t stream) {
    const long long n4 = count / 4;
    if (n4 <= 0) return hipSuccess;
    long long bx = (n4 + 255) / 256;
    if (bx > 256 * 32) bx = 256 * 32;
    hipLaunchKernelGGL(stream_kernel, dim3((unsigned)bx), dim3(256), 0, stream, (f32x4_s*)dst, (const f32x4_s*)src, n4,
                       scale);
    return hipGetLastError();
}

// ------------------------------------------------------------------ Gram matrix in fp64
// One 32 x 32 tile on or below the diagonal per wave and range of rows (2 x 2 fp64 MFMAs, v_mfma_f64_16x16x4), four
// tiles in row order per workgroup.  Both operands come as they lie in memory: a
// lane's element of a 4 x 16 operand is one float, four rows of 64 bytes per load, sixteen rows under way while the
// last sixteen are multiplied (1024 cycles of MFMAs against sixteen loads), so neither LDS nor more bandwidth is asked
// for: bound by the matrix cores' fp64 rate (168 matrices of together 467 000 rows, k = 528: 3.0 ms, 49 TFLOP/s; as four
// quadrants of a 64 x 64 tile, of which those above the diagonal and beyond the matrix leave a SIMD idle, 3.3 ms).
__global__ __launch_bounds__(256) void gram64_kernel(const Gram64Block* table, const Gram64Block single, const int workgroups) {
    typedef double d4_t __attribute__((ext_vector_type(4)));
    typedef const float __attribute__((address_space(1))) gfloat;
    Gram64Block b = single;
    if (table) b = table[blockIdx.y];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, li = lane & 15, lk = lane >> 4;
    const int split = blockIdx.x / workgroups, t = __builtin_amdgcn_readfirstlane(4 * (blockIdx.x % workgroups) + wave);
    int qi = (int)((sqrtf(8.0f * (float)t + 1.0f) - 1.0f) * 0.5f);
    while ((qi + 1) * (qi + 2) / 2 <= t) ++qi;
    while (qi * (qi + 1) / 2 > t) --qi;
    const int i0 = 32 * qi, j0 = 32 * (t - qi * (qi + 1) / 2);
    if (split >= b.splits || i0 >= b.k) return;
    const int begin = split * b.chunk, end = min(b.rows, begin + b.chunk);
    gfloat* X = (gfloat*)b.X;
    unsigned ci[2], cj[2];
#pragma unroll
    for (int f = 0; f < 2; ++f) {
        ci[f] = min(i0 + 16 * f + li, b.k - 1);
        cj[f] = min(j0 + 16 * f + li, b.k - 1);
    }
    d4_t acc[2][2] = {};
    float a[2][4][2], c[2][4][2];
    auto fetch = [&](int s, int r0) {                          // rows past the range: clamped here, cleared when used
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            gfloat* row = X + (size_t)min(r0 + 4 * q + lk, end - 1) * b.k;
#pragma unroll
            for (int f = 0; f < 2; ++f) { a[s][q][f] = row[ci[f]]; c[s][q][f] = row[cj[f]]; }
        }
    };
    auto multiply = [&](int s, int r0, bool whole) {           // (selects in the loop cost a tenth of the time)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const bool in = whole || r0 + 4 * q + lk < end;
            double x[2], y[2];
#pragma unroll
            for (int f = 0; f < 2; ++f) { x[f] = in ? (double)a[s][q][f] : 0.0; y[f] = in ? (double)c[s][q][f] : 0.0; }
#pragma unroll
            for (int f = 0; f < 2; ++f)
#pragma unroll
                for (int g = 0; g < 2; ++g) acc[f][g] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[f], y[g], acc[f][g], 0, 0, 0);
        }
    };
    if (begin < end) {
        fetch(0, begin);
        int r = begin;
        for (; r + 32 <= end; r += 32) {
            fetch(1, r + 16);
            multiply(0, r, true);
            fetch(0, r + 32);
            multiply(1, r + 16, true);
        }
        if (r < end) {
            fetch(1, r + 16);
            multiply(0, r, false);
            multiply(1, r + 16, false);
        }
    }
    double* out = b.splits > 1 ? b.part + (size_t)split * b.k * b.k : b.S;
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
        for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int i = i0 + 16 * f + 4 * v + lk, j = j0 + 16 * g + li;
                if (i < b.k && j <= i) out[(size_t)i * b.k + j] = acc[f][g][v];
            }
}

__global__ __launch_bounds__(256) void gram64_sum_kernel(const Gram64Block* table, const Gram64Block single) {
    Gram64Block b = single;
    if (table) b = table[blockIdx.y];
    const int n = b.k * b.k, i = blockIdx.x * 256 + threadIdx.x;
    if (b.splits <= 1 || i >= n || i % b.k > i / b.k) return;
    double s = 0.0;
    int p = 0;
    for (; p + 8 <= b.splits; p += 8) {
        double x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = b.part[(size_t)(p + u) * n + i];
#pragma unroll
        for (int u = 0; u < 8; ++u) s += x[u];
    }
    for (; p < b.splits; ++p) s += b.part[(size_t)p * n + i];
    b.S[i] = s;
}

hipError_t launch_gram64(const Gram64Block* table_dev, const Gram64Block* single, int blocks, int max_k, int max_splits,
                         hipStream_t stream) {
    if (blocks <= 0 || max_k <= 0) return hipSuccess;
    Gram64Block sb{};
    if (single) sb = *single;
    const int workgroups = gram64_workgroups(max_k);
    hipLaunchKernelGGL(gram64_kernel, dim3(workgroups * max_splits, blocks), dim3(256), 0, stream, table_dev, sb, workgroups);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || max_splits <= 1) return e;
    hipLaunchKernelGGL(gram64_sum_kernel, dim3((max_k * max_k + 255) / 256, blocks), dim3(256), 0, stream, table_dev, sb);
    return hipGetLastError();
}

// ------------------------------------------------------------------ product with the inverse factor in fp64
// One 64 x 64 tile of X Rinv per workgroup, 32 x 32 per wave, over the rows of Rinv that are not zero there.  Four
// columns of X per lane and load (a row's sixteen side by side), Rinv as it lies; k step q of a load is column 4 l + q
// for the lanes of group l, of either operand.  Bound by the matrix cores' fp64 rate like the Gram matrices.
// 168 matrices of together 467 000 rows, k = 528: 2.7 ms, 54 TFLOP/s (the Gram matrices of the same 3.0 ms); asking
// for fewer than four workgroups per compute unit lets the accumulators move through both register files in every
// step, 2.9 ms.  The refreshes of the 60M, 130M and 1B models take 3.99, 5.53 and 84.8 ms with the two fp64
// passes; 3.86, 5.30 and 79.3 ms with the products in two and three bf16 pieces, which lose weak directions (see
// ORTH_SHIFT in api.hip), and 4.52, 6.35 and 87.6 ms with three passes of those.
__global__ __launch_bounds__(256, 4) void apply64_kernel(const Apply64Block* table, const Apply64Block single, const int col_tiles) {
    typedef double d4_t __attribute__((ext_vector_type(4)));
    typedef float f4_t __attribute__((ext_vector_type(4)));
    typedef f4_t f4u_t __attribute__((aligned(4)));
    typedef const float __attribute__((address_space(1))) gfloat;
    typedef const f4u_t __attribute__((address_space(1))) gf4u;
    Apply64Block b = single;
    if (table) b = table[blockIdx.y];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, li = lane & 15, lk = lane >> 4, k = b.k;
    const int i0 = (int)(blockIdx.x / col_tiles) * 64 + (wave >> 1) * 32;
    const int j0 = (col_tiles - 1 - (int)(blockIdx.x % col_tiles)) * 64 + (wave & 1) * 32;      // (most work first)
    if (i0 >= b.rows || j0 >= k) return;
    const int end = min(k, j0 + 32), steps = min(end, k / 16 * 16) / 16;
    gfloat* X = (gfloat*)b.X;
    gfloat* R = (gfloat*)b.Rinv;
    size_t row[2];
    unsigned col[2];
#pragma unroll
    for (int f = 0; f < 2; ++f) {
        row[f] = (size_t)min(i0 + 16 * f + li, b.rows - 1) * k;
        col[f] = min(j0 + 16 * f + li, k - 1);
    }
    d4_t acc[2][2] = {};
    f4_t a[2][2];
    float c[2][4][2];
    auto fetch = [&](int s, int t) {
        const int kk = 16 * min(t, steps - 1) + 4 * lk;
#pragma unroll
        for (int f = 0; f < 2; ++f) a[s][f] = *(gf4u*)(X + row[f] + kk);
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int g = 0; g < 2; ++g) c[s][q][g] = R[(size_t)(kk + q) * k + col[g]];
    };
    auto multiply = [&](int s) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int f = 0; f < 2; ++f)
#pragma unroll
                for (int g = 0; g < 2; ++g)
                    acc[f][g] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)a[s][f][q], (double)c[s][q][g], acc[f][g], 0, 0, 0);
    };
    if (steps > 0) {
        fetch(0, 0);
        for (int t = 0; t + 1 < steps; t += 2) {
            fetch(1, t + 1);
            multiply(0);
            fetch(0, t + 2);
            multiply(1);
        }
        if (steps & 1) multiply(0);
    }
    if (16 * steps < end) {                                    // the last columns of X, fewer than sixteen
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int kk = 16 * steps + 4 * lk + q, at = min(kk, k - 1);
#pragma unroll
            for (int f = 0; f < 2; ++f) {
                a[0][f][q] = kk < k ? X[row[f] + at] : 0.0f;
                c[0][q][f] = kk < k ? R[(size_t)at * k + col[f]] : 0.0f;
            }
        }
        multiply(0);
    }
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
        for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int i = i0 + 16 * f + 4 * v + lk, j = j0 + 16 * g + li;
                if (i < b.rows && j < k) b.out[(size_t)i * k + j] = (float)acc[f][g][v];
            }
}

hipError_t launch_apply64(const Apply64Block* table_dev, const Apply64Block* single, int blocks, int max_rows, int max_k,
                          hipStream_t stream) {
    if (blocks <= 0 || max_rows <= 0 || max_k <= 0) return hipSuccess;
    Apply64Block sb{};
    if (single) sb = *single;
    const int ct = (max_k + 63) / 64;
    hipLaunchKernelGGL(apply64_kernel, dim3((max_rows + 63) / 64 * ct, blocks), dim3(256), 0, stream, table_dev, sb, ct);
    return hipGetLastError();
}

// ------------------------------------------------------------------ Cholesky + inverse
constexpr int SMALL_THREADS = 1024;
constexpr int SMALL_MAXK = 1024;

__device__ inline double gram_entry(const CholBlock& b, size_t at) { return b.S64 ? b.S64[at] : (double)b.S[at]; }

// shift_rel * (largest diagonal entry of the k x k matrix S), computed by the whole workgroup
__device__ inline double diagonal_shift(const CholBlock& b, int k, double shift_rel) {
    __shared__ double s_wave_max[SMALL_THREADS / 64];
    __shared__ double s_shift;
    const int tid = threadIdx.x, nt = blockDim.x;
    double mx = 0.0;
    for (int j = tid; j < k; j += nt) mx = fmax(mx, gram_entry(b, (size_t)j * k + j));
    for (int off = 32; off > 0; off >>= 1) mx = fmax(mx, __shfl_xor(mx, off));
    if ((tid & 63) == 0) s_wave_max[tid >> 6] = mx;
    __syncthreads();
    if (tid == 0) {
        double m = 0.0;
        for (int w = 0; w < (nt >> 6); ++w) m = fmax(m, s_wave_max[w]);
        s_shift = shift_rel * m;
    }
    __syncthreads();
    return s_shift;
}

__global__ __launch_bounds__(SMALL_THREADS) void chol_inv_kernel(const CholBlock* table, const CholBlock single,
                                                                 const double tol, const double shift_rel) {
    const CholBlock* blk = table ? table + blockIdx.x : &single;
    const int k = blk->k;
    double* A = blk->work;                     // lower triangle becomes L, S = L L^T
    double* X = blk->work + (size_t)k * k;     // X = L^-1 (lower)
    const int tid = threadIdx.x, nt = blockDim.x;
    const int lane = tid & 63, wave = tid >> 6, nw = nt >> 6;
    __shared__ double colj[SMALL_MAXK];
    __shared__ double s_invd;

    const double shift = diagonal_shift(*blk, k, shift_rel);
    for (int idx = tid; idx < k * k; idx += nt) A[idx] = gram_entry(*blk, idx) + ((idx / k == idx % k) ? shift : 0.0);
    __syncthreads();

    for (int j = 0; j < k; ++j) {
        if (tid == 0) {
            const double a = A[(size_t)j * k + j];
            const double s0 = gram_entry(*blk, (size_t)j * k + j);
            if (a > 0.0 && a > tol * s0) {
                const double d = sqrt(a);
                A[(size_t)j * k + j] = d;
                s_invd = 1.0 / d;
            } else {                            // dependent column: drop it
                A[(size_t)j * k + j] = 0.0;
                s_invd = 0.0;
            }
        }
        __syncthreads();
        const double invd = s_invd;
        for (int i = j + 1 + tid; i < k; i += nt) {
            const double v = A[(size_t)i * k + j] * invd;
            A[(size_t)i * k + j] = v;
            colj[i] = v;
        }
        __syncthreads();
        if (invd != 0.0) {
            for (int i = j + 1 + wave; i < k; i += nw) {
                const double li = colj[i];
                double* row = A + (size_t)i * k;
                for (int c = j + 1 + lane; c <= i; c += 64) row[c] -= li * colj[c];
            }
        }
        __syncthreads();
    }

    // X = L^-1 by forward substitution, one column per thread (entries above the diagonal
    // come out as exact zeros, which keeps every lane on the same (i, j))
    for (int c = tid; c < k; c += nt) {
        for (int i = 0; i < k; ++i) {
            double s = (i == c) ? 1.0 : 0.0;
            const double* row = A + (size_t)i * k;
            for (int j = 0; j < i; ++j) s -= row[j] * X[(size_t)j * k + c];
            const double d = row[i];
            X[(size_t)i * k + c] = (d != 0.0) ? s / d : 0.0;
        }
    }
    __syncthreads();

    // Rinv = X^T (upper triangular), fp32
    float* Rinv = blk->Rinv;
    for (int idx = tid; idx < k * k; idx += nt) {
        const int a = idx / k, b = idx % k;
        Rinv[idx] = (a <= b) ? (float)X[(size_t)b * k + a] : 0.0f;
    }
    // Rtot = R = L^T
    double* Rtot = blk->Rtot;
    if (Rtot != nullptr) {
        for (int idx = tid; idx < k * k; idx += nt) {
            const int a = idx / k, b = idx % k;
            Rtot[idx] = (a <= b) ? A[(size_t)b * k + a] : 0.0;
        }
    }
}

__device__ inline double readlane_f64(double v, int lane) {      // lane: a compile-time constant
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), lane);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), lane);
    return __hiloint2double(hi, lo);
}

// Variant for k <= 272, one launch: factor and inverse of one matrix in the registers of one workgroup.
// The lower triangle is cut into 16 x 16 tiles, each owned by a wave in the fp64 MFMA accumulator layout
// (v_mfma_f64_16x16x4: lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16], receives
// D[4 v + l / 16][l % 16]).  At step J the row and column through the diagonal tile J are finished
//     L_IJ = A_IJ Li_J^T (I > J)          X_Jc = Li_J E_Jc (c < J),   Li_J = L_JJ^-1
// and shared through LDS; then every tile below row J takes its update
//     A_IK -= L_IJ L_KJ^T (K > J)         E_Ic -= L_IJ X_Jc (c <= J)
// where the tile of column c, done as part of L after step c, holds E, the part of the inverse under way,
// from then on.  With the tiles and X held transposed both updates are the same product, slot K times the
// transpose of slot I.  So nothing but the input and the results touches memory, and the inverse costs no
// launches of its own.  What bounds it up to k = 144 is the serial chain of the diagonal tiles, above that the fp64
// products of the early steps (64 cycles of a SIMD per 16 x 16 x 4).  The last wave has
// no tiles of its own: it takes the next diagonal tile through LDS and factors it while the others work on theirs,
// four columns at a time with products between (3600 cycles; a column at a time, with broadcasts of every entry by
// v_readlane, took 7300, and 11 500 beside a wave with products).
// Per call, one matrix per compute unit, before -> with that: k = 72 29.5 -> 17.1 us (eight waves; with four 19.4),
// k = 136 63 -> 38.8 us, k = 264 172 -> 138 us (twelve waves; eight 161, sixteen 159).  272 is where the tiles fill
// the registers; larger matrices (up to 544) are cut in two:
//     [S11    ]   the kernel on S11 (PART 1), L21 = S21 Li1^T, S22 - L21 L21^T, the kernel on that (PART 2);
//     [S21 S22]   the inverse below the diagonal is -Li2 (L21 Li1).
// (In two halves from 160 on it takes 115 / 130 us for one matrix of k = 264, but 150 / 137 for 56 and at k = 200
// 87 / 83 and 103 / 88.)
// The products (fp64 MFMAs, 64 x 64 tiles over the whole chip) and Li1, Li2 go through `work`.  The variant this
// replaces, 32-wide block columns of a matrix in memory, spent one workgroup's chain on all of it.
// Per call at k = 528, 56 matrices, the other groups of a refresh running beside it: 1.29 + 0.69 + 0.18 ms in
// three launches -> 0.35 + 0.21 + 0.25 + 0.25 + 0.17 ms in five; refresh of the 1B model 107.8 -> 96.3 ms.
constexpr int CT = 16;
constexpr int CT_P = CT + 2;                   // LDS row: 144 bytes, operand reads free of bank conflicts
constexpr int CT_MAXK = 272;
constexpr int NEG_A = 1;                       // of a double-precision MFMA: the left operand negated

// Workgroup barrier that orders LDS only: the results on their way to global memory are not waited for.
__device__ inline void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Leading part of a matrix cut in two: whole tiles, both parts at most CT_MAXK for k up to 2 CT_MAXK.
__host__ __device__ inline int chol_lead(int k) { return min(((k + 1) / 2 + CT - 1) / CT * CT, k); }

// PART 0: the whole matrix; 1: its leading part; 2: the trailing part, whose lower triangle (less L21 L21^T) is
// in `work`.  Parts leave their inverse in the second half of `work` as well, in fp64.
template <int NT, int WAVES, int PART>
__global__ __launch_bounds__(64 * WAVES, 1) void chol_tiles_kernel(const CholBlock* table, const CholBlock single,
                                                                    const double tol, const double shift_rel) {
    constexpr int SLOTS = (NT * (NT + 1) / 2 + WAVES - 2) / (WAVES - 1);   // tiles per wave; the last wave has none
    constexpr int TILE = CT * CT_P * 8;                        // bytes of a tile in LDS
    typedef double d4_t __attribute__((ext_vector_type(4)));
    typedef double tile_t[CT][CT_P];
    extern __shared__ double smem[];
    // two buffers of NT tiles; slot x of step J: L_xJ (x > J), X_Jx^T (x <= J)
    tile_t* raw = (tile_t*)smem + 2 * NT;                      // the next diagonal tile, two buffers
    tile_t* low_diag = raw + 2;                                // L_JJ, two buffers
    double* s_diag = smem + (2 * NT + 4) * CT * CT_P;          // diagonal of S

    CholBlock cb = single;
    if (table) cb = table[blockIdx.x];
    const int ld = cb.k;
    const int lead = chol_lead(ld);
    const int k = PART == 0 ? ld : PART == 1 ? lead : ld - lead;
    if (k <= 0) return;
    const size_t first = PART == 2 ? (size_t)lead * ld + lead : 0;
    const int nt = (k + CT - 1) / CT;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, lk = lane >> 4;
    typedef const float __attribute__((address_space(1))) gfloat;
    typedef double __attribute__((address_space(1))) gdouble;
    gfloat* S = (gfloat*)cb.S;
    const gdouble* S64 = (const gdouble*)cb.S64;
    auto entry = [&](size_t at) { return S64 ? (double)S64[at] : (double)S[at]; };   // of the whole matrix
    float __attribute__((address_space(1)))* Rinv = (float __attribute__((address_space(1)))*)cb.Rinv + first;
    gdouble* Rtot = cb.Rtot ? (gdouble*)cb.Rtot + first : nullptr;
    const gdouble* A = (const gdouble*)cb.work + first;
    gdouble* X = (gdouble*)cb.work + (size_t)ld * ld + first;

    // diagonal of S to LDS; the shift; zeros below the block diagonal of both results
    auto diagonal_shift_tiles = [&]() {
        double mx = 0.0;
        for (int j = tid; j < nt * CT; j += 64 * WAVES) {
            const double d = (j < k) ? entry(first + (size_t)j * ld + j) : 1.0;
            s_diag[j] = d;
            if (PART == 0 && j < k) mx = fmax(mx, d);
        }
        if (PART != 0)                                         // the shift is one for the whole matrix
            for (int j = tid; j < ld; j += 64 * WAVES) mx = fmax(mx, entry((size_t)j * ld + j));
        for (int off = 32; off > 0; off >>= 1) mx = fmax(mx, __shfl_xor(mx, off));
        if (lane == 0) smem[wave] = mx;
        lds_barrier();
        mx = smem[0];
#pragma unroll
        for (int w = 1; w < WAVES; ++w) mx = fmax(mx, smem[w]);
        lds_barrier();
        for (int a = CT + wave; a < k; a += WAVES)
            for (int b = lane; b < a / CT * CT; b += 64) {
                Rinv[(size_t)a * ld + b] = 0.0f;
                if (Rtot) Rtot[(size_t)a * ld + b] = 0.0;
            }
        return shift_rel * mx;
    };
    auto put = [&](tile_t& d, const d4_t& x) {
#pragma unroll
        for (int v = 0; v < 4; ++v) d[4 * v + lk][li] = x[v];
    };
    // four k values of row li of a tile, k = 4 q + lk: a left operand, or the transpose as a right operand
    auto row4 = [&](const tile_t& d, double (&x)[4]) {
#pragma unroll
        for (int q = 0; q < 4; ++q) x[q] = d[li][4 * q + lk];
    };
    auto col4 = [&](const tile_t& d, double (&x)[4]) {
#pragma unroll
        for (int q = 0; q < 4; ++q) x[q] = d[4 * q + lk][li];
    };
    // Factor the diagonal tile t (symmetric, accumulator layout) and invert the factor, four columns at a time.
    // Register v of the accumulator layout, element [4 v + l / 16][l % 16], is by symmetry the four columns from
    // 4 v on in the layout of a left operand, and as it stands that of a right operand; so with X4 the inverse of
    // the 4 x 4 factor on the diagonal (every lane computes its factor, and column l / 16 of X4),
    //     L_v = T_v X4^T      T -= L_v L_v^T      X_v = X4 E_v      E -= L_v X_v      (E: the identity)
    // are one product each.  A dropped pivot leaves a zero column in L and a zero row and column in the inverse.
    auto factor = [&](int J, d4_t t, tile_t& inv_t, tile_t& low_t) {
        double low[CT];                                        // pivots up to here are dropped
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            low[c] = fmax(tol * s_diag[J * CT + c], 0.0);
            asm("" : "+v"(low[c]));                            // (a select below, not a branch on a uniform value)
        }
        d4_t E, Xv = {0.0, 0.0, 0.0, 0.0}, Lv, left;
#pragma unroll
        for (int v = 0; v < 4; ++v) E[v] = (4 * v + lk == li) ? 1.0 : 0.0;
        const d4_t zero = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            double d[4][4], x[4];
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
                for (int a = b; a < 4; ++a) d[a][b] = readlane_f64(t[v], 16 * b + 4 * v + a);
            double sel = 0.0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                // 1 / sqrt(pivot), zero for a dropped one: the hardware's first digits and one third-order step
                const double piv = d[j][j];
                const double r0 = __builtin_amdgcn_rsq(piv);
                const double e = fma(-(piv * r0), r0, 1.0);
                const double inv = (piv > low[4 * v + j]) ? fma(r0 * e, fma(0.375, e, 0.5), r0) : 0.0;
                double rhs = (lk == j) ? 1.0 : 0.0;            // column lk of X4
#pragma unroll
                for (int b = 0; b < j; ++b) rhs = fma(-d[j][b], x[b], rhs);
                x[j] = rhs * inv;
                sel = (li == 4 * v + j) ? x[j] : sel;
#pragma unroll
                for (int a = j + 1; a < 4; ++a) d[a][j] *= inv;
#pragma unroll
                for (int b = j + 1; b < 4; ++b)
#pragma unroll
                    for (int a = b; a < 4; ++a) d[a][b] = fma(-d[a][j], d[b][j], d[a][b]);
                // the inverse's update with the four columns before, in the shadow of this chain
                if (j == 1 && v > 0) {
                    __builtin_amdgcn_sched_barrier(0);
                    E = __builtin_amdgcn_mfma_f64_16x16x4f64(Lv[v - 1], Xv[v - 1], E, 0, 0, NEG_A);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            const double p = (li >= 4 * v) ? t[v] : 0.0;       // finished rows
            left = __builtin_amdgcn_mfma_f64_16x16x4f64(sel, p, zero, 0, 0, 0);
            Lv[v] = left[v];
            if (v < 3) t = __builtin_amdgcn_mfma_f64_16x16x4f64(Lv[v], Lv[v], t, 0, 0, NEG_A);
            __builtin_amdgcn_sched_barrier(0);
            left = __builtin_amdgcn_mfma_f64_16x16x4f64(sel, E[v], zero, 0, 0, 0);
            Xv[v] = left[v];
            low_t[li][4 * v + lk] = (4 * v + lk <= li) ? Lv[v] : 0.0;
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) inv_t[li][4 * v + lk] = Xv[v];
    };

    // ---- finish column J of L and row J of the inverse, the tiles dealt to all waves; slot J holds Li_J^T
    auto buffer = [&](int J) { return (tile_t*)smem + ((J & 1) ? NT : 0); };
    auto finish = [&](int J) {
        tile_t* cur = buffer(J);
        for (int y = wave; y + 1 < nt; y += WAVES) {
            const int x = y + (y >= J);
            double a[4], b[4];
            col4(cur[J], b);
            if (x > J) col4(cur[x], a);                    // A_xJ, there transposed
            else row4(cur[x], a);                          // E_Jx^T
            __builtin_amdgcn_sched_barrier(0);             // all operands on their way before the first product
            d4_t p = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int q = 0; q < 4; ++q) p = __builtin_amdgcn_mfma_f64_16x16x4f64(a[q], b[q], p, 0, 0, 0);
            put(cur[x], p);
        }
        lds_barrier();
    };

    // ---- results of step J to memory: L_xJ^T -> Rtot (x >= J), X_Jx^T -> Rinv (x <= J).
    auto results = [&](int J) {
        const tile_t* cur = buffer(J);
        // element (4 v + lk, li) of tile (R, C)
        auto store = [&](auto* dst, int R, int C, const double (&o)[4]) {
            const unsigned at = (R * CT + lk) * ld + C * CT + li, rows = 4 * ld;
            if ((max(R, C) + 1) * CT <= k) {
#pragma unroll
                for (int v = 0; v < 4; ++v) dst[at + v * rows] = o[v];
            } else if (C * CT + li < k) {
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (R * CT + lk + 4 * v < k) dst[at + v * rows] = o[v];
            }
        };
        for (int x = wave; x < nt; x += WAVES - 1) {
            double o[4];
            if (x <= J) {
                col4(cur[x], o);
                store(Rinv, x, J, o);
                if (PART != 0) {
                    row4(cur[x], o);
                    store(X, J, x, o);
                }
            }
            if (Rtot && x >= J) {
                row4(x == J ? low_diag[J & 1] : cur[x], o);
                store(Rtot, J, x, o);
            }
        }
    };

    if (wave == WAVES - 1) {
        (void)diagonal_shift_tiles();
        lds_barrier();
        for (int J = -1; J < nt; ++J) {
            if (J >= 0) finish(J);
            if (J + 1 >= nt) break;
            // ---- the next diagonal tile: update with step J, factor
            d4_t t;
#pragma unroll
            for (int v = 0; v < 4; ++v) t[v] = raw[(J + 1) & 1][4 * v + lk][li];
            __builtin_amdgcn_s_setprio(3);
            if (J >= 0) {
                double a[4];
                row4(buffer(J)[J + 1], a);
#pragma unroll
                for (int q = 0; q < 4; ++q) t = __builtin_amdgcn_mfma_f64_16x16x4f64(a[q], a[q], t, 0, 0, NEG_A);
            }
            factor(J + 1, t, buffer(J + 1)[J + 1], low_diag[(J + 1) & 1]);
            __builtin_amdgcn_s_setprio(0);
            lds_barrier();
        }
        return;
    }

    // ---- tiles of this wave: number wave + (WAVES - 1) s of the row-major triangle, (I, K) as the LDS offsets of
    // slots I and K.  Tile (I, K) is held transposed.
    unsigned tile_at[SLOTS];
    d4_t acc[SLOTS];
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) {
        const int t = s * (WAVES - 1) + wave;
        int I = (int)((sqrtf(8.0f * (float)t + 1.0f) - 1.0f) * 0.5f);
        while ((I + 1) * (I + 2) / 2 <= t) ++I;
        while (I * (I + 1) / 2 > t) --I;
        const int K = min(t - I * (I + 1) / 2, NT - 1);
        tile_at[s] = __builtin_amdgcn_readfirstlane((int)((unsigned)(I * TILE) | (unsigned)(K * TILE) << 16));
    }
    // A slot's coordinates, opaque to the compiler: it would otherwise keep the LDS addresses of every
    // slot in vector registers across the loop (and spill).
    auto coords = [&](int s, unsigned& I, unsigned& K) {
        unsigned x = tile_at[s];
        asm volatile("" : "+s"(x));
        I = x & 0xffff; K = x >> 16;
    };
    const unsigned end = nt * TILE;
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) {
        const int I = (tile_at[s] & 0xffff) / TILE, K = (tile_at[s] >> 16) / TILE;
        if (I >= nt) continue;                                 // uniform
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int i = I * CT + li, c = K * CT + 4 * v + lk;
            const bool in = i < k && c < k;
            const int lo = min(min(i, c), k - 1), hi = min(max(i, c), k - 1);    // the lower triangle of S is read
            const double x = PART == 2 ? A[(size_t)hi * ld + lo] : entry(first + (size_t)hi * ld + lo);
            acc[s][v] = in ? x : (i == c ? 1.0 : 0.0);
        }
    }
    const double shift = diagonal_shift_tiles();
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) {
        const unsigned I = tile_at[s] & 0xffff, K = tile_at[s] >> 16;
        if (I != K) continue;
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (4 * v + lk == li && (int)(I / TILE) * CT + li < k) acc[s][v] += shift;
    }
    if (wave == 0) put(raw[0], acc[0]);                        // the first diagonal tile
    lds_barrier();

    // the raw value of a tile that the next step finishes goes to LDS, and the diagonal tile of the step after it
    auto put_raw = [&](int s, int J) {
        unsigned I, K;
        coords(s, I, K);
        const unsigned next = (J + 1) * TILE;
        const bool column = K == next && I > next, row = I == next && K < next, diag = I == K && I == next + TILE;
        if (I < end && (column || row || diag)) {
            const char* d = diag ? (const char*)(raw + (J & 1)) : (const char*)buffer(J + 1) + (column ? I : K);
            put(*(tile_t*)d, acc[s]);
        }
    };
    // (the waves of a SIMD, four numbers apart, write results at different times: one before, one after the products)
    const bool early = (wave & 4) == 0;
    for (int J = -1; J < nt; ++J) {
        const tile_t* cur = buffer(J);
        if (J >= 0) {
            finish(J);
            if (early || J + 1 >= nt) results(J);
            if (J + 1 >= nt) break;
        }
        // ---- every tile below row J: minus slot K times the transpose of slot I.  A tile of column J starts from
        // zero, as a tile of E.  Two tiles at a time, their products interleaved; a wave's tiles come in row order.
        const unsigned at_J = J * TILE;
#pragma unroll
        for (int s = 0; s < SLOTS; s += 2) {
            constexpr int LAST = SLOTS - 1;
            const int s1 = s < LAST ? s + 1 : s;
            unsigned I0, K0, I1, K1;
            coords(s, I0, K0);
            coords(s1, I1, K1);
            if (J >= 0 && I1 > at_J && I0 < end) {
                double a[2][4], b[2][4];
                row4(*(const tile_t*)((const char*)cur + K0), a[0]);
                row4(*(const tile_t*)((const char*)cur + I0), b[0]);
                if (s < LAST) {
                    row4(*(const tile_t*)((const char*)cur + K1), a[1]);
                    row4(*(const tile_t*)((const char*)cur + I1), b[1]);
                }
                if (K0 == at_J) acc[s] = d4_t{0.0, 0.0, 0.0, 0.0};
                if (s < LAST && K1 == at_J) acc[s1] = d4_t{0.0, 0.0, 0.0, 0.0};
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    acc[s] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[0][q], b[0][q], acc[s], 0, 0, NEG_A);
                    if (s < LAST) acc[s1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[1][q], b[1][q], acc[s1], 0, 0, NEG_A);
                }
            }
            if (s >= 2) { put_raw(s - 2, J); put_raw(s - 1, J); }
        }
        constexpr int LEFT = (SLOTS - 1) / 2 * 2;
#pragma unroll
        for (int s = LEFT; s < SLOTS; ++s) put_raw(s, J);
        if (J >= 0 && !early) results(J);
        lds_barrier();
    }
}

// The products between the two parts, one 64 x 64 output tile per workgroup, 16-deep k-tiles through LDS (the
// next one in registers meanwhile).  With o = chol_lead(k), A the first and X the second half of `work`:
//   STAGE 0  A[o..][0..o) = L21 = S21 X11^T, its transpose to Rtot
//   STAGE 1  A[o..][o..) = S22 - L21 L21^T (tiles on and below the diagonal) and X[o..][0..o) = L21 X11
//   STAGE 2  -X22 (L21 X11), transposed, to Rinv; zeros below the diagonal of Rinv and Rtot
// Of X11 and X22 only the lower triangles are defined (and read).
constexpr int CG = 64, CG_K = 16, CG_P = CG_K + 2;

template <int STAGE>
__global__ __launch_bounds__(256) void chol_parts_kernel(const CholBlock* table, const CholBlock single, const int tiles) {
    typedef double d4_t __attribute__((ext_vector_type(4)));
    typedef double __attribute__((address_space(1))) gdouble;
    typedef float __attribute__((address_space(1))) gfloat;
    __shared__ double lds[2][2][CG][CG_P];                     // [buffer][operand][row][k]
    static_assert(sizeof(lds) >= sizeof(double) * CG * (CG + 1), "the output tile goes through the same memory");
    CholBlock cb = single;
    if (table) cb = table[blockIdx.y];
    const int ld = cb.k, o = chol_lead(ld), k2 = ld - o;
    const bool gram = STAGE == 1 && (int)blockIdx.x >= tiles * tiles;        // S22 - L21 L21^T
    const int t = blockIdx.x - (gram ? tiles * tiles : 0);
    const int i0 = t / tiles * CG, j0 = t % tiles * CG;
    if (i0 >= k2 || j0 >= (gram ? i0 + 1 : o)) return;         // the whole workgroup
    auto entry = [&](size_t at) { return cb.S64 ? (double)((const gdouble*)cb.S64)[at] : (double)((const gfloat*)cb.S)[at]; };
    gdouble* A = (gdouble*)cb.work;
    gdouble* X = A + (size_t)ld * ld;
    const int nrow = k2, ncol = gram ? k2 : o, depth = STAGE == 2 ? k2 : o;
    // where the triangular factor leaves nothing: k above the tile's last column or row, k below its first column
    const int kend = STAGE == 0 ? min(depth, j0 + CG) : STAGE == 2 ? min(depth, i0 + CG) : depth;
    const int kbeg = (STAGE == 1 && !gram) ? j0 : 0;
    const bool b_across = STAGE == 2 || (STAGE == 1 && !gram);               // the right operand is stored [k][column]

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, li = lane & 15, lk = lane >> 4;
    const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
    const int rr = tid >> 2, rk = (tid & 3) * 4;               // staging: row and first k; across: k and first column
    const int ck = tid >> 4, cc = (tid & 15) * 4;
    double ra[4], rb[4];
    auto fetch = [&](int kt) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int kk = kt + rk + q, i = i0 + rr;
            double v = 0.0;
            if (i < nrow && kk < depth) {
                if (STAGE == 0) v = entry((size_t)(o + i) * ld + kk);
                else if (STAGE == 1) v = A[(size_t)(o + i) * ld + kk];
                else if (kk <= i) v = X[(size_t)(o + i) * ld + o + kk];
            }
            ra[q] = v;
            v = 0.0;
            if (b_across) {
                const int k = kt + ck, j = j0 + cc + q;
                if (k < depth && j < ncol) {
                    if (STAGE == 2) v = X[(size_t)(o + k) * ld + j];
                    else if (j <= k) v = X[(size_t)k * ld + j];
                }
            } else {
                const int j = j0 + rr;
                if (j < ncol && kk < depth) {
                    if (gram) v = A[(size_t)(o + j) * ld + kk];
                    else if (kk <= j) v = X[(size_t)j * ld + kk];
                }
            }
            rb[q] = v;
        }
    };
    d4_t acc[2][2] = {};
    fetch(kbeg);
    int buf = 0;
    for (int kt = kbeg; kt < kend; kt += CG_K, buf ^= 1) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            lds[buf][0][rr][rk + q] = ra[q];
            if (b_across) lds[buf][1][cc + q][ck] = rb[q];
            else lds[buf][1][rr][rk + q] = rb[q];
        }
        __syncthreads();
        if (kt + CG_K < kend) fetch(kt + CG_K);
#pragma unroll
        for (int q = 0; q < CG_K / 4; ++q) {
            double a[2], b[2];
#pragma unroll
            for (int f = 0; f < 2; ++f) {
                a[f] = lds[buf][0][wm + f * 16 + li][4 * q + lk];
                b[f] = lds[buf][1][wn + f * 16 + li][4 * q + lk];
            }
#pragma unroll
            for (int f = 0; f < 2; ++f)
#pragma unroll
                for (int g = 0; g < 2; ++g) acc[f][g] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[f], b[g], acc[f][g], 0, 0, 0);
        }
    }
    __syncthreads();
    double (*out)[CG + 1] = (double (*)[CG + 1])&lds[0][0][0][0];
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
        for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int r = wm + f * 16 + 4 * v + lk, c = wn + g * 16 + li, i = i0 + r, j = j0 + c;
                const double x = acc[f][g][v];
                if (STAGE != 1) out[r][c] = x;
                if (i >= nrow || j >= ncol) continue;
                if (STAGE == 0) A[(size_t)(o + i) * ld + j] = x;
                else if (STAGE == 1 && gram) { if (j <= i) A[(size_t)(o + i) * ld + o + j] = entry((size_t)(o + i) * ld + o + j) - x; }
                else if (STAGE == 1) X[(size_t)(o + i) * ld + j] = x;
                else {
                    cb.Rinv[(size_t)(o + i) * ld + j] = 0.0f;
                    if (cb.Rtot) cb.Rtot[(size_t)(o + i) * ld + j] = 0.0;
                }
            }
    if (STAGE == 1) return;
    __syncthreads();
    for (int e = tid; e < CG * CG; e += 256) {                 // transposed outputs, rows of the tile running along i
        const int r = e & (CG - 1), c = e / CG, i = i0 + r, j = j0 + c;
        if (i >= nrow || j >= ncol) continue;
        if (STAGE == 0) { if (cb.Rtot) cb.Rtot[(size_t)j * ld + o + i] = out[r][c]; }
        else cb.Rinv[(size_t)j * ld + o + i] = (float)-out[r][c];
    }
}

template <int NT, int WAVES, int PART = 0>
static hipError_t launch_chol_tiles(const CholBlock* table_dev, const CholBlock& single, int blocks, double tol, double shift_rel,
                                    hipStream_t stream) {
    constexpr int lds = (2 * NT + 4) * CT * CT_P * 8 + NT * CT * 8;
    const hipError_t e = allow_lds((const void*)chol_tiles_kernel<NT, WAVES, PART>, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((chol_tiles_kernel<NT, WAVES, PART>), dim3(blocks), dim3(64 * WAVES), lds, stream, table_dev, single, tol, shift_rel);
    return hipGetLastError();
}

template <int NT, int WAVES>
static hipError_t launch_chol_parts(const CholBlock* table_dev, const CholBlock& single, int blocks, int max_k, double tol,
                                    double shift_rel, hipStream_t stream) {
    hipError_t e = launch_chol_tiles<NT, WAVES, 1>(table_dev, single, blocks, tol, shift_rel, stream);
    if (e != hipSuccess) return e;
    const int tiles = (chol_lead(max_k) + CG - 1) / CG;        // the trailing part is no larger
    hipLaunchKernelGGL(chol_parts_kernel<0>, dim3(tiles * tiles, blocks), dim3(256), 0, stream, table_dev, single, tiles);
    hipLaunchKernelGGL(chol_parts_kernel<1>, dim3(2 * tiles * tiles, blocks), dim3(256), 0, stream, table_dev, single, tiles);
    e = launch_chol_tiles<NT, WAVES, 2>(table_dev, single, blocks, tol, shift_rel, stream);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(chol_parts_kernel<2>, dim3(tiles * tiles, blocks), dim3(256), 0, stream, table_dev, single, tiles);
    return hipGetLastError();
}

hipError_t launch_chol_inv(const CholBlock* table_dev, const CholBlock* single, int blocks, int max_k, double tol,
                           double shift_rel, hipStream_t stream) {
    if (blocks <= 0) return hipSuccess;
    CholBlock sb{};
    if (single) sb = *single;
    if (max_k <= 5 * CT) return launch_chol_tiles<5, 8>(table_dev, sb, blocks, tol, shift_rel, stream);
    if (max_k <= 9 * CT) return launch_chol_tiles<9, 8>(table_dev, sb, blocks, tol, shift_rel, stream);
    if (max_k <= CT_MAXK) return launch_chol_tiles<17, 12>(table_dev, sb, blocks, tol, shift_rel, stream);
    // both parts fit the tile counts of the two halves of max_k, whatever the other matrices of the launch
    if (max_k <= 2 * 9 * CT) return launch_chol_parts<9, 8>(table_dev, sb, blocks, max_k, tol, shift_rel, stream);
    if (max_k <= 2 * CT_MAXK) return launch_chol_parts<17, 12>(table_dev, sb, blocks, max_k, tol, shift_rel, stream);
    hipLaunchKernelGGL(chol_inv_kernel, dim3(blocks), dim3(SMALL_THREADS), 0, stream, table_dev, sb, tol, shift_rel);
    return hipGetLastError();
}

// ------------------------------------------------------------------ Jacobi SVD
__device__ inline double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}


// SVD of the k x k factor R through the symmetric eigenproblem of its Gram matrix, all in
// fp64 inside one workgroup:
//   T = R R^T ;  T = E diag(lambda) E^T  (Householder tridiagonalization + implicit QL with
//   accumulation of E^T) ;  rows of E^T R are mutually orthogonal with norms sigma_i.
// Squaring costs relative accuracy of singular values below 1e-8 sigma_1, far below the fp32
// data R was built from.  Compared with sweeping Jacobi rotations over full rows this needs
// about k^2 rotations in total (each applied to one k-vector held across the threads) instead
// of ~10 sweeps of k^2/2 rotations on 2k-vectors, and everything else is matrix products.
// Outputs as before: R is overwritten by E^T R, Gacc = E^T.
constexpr int QL_MAX_ITER = 60;
constexpr int JAC_PARTS = 4;            // pieces a long sum is cut into (k <= JAC_SPLIT_MAXK)
constexpr int JAC_SPLIT_MAXK = 544;
#define JAC_SPLIT_MAXK_OR(k) JAC_SPLIT_MAXK

__global__ __launch_bounds__(SMALL_THREADS) void jacobi_kernel(const JacobiBlock* table, const JacobiBlock single) {
    const JacobiBlock* blk = table ? table + blockIdx.x : &single;
    const int k = blk->k, r = blk->r;
    double* R = blk->R;
    double* W = blk->Gacc;              // rows become the eigenvectors (E^T)
    double* T = blk->tmp;               // Gram matrix, later E^T R
    const int tid = threadIdx.x, nt = blockDim.x;
    const int lane = tid & 63, wave = tid >> 6, nw = nt >> 6;
    __shared__ double s_d[SMALL_MAXK];      // diagonal, later eigenvalues / singular values
    __shared__ double s_e[SMALL_MAXK];      // sub-diagonal
    __shared__ double s_v[SMALL_MAXK];      // Householder vector / rotation cosines
    __shared__ double s_w[SMALL_MAXK];      // work vector / rotation sines
    __shared__ double s_rc[SMALL_MAXK];     // second buffer of rotation cosines
    __shared__ double s_rs[SMALL_MAXK];     // second buffer of rotation sines
    __shared__ double s_part[JAC_PARTS * JAC_SPLIT_MAXK];   // partial sums of the split loops
    __shared__ double s_red[SMALL_THREADS / 64];
    __shared__ int s_job[2][4];
    __shared__ int s_rank[SMALL_MAXK];

    auto block_sum = [&](double v) -> double {      // sum over the workgroup, result to all
        v = wave_sum(v);
        __syncthreads();
        if (lane == 0) s_red[wave] = v;
        __syncthreads();
        double t = 0.0;
        for (int i = 0; i < nw; ++i) t += s_red[i];
        return t;
    };

    // ---- T = R R^T (4 x 4 register tiles), W = I.  R is upper triangular: the sum for T[i][j]
    // starts at column max(i, j).  R^T goes to W first so that the tiles read along rows.
    {
        for (int idx = tid; idx < k * k; idx += nt) W[(size_t)(idx % k) * k + idx / k] = R[idx];
        __syncthreads();
        const int tiles = (k + 3) >> 2;
        for (int q = tid; q < tiles * tiles; q += nt) {
            const int i0 = (q / tiles) * 4, j0 = (q % tiles) * 4;
            if (j0 < i0) continue;                             // the mirror image is written below
            double acc[4][4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[u][v] = 0.0;
#pragma unroll 2
            for (int c = j0; c < k; ++c) {                     // columns before j0 hold zeros of rows j0..
                double a[4], b[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    a[u] = (i0 + u < k) ? W[(size_t)c * k + i0 + u] : 0.0;
                    b[u] = (j0 + u < k) ? W[(size_t)c * k + j0 + u] : 0.0;
                }
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int v = 0; v < 4; ++v) acc[u][v] += a[u] * b[v];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (i0 + u < k && j0 + v < k) {
                        T[(size_t)(i0 + u) * k + j0 + v] = acc[u][v];
                        T[(size_t)(j0 + v) * k + i0 + u] = acc[u][v];
                    }
        }
        __syncthreads();
        for (int idx = tid; idx < k * k; idx += nt) W[idx] = (idx / k == idx % k) ? 1.0 : 0.0;
    }
    __syncthreads();

    // ---- Householder tridiagonalization of T (full symmetric storage), W <- H_j W as we go.
    // The two long loops of a step (the product T22 v and the update of W) have only n1 or k
    // independent outputs; each output's sum is cut into `parts` pieces so that all threads
    // carry loads (the step is bound by memory latency, not by arithmetic).
    const int parts = (k <= JAC_SPLIT_MAXK) ? JAC_PARTS : 1;
    const int tpp = nt / parts;                          // threads per part
    const int part = tid / tpp, li = tid % tpp;
    for (int j = 0; j + 2 < k; ++j) {
        const int n1 = k - j - 1;                       // length of the column below the diagonal
        // x = T[j+1.., j]; alpha = -sign(x0) |x|; v = x - alpha e1; H = I - beta v v^T
        double psum = 0.0;
        for (int i = tid; i < n1; i += nt) { const double x = T[(size_t)(j + 1 + i) * k + j]; s_v[i] = x; psum += x * x; }
        const double xnorm2 = block_sum(psum);
        const double x0 = s_v[0];
        const double xn = sqrt(xnorm2);
        double alpha = (x0 >= 0.0) ? -xn : xn;
        const double vnorm2 = xnorm2 - 2.0 * alpha * x0 + alpha * alpha;     // |x - alpha e1|^2
        const bool skip = (xnorm2 - x0 * x0 <= TRIDIAG_ZERO) || vnorm2 <= 0.0;        // already tridiagonal here
        if (skip) alpha = x0;
        __syncthreads();
        if (tid == 0) { s_d[j] = T[(size_t)j * k + j]; s_e[j] = alpha; if (!skip) s_v[0] = x0 - alpha; }
        __syncthreads();
        if (skip) continue;
        const double beta = 2.0 / vnorm2;
        const int seg = (n1 + parts - 1) / parts;
        const int c_lo = min(n1, part * seg), c_hi = min(n1, c_lo + seg);
        // p = beta T22 v   (T22 symmetric: read columns as rows, coalesced over the output index)
        for (int i = li; i < n1; i += tpp) {
            // eight independent partial sums keep eight loads in flight (the sum is a serial chain)
            double acc[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
            const double* col = T + (size_t)(j + 1) * k + (j + 1 + i);
            int c = c_lo;
            for (; c + 8 <= c_hi; c += 8) {
                double x[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) x[u] = col[(size_t)(c + u) * k];
#pragma unroll
                for (int u = 0; u < 8; ++u) acc[u] += x[u] * s_v[c + u];
            }
            for (; c < c_hi; ++c) acc[0] += col[(size_t)c * k] * s_v[c];
            s_part[part * JAC_SPLIT_MAXK_OR(k) + i] = ((acc[0] + acc[1]) + (acc[2] + acc[3])) + ((acc[4] + acc[5]) + (acc[6] + acc[7]));
        }
        __syncthreads();
        double pv = 0.0;
        for (int i = tid; i < n1; i += nt) {
            double t = 0.0;
            for (int q = 0; q < parts; ++q) t += s_part[q * JAC_SPLIT_MAXK_OR(k) + i];
            t *= beta;
            s_w[i] = t;
            pv += t * s_v[i];
        }
        const double kk2 = 0.5 * beta * block_sum(pv);
        for (int i = tid; i < n1; i += nt) s_w[i] -= kk2 * s_v[i];           // w = p - (beta/2)(p.v) v
        __syncthreads();
        // T22 -= v w^T + w v^T
        for (int idx = tid; idx < n1 * n1; idx += nt) {
            const int i = idx / n1, c = idx % n1;
            T[(size_t)(j + 1 + i) * k + j + 1 + c] -= s_v[i] * s_w[c] + s_w[i] * s_v[c];
        }
        // W[j+1.., :] -= beta v (v^T W[j+1.., :]): partial column dots first ...
        for (int c = li; c < k; c += tpp) {
            const double* wc = W + (size_t)(j + 1) * k + c;
            double acc[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
            int i = c_lo;
            for (; i + 8 <= c_hi; i += 8) {
                double x[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) x[u] = wc[(size_t)(i + u) * k];
#pragma unroll
                for (int u = 0; u < 8; ++u) acc[u] += x[u] * s_v[i + u];
            }
            for (; i < c_hi; ++i) acc[0] += wc[(size_t)i * k] * s_v[i];
            s_part[part * JAC_SPLIT_MAXK_OR(k) + c] = ((acc[0] + acc[1]) + (acc[2] + acc[3])) + ((acc[4] + acc[5]) + (acc[6] + acc[7]));
        }
        __syncthreads();
        // ... then every part updates its own rows
        for (int c = li; c < k; c += tpp) {
            double* wc = W + (size_t)(j + 1) * k + c;
            double y = 0.0;
            for (int q = 0; q < parts; ++q) y += s_part[q * JAC_SPLIT_MAXK_OR(k) + c];
            y *= beta;
            int i = c_lo;
            for (; i + 8 <= c_hi; i += 8) {
                double x[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) x[u] = wc[(size_t)(i + u) * k];
#pragma unroll
                for (int u = 0; u < 8; ++u) wc[(size_t)(i + u) * k] = x[u] - s_v[i + u] * y;
            }
            for (; i < c_hi; ++i) wc[(size_t)i * k] -= s_v[i] * y;
        }
        __syncthreads();
    }
    if (tid == 0) {
        if (k >= 2) { s_d[k - 2] = T[(size_t)(k - 2) * k + k - 2]; s_e[k - 2] = T[(size_t)(k - 1) * k + k - 2]; }
        s_d[k - 1] = T[(size_t)(k - 1) * k + k - 1];
        s_e[k - 1] = 0.0;
    }
    __syncthreads();

    // ---- implicit QL on (d, e); every rotation (c, s) of rows (i, i+1) is applied to W.
    // The scalar recurrences of a QL sweep are one serial chain and touch only (d, e); applying
    // the sweep's rotations to W touches only W.  So wave 0 produces sweeps (its lanes look for
    // the first negligible sub-diagonal entry at or after l, its lane 0 runs the recurrences,
    // operands prefetched one step ahead, the hypotenuse from a reciprocal square root, and
    // records the rotations) while the other waves apply the previous sweep to their columns of
    // W; one barrier per sweep hands the buffers over.
    {
        int l = 0, iter = 0;                              // producer state (wave 0, uniform)
        // job[b] = {m, lo, kind}; kind 1: apply rotations lo..m-1 from buffer b, 2: finished
        auto produce = [&](int b) {
            for (;;) {
                if (l >= k) { if (lane == 0) { s_job[b][2] = 2; } return; }
                int m = k - 1;
                for (int i = l + lane; i < k - 1; i += 64) {
                    const double dd = fabs(s_d[i]) + fabs(s_d[i + 1]);
                    if (fabs(s_e[i]) <= 2.3e-16 * dd) { m = i; break; }
                }
#pragma unroll
                for (int o = 32; o > 0; o >>= 1) m = min(m, __shfl_xor(m, o, 64));
                if (m == l || iter >= QL_MAX_ITER) { ++l; iter = 0; continue; }
                ++iter;
                if (lane == 0) {
                    double* rc = b ? s_rc : s_v;
                    double* rs = b ? s_rs : s_w;
                    int lo = m;                                   // rotations recorded for rows lo .. m-1
                    double g = (s_d[l + 1] - s_d[l]) / (2.0 * s_e[l]);
                    double rr = sqrt(g * g + 1.0);
                    g = s_d[m] - s_d[l] + s_e[l] / (g + ((g >= 0.0) ? fabs(rr) : -fabs(rr)));
                    double sn = 1.0, cs = 1.0, pp = 0.0;
                    double e_i = s_e[m - 1], d_i = s_d[m - 1], d_ip1 = s_d[m];
                    bool under = false;
                    for (int i = m - 1; i >= l; --i) {
                        // next step's operands, fetched without a branch (the values read at the
                        // last step, i == l, are not used) so that the wait for them can sit
                        // at their first use, one step later
                        const int ip = max(i - 1, 0);
                        const double e_n = s_e[ip];
                        const double d_n = s_d[ip];
                        const double f = sn * e_i;
                        const double bb = cs * e_i;
                        const double h2 = f * f + g * g;
                        if (h2 == 0.0) { s_e[i + 1] = 0.0; s_d[i + 1] -= pp; s_e[m] = 0.0; under = true; break; }
                        double rinv = __builtin_amdgcn_rsq(h2);
                        const double hh = 0.5 * h2;
                        rinv = rinv * (1.5 - hh * rinv * rinv);
                        rinv = rinv * (1.5 - hh * rinv * rinv);
                        s_e[i + 1] = h2 * rinv;
                        sn = f * rinv; cs = g * rinv;
                        g = d_ip1 - pp;
                        rr = (d_i - g) * sn + 2.0 * cs * bb;
                        pp = sn * rr;
                        s_d[i + 1] = g + pp;
                        g = cs * rr - bb;
                        rc[i] = cs; rs[i] = sn;
                        lo = i;
                        d_ip1 = d_i; d_i = d_n; e_i = e_n;
                    }
                    if (!under) { s_d[l] -= pp; s_e[l] = g; s_e[m] = 0.0; }
                    s_job[b][0] = m; s_job[b][1] = lo; s_job[b][2] = 1;
                }
                // lane 0's updates of (d, e) must be visible to the whole wave's next search
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
                __builtin_amdgcn_wave_barrier();
                return;
            }
        };
        const int n_cons = nt - 64;                      // threads that apply rotations
        if (wave == 0) produce(0);
        __syncthreads();
        for (int cur = 0;; cur ^= 1) {
            const int kind = s_job[cur][2];
            if (kind == 2) break;
            if (wave == 0) {
                produce(cur ^ 1);
            } else {
                const int m = s_job[cur][0], lo = s_job[cur][1];
                const double* rc = cur ? s_rc : s_v;
                const double* rs = cur ? s_rs : s_w;
                for (int c = tid - 64; c < k; c += n_cons) {
                    double* wc = W + c;
                    double hi = wc[(size_t)m * k];                 // current row i+1, starting with i = m-1
                    int i = m - 1;
                    for (; i - 7 >= lo; i -= 8) {                  // eight rows fetched together
                        double a[8];
#pragma unroll
                        for (int u = 0; u < 8; ++u) a[u] = wc[(size_t)(i - u) * k];
#pragma unroll
                        for (int u = 0; u < 8; ++u) {
                            const double cs = rc[i - u], sn = rs[i - u];
                            wc[(size_t)(i - u + 1) * k] = sn * a[u] + cs * hi;
                            hi = cs * a[u] - sn * hi;
                        }
                    }
                    for (; i >= lo; --i) {
                        const double cs = rc[i], sn = rs[i];
                        const double a = wc[(size_t)i * k];
                        wc[(size_t)(i + 1) * k] = sn * a + cs * hi;
                        hi = cs * a - sn * hi;
                    }
                    wc[(size_t)lo * k] = hi;
                }
            }
            __syncthreads();
        }
    }
    __syncthreads();

    // ---- T <- W R  (rows of E^T R), 4 x 4 register tiles
    {
        const int tiles = (k + 3) >> 2;
        for (int q = tid; q < tiles * tiles; q += nt) {
            const int i0 = (q / tiles) * 4, c0 = (q % tiles) * 4;
            double acc[4][4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[u][v] = 0.0;
            const int jend = min(k, c0 + 4);                   // R is upper triangular
#pragma unroll 2
            for (int j = 0; j < jend; ++j) {
                double a[4], b[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    a[u] = (i0 + u < k) ? W[(size_t)(i0 + u) * k + j] : 0.0;
                    b[u] = (c0 + u < k) ? R[(size_t)j * k + c0 + u] : 0.0;
                }
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int v = 0; v < 4; ++v) acc[u][v] += a[u] * b[v];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (i0 + u < k && c0 + v < k) T[(size_t)(i0 + u) * k + c0 + v] = acc[u][v];
        }
    }
    __syncthreads();

    // singular values = row norms of E^T R; order descending (ties by index)
    for (int j = wave; j < k; j += nw) {
        double a = 0.0;
        for (int c = lane; c < k; c += 64) { const double v = T[(size_t)j * k + c]; a += v * v; }
        a = wave_sum(a);
        if (lane == 0) s_d[j] = sqrt(a);
    }
    __syncthreads();
    for (int j = tid; j < k; j += nt) {
        const double sj = s_d[j];
        int rank = 0;
        for (int i = 0; i < k; ++i) {
            const double si = s_d[i];
            rank += (si > sj || (si == sj && i < j)) ? 1 : 0;
        }
        s_rank[j] = rank;
        if (blk->sigma) blk->sigma[rank] = (float)sj;
    }
    __syncthreads();
    for (int j = wave; j < k; j += nw) {
        const int rank = s_rank[j];
        if (rank >= r) continue;
        const double sj = s_d[j];
        double top = 0.0;
        for (int i = lane; i < k; i += 64) top = fmax(top, s_d[i]);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) top = fmax(top, __shfl_xor(top, o, 64));
        const bool null = sj <= SVD_NULL * top;              // (not a NaN, which is passed on)
        const double inv = null ? 0.0 : 1.0 / sj;
        for (int c = lane; c < k; c += 64) {
            blk->XrT[(size_t)rank * k + c] = (float)(T[(size_t)j * k + c] * inv);
            blk->GrT[(size_t)rank * k + c] = null ? 0.0f : (float)W[(size_t)j * k + c];
        }
    }
}

hipError_t launch_jacobi(const JacobiBlock* table_dev, const JacobiBlock* single, int blocks, int max_k,
                         hipStream_t stream) {
    if (blocks <= 0) return hipSuccess;
    if (max_k > SMALL_MAXK) return hipErrorInvalidValue;
    JacobiBlock sb{};
    if (single) sb = *single;
    hipLaunchKernelGGL(jacobi_kernel, dim3(blocks), dim3(SMALL_THREADS), 0, stream, table_dev, sb);
    return hipGetLastError();
}

}  // namespace tsr
