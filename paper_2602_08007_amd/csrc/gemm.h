// Grouped tall-skinny GEMM family on the gfx950 matrix cores (internal interface).
//
// One launch computes, for every tile in a tile list,
//     C[tile] = alpha * op(A) op(B) [tile] + beta * C[tile]          (fp32 output)
// with op(A) M x K and op(B) K x N taken from row-major storage in either orientation.
// Operands are fp32 (A may also be bf16); they are cut into 1..3 bf16 pieces and the
// leading cross products are accumulated in fp32 by v_mfma_f32_32x32x16_bf16.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tsr {

struct GemmProblem {
    const void* A;      // k-contiguous: element (i,k) at A[i*lda + k]; k-strided: A[k*lda + i]
    const float* B;     // k-contiguous: element (j,k) at B[j*ldb + k]; k-strided: B[k*ldb + j]
    float* C;           // row-major M x N, leading dimension ldc
    long long lda, ldb, ldc;
    long long c_split_stride;  // elements between the partial outputs of consecutive k-splits
    int M, N, K;
    int kchunk;         // K range handled by one tile (multiple of 32); K if no split; negative (no split): B is upper
                        // triangular, element (j, k) zero for k > j
};

struct GemmTile {       // one workgroup's work
    int prob, tm, tn, ks;
};

struct GemmLaunch {
    const GemmProblem* probs;  // device array (grouped) or nullptr
    const GemmTile* tiles;     // device array (grouped) or nullptr
    GemmProblem single;        // used when tiles == nullptr
    int tiles_m, tiles_n, ksplit;  // decode of blockIdx when tiles == nullptr
    int n_tiles;               // grid size
    float alpha, beta;         // epilogue scalars of the whole launch; beta == 0: C is not read
};

// Operand layout / precision of one instantiation.
struct GemmVariant {
    int a_kstrided;   // 0: A stored M x K (k contiguous), 1: A stored K x M
    int b_kstrided;   // 0: B stored N x K (k contiguous), 1: B stored K x N
    int a_bf16;       // A elements are bf16 (then a_pieces must be 1)
    int a_pieces;     // 1..3
    int b_pieces;     // 1..3
    int shape;        // GemmShape
};

enum GemmShape { GEMM_128x128 = 0, GEMM_128x64 = 1, GEMM_64x64 = 2, GEMM_SHAPES = 3 };
inline int gemm_tile_m(int shape) { return shape == GEMM_64x64 ? 64 : 128; }
inline int gemm_tile_n(int shape) { return shape == GEMM_128x128 ? 128 : 64; }

// Enqueue one grouped GEMM.  Returns hipSuccess or the launch error; an unsupported
// variant returns hipErrorInvalidValue.
hipError_t launch_gemm(const GemmLaunch& L, const GemmVariant& v, hipStream_t stream);

// out[i] = alpha * sum_{s<splits} part[s*stride + i] + beta * out[i], i over an M x N
// matrix with leading dimension ldc (partials are dense M x N).  Summed in split order.
struct ReduceProblem {
    const float* part; float* out;
    long long stride, ldc;
    int M, N, splits;
};
// max_elems, max_splits: of the problems.
hipError_t launch_splitk_reduce(const ReduceProblem* probs_dev, const ReduceProblem* single,
                                int count, int max_elems, int max_splits, float alpha, float beta, hipStream_t stream);

// The step of one small matrix, r <= ONE_MAX_R.  Projection: workgroup (slab, chunk), slab-major, leaves
// U_s^T (G_sc V_c), r x r, for 64 rows s and kchunk columns c (a multiple of 32) in part[workgroup].
constexpr int ONE_MAX_R = 128;
struct ProjectOne {
    const void* G; const float* U; const float* V; float* part;
    long long ldg;
    int m, n, r, chunks, kchunk;
};
hipError_t launch_project_one(const ProjectOne& q, int g_bf16, int split, int blocks, hipStream_t stream);
// Lift: W = beta W + alpha U D V^T; workgroup (slab, group), slab-major: 64 rows, per_group tiles of 64 columns.
struct LiftOne {
    float* W; const float* U; const float* V; const float* D;
    long long ldw;
    int m, n, r, groups, per_group;
    float alpha, beta;
};
hipError_t launch_lift_one(const LiftOne& q, int split, int blocks, hipStream_t stream);

}  // namespace tsr
