// SVD of the k x k triangular factor R of the refresh (the "small SVD" of the randomized SVD,
// Algorithm 1's refresh step) as a chain of launches, for k <= EIG_MAXK:
//   1. T = R R^T                        fp64 MFMA GEMM, 64 x 64 tiles over the whole chip
//   2. per matrix, one workgroup:       Householder tridiagonalization of T (reflectors parked in
//      the rows of T they cleared), the last 288 columns in registers; then eigenvalues by Sturm-count multisection (chip-wide),
//      eigenvectors of the tridiagonal matrix by inverse iteration (one per thread, pivoted LU
//      of T - lambda I), Gram-Schmidt inside groups of numerically equal eigenvalues
//   3. E = H_0 H_1 ... Z                reflectors in blocks of sixteen, products on fp64 MFMAs with the
//      vectors held in registers
//   4. E^T R                            fp64 MFMA GEMM
//   5. singular values = row norms of E^T R, ordering, fp32 outputs
// Nothing here is a serial chain longer than k steps, which is what separates it from the QL
// sweeps of the single-kernel variant (about k^2 dependent rotations per matrix).
#include <hip/hip_runtime.h>

#include "device_lds.h"
#include "small.h"

namespace tsr {
namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
constexpr int EIG_THREADS = 1024;
constexpr double EIG_EPS = 2.220446049250313e-16;
// Solves per eigenvector.  With an eigenvalue good to a few ulps of the spectral radius one solve
// from a random start already carries the vector to the accuracy the gap allows (its component
// along the wanted vector is amplified by 1 / ulp relative to the others); the second covers an
// unlucky start and the third is margin (two measured 0.25 ms less per refresh of 84 matrices
// and passed every test; kept at three).
constexpr int EIG_INVIT_ROUNDS = 3;

__device__ inline double eig_wave_sum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Cross-lane sums without LDS: data-parallel moves inside the 16-lane rows, row and half swaps beyond.
template <int CTRL> __device__ inline double eig_dpp(double x) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(x), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(x), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
constexpr int DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E, DPP_MIRROR8 = 0x141, DPP_MIRROR16 = 0x140, DPP_ROR8 = 0x128;
// (a, b) -> (a of the lower 32 lanes, b of the lower 32 lanes) + (a of the upper, b of the upper): the sum of
// a over the halves in lanes 0-31, that of b in lanes 32-63
__device__ inline double eig_sum32(double a, double b) {
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(a), (unsigned)__double2loint(b), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(a), (unsigned)__double2hiint(b), false, false);
    return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}
// likewise over the two 16-lane rows of a half: a's sum in the even rows, b's in the odd ones
__device__ inline double eig_sum16(double a, double b) {
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)__double2loint(a), (unsigned)__double2loint(b), false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)__double2hiint(a), (unsigned)__double2hiint(b), false, false);
    return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}
__device__ inline double eig_wave_sum_dpp(double x) {         // result in every lane
    x += eig_dpp<DPP_XOR1>(x);
    x += eig_dpp<DPP_XOR2>(x);
    x += eig_dpp<DPP_MIRROR8>(x);
    x += eig_dpp<DPP_MIRROR16>(x);
    x = eig_sum16(x, x);
    return eig_sum32(x, x);
}

// 1 / x to full precision for finite non-zero x of ordinary size (no scaling, no fix-up)
__device__ inline double eig_rcp(double x) {
    double r = __builtin_amdgcn_rcp(x);
    r = fma(fma(-x, r, 1.0), r, r);
    r = fma(fma(-x, r, 1.0), r, r);
    return r;
}

// Kernels that cut a matrix into chunks run one workgroup per (block b, chunk c) on a 1-D grid.
// Workgroups are handed to the eight XCDs in turn.  Chunk-major numbering spreads the chunks of
// a block over the XCDs; "pinned" numbering (block index fastest, padded to a multiple of
// eight) keeps block b on XCD b % 8, where the one-workgroup-per-block kernels also run it.
struct EigGrid { int n_blocks, chunks, pinned; };
__device__ inline bool eig_decode(const EigGrid g, int& b, int& c) {
    const int lin = blockIdx.x;
    if (g.pinned) { const int bx = (g.n_blocks + 7) / 8 * 8; b = lin % bx; c = lin / bx; }
    else { c = lin % g.chunks; b = lin / g.chunks; }
    return b < g.n_blocks && c < g.chunks;
}
inline dim3 eig_grid(const EigGrid g) {
    return dim3((unsigned)((g.pinned ? (g.n_blocks + 7) / 8 * 8 : g.n_blocks) * g.chunks));
}

// ------------------------------------------------------------------ fp64 MFMA GEMMs
// v_mfma_f64_16x16x4: lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16] and receives
// D[4 v + l / 16][l % 16] in element v.  One wave owns a 32 x 32 patch (2 x 2 MFMA tiles), a
// workgroup of four waves a 64 x 64 tile; operands come straight from L2 (the matrices are a
// few hundred KB), 16 k-values per round.
// WHICH = 0: T = R R^T (R upper triangular: the sum for T[i][j] starts at max(i, j));
// WHICH = 1: E^T R into the second half of tmp (the sum for column c ends at c);
// WHICH = 2: R = R2 R1 with R2 in Gacc, both upper triangular (the sum runs from i to j).
template <int WHICH>
__global__ __launch_bounds__(256) void eig_gemm_kernel(const JacobiBlock* table, const JacobiBlock single, const EigGrid grid) {
    JacobiBlock jb = single;
    int gb, gc;
    if (!eig_decode(grid, gb, gc)) return;
    if (table) jb = table[gb];
    const JacobiBlock* blk = &jb;
    const int k = blk->k;
    const int tiles = (k + 63) >> 6;
    if (gc >= tiles * tiles) return;
    const int tm = gc / tiles, tn = gc % tiles;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int m0 = tm * 64 + (wave >> 1) * 32, n0 = tn * 64 + (wave & 1) * 32;
    if (m0 >= k || n0 >= k) return;
    typedef const double __attribute__((address_space(1))) cgdouble;
    typedef double __attribute__((address_space(1))) gdouble;
    cgdouble* A;
    cgdouble* B = (WHICH == 2) ? (cgdouble*)blk->R1 : (cgdouble*)blk->R;
    gdouble* C;
    long long sam, sak, sbk, sbn;
    int k_lo = 0, k_hi = k;
    if (WHICH == 0) { A = (cgdouble*)blk->R; sam = k; sak = 1; sbk = 1; sbn = k; C = (gdouble*)blk->tmp; k_lo = max(m0, n0) & ~3; }
    else if (WHICH == 1) { A = (cgdouble*)blk->Gacc; sam = k; sak = 1; sbk = k; sbn = 1; C = (gdouble*)blk->tmp + (size_t)k * k; k_hi = min(k, n0 + 32); }
    else { A = (cgdouble*)blk->Gacc; sam = k; sak = 1; sbk = k; sbn = 1; C = (gdouble*)blk->R; k_lo = m0 & ~3; k_hi = min(k, n0 + 32); }
    const int li = lane & 15, lk = lane >> 4;
    d4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = d4{0.0, 0.0, 0.0, 0.0};
    long long arow[2], bcol[2];
    bool aok[2], bok[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int row = m0 + 16 * i + li, col = n0 + 16 * i + li;
        aok[i] = row < k; bok[i] = col < k;
        arow[i] = (long long)min(row, k - 1) * sam;
        bcol[i] = (long long)min(col, k - 1) * sbn;
    }
    // sixteen k at a time, the next sixteen on their way (values past the range are cleared when they are used)
    double a[2][4][2], b[2][4][2];
    auto fetch = [&](int s, int kk) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const long long kcc = min(kk + 4 * u + lk, k - 1);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                a[s][u][i] = A[arow[i] + kcc * sak];
                b[s][u][i] = B[kcc * sbk + bcol[i]];
            }
        }
    };
    auto multiply = [&](int s, int kk) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const bool kok = kk + 4 * u + lk < k_hi;
            double x[2], y[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                x[i] = (kok && aok[i]) ? a[s][u][i] : 0.0;
                y[i] = (kok && bok[i]) ? b[s][u][i] : 0.0;
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[i], y[j], acc[i][j], 0, 0, 0);
        }
    };
    fetch(0, k_lo);
    for (int kk = k_lo; kk < k_hi; kk += 32) {
        fetch(1, kk + 16);
        multiply(0, kk);
        fetch(0, kk + 32);
        multiply(1, kk + 16);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = m0 + 16 * i + 4 * v + lk, col = n0 + 16 * j + li;
                if (row < k && col < k) C[(size_t)row * k + col] = acc[i][j][v];
            }
}

// ------------------------------------------------------------------ tridiagonal eigenproblem
// Start vector of the inverse iteration: a fixed pseudo-random value in (-0.5, 0.5) per entry
// (integer finalizer of the published MurmurHash3).
__device__ inline double eig_start_value(unsigned i, unsigned j) {
    unsigned h = i * 2654435761u ^ (j * 40503u + 0x9E3779B9u);
    h ^= h >> 16; h *= 0x85EBCA6Bu; h ^= h >> 13; h *= 0xC2B2AE35u; h ^= h >> 16;
    return (double)h * (1.0 / 4294967296.0) - 0.5 + 1.0 / 8589934592.0;
}

// Householder tridiagonalization of matrices too large for registers (k > EIG_TILES_K), down to a trailing
// matrix of EIG_TILES_K columns that eig_tridiag_tiles_kernel takes on.  Reflector t, H_t = I - beta v v^T
// on indices t+1..k-1, clears column t below the sub-diagonal; v goes to row t of T (columns t+1..), beta to
// T[t][t].  The rank-two update of reflector t-1,  T -= v w^T + w v^T, is still pending when reflector t is
// formed: column t is corrected on the fly, and one pass over the lower triangle of the trailing matrix then
// applies the pending update and multiplies the updated matrix with the new v.  The pass runs at the rate
// one CU moves data to and from L2.  The rows are dealt to the waves in turn, a wave sweeps its row up to the
// diagonal in strips of 64 columns, and an entry (c, i) below the diagonal adds to two sums of p = T v, p_i
// (kept per lane and strip over all rows of the wave, summed over the waves through LDS at the end) and p_c
// (summed over the lanes once per row); the upper triangle is dead storage but for the reflectors.
// (v, w) are indexed from t for the pending pair and from t+1 for the new one.  The sums over the lanes go by
// data-parallel moves; through LDS, six round trips a row, they were a tenth of it (56 matrices of k = 528 9.45 -> 8.52 ms,
// refresh step of the 1B model 86.5 -> 85.1 ms).  Slower: three rows in flight a wave instead of two (registers spill),
// eight waves with the vectors in registers (10.2 ms).
constexpr int EIG_TILES_K = 288;
__global__ __launch_bounds__(EIG_THREADS) void eig_tridiag_kernel(const JacobiBlock* table, const JacobiBlock single) {
    JacobiBlock jb = single;
    if (table) jb = table[blockIdx.x];
    const JacobiBlock* blk = &jb;
    const int k = blk->k;
    const int stop = k - EIG_TILES_K;           // columns reduced here
    if (stop <= 0) return;
    // (marked as global memory: a generic access would count as one to LDS, too)
    typedef double __attribute__((address_space(1))) gdouble;
    gdouble* T = (gdouble*)blk->tmp;            // symmetric; afterwards the reflectors
    const int tid = threadIdx.x, nt = blockDim.x;
    const int lane = tid & 63, wave = tid >> 6, nw = nt >> 6;
    __shared__ double s_d[EIG_MAXK];            // diagonal
    __shared__ double s_e[EIG_MAXK];            // sub-diagonal, s_e[i] couples i and i + 1
    __shared__ double s_v[EIG_MAXK];            // Householder vector v and companion w of two
    __shared__ double s_w[EIG_MAXK];            //   consecutive reflectors (pending / being formed)
    __shared__ double s_vn[EIG_MAXK];
    __shared__ double s_wn[EIG_MAXK];
    __shared__ double s_part[(EIG_THREADS / 128) * EIG_MAXK];   // column sums of the waves, two waves per slot
    __shared__ double s_prow[EIG_MAXK];                         // row sums
    __shared__ double s_red[EIG_THREADS / 64];

    auto block_sum = [&](double v) -> double {
        v = eig_wave_sum_dpp(v);
        __syncthreads();
        if (lane == 0) s_red[wave] = v;
        __syncthreads();
        double t = 0.0;
        for (int i = 0; i < nw; ++i) t += s_red[i];
        return t;
    };

    constexpr int STRIPS = (EIG_MAXK + 63) / 64;
    for (int i = tid; i < k; i += nt) { s_v[i] = 0.0; s_w[i] = 0.0; }
    __syncthreads();
    double* pv_ = s_v; double* pw_ = s_w;      // pending pair
    double* nv_ = s_vn; double* nw_ = s_wn;    // pair being formed
    for (int t = 0; t < stop; ++t) {
        const int n1 = k - t - 1;
        const double v0 = pv_[0], w0 = pw_[0];
        // column t below the diagonal
        double psum = 0.0;
        for (int i = tid; i < n1; i += nt) {
            const double x = T[(size_t)(t + 1 + i) * k + t] - v0 * pw_[1 + i] - w0 * pv_[1 + i];
            nv_[i] = x;
            psum += x * x;
        }
        const double dnew = T[(size_t)t * k + t] - 2.0 * v0 * w0;
        const double xnorm2 = block_sum(psum);
        const double x0 = nv_[0];
        const double xn = sqrt(xnorm2);
        double alpha = (x0 >= 0.0) ? -xn : xn;
        const double vnorm2 = xnorm2 - 2.0 * alpha * x0 + alpha * alpha;     // |x - alpha e1|^2
        const bool skip = (xnorm2 - x0 * x0 <= TRIDIAG_ZERO) || vnorm2 <= 0.0;        // already tridiagonal here
        if (skip) alpha = x0;
        const double beta = skip ? 0.0 : 2.0 / vnorm2;
        __syncthreads();
        if (tid == 0) { s_d[t] = dnew; s_e[t] = alpha; T[(size_t)t * k + t] = beta; nv_[0] = x0 - alpha; }
        if (skip) { for (int i = tid; i < n1; i += nt) nv_[i] = 0.0; }       // no reflector: only the pending update runs
        __syncthreads();
        if (!skip) { for (int i = tid; i < n1; i += nt) T[(size_t)t * k + t + 1 + i] = nv_[i]; }
        double pv = 0.0;
        // entry (c, i), i <= c, of the trailing matrix: pending update, then its terms of p = T v
        double colacc[STRIPS];
#pragma unroll
        for (int q = 0; q < STRIPS; ++q) colacc[q] = 0.0;
        // (the next row of a wave is fetched while the current one is worked on)
        auto fetch = [&](int c, double* x) {
            const gdouble* row = T + (size_t)(t + 1 + c) * k + (t + 1);
#pragma unroll
            for (int q = 0; q < STRIPS; ++q) {
                const int i = 64 * q + lane;
                x[q] = (c < n1 && i <= c) ? row[i] : 0.0;
            }
        };
        double xa[STRIPS], xb[STRIPS];
        fetch(wave, xa);
        auto work = [&](int c, const double* x) {
            const double vc = pv_[1 + c], wc = pw_[1 + c], nc = nv_[c];
            gdouble* row = T + (size_t)(t + 1 + c) * k + (t + 1);
            double rowacc = 0.0;
#pragma unroll
            for (int q = 0; q < STRIPS; ++q) {
                const int i = 64 * q + lane;
                if (i <= c) {
                    const double xi = x[q] - (vc * pw_[1 + i] + wc * pv_[1 + i]);
                    row[i] = xi;
                    colacc[q] += xi * nc;
                    if (i < c) rowacc += xi * nv_[i];
                }
            }
            rowacc = eig_wave_sum_dpp(rowacc);
            if (lane == 0) s_prow[c] = rowacc;
        };
        for (int c = wave; c < n1; c += 2 * nw) {
            fetch(c + nw, xb);
            work(c, xa);
            if (c + nw < n1) {
                fetch(c + 2 * nw, xa);
                work(c + nw, xb);
            }
        }
        // column sums of the waves: the first half of the waves store theirs, the second half add to them
        if (wave < nw / 2) {
#pragma unroll
            for (int q = 0; q < STRIPS; ++q)
                if (64 * q + lane < n1) s_part[wave * EIG_MAXK + 64 * q + lane] = colacc[q];
        }
        __syncthreads();
        if (wave >= nw / 2) {
#pragma unroll
            for (int q = 0; q < STRIPS; ++q)
                if (64 * q + lane < n1) s_part[(wave - nw / 2) * EIG_MAXK + 64 * q + lane] += colacc[q];
        }
        __syncthreads();
        for (int i = tid; i < n1; i += nt) {
            double a = s_prow[i];
            for (int q = 0; q < nw / 2; ++q) a += s_part[q * EIG_MAXK + i];
            a *= beta;
            nw_[i] = a;
            pv += a * nv_[i];
        }
        const double kk2 = 0.5 * beta * block_sum(pv);
        for (int i = tid; i < n1; i += nt) nw_[i] -= kk2 * nv_[i];           // w = p - (beta/2)(p.v) v
        __syncthreads();
        double* sw;
        sw = pv_; pv_ = nv_; nv_ = sw;
        sw = pw_; pw_ = nw_; nw_ = sw;
    }
    // the last pending update
    for (int c = wave; c < EIG_TILES_K; c += nw) {
        const double vc = pv_[c], wc = pw_[c];
        gdouble* row = T + (size_t)(stop + c) * k + stop;
        for (int i = lane; i <= c; i += 64) row[i] -= vc * pw_[i] + wc * pv_[i];
    }
    // the tridiagonal matrix travels to the next launches behind the LU scratch
    double* DE = blk->scratch + eig_tridiag_at(k);
    for (int i = tid; i < stop; i += nt) { DE[i] = s_d[i]; DE[k + i] = s_e[i]; }
}

// ---- Tridiagonalization with the matrix in registers, for the trailing part of at most 288 columns.
// Barrier that orders LDS only (the reflectors on their way to memory are not waited for).
__device__ inline void eig_lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The lower triangle in 32 x 32 tiles (diagonal tiles whole), dealt to the waves in turn; lane 8 a + b of a
// wave holds the 4 x 4 patch of a tile at row 4 a, column 4 b.  Per reflector v of column t:
//   every wave: norm of the column (in LDS), the reflector's scalars; row sums (A v) and column sums (A^T v)
//     of its tiles, reduced over the lanes; v^T A v                                       -> LDS, barrier
//   p = beta A v, an entry per thread, the sums of its tiles added                         -> LDS, barrier
//   every wave: w = p - (beta/2)(p.v) v, A -= v w^T + w v^T in registers; column t + 1     -> LDS, barrier
// so a reflector costs three barriers and no memory traffic but its own entries: it is bound by the latency
// of these steps.  The 4 x 4 patches keep that short: eight vector entries read from LDS, two reductions and
// a branch serve sixteen entries (16 x 16 tiles with four entries per lane took 1.8 times as long at k = 264).
// One matrix per compute unit, the pass over the matrix in L2 -> this: k = 72 304 -> 123 us, k = 136 725 -> 315 us,
// k = 264 2.65 -> 0.97 ms.  288 is what the registers hold (45 tiles over eight waves, 192 registers a lane).
constexpr int TT = 32;
template <int NB, int WAVES>
__global__ __launch_bounds__(64 * WAVES, 1) void eig_tridiag_tiles_kernel(const JacobiBlock* table, const JacobiBlock single) {
    constexpr int SLOTS = (NB * (NB + 1) / 2 + WAVES - 1) / WAVES;
    constexpr int N = NB * TT;
    typedef double d2_t __attribute__((ext_vector_type(2)));
    JacobiBlock jb = single;
    if (table) jb = table[blockIdx.x];
    const int kfull = jb.k;
    const int first = kfull > N ? kfull - N : 0;               // the columns before it are reduced already
    const int k = kfull - first;
    typedef double __attribute__((address_space(1))) gdouble;
    gdouble* T = (gdouble*)jb.tmp + (size_t)first * kfull + first;
    const int nb = (k + TT - 1) / TT;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int la = lane >> 3, lb = lane & 7;
    __shared__ __attribute__((aligned(16))) double s_x[2][N];           // column being reduced / the next one
    __shared__ __attribute__((aligned(16))) double s_p[N];
    __shared__ double s_part[NB][NB][TT];       // [block][other block of the tile]: the tile's sums for the block
    __shared__ double s_q[WAVES];               // v^T A v
    __shared__ double s_d[N], s_e[N];

    int tI[SLOTS], tK[SLOTS];
    double a[SLOTS][4][4];
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) {
        const int t = s * WAVES + wave;
        int I = (int)((sqrtf(8.0f * (float)t + 1.0f) - 1.0f) * 0.5f);
        while ((I + 1) * (I + 2) / 2 <= t) ++I;
        while (I * (I + 1) / 2 > t) --I;
        tI[s] = __builtin_amdgcn_readfirstlane(I);
        tK[s] = __builtin_amdgcn_readfirstlane(t - I * (I + 1) / 2);
    }
    auto coords = [&](int s, int& I, int& K) {   // opaque: keeps LDS addresses of all slots out of the registers
        I = tI[s]; K = tK[s];
        asm volatile("" : "+s"(I), "+s"(K));
    };
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) {
        if (tI[s] >= nb) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int i = tI[s] * TT + 4 * la + r, j = tK[s] * TT + 4 * lb + c;
                const double x = T[(size_t)min(max(i, j), k - 1) * kfull + min(min(i, j), k - 1)];
                a[s][r][c] = (i < k && j < k) ? x : 0.0;
            }
    }
    // column c of the matrix below the diagonal -> LDS, zeros up to the diagonal; the diagonal entry -> s_d
    auto put_column = [&](int c, double* dst) {
        const int Kc = c / TT, bc = (c % TT) / 4, cc = c % 4;
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            int I, K;
            coords(s, I, K);
            if (K != Kc || I >= nb) continue;
            if (lb == bc) {
                double y[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    // (selected by value: an array indexed by a variable would have to live in memory)
                    const double y0 = a[s][r][0], y1 = a[s][r][1], y2 = a[s][r][2], y3 = a[s][r][3];
                    y[r] = cc == 0 ? y0 : cc == 1 ? y1 : cc == 2 ? y2 : y3;
                }
                if (I == Kc) {
                    const int i = I * TT + 4 * la;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        if (i + r == c) s_d[c] = y[r];
                        y[r] = (i + r > c) ? y[r] : 0.0;
                    }
                }
                d2_t* d = (d2_t*)(dst + I * TT + 4 * la);
                d[0] = d2_t{y[0], y[1]};
                d[1] = d2_t{y[2], y[3]};
            }
        }
    };
    put_column(0, s_x[0]);
    __syncthreads();                            // (every wave has its tiles: the reflectors overwrite parts of T)

    for (int t = 0; t + 2 < k; ++t) {
        const double* x = s_x[t & 1];
        const int T0 = (t + 1) / TT;
        // ---- norm of the column below the diagonal, scalars of the reflector (every wave the same)
        double psum = 0.0;
#pragma unroll
        for (int q = 0; q < (N + 63) / 64; ++q) {
            const int i = 64 * q + lane;
            const double xi = (i >= T0 * TT && i < nb * TT) ? x[min(i, N - 1)] : 0.0;
            psum = fma(xi, xi, psum);
        }
        const double x0 = x[t + 1];
        const double xnorm2 = eig_wave_sum_dpp(psum);
        const bool skip = !(xnorm2 - x0 * x0 > TRIDIAG_ZERO);  // already tridiagonal here
        // alpha = -sign(x0) |x|, beta = 2 / |x - alpha e1|^2 = 1 / (|x|^2 + |x0| |x|)
        double rs = __builtin_amdgcn_rsq(xnorm2);
        {
            const double e = fma(-(xnorm2 * rs), rs, 1.0);
            rs = fma(rs * e, fma(0.375, e, 0.5), rs);
        }
        const double xn = xnorm2 * rs;
        const double alpha = skip ? x0 : (x0 >= 0.0 ? -xn : xn);
        const double beta = skip ? 0.0 : eig_rcp(fma(fabs(x0), xn, xnorm2));
        const double v0 = x0 - alpha;
        if (wave == WAVES - 1 && lane == 0) {
            s_e[t] = alpha;
            T[(size_t)t * kfull + t] = beta;
        }
        if (!skip)
            for (int i = t + 1 + tid; i < k; i += 64 * WAVES) T[(size_t)t * kfull + i] = (i == t + 1) ? v0 : x[i];

        // four entries from 4 g on within block B; in a vector v, entry t + 1 has to be put right afterwards
        auto load4 = [&](double (&v)[4], const double* src, int B, int g) {
            const d2_t* p = (const d2_t*)(src + B * TT + 4 * g);
            const d2_t u0 = p[0], u1 = p[1];
            v[0] = u0[0]; v[1] = u0[1]; v[2] = u1[0]; v[3] = u1[1];
        };
        auto fix = [&](double (&v)[4], int B, int g) {
            if (B == T0) {
                const int i = t + 1 - (B * TT + 4 * g);
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] = (i == r) ? v0 : v[r];
            }
        };

        // ---- sums of the tiles
        double q1 = 0.0;
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            int I, K;
            coords(s, I, K);
            if (I >= nb || K < T0 || skip) continue;           // uniform
            double vI[4], vK[4], R[4];
            load4(vK, x, K, lb);
            load4(vI, x, I, la);
            __builtin_amdgcn_sched_barrier(0);
            fix(vK, K, lb);
            fix(vI, I, la);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                R[r] = a[s][r][0] * vK[0];
#pragma unroll
                for (int c = 1; c < 4; ++c) R[r] = fma(a[s][r][c], vK[c], R[r]);
                q1 = fma(R[r], vI[r], q1);
            }
            {   // over the eight lanes of a patch row: lane b ends up with row b / 2
                const bool hi = lb >= 4, up = (lb & 2) != 0;
                double k0 = (hi ? R[2] : R[0]) + eig_dpp<DPP_MIRROR8>(hi ? R[0] : R[2]);
                double k1 = (hi ? R[3] : R[1]) + eig_dpp<DPP_MIRROR8>(hi ? R[1] : R[3]);
                double y = (up ? k1 : k0) + eig_dpp<DPP_XOR2>(up ? k0 : k1);
                y += eig_dpp<DPP_XOR1>(y);
                if ((lb & 1) == 0) s_part[I][K][4 * la + (lb >> 1)] = y;
            }
            if (I != K) {
                double C[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    C[c] = a[s][0][c] * vI[0];
#pragma unroll
                    for (int r = 1; r < 4; ++r) C[c] = fma(a[s][r][c], vI[r], C[c]);
                    q1 = fma(C[c], vK[c], q1);
                }
                // over the eight patches of a column: rows of lanes 0, 1, 2, 3 end up with columns 0, 2, 1, 3
                double y = eig_sum16(eig_sum32(C[0], C[1]), eig_sum32(C[2], C[3]));
                y += eig_dpp<DPP_ROR8>(y);
                const int c = ((lane >> 4) & 1) * 2 + (lane >> 5);
                if ((lane & 8) == 0) s_part[K][I][4 * lb + c] = y;
            }
        }
        q1 = eig_wave_sum_dpp(q1);
        if (lane == 0) s_q[wave] = q1;
        eig_lds_barrier();

        // ---- p, an entry per thread
        for (int i = T0 * TT + tid; i < nb * TT; i += 64 * WAVES) {
            double y[NB], p = 0.0;
#pragma unroll
            for (int X = 0; X < NB; ++X) y[X] = s_part[i / TT][X][i % TT];
#pragma unroll
            for (int X = 0; X < NB; ++X) p += (X >= T0 && X < nb) ? y[X] : 0.0;
            s_p[i] = (i > t && !skip) ? beta * p : 0.0;
        }
        eig_lds_barrier();

        // ---- w and the rank-two update
        double pv = 0.0;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) pv += s_q[w];
        const double kk2 = 0.5 * beta * (beta * pv);
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
            int I, K;
            coords(s, I, K);
            if (I >= nb || K < T0 || skip) continue;
            double vI[4], vK[4], wI[4], wK[4];
            load4(vK, x, K, lb);
            load4(vI, x, I, la);
            load4(wK, s_p, K, lb);
            load4(wI, s_p, I, la);
            __builtin_amdgcn_sched_barrier(0);
            fix(vK, K, lb);
            fix(vI, I, la);
#pragma unroll
            for (int r = 0; r < 4; ++r) { wK[r] = fma(-kk2, vK[r], wK[r]); wI[r] = fma(-kk2, vI[r], wI[r]); }
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int c = 0; c < 4; ++c) a[s][r][c] = fma(-wI[r], vK[c], fma(-vI[r], wK[c], a[s][r][c]));
        }
        put_column(t + 1, s_x[(t + 1) & 1]);
        eig_lds_barrier();
    }
    // the last two columns (column k - 2 is in LDS, its diagonal entry in s_d)
    if (k >= 2) put_column(k - 1, s_p);
    if (tid == 0) {
        if (k >= 2) s_e[k - 2] = s_x[(k - 2) & 1][k - 1];
        s_e[k - 1] = 0.0;
    }
    eig_lds_barrier();
    double* DE = jb.scratch + eig_tridiag_at(kfull);
    for (int i = tid; i < k; i += 64 * WAVES) { DE[first + i] = s_d[i]; DE[kfull + first + i] = s_e[i]; }
}

// Eigenvalues and eigenvectors of the tridiagonal matrix (d, e) left by eig_tridiag_kernel, in
// three launches: eigenvalues (chip-wide), inverse iteration (one wave per workgroup),
// orthogonalisation inside groups of numerically equal eigenvalues (one workgroup per matrix).
// The scratch is laid out by eig_layout.h; a radius of zero marks a zero or non-finite matrix.

// Sturm-count multisection: 2^LP threads of a workgroup share an eigenvalue; their 2^LP - 1 probes cut its
// bracket into 2^LP pieces per pass, and the number of eigenvalues below a probe tells on which side of it the
// wanted one lies.  The count is the number of sign changes in the sequence of leading principal minors
//     p_i = (d_i - x) p_{i-1} - e_{i-1}^2 p_{i-2}
// of the matrix scaled to unit norm (Givens; as stable as the recurrence of the pivots p_i / p_{i-1}, which
// needs a division per step: two dependent operations a step here against eight there), rescaled every eight
// steps.  A minor that vanishes has the sign that the count of a slightly larger probe gives it; d_i - x is kept
// from vanishing by a shift of 1e-34 of the norm.  The chain of k steps is what bounds it: more probes per
// pass (fewer passes) as long as the chip has room.  One matrix, eight threads each -> this: k = 72 90 -> 23 us,
// k = 136 153 -> 38 us; 19 matrices at k = 264 288 -> 136 us.
template <int LP>
__global__ __launch_bounds__(256) void eig_values_kernel(const JacobiBlock* table, const JacobiBlock single, const EigGrid grid) {
    constexpr int P = 1 << LP, PER_WG = 256 / P, S = P - 1;
    JacobiBlock jb = single;
    int gb, gc;
    if (!eig_decode(grid, gb, gc)) return;
    if (table) jb = table[gb];
    const JacobiBlock* blk = &jb;
    const int k = blk->k;
    const int e0 = gc * PER_WG;
    if (e0 >= k) return;
    const double* DE = blk->scratch + eig_tridiag_at(k);
    double* LAM = blk->scratch + eig_tridiag_at(k) + 2 * k;
    const int tid = threadIdx.x, nt = blockDim.x;
    const int lane = tid & 63, wave = tid >> 6, nw = nt >> 6;
    typedef double d2_t __attribute__((ext_vector_type(2)));
    __shared__ __attribute__((aligned(16))) d2_t s_dw[EIG_MAXK + 8];   // d_i, e_{i-1}^2 of the scaled matrix
    __shared__ int s_cnt[256];                  // Sturm counts of the probes
    __shared__ double s_red[4];
    auto block_max = [&](double v) -> double {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
        __syncthreads();
        if (lane == 0) s_red[wave] = v;
        __syncthreads();
        double t = s_red[0];
        for (int i = 1; i < nw; ++i) t = fmax(t, s_red[i]);
        return t;
    };
    double gl, gu;
    {
        double lo = 1e300, hi = -1e300;
        for (int i = tid; i < k; i += nt) {
            const double di = DE[i], ei = DE[k + i];
            const double rad = ((i > 0) ? fabs(DE[k + i - 1]) : 0.0) + ((i < k - 1) ? fabs(ei) : 0.0);
            lo = fmin(lo, di - rad);
            hi = fmax(hi, di + rad);
        }
        gu = block_max(hi);
        gl = -block_max(-lo);
    }
    double tnorm = fmax(fabs(gl), fabs(gu));
    const bool degenerate = !(tnorm > 0.0) || !(tnorm < 1e300);   // zero (or non-finite) matrix
    if (degenerate) tnorm = 0.0;
    if (gc == 0 && tid == 0) LAM[k] = tnorm;
    if (degenerate) {
        if (tid < PER_WG && e0 + tid < k) LAM[e0 + tid] = 0.0;
        return;
    }
    const double inv = 1.0 / tnorm;
    for (int i = tid; i < k + 8; i += nt) {     // (eight idle steps at the end: rows that change no sign)
        const double e1 = (i > 0 && i < k) ? DE[k + i - 1] * inv : 0.0;
        s_dw[i] = (i < k) ? d2_t{DE[i] * inv, e1 * e1} : d2_t{4.0, 0.0};
    }
    gl *= inv; gu *= inv;
    {
        const double margin = 2.0 * EIG_EPS * (double)k + 2e-32;
        gl -= margin; gu += margin;
    }
    const int el = tid / P, es = tid % P;
    const int ej = e0 + el;
    const bool eact = ej < k && es < S;
    double lo = gl, hi = gu;                                 // bracket, kept by each of the eigenvalue's threads
    __syncthreads();
    constexpr int PASSES = (57 + LP - 1) / LP;               // 2^-57 of the bracket
    for (int pass = 0; pass < PASSES; ++pass) {
        const double step = (hi - lo) * (1.0 / (double)P);
        if (eact) {
            const double x = lo + (double)(es + 1) * step;
            double p1 = 1.0, p2 = 0.0;                       // p_{i-1}, p_{i-2}
            int cnt = 0;
            unsigned signs = 0;
            for (int i0 = 0; i0 < k; i0 += 8) {
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const d2_t dw = s_dw[i0 + u];
                    const double dx = (dw[0] - x) - 1e-34;
                    const double p = fma(dx, p1, -(dw[1] * p2));
                    p2 = p1; p1 = p;
                    signs = __builtin_amdgcn_alignbit(signs, (unsigned)__double2hiint(p), 31);
                }
                cnt += __popc((signs ^ (signs >> 1)) & 0xffu);
                const int ex = -max(__builtin_amdgcn_frexp_exp(p1), __builtin_amdgcn_frexp_exp(p2));
                p1 = __builtin_amdgcn_ldexp(p1, ex);
                p2 = __builtin_amdgcn_ldexp(p2, ex);
            }
            s_cnt[tid] = cnt;
        }
        __syncthreads();
        if (ej < k) {
            const int* c = s_cnt + el * P;
            int m = 0;                                       // leading probes at or below eigenvalue ej: counts ascend
#pragma unroll
            for (int h = P / 2; h > 0; h >>= 1)
                if (c[m + h - 1] <= ej) m += h;
            if (m < S) hi = lo + (double)(m + 1) * step;
            if (m > 0) lo = lo + (double)m * step;
        }
        __syncthreads();
    }
    if (ej < k && es == 0) LAM[ej] = 0.5 * (lo + hi) * tnorm;
}

// Eigenvectors by inverse iteration, vector j on its own thread, one wave per workgroup.  The matrix scaled to
// unit norm, T - lambda I = P L U with partial pivoting; U (three diagonals, pivots as reciprocals) and the
// multipliers of L (the exchange of rows in their lowest bit) are kept in memory, so that the later rounds
// repeat no division.  The recurrences are serial in the row index: without branches, and the rows they need
// travel two batches of eight ahead.  The rows fetched batch by batch, a
// division in every round -> this: k = 72 111 -> 62 us, k = 264 (19 matrices) 496 -> 209 us.
__global__ __launch_bounds__(64) void eig_invit_kernel(const JacobiBlock* table, const JacobiBlock single, const EigGrid grid) {
    constexpr int B = 8, NB = 2;                // rows per batch, batches in flight
    JacobiBlock jb = single;
    int gb, gc;
    if (!eig_decode(grid, gb, gc)) return;
    if (table) jb = table[gb];
    const int k = jb.k;
    if (gc * 64 >= k) return;
    typedef double __attribute__((address_space(1))) gdouble;
    gdouble* Z = (gdouble*)jb.tmp + (size_t)k * k;     // eigenvectors of the tridiagonal matrix, Z[i][j] = j-th vector
    gdouble* U0 = (gdouble*)jb.scratch;         // per thread j: reciprocal pivots, first and second
    gdouble* U1 = U0 + (size_t)k * k;           //   super-diagonal of the LU factor, entry [i][j]
    gdouble* U2 = U1 + (size_t)k * k;
    gdouble* LM = (gdouble*)jb.Gacc;            // multipliers (Gacc receives the eigenvectors later)
    const double* DE = jb.scratch + eig_tridiag_at(k);
    const double* LAM = DE + 2 * k;
    const int tid = threadIdx.x;
    const int j = gc * 64 + tid;
    __shared__ double s_d[EIG_MAXK + 1];        // diagonal
    __shared__ double s_e[EIG_MAXK + 1];        // sub-diagonal, s_e[i] couples i and i + 1
    const double tnorm = LAM[k];
    if (tnorm == 0.0) {
        // zero (or non-finite) matrix: every orthonormal basis is one of eigenvectors
        if (j < k) for (int i = 0; i < k; ++i) Z[(size_t)i * k + j] = (i == j) ? 1.0 : 0.0;
        return;
    }
    const double inv_norm = 1.0 / tnorm;
    for (int i = tid; i <= k; i += 64) {
        s_d[i] = (i < k) ? DE[i] * inv_norm : 0.0;
        s_e[i] = (i < k - 1) ? DE[k + i] * inv_norm : 0.0;
    }
    __syncthreads();
    const double tiny = EIG_EPS;                         // floor of an LU pivot
    const int jc = min(j, k - 1);                        // idle lanes repeat the last vector and store nothing
    const bool act = j < k;
    const double lam = LAM[jc] * inv_norm;
    auto floored = [&](double p) -> double { return (fabs(p) < tiny) ? copysign(tiny, p) : p; };
    auto at = [&](int i) -> size_t { return (size_t)i * k + jc; };
    double scale = 1.0, ss = 0.0;
    for (int round = 0; round < EIG_INVIT_ROUNDS; ++round) {
        // ---- forward: y = L^-1 P (start vector / previous x); the first round forms the factors
        double ycur;
        if (round == 0) {
            ycur = eig_start_value(0u, (unsigned)jc);
            double a = s_d[0] - lam, b = s_e[0];
            for (int i = 0; i + 1 < k; ++i) {
                const double c = s_e[i], dn = s_d[i + 1] - lam, en = s_e[i + 1];
                const double ynext = eig_start_value((unsigned)(i + 1), (unsigned)jc);
                const bool sw = fabs(a) < fabs(c);
                const double inv = eig_rcp(floored(sw ? c : a));
                double mult = (sw ? a : c) * inv;
                mult = __hiloint2double(__double2hiint(mult), (__double2loint(mult) & ~1) | (sw ? 1 : 0));
                const double p1 = sw ? dn : b, p2 = sw ? en : 0.0;
                const double yp = sw ? ynext : ycur, yo = sw ? ycur : ynext;
                if (act) { U0[at(i)] = inv; U1[at(i)] = p1; U2[at(i)] = p2; LM[at(i)] = mult; Z[at(i)] = yp; }
                a = fma(-mult, p1, sw ? b : dn);
                b = sw ? -mult * en : en;
                ycur = fma(-mult, yp, yo);
            }
            if (act) { U0[at(k - 1)] = eig_rcp(floored(a)); U1[at(k - 1)] = 0.0; U2[at(k - 1)] = 0.0; }
        } else {
            double zb[NB][B], lb[NB][B];
            auto fetch = [&](int s, int i0) {            // z of rows i0 + 1 .., multipliers of rows i0 ..
#pragma unroll
                for (int u = 0; u < B; ++u) {
                    zb[s][u] = Z[at(min(i0 + 1 + u, k - 1))];
                    lb[s][u] = LM[at(min(i0 + u, k - 2 > 0 ? k - 2 : 0))];
                }
            };
            ycur = scale * Z[at(0)];
#pragma unroll
            for (int s = 0; s < NB; ++s) fetch(s, s * B);
            for (int i0 = 0; i0 + 1 < k; i0 += NB * B) {
#pragma unroll
                for (int s = 0; s < NB; ++s) {
                    double yp[B];
#pragma unroll
                    for (int u = 0; u < B; ++u) {
                        if (i0 + s * B + u + 1 < k) {    // uniform
                            const double mult = lb[s][u], ynext = scale * zb[s][u];
                            const bool sw = (__double2loint(mult) & 1) != 0;
                            yp[u] = sw ? ynext : ycur;
                            ycur = fma(-mult, yp[u], sw ? ycur : ynext);
                        }
                    }
                    fetch(s, i0 + (NB + s) * B);
#pragma unroll
                    for (int u = 0; u < B; ++u)
                        if (act && i0 + s * B + u + 1 < k) Z[at(i0 + s * B + u)] = yp[u];
                }
            }
        }
        if (act) Z[at(k - 1)] = ycur;
        // ---- backward: U x = y
        double x1 = 0.0, x2 = 0.0, amax = 0.0;          // x[i+1], x[i+2]
        bool bad = false;
        ss = 0.0;
        double y[NB][B], p0[NB][B], p1[NB][B], p2[NB][B];
        auto fetch = [&](int s, int i0) {                // rows i0, i0 - 1, ...
#pragma unroll
            for (int u = 0; u < B; ++u) {
                const size_t o = at(max(i0 - u, 0));
                y[s][u] = Z[o]; p0[s][u] = U0[o]; p1[s][u] = U1[o]; p2[s][u] = U2[o];
            }
        };
#pragma unroll
        for (int s = 0; s < NB; ++s) fetch(s, k - 1 - s * B);
        for (int i0 = k - 1; i0 >= 0; i0 -= NB * B) {
#pragma unroll
            for (int s = 0; s < NB; ++s) {
                double xs[B];
#pragma unroll
                for (int u = 0; u < B; ++u) {
                    if (i0 - s * B - u >= 0) {           // uniform
                        const double x = fma(-p1[s][u], x1, fma(-p2[s][u], x2, y[s][u])) * p0[s][u];
                        xs[u] = x;
                        amax = fmax(amax, fabs(x));
                        bad = bad || !(fabs(x) <= 1e300);
                        ss = fma(x, x, ss);
                        x2 = x1; x1 = x;
                    }
                }
                fetch(s, i0 - (NB + s) * B);
#pragma unroll
                for (int u = 0; u < B; ++u)
                    if (act && i0 - s * B - u >= 0) Z[at(i0 - s * B - u)] = xs[u];
            }
        }
        if (bad || !(amax > 0.0)) {
            // overflow or a vanished vector (the floored pivots are meant to rule both out):
            // go on from the unit vector rather than carry a non-finite value
            if (act) for (int q = 0; q < k; ++q) Z[at(q)] = (q == jc) ? 1.0 : 0.0;
            amax = 1.0;
            ss = 1.0;
        }
        scale = 1.0 / amax;
    }
    const double nrm = 1.0 / sqrt(ss);
    for (int i0 = 0; i0 < k; i0 += 16) {
        double x[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) x[u] = Z[at(min(i0 + u, k - 1))];
#pragma unroll
        for (int u = 0; u < 16; ++u)
            if (act && i0 + u < k) Z[at(i0 + u)] = nrm * x[u];
    }
}

// The same with everything a vector needs in LDS: reciprocal pivots, the row that stays (the first super-diagonal of a
// row without exchange), multipliers and the vector, V vectors to a workgroup of one wave.  What a recurrence waits for
// is then its own few operations (the rows of the others come from memory, two trips a round and batch): one matrix of
// k = 72 62 -> 43 us, two of k = 136 114 -> 76 us.  A workgroup fills the LDS of a compute unit, so this is for
// launches that fit the chip at once: 19 matrices of k = 264, sixteen vectors each, took 322 us instead of 207.
constexpr int EIG_INVIT_LDS = 150 * 1024;
constexpr int EIG_INVIT_LDS_K = 144;
constexpr int eig_invit_vectors(int k) { return 4 * 8 * 64 * k <= EIG_INVIT_LDS ? 64 : 32; }
template <int V>
__global__ __launch_bounds__(64) void eig_invit_lds_kernel(const JacobiBlock* table, const JacobiBlock single, const EigGrid grid,
                                                           const int max_k) {
    constexpr int B = 8;                        // rows per batch
    JacobiBlock jb = single;
    int gb, gc;
    if (!eig_decode(grid, gb, gc)) return;
    if (table) jb = table[gb];
    const int k = jb.k;
    if (gc * V >= k) return;
    typedef double __attribute__((address_space(1))) gdouble;
    gdouble* Z = (gdouble*)jb.tmp + (size_t)k * k;     // eigenvectors of the tridiagonal matrix, Z[i][j] = j-th vector
    const double* DE = jb.scratch + eig_tridiag_at(k);
    const double* LAM = DE + 2 * k;
    const int tid = threadIdx.x;
    const int v = tid % V, j = gc * V + v;      // (further lanes do as the first V)
    __shared__ double s_d[EIG_INVIT_LDS_K + 2];        // diagonal
    __shared__ double s_e[EIG_INVIT_LDS_K + 2];        // sub-diagonal, s_e[i] couples i and i + 1
    extern __shared__ double s_vec[];
    double* U0 = s_vec + v;                     // row i at i V
    double* U1 = U0 + (size_t)max_k * V;
    double* LM = U1 + (size_t)max_k * V;
    double* X = LM + (size_t)max_k * V;
    const double tnorm = LAM[k];
    if (tnorm == 0.0) {
        // zero (or non-finite) matrix: every orthonormal basis is one of eigenvectors
        if (tid < V && j < k) for (int i = 0; i < k; ++i) Z[(size_t)i * k + j] = (i == j) ? 1.0 : 0.0;
        return;
    }
    const double inv_norm = 1.0 / tnorm;
    for (int i = tid; i <= k; i += 64) {
        s_d[i] = (i < k) ? DE[i] * inv_norm : 0.0;
        s_e[i] = (i < k - 1) ? DE[k + i] * inv_norm : 0.0;
    }
    __syncthreads();
    const double tiny = EIG_EPS;                         // floor of an LU pivot
    const int jc = min(j, k - 1);                        // idle lanes repeat the last vector and store nothing
    const double lam = LAM[jc] * inv_norm;
    auto floored = [&](double p) -> double { return (fabs(p) < tiny) ? copysign(tiny, p) : p; };
    double scale = 1.0, ss = 0.0;
    for (int round = 0; round < EIG_INVIT_ROUNDS; ++round) {
        // ---- forward: y = L^-1 P (start vector / previous x); the first round forms the factors
        double ycur;
        if (round == 0) {
            ycur = eig_start_value(0u, (unsigned)jc);
            double a = s_d[0] - lam, b = s_e[0];
            for (int i = 0; i + 1 < k; ++i) {
                const double c = s_e[i], dn = s_d[i + 1] - lam, en = s_e[i + 1];
                const double ynext = eig_start_value((unsigned)(i + 1), (unsigned)jc);
                const bool sw = fabs(a) < fabs(c);
                const double inv = eig_rcp(floored(sw ? c : a));
                double mult = (sw ? a : c) * inv;
                mult = __hiloint2double(__double2hiint(mult), (__double2loint(mult) & ~1) | (sw ? 1 : 0));
                const double p1 = sw ? dn : b;
                const double yp = sw ? ynext : ycur, yo = sw ? ycur : ynext;
                U0[i * V] = inv; U1[i * V] = b; LM[i * V] = mult; X[i * V] = yp;
                a = fma(-mult, p1, sw ? b : dn);
                b = sw ? -mult * en : en;
                ycur = fma(-mult, yp, yo);
            }
            U0[(k - 1) * V] = eig_rcp(floored(a)); U1[(k - 1) * V] = 0.0; LM[(k - 1) * V] = 0.0;
        } else {
            ycur = scale * X[0];
            for (int i0 = 0; i0 + 1 < k; i0 += B) {
                double zb[B], lb[B];
#pragma unroll
                for (int u = 0; u < B; ++u) { zb[u] = X[min(i0 + 1 + u, k - 1) * V]; lb[u] = LM[min(i0 + u, k - 1) * V]; }
#pragma unroll
                for (int u = 0; u < B; ++u) {
                    if (i0 + u + 1 < k) {                // uniform
                        const double mult = lb[u], ynext = scale * zb[u];
                        const bool sw = (__double2loint(mult) & 1) != 0;
                        const double yp = sw ? ynext : ycur;
                        ycur = fma(-mult, yp, sw ? ycur : ynext);
                        X[(i0 + u) * V] = yp;
                    }
                }
            }
        }
        X[(k - 1) * V] = ycur;
        // ---- backward: U x = y
        double x1 = 0.0, x2 = 0.0, amax = 0.0;          // x[i+1], x[i+2]
        bool bad = false;
        ss = 0.0;
        for (int i0 = k - 1; i0 >= 0; i0 -= B) {
            double y[B], p0[B], p1[B], m[B], dn[B], en[B];
#pragma unroll
            for (int u = 0; u < B; ++u) {
                const int i = max(i0 - u, 0);
                y[u] = X[i * V]; p0[u] = U0[i * V]; p1[u] = U1[i * V]; m[u] = LM[i * V];
                dn[u] = s_d[i + 1]; en[u] = s_e[i + 1];
            }
#pragma unroll
            for (int u = 0; u < B; ++u) {
                if (i0 - u >= 0) {                       // uniform
                    const bool sw = (__double2loint(m[u]) & 1) != 0;
                    const double q1 = sw ? dn[u] - lam : p1[u], q2 = sw ? en[u] : 0.0;
                    const double x = fma(-q1, x1, fma(-q2, x2, y[u])) * p0[u];
                    X[(i0 - u) * V] = x;
                    amax = fmax(amax, fabs(x));
                    bad = bad || !(fabs(x) <= 1e300);
                    ss = fma(x, x, ss);
                    x2 = x1; x1 = x;
                }
            }
        }
        if (bad || !(amax > 0.0)) {
            // overflow or a vanished vector (the floored pivots are meant to rule both out):
            // go on from the unit vector rather than carry a non-finite value
            for (int q = 0; q < k; ++q) X[q * V] = (q == jc) ? 1.0 : 0.0;
            amax = 1.0;
            ss = 1.0;
        }
        scale = 1.0 / amax;
    }
    const double nrm = 1.0 / sqrt(ss);
    __syncthreads();
    // V neighbouring vectors per row, 64 / V rows at a time
    if (j < k)
        for (int i = tid / V; i < k; i += 64 / V) Z[(size_t)i * k + j] = nrm * X[i * V];
}

template <int V>
hipError_t launch_invit_lds(const JacobiBlock* table_dev, const JacobiBlock& single, int blocks, int max_k, hipStream_t stream) {
    const int lds = 4 * max_k * V * (int)sizeof(double);
    const hipError_t e = allow_lds((const void*)eig_invit_lds_kernel<V>, EIG_INVIT_LDS);
    if (e != hipSuccess) return e;
    const EigGrid g{blocks, (max_k + V - 1) / V, 1};
    hipLaunchKernelGGL(eig_invit_lds_kernel<V>, eig_grid(g), dim3(64), lds, stream, table_dev, single, g, max_k);
    return hipGetLastError();
}

// Eigenvalues closer than ortol form a group; inside a group the vectors of the inverse
// iteration span the right subspace but need not be orthogonal: Gram-Schmidt (two passes) in
// order.  One workgroup per matrix; returns at once when there is no group.
__global__ __launch_bounds__(EIG_THREADS) void eig_groups_kernel(const JacobiBlock* table, const JacobiBlock single) {
    JacobiBlock jb = single;
    if (table) jb = table[blockIdx.x];
    const JacobiBlock* blk = &jb;
    const int k = blk->k;
    double* Z = blk->tmp + (size_t)k * k;
    const double* LAM = blk->scratch + eig_tridiag_at(k) + 2 * k;
    const int tid = threadIdx.x, nt = blockDim.x;
    const int lane = tid & 63, wave = tid >> 6, nw = nt >> 6;
    __shared__ double s_v[EIG_MAXK];            // eigenvalues, ascending
    __shared__ double s_part[EIG_MAXK];         // Gram-Schmidt coefficients
    __shared__ double s_red[EIG_THREADS / 64];
    __shared__ int s_first[EIG_MAXK];           // first member of the group an eigenvalue belongs to
    __shared__ int s_any;
    auto block_sum = [&](double v) -> double {
        v = eig_wave_sum(v);
        __syncthreads();
        if (lane == 0) s_red[wave] = v;
        __syncthreads();
        double t = 0.0;
        for (int i = 0; i < nw; ++i) t += s_red[i];
        return t;
    };
    const double tnorm = LAM[k];
    if (tnorm == 0.0) return;
    if (tid == 0) s_any = 0;
    for (int i = tid; i < k; i += nt) s_v[i] = LAM[i];
    __syncthreads();
    {
        const double ortol0 = 1e-9 * tnorm;
        for (int i = 1 + tid; i < k; i += nt) if (s_v[i] - s_v[i - 1] <= ortol0) s_any = 1;
    }
    __syncthreads();
    if (s_any == 0) return;
    // ---- eigenvalues closer than ortol form a group; inside a group the vectors found above
    // span the right subspace but need not be orthogonal: Gram-Schmidt (two passes) in order.
    {
        const double ortol = 1e-9 * tnorm;
        if (tid == 0) {
            s_first[0] = 0;
            for (int j = 1; j < k; ++j) s_first[j] = (s_v[j] - s_v[j - 1] <= ortol) ? s_first[j - 1] : j;
        }
        __syncthreads();
        double* coef = s_part;
        // Groups from the top down.  Where little of a vector is left (the null space of a matrix of much lower rank:
        // inverse iteration finds few directions there), its rounding grows as it is brought back to length, with that
        // its share of the vectors above the group: it is freed of these as well (singular values of 6e-2 sigma_1 came
        // out beyond the rank, k = 516, rank 20).
        for (int end = k; end > 0; end = s_first[end - 1]) {
            const int cs = s_first[end - 1];
            for (int j = cs + 1; j < end; ++j) {
                auto remove = [&](int above) {           // from vector j what it has of the group's before it, and of those above
                    const int before = j - cs, total = before + above;
                    for (int q = wave; q < total; q += nw) {
                        const int i = q < before ? cs + q : end + (q - before);
                        double a = 0.0;
                        for (int t = lane; t < k; t += 64) a += Z[(size_t)t * k + i] * Z[(size_t)t * k + j];
                        a = eig_wave_sum(a);
                        if (lane == 0) coef[q] = a;
                    }
                    __syncthreads();
                    for (int t = tid; t < k; t += nt) {
                        double a = 0.0;
                        for (int q = 0; q < before; ++q) a += coef[q] * Z[(size_t)t * k + cs + q];
                        for (int q = 0; q < above; ++q) a += coef[before + q] * Z[(size_t)t * k + end + q];
                        Z[(size_t)t * k + j] -= a;
                    }
                    __syncthreads();
                };
                auto normalise = [&]() -> double {       // returns the square of the length
                    double ss = 0.0;
                    for (int t = tid; t < k; t += nt) { const double x = Z[(size_t)t * k + j]; ss += x * x; }
                    ss = block_sum(ss);
                    const double inv = (ss > 0.0) ? 1.0 / sqrt(ss) : 0.0;
                    for (int t = tid; t < k; t += nt)
                        Z[(size_t)t * k + j] = (ss > 0.0) ? Z[(size_t)t * k + j] * inv : eig_start_value((unsigned)t, (unsigned)(k + j));
                    __syncthreads();
                    return ss;
                };
                remove(0);
                remove(0);
                if (normalise() < 1e-2) {                // (uniform)
                    remove(k - end);
                    remove(k - end);
                    normalise();
                }
            }
        }
    }
}

// ------------------------------------------------------------------ back-transformation
// E = H_0 H_1 ... H_{k-3} Z in blocks of sixteen reflectors, H_j0 ... H_j0+15 = I - V T V^T (compact WY form), so
// that the work is products on fp64 MFMAs.  First launch: the triangular factors T of all blocks, one wave each:
// T(:,r) = -beta_r T (V^T v_r) above the diagonal, beta_r on it; they take the place of the LU factors.
// (Only the rows and columns of reflectors that exist are stored; see eig_wy_at.)
__device__ inline bool eig_has_reflector(int j, int k) { return j + 2 < k; }
__global__ __launch_bounds__(64) void eig_wy_kernel(const JacobiBlock* table, const JacobiBlock single, const EigGrid grid) {
    JacobiBlock jb = single;
    int gb, b;
    if (!eig_decode(grid, gb, b)) return;
    if (table) jb = table[gb];
    const int k = jb.k;
    const int j0 = 16 * b;
    if (!eig_has_reflector(j0, k)) return;
    typedef const double __attribute__((address_space(1))) cgdouble;
    typedef double __attribute__((address_space(1))) gdouble;
    cgdouble* T = (cgdouble*)jb.tmp;
    const int lane = threadIdx.x, li = lane & 15, lk = lane >> 4;
    __shared__ double s_m[16][17];
    __shared__ double s_beta[16];
    const int j = j0 + li;                                   // this lane's reflector
    const bool valid = eig_has_reflector(j, k);
    const double beta = valid ? T[(size_t)j * k + j] : 0.0;
    cgdouble* row = T + (size_t)min(j, k - 1) * k;
    const bool live = valid && beta != 0.0;                  // (a step without a reflector leaves no entries)
    d4 m = {0.0, 0.0, 0.0, 0.0};
    for (int t = b; 16 * t < k; ++t) {
        double a[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int i = 16 * t + 4 * q + lk;
            const double x = row[min(i, k - 1)];
            a[q] = (live && i > j && i < k) ? x : 0.0;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) m = __builtin_amdgcn_mfma_f64_16x16x4f64(a[q], a[q], m, 0, 0, 0);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) s_m[4 * v + lk][li] = m[v];
    if (lk == 0) s_beta[li] = beta;
    __syncthreads();
    double x[16];                                            // row li of T
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        double sum = 0.0;
#pragma unroll
        for (int c = 0; c < r; ++c) sum = fma(x[c], s_m[c][r], sum);
        const double br = s_beta[r];
        x[r] = (li < r) ? -br * sum : (li == r) ? br : 0.0;
    }
    gdouble* out = (gdouble*)jb.scratch;
    const int rank = eig_wy_rank(k, b);
    if (lk == 0 && li < rank) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
            if (r < rank) out[eig_wy_at(b, li, r)] = x[r];
    }
}

// Second launch: Z <- Z - V (T (V^T Z)) block by block, sixteen columns of Z per wave in the accumulator layout of
// v_mfma_f64_16x16x4 (element v of lane l: row 4 v + l / 16, column l % 16), which is also the layout of its right
// operand: Z and the two small products go from one product to the next without a move.  V is shared by the four
// waves through LDS, the next block on its way in registers.  E is written transposed (row j of Gacc = j-th
// eigenvector).  One reflector after the other (a barrier and a sum across waves each) took 83 us at k = 72,
// 247 at 136, 588 at 264 (19 matrices) and 4.0 ms at 528 (56); both launches now 23, 55, 176 us and 1.8 ms.
template <int RT>
__global__ __launch_bounds__(256, 1) void eig_backtransform_kernel(const JacobiBlock* table, const JacobiBlock single, const EigGrid grid) {
    constexpr int PITCH = (16 * RT + 13) / 32 * 32 + 18;     // row of V: 18 modulo 32 doubles, no bank conflicts
    constexpr int PER = RT;                                  // entries of a block of V per thread (16 x 16 RT / 256)
    JacobiBlock jb = single;
    int gb, gc;
    if (!eig_decode(grid, gb, gc)) return;
    if (table) jb = table[gb];
    const int k = jb.k;
    if (gc * 64 >= k) return;
    typedef const double __attribute__((address_space(1))) cgdouble;
    typedef double __attribute__((address_space(1))) gdouble;
    cgdouble* T = (cgdouble*)jb.tmp;
    cgdouble* Z = T + (size_t)k * k;
    cgdouble* TF = (cgdouble*)jb.scratch;
    gdouble* E = (gdouble*)jb.Gacc;
    extern __shared__ double s_v[];                          // [16][PITCH]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, li = lane & 15, lk = lane >> 4;
    const int nt = (k + 15) / 16;
    const int col = gc * 64 + wave * 16 + li;
    d4 z[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int i = 16 * t + 4 * v + lk;
            z[t][v] = (i < k && col < k) ? Z[(size_t)min(i, k - 1) * k + min(col, k - 1)] : 0.0;
        }
    // block b of V: thread tid takes entry tid % 16 of every row tile of reflector tid / 16
    double vr[PER], tf[4], tn[4];
    auto fetch = [&](int b) {
        const int j = 16 * b + (tid >> 4);
        const bool valid = eig_has_reflector(j, k);
        cgdouble* row = T + (size_t)min(j, k - 1) * k;
        const bool live = valid && row[min(j, k - 1)] != 0.0;
#pragma unroll
        for (int t = 0; t < PER; ++t) {
            const int i = 16 * t + (tid & 15);
            if (t >= b) {                                    // uniform
                const double x = row[min(i, k - 1)];
                vr[t] = (live && i > j && i < k) ? x : 0.0;
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) tn[q] = (li < eig_wy_rank(k, b) && 4 * q + lk < eig_wy_rank(k, b)) ? TF[eig_wy_at(b, li, 4 * q + lk)] : 0.0;
    };
    const int last = (k >= 3) ? (k - 3) / 16 : -1;
    if (last >= 0) fetch(last);
    for (int b = last; b >= 0; --b) {
#pragma unroll
        for (int t = 0; t < PER; ++t)
            if (t >= b) s_v[(tid >> 4) * PITCH + 16 * t + (tid & 15)] = vr[t];
#pragma unroll
        for (int q = 0; q < 4; ++q) tf[q] = tn[q];
        eig_lds_barrier();
        if (b > 0) fetch(b - 1);
        // W = V^T Z, two tiles at a time
        d4 w0 = {0.0, 0.0, 0.0, 0.0}, w1 = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int t = 0; t < RT; t += 2) {
            if (t + 1 >= b && t < nt) {
                double a0[4], a1[4];
                const bool two = t + 1 < RT;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    a0[q] = (t >= b) ? s_v[li * PITCH + 16 * t + 4 * q + lk] : 0.0;
                    a1[q] = (two && t + 1 < nt) ? s_v[li * PITCH + 16 * (t + 1) + 4 * q + lk] : 0.0;
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    w0 = __builtin_amdgcn_mfma_f64_16x16x4f64(a0[q], z[t][q], w0, 0, 0, 0);
                    if (two) w1 = __builtin_amdgcn_mfma_f64_16x16x4f64(a1[q], z[t + 1 < RT ? t + 1 : t][q], w1, 0, 0, 0);
                }
            }
        }
        w0 += w1;
        d4 sm = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int q = 0; q < 4; ++q) sm = __builtin_amdgcn_mfma_f64_16x16x4f64(tf[q], w0[q], sm, 0, 0, 0);
        sm = -sm;
#pragma unroll
        for (int t = 0; t < RT; t += 2) {
            if (t + 1 >= b && t < nt) {
                double a0[4], a1[4];
                const bool two = t + 1 < RT;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    a0[q] = (t >= b) ? s_v[(4 * q + lk) * PITCH + 16 * t + li] : 0.0;
                    a1[q] = (two && t + 1 < nt) ? s_v[(4 * q + lk) * PITCH + 16 * (t + 1) + li] : 0.0;
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    z[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0[q], sm[q], z[t], 0, 0, 0);
                    if (two) z[t + 1 < RT ? t + 1 : t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1[q], sm[q], z[t + 1 < RT ? t + 1 : t], 0, 0, 0);
                }
            }
        }
        eig_lds_barrier();
    }
    if (col < k) {
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int i = 16 * t + 4 * v + lk;
                if (i < k) E[(size_t)col * k + i] = z[t][v];
            }
    }
}

template <int RT>
hipError_t launch_backtransform(const JacobiBlock* table_dev, const JacobiBlock& single, int blocks, int max_k, hipStream_t stream) {
    constexpr int lds = 16 * ((16 * RT + 13) / 32 * 32 + 18) * 8;
    const hipError_t e = allow_lds((const void*)eig_backtransform_kernel<RT>, lds);
    if (e != hipSuccess) return e;
    const EigGrid g{blocks, (max_k + 63) / 64, 0};
    hipLaunchKernelGGL(eig_backtransform_kernel<RT>, eig_grid(g), dim3(256), lds, stream, table_dev, single, g);
    return hipGetLastError();
}

// ------------------------------------------------------------------ ordering and outputs
// Rows of E^T R (second half of tmp) are mutually orthogonal with norms sigma_i: the norms go behind the
// eigenvalues' place, one wave per row ...
__global__ __launch_bounds__(256) void eig_norms_kernel(const JacobiBlock* table, const JacobiBlock single, const EigGrid grid) {
    JacobiBlock jb = single;
    int gb, gc;
    if (!eig_decode(grid, gb, gc)) return;
    if (table) jb = table[gb];
    const int k = jb.k;
    const int lane = threadIdx.x & 63, j = gc * 4 + (threadIdx.x >> 6);
    if (j >= k) return;
    typedef const double __attribute__((address_space(1))) cgdouble;
    cgdouble* row = (cgdouble*)jb.tmp + (size_t)k * k + (size_t)j * k;
    double a = 0.0;
    for (int c = lane; c < k; c += 64) a = fma(row[c], row[c], a);
    a = eig_wave_sum_dpp(a);
    if (lane == 0) jb.scratch[eig_tridiag_at(k) + j] = sqrt(a);      // (the tridiagonal matrix is not needed any more)
}

// ... and every wave then finds the place of its row among them and writes the row's outputs.
__global__ __launch_bounds__(256) void eig_finish_kernel(const JacobiBlock* table, const JacobiBlock single, const EigGrid grid) {
    JacobiBlock jb = single;
    int gb, gc;
    if (!eig_decode(grid, gb, gc)) return;
    if (table) jb = table[gb];
    const int k = jb.k, r = jb.r;
    const int lane = threadIdx.x & 63, j = gc * 4 + (threadIdx.x >> 6);
    if (j >= k) return;
    typedef const double __attribute__((address_space(1))) cgdouble;
    typedef float __attribute__((address_space(1))) gfloat;
    cgdouble* ER = (cgdouble*)jb.tmp + (size_t)k * k + (size_t)j * k;
    cgdouble* E = (cgdouble*)jb.Gacc + (size_t)j * k;
    cgdouble* sig = (cgdouble*)jb.scratch + eig_tridiag_at(k);
    const double sj = sig[j];
    int rank = 0;                                            // descending, ties by index
    double top = 0.0;
    for (int i = lane; i < k; i += 64) {
        const double si = sig[i];
        rank += (si > sj || (si == sj && i < j)) ? 1 : 0;
        top = fmax(top, si);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        rank += __shfl_xor(rank, o, 64);
        top = fmax(top, __shfl_xor(top, o, 64));
    }
    if (lane == 0 && jb.sigma) jb.sigma[rank] = (float)sj;
    if (rank >= r) return;
    const bool null = sj <= SVD_NULL * top;                  // (not a NaN, which is passed on)
    const double inv = null ? 0.0 : 1.0 / sj;
    gfloat* xr = (gfloat*)jb.XrT + (size_t)rank * k;
    gfloat* gr = (gfloat*)jb.GrT + (size_t)rank * k;
    for (int c = lane; c < k; c += 64) {
        xr[c] = (float)(ER[c] * inv);
        gr[c] = null ? 0.0f : (float)E[c];
    }
}

}  // namespace

hipError_t launch_rtot_product(const JacobiBlock* table_dev, const JacobiBlock* single, int blocks, int max_k,
                               hipStream_t stream) {
    if (blocks <= 0 || max_k < 1) return hipSuccess;
    JacobiBlock sb{};
    if (single) sb = *single;
    const int tiles = (max_k + 63) / 64;
    const EigGrid gt{blocks, tiles * tiles, 0};
    hipLaunchKernelGGL(eig_gemm_kernel<2>, eig_grid(gt), dim3(256), 0, stream, table_dev, sb, gt);
    return hipGetLastError();
}

hipError_t launch_eig_svd(const JacobiBlock* table_dev, const JacobiBlock* single, int blocks, int max_k,
                          hipStream_t stream) {
    if (blocks <= 0) return hipSuccess;
    if (max_k > EIG_MAXK || max_k < 1) return hipErrorInvalidValue;
    JacobiBlock sb{};
    if (single) sb = *single;
    const int tiles = (max_k + 63) / 64;
    const EigGrid gt{blocks, tiles * tiles, 0};
    const EigGrid gi{blocks, (max_k + 63) / 64, 1};      // measured: pinned 0.70 ms, chunk-major 0.74 (84 blocks, k = 264)
    hipLaunchKernelGGL(eig_gemm_kernel<0>, eig_grid(gt), dim3(256), 0, stream, table_dev, sb, gt);
    // tile rows of the register kernel by the largest matrix of the launch
    if (max_k > EIG_TILES_K) hipLaunchKernelGGL(eig_tridiag_kernel, dim3(blocks), dim3(EIG_THREADS), 0, stream, table_dev, sb);
    if (max_k <= 3 * TT) hipLaunchKernelGGL((eig_tridiag_tiles_kernel<3, 6>), dim3(blocks), dim3(384), 0, stream, table_dev, sb);
    else if (max_k <= 5 * TT) hipLaunchKernelGGL((eig_tridiag_tiles_kernel<5, 8>), dim3(blocks), dim3(512), 0, stream, table_dev, sb);
    else if (max_k <= 7 * TT) hipLaunchKernelGGL((eig_tridiag_tiles_kernel<7, 8>), dim3(blocks), dim3(512), 0, stream, table_dev, sb);
    else hipLaunchKernelGGL((eig_tridiag_tiles_kernel<9, 8>), dim3(blocks), dim3(512), 0, stream, table_dev, sb);
    // threads per eigenvalue: up to a wave, as long as the launch stays within two waves per SIMD
    int lp = 6;
    while (lp > 3 && ((long long)blocks * max_k << lp) > 2LL * 1024 * 64) --lp;
    const EigGrid gv{blocks, ((max_k << lp) + 255) / 256, 0};
    if (lp == 6) hipLaunchKernelGGL(eig_values_kernel<6>, eig_grid(gv), dim3(256), 0, stream, table_dev, sb, gv);
    else if (lp == 5) hipLaunchKernelGGL(eig_values_kernel<5>, eig_grid(gv), dim3(256), 0, stream, table_dev, sb, gv);
    else if (lp == 4) hipLaunchKernelGGL(eig_values_kernel<4>, eig_grid(gv), dim3(256), 0, stream, table_dev, sb, gv);
    else hipLaunchKernelGGL(eig_values_kernel<3>, eig_grid(gv), dim3(256), 0, stream, table_dev, sb, gv);
    const int vectors = eig_invit_vectors(max_k);
    if (max_k <= EIG_INVIT_LDS_K && (long long)blocks * ((max_k + vectors - 1) / vectors) <= 256) {
        const hipError_t e = vectors == 64 ? launch_invit_lds<64>(table_dev, sb, blocks, max_k, stream)
                                           : launch_invit_lds<32>(table_dev, sb, blocks, max_k, stream);
        if (e != hipSuccess) return e;
    } else {
        hipLaunchKernelGGL(eig_invit_kernel, eig_grid(gi), dim3(64), 0, stream, table_dev, sb, gi);
    }
    hipLaunchKernelGGL(eig_groups_kernel, dim3(blocks), dim3(EIG_THREADS), 0, stream, table_dev, sb);
    const EigGrid gwy{blocks, (max_k + 15) / 16, 0}, gr{blocks, (max_k + 3) / 4, 0};
    hipLaunchKernelGGL(eig_wy_kernel, eig_grid(gwy), dim3(64), 0, stream, table_dev, sb, gwy);
    const hipError_t bt = (max_k <= 80) ? launch_backtransform<5>(table_dev, sb, blocks, max_k, stream)
                          : (max_k <= 144) ? launch_backtransform<9>(table_dev, sb, blocks, max_k, stream)
                          : (max_k <= 288) ? launch_backtransform<18>(table_dev, sb, blocks, max_k, stream)
                                           : launch_backtransform<34>(table_dev, sb, blocks, max_k, stream);
    if (bt != hipSuccess) return bt;
    hipLaunchKernelGGL(eig_gemm_kernel<1>, eig_grid(gt), dim3(256), 0, stream, table_dev, sb, gt);
    hipLaunchKernelGGL(eig_norms_kernel, eig_grid(gr), dim3(256), 0, stream, table_dev, sb, gr);
    hipLaunchKernelGGL(eig_finish_kernel, eig_grid(gr), dim3(256), 0, stream, table_dev, sb, gr);
    return hipGetLastError();
}

}  // namespace tsr
