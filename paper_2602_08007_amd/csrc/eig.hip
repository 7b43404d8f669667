// SVD of the k x k triangular factor R of the refresh (the "small SVD" of the randomized SVD,
// Algorithm 1's refresh step) as a chain of launches, for k <= EIG_MAXK:
//   1. T = R R^T                        fp64 MFMA GEMM, 64 x 64 tiles over the whole chip
//   2. per matrix, one workgroup:       Householder tridiagonalization of T (reflectors parked in
//      the rows of T they cleared), the last 288 columns in registers; then eigenvalues by Sturm-count multisection (chip-wide),
//      eigenvectors of the tridiagonal matrix by inverse iteration (one per thread, pivoted LU
//      of T - lambda I), Gram-Schmidt inside groups of numerically equal eigenvalues
//   3. E = H_0 H_1 ... Z                reflectors applied to 64 eigenvectors per workgroup, the
//      vectors held in registers
//   4. E^T R                            fp64 MFMA GEMM
//   5. singular values = row norms of E^T R, ordering, fp32 outputs
// Nothing here is a serial chain longer than k steps, which is what separates it from the QL
// sweeps of the single-kernel variant (about k^2 dependent rotations per matrix).
#include <hip/hip_runtime.h>

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
    const double* __restrict__ A;
    const double* __restrict__ B = (WHICH == 2) ? blk->R1 : blk->R;
    double* __restrict__ C;
    long long sam, sak, sbk, sbn;
    int k_lo = 0, k_hi = k;
    if (WHICH == 0) { A = blk->R; sam = k; sak = 1; sbk = 1; sbn = k; C = blk->tmp; k_lo = max(m0, n0) & ~3; }
    else if (WHICH == 1) { A = blk->Gacc; sam = 1; sak = k; sbk = k; sbn = 1; C = blk->tmp + (size_t)k * k; k_hi = min(k, n0 + 32); }
    else { A = blk->Gacc; sam = k; sak = 1; sbk = k; sbn = 1; C = blk->R; k_lo = m0 & ~3; k_hi = min(k, n0 + 32); }
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
    for (int kk = k_lo; kk < k_hi; kk += 16) {
        double a[4][2], b[4][2];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int kc = kk + 4 * u + lk;
            const bool kok = kc < k_hi;
            const long long kcc = min(kc, k - 1);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const double av = A[arow[i] + kcc * sak];
                const double bv = B[kcc * sbk + bcol[i]];
                a[u][i] = (kok && aok[i]) ? av : 0.0;
                b[u][i] = (kok && bok[i]) ? bv : 0.0;
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u][i], b[u][j], acc[i][j], 0, 0, 0);
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
// (v, w) are indexed from t for the pending pair and from t+1 for the new one.
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
        v = eig_wave_sum(v);
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
        const bool skip = (xnorm2 - x0 * x0 <= 0.0) || vnorm2 <= 0.0;        // already tridiagonal here
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
            rowacc = eig_wave_sum(rowacc);
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
    double* DE = blk->scratch + (size_t)3 * k * k;
    for (int i = tid; i < stop; i += nt) { DE[i] = s_d[i]; DE[k + i] = s_e[i]; }
}

// ---- Tridiagonalization with the matrix in registers, for the trailing part of at most 288 columns.
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
        const bool skip = !(xnorm2 - x0 * x0 > 0.0);           // already tridiagonal here
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
    double* DE = jb.scratch + (size_t)3 * kfull * kfull;
    for (int i = tid; i < k; i += 64 * WAVES) { DE[first + i] = s_d[i]; DE[kfull + first + i] = s_e[i]; }
}

// Eigenvalues and eigenvectors of the tridiagonal matrix (d, e) left by eig_tridiag_kernel, in
// three launches: eigenvalues (chip-wide), inverse iteration (one wave per workgroup),
// orthogonalisation inside groups of numerically equal eigenvalues (one workgroup per matrix).
// Behind the LU scratch (3 k^2 doubles) sit d (k), e (k), the eigenvalues (k, ascending) and the
// radius of the spectrum's bracket (1; zero marks a zero or non-finite matrix).

// Sturm-count multisection: 32 eigenvalues per workgroup, 8 threads each; 7 probes cut an
// eigenvalue's bracket into 8 pieces per pass, and the number of eigenvalues below a probe
// tells on which side of it the wanted one lies.
constexpr int EIG_VAL_PER_WG = 32;
__global__ __launch_bounds__(256) void eig_values_kernel(const JacobiBlock* table, const JacobiBlock single, const EigGrid grid) {
    JacobiBlock jb = single;
    int gb, gc;
    if (!eig_decode(grid, gb, gc)) return;
    if (table) jb = table[gb];
    const JacobiBlock* blk = &jb;
    const int k = blk->k;
    const int e0 = gc * EIG_VAL_PER_WG;
    if (e0 >= k) return;
    const double* DE = blk->scratch + (size_t)3 * k * k;
    double* LAM = blk->scratch + (size_t)3 * k * k + 2 * k;
    const int tid = threadIdx.x, nt = blockDim.x;
    const int lane = tid & 63, wave = tid >> 6, nw = nt >> 6;
    __shared__ double s_d[EIG_MAXK];            // diagonal
    __shared__ double s_w[EIG_MAXK];            // squared sub-diagonal
    __shared__ double s_lo[EIG_VAL_PER_WG];     // eigenvalue brackets
    __shared__ double s_hi[EIG_VAL_PER_WG];
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
    double gl = 0.0, gu = 0.0;
    {
        double lo = 1e300, hi = -1e300;
        for (int i = tid; i < k; i += nt) {
            const double di = DE[i], ei = DE[k + i];
            const double rad = ((i > 0) ? fabs(DE[k + i - 1]) : 0.0) + ((i < k - 1) ? fabs(ei) : 0.0);
            lo = fmin(lo, di - rad);
            hi = fmax(hi, di + rad);
            s_d[i] = di;
            s_w[i] = ei * ei;
        }
        gu = block_max(hi);
        gl = -block_max(-lo);
    }
    double tnorm = fmax(fabs(gl), fabs(gu));
    const bool degenerate = !(tnorm > 0.0) || !(tnorm < 1e300);   // zero (or non-finite) matrix
    if (degenerate) tnorm = 0.0;
    if (gc == 0 && tid == 0) LAM[k] = tnorm;
    if (degenerate) {
        if (tid < EIG_VAL_PER_WG && e0 + tid < k) LAM[e0 + tid] = 0.0;
        return;
    }
    const double pivmin = fmax(1e-290, 1e-32 * tnorm);
    {
        const double margin = 2.0 * EIG_EPS * tnorm * (double)k + 2.0 * pivmin;
        gl -= margin; gu += margin;
    }
    constexpr int S = 7;
    const int el = tid >> 3, es = tid & 7;
    const int ej = e0 + el;
    const bool eact = ej < k && es < S;
    int passes = 0;
    for (double shrink = 1.0; shrink < 1.5e17; shrink *= (double)(S + 1)) ++passes;       // 2^-57 of the bracket
    if (tid < EIG_VAL_PER_WG) { s_lo[tid] = gl; s_hi[tid] = gu; }
    __syncthreads();
    const double inv_pieces = 1.0 / (double)(S + 1);
    for (int pass = 0; pass < passes; ++pass) {
        if (eact) {
            const double lo = s_lo[el], hi = s_hi[el];
            const double x = lo + (double)(es + 1) * ((hi - lo) * inv_pieces);
            double q = s_d[0] - x;
            if (fabs(q) < pivmin) q = -pivmin;
            int cnt = (q < 0.0) ? 1 : 0;
            for (int i = 1; i < k; ++i) {
                q = (s_d[i] - x) - s_w[i - 1] * eig_rcp(q);
                if (fabs(q) < pivmin) q = -pivmin;
                cnt += (q < 0.0) ? 1 : 0;
            }
            s_cnt[tid] = cnt;
        }
        __syncthreads();
        if (eact && es == 0) {
            const double lo = s_lo[el], hi = s_hi[el];
            const double step = (hi - lo) * inv_pieces;
            int m = 0;                                       // leading probes at or below eigenvalue ej
            while (m < S && s_cnt[tid + m] <= ej) ++m;
            if (m > 0) s_lo[el] = lo + (double)m * step;
            if (m < S) s_hi[el] = lo + (double)(m + 1) * step;
        }
        __syncthreads();
    }
    if (tid < EIG_VAL_PER_WG && e0 + tid < k) LAM[e0 + tid] = 0.5 * (s_lo[tid] + s_hi[tid]);
}

// Eigenvectors by inverse iteration, vector j on its own thread, one wave per workgroup (the
// recurrences are serial in the row index and wait on L2 for their operands: a wave alone on
// its SIMD; up to sixteen rows are fetched at a time).  T - lambda I = P L U with
// partial pivoting; U (three diagonals, pivots as reciprocals) is kept, L is applied to the
// right-hand side while it is formed and formed again in every round.
__global__ __launch_bounds__(64) void eig_invit_kernel(const JacobiBlock* table, const JacobiBlock single, const EigGrid grid) {
    JacobiBlock jb = single;
    int gb, gc;
    if (!eig_decode(grid, gb, gc)) return;
    if (table) jb = table[gb];
    const JacobiBlock* blk = &jb;
    const int k = blk->k;
    if (gc * 64 >= k) return;
    double* Z = blk->tmp + (size_t)k * k;       // eigenvectors of the tridiagonal matrix, Z[i][j] = j-th vector
    double* U0 = blk->scratch;                  // per thread j: reciprocal pivots, first and second
    double* U1 = U0 + (size_t)k * k;            //   super-diagonal of the LU factor, entry [i][j]
    double* U2 = U1 + (size_t)k * k;
    const double* DE = blk->scratch + (size_t)3 * k * k;
    const double* LAM = DE + 2 * k;
    const int tid = threadIdx.x;
    const int j = gc * 64 + tid;
    __shared__ double s_d[EIG_MAXK];            // diagonal
    __shared__ double s_e[EIG_MAXK];            // sub-diagonal, s_e[i] couples i and i + 1
    for (int i = tid; i < k; i += 64) { s_d[i] = DE[i]; s_e[i] = DE[k + i]; }
    __syncthreads();
    const double tnorm = LAM[k];
    if (tnorm == 0.0) {
        // zero (or non-finite) matrix: every orthonormal basis is one of eigenvectors
        if (j < k) for (int i = 0; i < k; ++i) Z[(size_t)i * k + j] = (i == j) ? 1.0 : 0.0;
        return;
    }
    const double tiny = EIG_EPS * tnorm;                 // floor of an LU pivot
    int vz;                                              // a zero the compiler keeps in a vector register
    asm volatile("v_mov_b32 %0, 0" : "=v"(vz));
    if (j < k) {
        const double lam = LAM[j];
        double* zc = Z + j;
        double* u0 = U0 + j; double* u1 = U1 + j; double* u2 = U2 + j;
        double scale = 1.0;
        for (int round = 0; round < EIG_INVIT_ROUNDS; ++round) {
            // forward: eliminate, apply to y (first time round: the start vector, later scale * previous x)
            auto yval = [&](int i) -> double {
                return (round == 0) ? eig_start_value((unsigned)i, (unsigned)j) : scale * zc[(size_t)i * k];
            };
            double a = s_d[0] - lam, b = (k > 1) ? s_e[0] : 0.0;
            double ycur = yval(0);
            auto step = [&](int i, double ynext) {
                const double c = s_e[i];
                const double dn = s_d[i + 1] - lam;
                const double en = (i + 2 < k) ? s_e[i + 1] : 0.0;
                const size_t o = (size_t)i * k;
                if (fabs(a) >= fabs(c)) {
                    double piv = a;
                    if (fabs(piv) < tiny) piv = (piv < 0.0) ? -tiny : tiny;
                    const double inv = eig_rcp(piv);
                    const double mult = c * inv;
                    if (round == 0) { u0[o] = inv; u1[o] = b; u2[o] = 0.0; }
                    zc[o] = ycur;
                    a = dn - mult * b; b = en;
                    ycur = ynext - mult * ycur;
                } else {
                    double piv = c;
                    if (fabs(piv) < tiny) piv = (piv < 0.0) ? -tiny : tiny;
                    const double inv = eig_rcp(piv);
                    const double mult = a * inv;
                    if (round == 0) { u0[o] = inv; u1[o] = dn; u2[o] = en; }
                    zc[o] = ynext;
                    a = b - mult * dn; b = -mult * en;
                    ycur = ycur - mult * ynext;
                }
            };
            {
                int i = 0;
                for (; i + 16 < k; i += 16) {                // rows i+1 .. i+16 fetched together
                    double yn[16];
#pragma unroll
                    for (int u = 0; u < 16; ++u) yn[u] = yval(i + 1 + u);
#pragma unroll
                    for (int u = 0; u < 16; ++u) step(i + u, yn[u]);
                }
                for (; i + 1 < k; ++i) step(i, yval(i + 1));
            }
            {
                double piv = a;
                if (fabs(piv) < tiny) piv = (piv < 0.0) ? -tiny : tiny;
                if (round == 0) { u0[(size_t)(k - 1) * k] = eig_rcp(piv); u1[(size_t)(k - 1) * k] = 0.0; u2[(size_t)(k - 1) * k] = 0.0; }
                zc[(size_t)(k - 1) * k] = ycur;
            }
            // backward: U x = y, sixteen rows fetched together (row offsets kept in vector registers:
            // as wave-uniform values they would need more scalar registers than there are)
            double x1 = 0.0, x2 = 0.0, amax = 0.0;      // x[i+1], x[i+2]
            bool bad = false;
            int i = k - 1;
            for (; i >= 15; i -= 16) {
                double y[16], p0[16], p1[16], p2[16];
#pragma unroll
                for (int u = 0; u < 16; ++u) {
                    const size_t o = (size_t)(i - u + vz) * k;
                    y[u] = zc[o]; p0[u] = u0[o]; p1[u] = u1[o]; p2[u] = u2[o];
                }
#pragma unroll
                for (int u = 0; u < 16; ++u) {
                    const double x = (y[u] - p1[u] * x1 - p2[u] * x2) * p0[u];
                    zc[(size_t)(i - u) * k] = x;
                    amax = fmax(amax, fabs(x));
                    bad = bad || !(fabs(x) <= 1e300);
                    x2 = x1; x1 = x;
                }
            }
            for (; i >= 0; --i) {
                const size_t o = (size_t)i * k;
                const double x = (zc[o] - u1[o] * x1 - u2[o] * x2) * u0[o];
                zc[o] = x;
                amax = fmax(amax, fabs(x));
                bad = bad || !(fabs(x) <= 1e300);
                x2 = x1; x1 = x;
            }
            if (bad || !(amax > 0.0)) {
                // overflow or a vanished vector (the floored pivots are meant to rule both out):
                // go on from the unit vector rather than carry a non-finite value
                for (int q = 0; q < k; ++q) zc[(size_t)q * k] = (q == j) ? 1.0 : 0.0;
                amax = 1.0;
            }
            scale = 1.0 / amax;
        }
        double ss = 0.0;
        for (int i = 0; i < k; ++i) { const double x = scale * zc[(size_t)i * k]; ss += x * x; }
        const double nrm = scale / sqrt(ss);
        for (int i = 0; i < k; ++i) zc[(size_t)i * k] *= nrm;
    }
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
    const double* LAM = blk->scratch + (size_t)3 * k * k + 2 * k;
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
        for (int j = 1; j < k; ++j) {
            const int cs = s_first[j];
            if (cs == j) continue;                       // uniform
            for (int pass = 0; pass < 2; ++pass) {
                for (int i = cs + wave; i < j; i += nw) {
                    double a = 0.0;
                    for (int t = lane; t < k; t += 64) a += Z[(size_t)t * k + i] * Z[(size_t)t * k + j];
                    a = eig_wave_sum(a);
                    if (lane == 0) coef[i - cs] = a;
                }
                __syncthreads();
                for (int t = tid; t < k; t += nt) {
                    double a = 0.0;
                    for (int i = cs; i < j; ++i) a += coef[i - cs] * Z[(size_t)t * k + i];
                    Z[(size_t)t * k + j] -= a;
                }
                __syncthreads();
            }
            double ss = 0.0;
            for (int t = tid; t < k; t += nt) { const double x = Z[(size_t)t * k + j]; ss += x * x; }
            ss = block_sum(ss);
            const double inv = (ss > 0.0) ? 1.0 / sqrt(ss) : 0.0;
            for (int t = tid; t < k; t += nt) Z[(size_t)t * k + j] *= inv;
            __syncthreads();
        }
    }
}

// ------------------------------------------------------------------ back-transformation
// E = H_0 H_1 ... H_{k-3} Z for 64 columns of Z per workgroup: lane = column, each of the WAVES
// waves owns EPT consecutive rows (in registers); the reflector entries are uniform over a
// wave.  One barrier per reflector (the dot product spans the waves).
template <int EPT, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void eig_backtransform_kernel(const JacobiBlock* table, const JacobiBlock single, const EigGrid grid) {
    JacobiBlock jb = single;
    int gb, gc;
    if (!eig_decode(grid, gb, gc)) return;
    if (table) jb = table[gb];
    const JacobiBlock* blk = &jb;
    const int k = blk->k;
    const int c0 = gc * 64;
    if (c0 >= k) return;
    typedef const double __attribute__((address_space(1))) gdouble;
    typedef double d8 __attribute__((ext_vector_type(8)));
    typedef d8 __attribute__((aligned(8))) d8u;
    typedef const d8u __attribute__((address_space(1))) cd8u;
    static_assert(EPT % 8 == 0, "rows per wave come in chunks of eight");
    // the reflector entries have wave-uniform addresses: they travel through the scalar data path
    const gdouble* __restrict__ T = (const gdouble*)blk->tmp;
    const double* __restrict__ Z = blk->tmp + (size_t)k * k;
    double* __restrict__ E = blk->Gacc;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = c0 + lane;
    const bool colok = col < k;
    const int i0 = wave * EPT;
    __shared__ double s_dot[2][WAVES][64];
    double x[EPT];
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        const int i = i0 + e;
        x[e] = (colok && i < k) ? Z[(size_t)min(i, k - 1) * k + min(col, k - 1)] : 0.0;
    }
    int par = 0;
    for (int j = k - 3; j >= 0; --j) {
        const double beta = T[(size_t)j * k + j];
        if (beta == 0.0) continue;                          // uniform: no reflector at this step
        const gdouble* __restrict__ vrow = T + (size_t)j * k;
        const bool active = i0 + EPT > j + 1 && i0 < k;     // uniform over the wave
        // eight reflector entries per fetch; chunks that end at or before j hold no entry of v.
        // (A chunk may reach past column k-1: what it reads there is still inside tmp, which
        // carries 64 doubles of padding for the smallest k, and is masked out.)
        double part = 0.0;
        if (active) {
#pragma unroll
            for (int c = 0; c < EPT / 8; ++c) {
                const int ib = i0 + 8 * c;
                if (ib > j && ib + 7 < k) {                 // whole chunk inside the reflector
                    const d8u v8 = *(const cd8u*)(vrow + ib);
#pragma unroll
                    for (int u = 0; u < 8; ++u) part += v8[u] * x[8 * c + u];
                } else if (ib + 7 > j && ib < k) {
                    const d8u v8 = *(const cd8u*)(vrow + ib);
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const double v = (ib + u > j && ib + u < k) ? v8[u] : 0.0;
                        part += v * x[8 * c + u];
                    }
                }
            }
        }
        s_dot[par][wave][lane] = part;
        __syncthreads();
        double tot = 0.0;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) tot += s_dot[par][w][lane];
        const double s = beta * tot;
        if (active) {
#pragma unroll
            for (int c = 0; c < EPT / 8; ++c) {
                const int ib = i0 + 8 * c;
                if (ib > j && ib + 7 < k) {
                    const d8u v8 = *(const cd8u*)(vrow + ib);
#pragma unroll
                    for (int u = 0; u < 8; ++u) x[8 * c + u] -= s * v8[u];
                } else if (ib + 7 > j && ib < k) {
                    const d8u v8 = *(const cd8u*)(vrow + ib);
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const double v = (ib + u > j && ib + u < k) ? v8[u] : 0.0;
                        x[8 * c + u] -= s * v;
                    }
                }
            }
        }
        par ^= 1;
    }
    if (colok) {
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            const int i = i0 + e;
            if (i < k) E[(size_t)i * k + col] = x[e];
        }
    }
}

// ------------------------------------------------------------------ ordering and outputs
// Rows of E^T R (second half of tmp) are mutually orthogonal with norms sigma_i.
__global__ __launch_bounds__(EIG_THREADS) void eig_finish_kernel(const JacobiBlock* table, const JacobiBlock single) {
    JacobiBlock jb = single;
    if (table) jb = table[blockIdx.x];
    const JacobiBlock* blk = &jb;
    const int k = blk->k, r = blk->r;
    const double* __restrict__ ER = blk->tmp + (size_t)k * k;
    const double* __restrict__ E = blk->Gacc;
    const int tid = threadIdx.x, nt = blockDim.x;
    const int lane = tid & 63, wave = tid >> 6, nw = nt >> 6;
    __shared__ double s_sig[EIG_MAXK];
    __shared__ int s_rank[EIG_MAXK];
    for (int j = wave; j < k; j += nw) {
        double a = 0.0;
        for (int c = lane; c < k; c += 64) { const double v = ER[(size_t)j * k + c]; a += v * v; }
        a = eig_wave_sum(a);
        if (lane == 0) s_sig[j] = sqrt(a);
    }
    __syncthreads();
    for (int j = tid; j < k; j += nt) {
        const double sj = s_sig[j];
        int rank = 0;
        for (int i = 0; i < k; ++i) {
            const double si = s_sig[i];
            rank += (si > sj || (si == sj && i < j)) ? 1 : 0;
        }
        s_rank[j] = rank;
        if (blk->sigma) blk->sigma[rank] = (float)sj;
    }
    __syncthreads();
    for (int j = wave; j < k; j += nw) {
        const int rank = s_rank[j];
        if (rank >= r) continue;
        const double sj = s_sig[j];
        const double inv = (sj > 0.0) ? 1.0 / sj : 0.0;
        for (int c = lane; c < k; c += 64) {
            blk->XrT[(size_t)rank * k + c] = (float)(ER[(size_t)j * k + c] * inv);
            blk->GrT[(size_t)rank * k + c] = (float)E[(size_t)c * k + j];
        }
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
    const EigGrid gv{blocks, (max_k + EIG_VAL_PER_WG - 1) / EIG_VAL_PER_WG, 0};
    const EigGrid gi{blocks, (max_k + 63) / 64, 1};      // measured: pinned 0.70 ms, chunk-major 0.74 (84 blocks, k = 264)
    hipLaunchKernelGGL(eig_gemm_kernel<0>, eig_grid(gt), dim3(256), 0, stream, table_dev, sb, gt);
    // tile rows of the register kernel by the largest matrix of the launch
    if (max_k > EIG_TILES_K) hipLaunchKernelGGL(eig_tridiag_kernel, dim3(blocks), dim3(EIG_THREADS), 0, stream, table_dev, sb);
    if (max_k <= 3 * TT) hipLaunchKernelGGL((eig_tridiag_tiles_kernel<3, 6>), dim3(blocks), dim3(384), 0, stream, table_dev, sb);
    else if (max_k <= 5 * TT) hipLaunchKernelGGL((eig_tridiag_tiles_kernel<5, 8>), dim3(blocks), dim3(512), 0, stream, table_dev, sb);
    else if (max_k <= 7 * TT) hipLaunchKernelGGL((eig_tridiag_tiles_kernel<7, 8>), dim3(blocks), dim3(512), 0, stream, table_dev, sb);
    else hipLaunchKernelGGL((eig_tridiag_tiles_kernel<9, 8>), dim3(blocks), dim3(512), 0, stream, table_dev, sb);
    hipLaunchKernelGGL(eig_values_kernel, eig_grid(gv), dim3(256), 0, stream, table_dev, sb, gv);
    hipLaunchKernelGGL(eig_invit_kernel, eig_grid(gi), dim3(64), 0, stream, table_dev, sb, gi);
    hipLaunchKernelGGL(eig_groups_kernel, dim3(blocks), dim3(EIG_THREADS), 0, stream, table_dev, sb);
    const EigGrid gbt{blocks, tiles, 0};
    const dim3 bt_grid = eig_grid(gbt);
    if (max_k <= 32) hipLaunchKernelGGL((eig_backtransform_kernel<8, 4>), bt_grid, dim3(256), 0, stream, table_dev, sb, gbt);
    else if (max_k <= 96) hipLaunchKernelGGL((eig_backtransform_kernel<24, 4>), bt_grid, dim3(256), 0, stream, table_dev, sb, gbt);
    else if (max_k <= 160) hipLaunchKernelGGL((eig_backtransform_kernel<40, 4>), bt_grid, dim3(256), 0, stream, table_dev, sb, gbt);
    else if (max_k <= 320) hipLaunchKernelGGL((eig_backtransform_kernel<40, 8>), bt_grid, dim3(512), 0, stream, table_dev, sb, gbt);
    else hipLaunchKernelGGL((eig_backtransform_kernel<40, 16>), bt_grid, dim3(1024), 0, stream, table_dev, sb, gbt);
    hipLaunchKernelGGL(eig_gemm_kernel<1>, eig_grid(gt), dim3(256), 0, stream, table_dev, sb, gt);
    hipLaunchKernelGGL(eig_finish_kernel, dim3(blocks), dim3(EIG_THREADS), 0, stream, table_dev, sb);
    return hipGetLastError();
}

}  // namespace tsr
