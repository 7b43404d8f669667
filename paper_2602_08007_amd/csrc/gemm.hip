// Grouped tall-skinny GEMM on gfx950 matrix cores: TM x TN output tile (128 x 128, 128 x 64 or 64 x 64)
// per 256-thread workgroup, 32-deep k-tiles staged through LDS as bf16 pieces, fp32 accumulation with
// v_mfma_f32_32x32x16_bf16 (the four waves own the four quadrants of the tile).
//
// Global -> registers (two or three k-tiles ahead) -> split into bf16 pieces -> LDS in [row][k] order ->
// 16-byte fragment reads.  Both operand orientations end up in the same LDS layout, so the MFMA loop is
// shared by all variants.
//
// What bounds it: with few tiles per compute unit the trips to memory, with many the LDS traffic (with
// two pieces per operand 64 KB of fragment reads and 40 KB of stores per k-tile against 768 cycles of
// MFMAs) and the conversions.  Hence two register stages, branch-free loads in the loop (edges by clamped
// addresses, the rest of a partial k-tile by a mask when it is stored), two LDS buffers with one barrier per
// k-tile where they fit twice into a compute unit, the next k-tile converted and stored behind the products
// of the current one, and for operands stored across k a lane layout (eight lanes along k, eight along the
// rows) whose transposing LDS stores touch every bank once: with the lanes along the rows the stores met in
// two banks and took sixteen passes.  Measured (with one stage, per-element guards and element-by-element
// read-modify-write -> two stages -> W read early -> stores behind the products): the step of the 60M model in
// fp32 at rank 256, 643 -> 304 -> 289 -> 271 us; of a 32000 x 2048 embedding and LM head at rank 128,
// 1060 -> 551 -> 512 -> 475 us; the refresh of the latter 3608 -> 3399 us by the last of these (each pair on one
// card; cards differ by some 3 %).  The hint on W further down takes the two steps to 269 and 460 us.
#include "gemm.h"

#include <type_traits>

namespace tsr {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;
// the same with the alignment the operands are guaranteed to have (the hardware loads any address)
typedef f32x4 __attribute__((aligned(4))) f32x4_u;
typedef u32x4 __attribute__((aligned(2))) u32x4_u;
typedef u32x2 __attribute__((aligned(2))) u32x2_u;

// Addresses that come out of a descriptor are marked as global memory: a generic (flat) access counts as
// an LDS access too, and every wait for LDS would then wait for the loads in flight.
#define TSR_GLOBAL __attribute__((address_space(1)))
typedef const TSR_GLOBAL char* gcptr;

constexpr int BK = 32;          // k-tile depth
// Place of element (row, k) in an LDS operand.  ROT: rows of 64 bytes that rotate within their group of four, and
// 16-byte chunks exchanged within the row, both by the group's number; else rows padded to 80 bytes.  Either way
// sixteen consecutive rows at one k (fragment reads) and eight rows four apart over all k (transposing stores)
// touch every bank equally.
template <bool ROT> constexpr int lds_pitch() { return ROT ? BK : BK + 8; }
// The row is first + row, `first` a multiple of 16.
template <bool ROT> __device__ inline int lds_at(int first, int row, int k) {
    if (!ROT) return (first + row) * lds_pitch<ROT>() + k;
    const int g = row >> 2;
    return first * BK + ((row & ~3) | ((row + g) & 3)) * BK + ((((k >> 3) ^ g) & 3) << 3) + (k & 7);
}
constexpr int NTHREADS = 256;

// ------------------------------------------------------------------ operand staging
// One operand's share of a k-tile, ROWS x 32 elements, in the registers of the workgroup.
//   k-contiguous, fp32: chunks of 4 k (eight lanes cover the 128 bytes of a row), rows 32 apart;
//   k-contiguous, bf16: chunks of 8 k (four lanes per row), rows 64 apart;
//   k-strided: a micro-tile of KPT k x 4 rows per thread, the lanes running along k first.
template <bool KS, bool BF16, int ROWS, bool ROT> struct Operand {
    static constexpr int KPT = KS ? ROWS / 32 : (BF16 ? 8 : 4);       // k values per chunk
    static constexpr int KL = BK / KPT;                               // lanes along k
    static constexpr int NCH = KS ? KPT : ROWS * KL / NTHREADS;       // loads per thread and k-tile
    static constexpr int ESZ = BF16 ? 2 : 4;
    static constexpr int TILE = ROWS * lds_pitch<ROT>();              // one piece of one LDS buffer
    typedef typename std::conditional<BF16, typename std::conditional<KS, u32x2, u32x4>::type, f32x4>::type Reg;

    gcptr base;            // first element of the k range; k-contiguous: of the tile's first row
    long long pitch;       // row pitch, bytes
    unsigned ldb;          // the same for the vector loads
    int klen;              // k range
    int rows, row0;        // rows of the operand, first row of the tile
    int kl, rl;            // this thread's lane along k, and along the rows
    unsigned roff[KS ? 1 : NCH];

    __device__ inline void init(const void* p, long long ld, int rows_, int row0_, int kbeg, int klen_, int tid) {
        pitch = ld * ESZ; ldb = (unsigned)pitch; klen = klen_; rows = rows_; row0 = row0_;
        kl = tid % KL; rl = tid / KL;
        if constexpr (KS) {
            base = (gcptr)p + (long long)kbeg * ld * ESZ;
            roff[0] = (unsigned)min(row0 + rl * 4, max(rows - 4, 0)) * ESZ;
        } else {
            base = (gcptr)p + ((long long)row0 * ld + kbeg) * ESZ;
#pragma unroll
            for (int it = 0; it < NCH; ++it) roff[it] = (unsigned)min(rl + it * (NTHREADS / KL), rows - 1 - row0) * ldb;
        }
    }
    // smallest extents the vector loads work on, and the largest pitch for which their 32-bit offsets hold
    // (up to 127 rows and a place within a row)
    __device__ inline bool vector_ok() const { return (KS ? rows >= 4 : klen >= KPT) && pitch <= (1 << 24); }

    __device__ inline void load(Reg (&v)[NCH], int t) const {
        if constexpr (KS) {
            const gcptr b = base + (long long)(t * BK) * ldb;
            const int last = klen - 1 - t * BK;
#pragma unroll
            for (int kk = 0; kk < NCH; ++kk) {
                const unsigned off = (unsigned)min(kl * KPT + kk, last) * ldb + roff[0];
                if constexpr (BF16) v[kk] = *(const TSR_GLOBAL u32x2_u*)(b + off);
                else v[kk] = *(const TSR_GLOBAL f32x4_u*)(b + off);
            }
        } else {
            const unsigned ko = (unsigned)min(t * BK + kl * KPT, klen - KPT) * ESZ;
#pragma unroll
            for (int it = 0; it < NCH; ++it) {
                if constexpr (BF16) v[it] = *(const TSR_GLOBAL u32x4_u*)(base + (roff[it] + ko));
                else v[it] = *(const TSR_GLOBAL f32x4_u*)(base + (roff[it] + ko));
            }
        }
    }
    // the same element by element, for extents below a vector's
    __device__ inline void load_scalar(Reg (&v)[NCH], int t) const {
        auto at = [&](int r, int k) -> float {        // bf16: the bits in the upper half
            r = min(r, rows - 1);
            const bool ok = k < klen;
            k = min(k, klen - 1);
            const gcptr p = KS ? base + k * pitch + (long long)r * ESZ
                               : base + (r - row0) * pitch + (long long)k * ESZ;
            const float x = BF16 ? __uint_as_float((unsigned)*(const TSR_GLOBAL unsigned short*)p << 16) : *(const TSR_GLOBAL float*)p;
            return ok ? x : 0.0f;
        };
#pragma unroll
        for (int it = 0; it < NCH; ++it) {
            constexpr int N = KS ? 4 : KPT;
            float e[N];
#pragma unroll
            for (int j = 0; j < N; ++j)
                e[j] = KS ? at(row0 + rl * 4 + j, t * BK + kl * KPT + it)
                          : at(row0 + rl + it * (NTHREADS / KL), t * BK + kl * KPT + j);
            if constexpr (BF16) {
#pragma unroll
                for (int j = 0; j < N / 2; ++j) v[it][j] = (__float_as_uint(e[2 * j]) >> 16) | (__float_as_uint(e[2 * j + 1]) & 0xffff0000u);
            } else {
#pragma unroll
                for (int j = 0; j < N; ++j) v[it][j] = e[j];
            }
        }
    }

    // Registers -> NS pieces in LDS.  partial: the k-tile reaches past the k range (its loads were clamped,
    // unless they were load_scalar's); edge: (k-strided) the tile reaches past the last row likewise.
    template <int NS>
    __device__ inline void store(Reg (&v)[NCH], unsigned short* lds, int t, bool partial, bool edge) const {
        if (partial) mask_k(v, t);
        if constexpr (KS) {
            const int r = (edge ? min(row0 + rl * 4, rows - 4) - row0 : rl * 4);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (edge && r + j < 0) continue;
                unsigned short* d = lds + lds_at<ROT>(0, r + j, kl * KPT);
                if constexpr (BF16) {
                    unsigned h[KPT / 2];
#pragma unroll
                    for (int q = 0; q < KPT / 2; ++q) {
                        const unsigned a = v[2 * q][j >> 1], b = v[2 * q + 1][j >> 1];
                        h[q] = (j & 1) ? (a >> 16) | (b & 0xffff0000u) : (a & 0xffffu) | (b << 16);
                    }
                    if constexpr (KPT == 4) *(u32x2*)d = u32x2{h[0], h[1]};
                    else *(unsigned*)d = h[0];
                } else {
                    float x[KPT];
#pragma unroll
                    for (int kk = 0; kk < KPT; ++kk) x[kk] = v[kk][j];
                    put<NS, KPT>(x, d);
                }
            }
        } else {
#pragma unroll
            for (int it = 0; it < NCH; ++it) {
                unsigned short* d = lds + lds_at<ROT>(it * (NTHREADS / KL), rl, kl * KPT);
                if constexpr (BF16) {
                    *(u32x4*)d = v[it];
                } else {
                    float x[KPT];
#pragma unroll
                    for (int j = 0; j < KPT; ++j) x[j] = v[it][j];
                    put<NS, KPT>(x, d);
                }
            }
        }
    }

private:
    template <int NS, int N> __device__ static inline void put(float (&x)[N], unsigned short* d) {
        typedef __attribute__((ext_vector_type(N))) __bf16 hv;
#pragma unroll
        for (int p = 0; p < NS; ++p) {
            hv h;
#pragma unroll
            for (int j = 0; j < N; ++j) {
                h[j] = (__bf16)x[j];
                if (p + 1 < NS) x[j] -= (float)h[j];
            }
            *(hv*)(d + p * TILE) = h;
        }
    }
    // what lies past the k range becomes zero; a clamped k-contiguous chunk is moved back into place
    __device__ inline void mask_k(Reg (&v)[NCH], int t) const {
        if constexpr (KS) {
#pragma unroll
            for (int kk = 0; kk < NCH; ++kk)
                if (t * BK + kl * KPT + kk >= klen)
#pragma unroll
                    for (int j = 0; j < 4; ++j) { if (j < (int)(sizeof(Reg) / 4)) v[kk][j] = 0; }
        } else {
            const int k0 = t * BK + kl * KPT;
            const int sh = k0 - min(k0, klen - KPT);          // elements the load was moved down by
#pragma unroll
            for (int it = 0; it < NCH; ++it) {
                float e[KPT], o[KPT];
#pragma unroll
                for (int j = 0; j < KPT; ++j) {
                    if constexpr (BF16) e[j] = __uint_as_float((j & 1) ? (v[it][j >> 1] & 0xffff0000u) : (v[it][j >> 1] << 16));
                    else e[j] = v[it][j];
                }
#pragma unroll
                for (int j = 0; j < KPT; ++j) {
                    o[j] = 0.0f;
#pragma unroll
                    for (int q = j; q < KPT; ++q) o[j] = (q - j == sh) ? e[q] : o[j];
                }
                if constexpr (BF16) {
#pragma unroll
                    for (int j = 0; j < KPT / 2; ++j) v[it][j] = (__float_as_uint(o[2 * j]) >> 16) | (__float_as_uint(o[2 * j + 1]) & 0xffff0000u);
                } else {
#pragma unroll
                    for (int j = 0; j < KPT; ++j) v[it][j] = o[j];
                }
            }
        }
    }
};

// ------------------------------------------------------------------ the kernel
template <bool A_KS, bool B_KS, bool A_BF16, int NSA, int NSB, int TM, int TN>
__global__ __launch_bounds__(NTHREADS, 2) void gemm_kernel(const GemmLaunch L) {
    constexpr bool KS = A_KS || B_KS;
    // Three pieces fit twice into LDS (128 x 64 tiles, two workgroups per compute unit) only without padding.  With
    // fewer the padded rows are the faster ones (fewer address instructions: step of the 60M model in fp32 271
    // against 288 us, of the embedding and LM head 475 against 537).
    constexpr bool ROT = KS && (NSA > 2 || NSB > 2);
    typedef Operand<A_KS, A_BF16, TM, ROT> OpA;
    typedef Operand<B_KS, false, TN, ROT> OpB;
    constexpr int A_ELEMS = NSA * OpA::TILE, BUF = A_ELEMS + NSB * OpB::TILE;
    constexpr int NBUF = (BUF * 4 <= 80 * 1024) ? 2 : 1;       // two workgroups per compute unit either way
    constexpr int FM = TM / 64, FN = TN / 64;
    // The weight update (both operands k-contiguous) is bound by W's traffic at a short contraction: W's tile
    // is fetched behind the first two k-tiles, so that it travels while they are multiplied.  Fetched after the
    // last k-tile -> here: step of a 32000 x 2048 embedding and LM head (rank 128) 557 -> 511 us, of the 60M
    // model in fp32 (rank 256) 310 -> 292 us.  Three pieces leave no registers for it (and nothing uses it there).
    // W passes through once, with the non-temporal hint, so that it does not push the factors out of L2: 489 -> 461
    // and 273 -> 269 us for the same two (three comparisons in turn on one card, 487-491 -> 460-462, 273.3 -> 269.5).
    // The weight update keeps the plain order: its short contraction is behind the read of W, which fills the registers.
    constexpr bool AHEAD = NBUF == 2 && KS;
    constexpr bool EARLY = !A_KS && !B_KS && NSA <= 2 && NSB <= 2;
    __shared__ __attribute__((aligned(16))) unsigned short lds[NBUF * BUF];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;

    // Workgroups go to the eight XCDs in turn: neighbouring tiles, which share operand panels, are
    // given to workgroups of one XCD (and its L2).
    int tile;
    {
        const int n = gridDim.x, x = blockIdx.x % 8, q = n / 8, rem = n % 8;
        tile = x * q + min(x, rem) + blockIdx.x / 8;
    }
    int tm, tn, ks;
    const GemmProblem* pp;
    if (L.tiles != nullptr) {
        const GemmTile t = L.tiles[tile];
        tm = t.tm; tn = t.tn; ks = t.ks;
        pp = L.probs + t.prob;
    } else {
        tn = tile % L.tiles_n;
        tm = (tile / L.tiles_n) % L.tiles_m;
        ks = tile / (L.tiles_n * L.tiles_m);
        pp = &L.single;
    }
    const long long ldc = pp->ldc;
    const int M = pp->M, N = pp->N;
    const float alpha = L.alpha, beta = L.beta;
    TSR_GLOBAL float* C = (TSR_GLOBAL float*)pp->C + (long long)ks * pp->c_split_stride;
    const int kbeg = ks * pp->kchunk;
    const int row0 = tm * TM, col0 = tn * TN;
    int klen = min(pp->K - kbeg, abs(pp->kchunk));
    // A third of the work of X R^-1 at k = 264 and 528 (below the diagonal of the factor: zeros).  Told by a sign: a
    // word of its own in the launch is one more trip of the scalar loads, 0.1 us of every launch.
    if (pp->kchunk < 0) klen = min(klen, col0 + TN);

    f32x16 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

    OpA a; OpB b;
    a.init(pp->A, pp->lda, M, row0, kbeg, klen, tid);
    b.init(pp->B, pp->ldb, N, col0, kbeg, klen, tid);
    const int nt = (klen + BK - 1) / BK;
    const bool early_done = EARLY && nt > 0 && a.vector_ok() && b.vector_ok();
    const bool edge_a = row0 + TM > M, edge_b = col0 + TN > N;

    // Where this lane's accumulators go: column (lane & 31), rows 8*(e/4) + 4*(lane>>5) + e%4 of each 32x32 tile.
    const int rbase = row0 + wm * (TM / 2) + (lane >> 5) * 4, cbase = col0 + wn * (TN / 2) + (lane & 31);
    f32x16 old[FM][FN];
    auto load_old = [&] {          // edges by clamped addresses
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const TSR_GLOBAL float* c = C + (long long)min(rbase + i * 32 + (e >> 2) * 8 + (e & 3), M - 1) * ldc;
#pragma unroll
                for (int j = 0; j < FN; ++j) old[i][j][e] = __builtin_nontemporal_load(c + min(cbase + j * 32, N - 1));
            }
    };

    typename OpA::Reg sa[2][OpA::NCH];
    typename OpB::Reg sb[2][OpB::NCH];

    auto compute = [&](const unsigned short* sA) {
        const unsigned short* sB = sA + A_ELEMS;
#pragma unroll
        for (int kk = 0; kk < BK / 16; ++kk) {
            const int kofs = kk * 16 + (lane >> 5) * 8;
            bf16x8 fa[NSA][FM], fb[NSB][FN];
#pragma unroll
            for (int p = 0; p < NSA; ++p)
#pragma unroll
                for (int i = 0; i < FM; ++i)
                    fa[p][i] = *(const bf16x8*)(sA + p * OpA::TILE + lds_at<ROT>(wm * (TM / 2) + i * 32, lane & 31, kofs));
#pragma unroll
            for (int p = 0; p < NSB; ++p)
#pragma unroll
                for (int j = 0; j < FN; ++j)
                    fb[p][j] = *(const bf16x8*)(sB + p * OpB::TILE + lds_at<ROT>(wn * (TN / 2) + j * 32, lane & 31, kofs));
            // cross products of the pieces, smallest terms first; keep those of total order
            // below max(NSA, NSB)
            constexpr int ORD = (NSA > NSB) ? NSA : NSB;
#pragma unroll
            for (int o = ORD - 1; o >= 0; --o)
#pragma unroll
                for (int pa = 0; pa < NSA; ++pa) {
                    const int pb = o - pa;
                    if (pb < 0 || pb >= NSB) continue;
#pragma unroll
                    for (int i = 0; i < FM; ++i)
#pragma unroll
                        for (int j = 0; j < FN; ++j)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[pa][i], fb[pb][j], acc[i][j], 0, 0, 0);
                }
        }
    };
    // One k-tile: register stage S (holding tile t) -> LDS, the stage refilled with tile t + 2, multiply.
    auto step = [&](auto slot, auto refill, int t) {
        constexpr int S = decltype(slot)::value;
        unsigned short* d = lds + (NBUF == 2 ? S : 0) * BUF;
        const bool partial = !decltype(refill)::value && (t + 1) * BK > klen;
        a.template store<NSA>(sa[S], d, t, partial, edge_a);
        b.template store<NSB>(sb[S], d + A_ELEMS, t, partial, edge_b);
        __syncthreads();
        if constexpr (decltype(refill)::value) { a.load(sa[S], t + 2); b.load(sb[S], t + 2); }
        compute(d);
        if constexpr (NBUF == 1) __syncthreads();
    };
    // AHEAD: tile t is multiplied from its buffer while tile t + 1 is converted and stored into the other one
    // and its register stage refilled with tile t + 3 (all: tiles up to t + 3 exist and none of them is partial).
    auto step_ahead = [&](auto slot, auto all, int t) {
        constexpr int S = decltype(slot)::value;
        __syncthreads();
        compute(lds + S * BUF);
        if (decltype(all)::value || t + 1 < nt) {
            unsigned short* d = lds + (S ^ 1) * BUF;
            const bool partial = !decltype(all)::value && (t + 2) * BK > klen;
            a.template store<NSA>(sa[S ^ 1], d, t + 1, partial, edge_a);
            b.template store<NSB>(sb[S ^ 1], d + A_ELEMS, t + 1, partial, edge_b);
        }
        if (decltype(all)::value || t + 3 < nt) { a.load(sa[S ^ 1], t + 3); b.load(sb[S ^ 1], t + 3); }
    };
    typedef std::integral_constant<int, 0> S0;
    typedef std::integral_constant<int, 1> S1;
    if (nt > 0) {
        if (a.vector_ok() && b.vector_ok()) {
            a.load(sa[0], 0); b.load(sb[0], 0);
            if (nt > 1) { a.load(sa[1], 1); b.load(sb[1], 1); }
            if constexpr (EARLY) { if (beta != 0.0f) load_old(); }
            int t = 0;
            if constexpr (AHEAD) {
                const bool partial = BK > klen;
                a.template store<NSA>(sa[0], lds, 0, partial, edge_a);
                b.template store<NSB>(sb[0], lds + A_ELEMS, 0, partial, edge_b);
                if (nt > 2) { a.load(sa[0], 2); b.load(sb[0], 2); }
                for (; t + 4 < nt; t += 2) {
                    step_ahead(S0{}, std::true_type{}, t);
                    step_ahead(S1{}, std::true_type{}, t + 1);
                }
                for (; t < nt; t += 2) {                       // the last one to four
                    step_ahead(S0{}, std::false_type{}, t);
                    if (t + 1 < nt) step_ahead(S1{}, std::false_type{}, t + 1);
                }
            } else {
                for (; t + 3 < nt; t += 2) {
                    step(S0{}, std::true_type{}, t);
                    step(S1{}, std::true_type{}, t + 1);
                }
                if (nt - t == 3) {
                    step(S0{}, std::true_type{}, t);
                    step(S1{}, std::false_type{}, t + 1);
                    step(S0{}, std::false_type{}, t + 2);
                } else {
                    step(S0{}, std::false_type{}, t);
                    if (nt - t == 2) step(S1{}, std::false_type{}, t + 1);
                }
            }
        } else {
            for (int t = 0; t < nt; ++t) {
                a.load_scalar(sa[0], t); b.load_scalar(sb[0], t);
                a.template store<NSA>(sa[0], lds, t, false, false);
                b.template store<NSB>(sb[0], lds + A_ELEMS, t, false, false);
                __syncthreads();
                compute(lds);
                __syncthreads();
            }
        }
    }

    // epilogue; with beta the whole tile is read before the first element is written (one trip to memory)
    auto write = [&](auto&& value) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int row = rbase + i * 32 + (e >> 2) * 8 + (e & 3), col = cbase + j * 32;
                    if (row < M && col < N) {
                        TSR_GLOBAL float* c = C + (long long)row * ldc + col;
                        if constexpr (EARLY) __builtin_nontemporal_store(value(i, j, e), c);
                        else *c = value(i, j, e);
                    }
                }
    };
    if (beta != 0.0f) {
        if (!EARLY || !early_done) load_old();
        write([&](int i, int j, int e) { return alpha * acc[i][j][e] + beta * old[i][j][e]; });
    } else {
        write([&](int i, int j, int e) { return alpha * acc[i][j][e]; });
    }
}

// ------------------------------------------------------------------ dispatch
typedef void (*gemm_fn)(const GemmLaunch);
struct Entry { GemmVariant v; gemm_fn fn[GEMM_SHAPES]; };

#define TSR_GEMM(aks, bks, abf, nsa, nsb) \
    { {aks, bks, abf, nsa, nsb}, {gemm_kernel<(aks) != 0, (bks) != 0, (abf) != 0, nsa, nsb, 128, 128>, \
                                  gemm_kernel<(aks) != 0, (bks) != 0, (abf) != 0, nsa, nsb, 128, 64>, \
                                  gemm_kernel<(aks) != 0, (bks) != 0, (abf) != 0, nsa, nsb, 64, 64>} }

static const Entry kTable[] = {
    // A = G (k contiguous), B k-strided: G V, G Omega, G Qrow; also U D, Y Rinv, Q X
    TSR_GEMM(0, 1, 1, 1, 1), TSR_GEMM(0, 1, 1, 1, 2),
    TSR_GEMM(0, 1, 0, 1, 1), TSR_GEMM(0, 1, 0, 2, 2), TSR_GEMM(0, 1, 0, 3, 3),
    // A k-strided, B k-strided: U^T P, Y^T Y, G^T Q
    TSR_GEMM(1, 1, 0, 1, 1), TSR_GEMM(1, 1, 0, 2, 2), TSR_GEMM(1, 1, 0, 3, 3),
    TSR_GEMM(1, 1, 1, 1, 1), TSR_GEMM(1, 1, 1, 1, 2),
    // A k-contiguous, B k-contiguous: T V^T
    TSR_GEMM(0, 0, 0, 1, 1), TSR_GEMM(0, 0, 0, 2, 2), TSR_GEMM(0, 0, 0, 3, 3),
};

hipError_t launch_gemm(const GemmLaunch& L, const GemmVariant& v, hipStream_t stream) {
    if (L.n_tiles <= 0) return hipSuccess;
    if (v.shape < 0 || v.shape >= GEMM_SHAPES) return hipErrorInvalidValue;
    for (const Entry& e : kTable) {
        if (e.v.a_kstrided == v.a_kstrided && e.v.b_kstrided == v.b_kstrided && e.v.a_bf16 == v.a_bf16 &&
            e.v.a_pieces == v.a_pieces && e.v.b_pieces == v.b_pieces) {
            hipLaunchKernelGGL(e.fn[v.shape], dim3(L.n_tiles), dim3(NTHREADS), 0, stream, L);
            return hipGetLastError();
        }
    }
    return hipErrorInvalidValue;
}

// ------------------------------------------------------------------ the step of one small matrix
// A single call on a small matrix is bound by its launches, on the host (3-4 us each) as on the device (3-6 us each,
// of which the trips to memory are the most).  So the two products of the projection are one launch here (and the
// sum of its partial cores a second), and the two products of the lift one: seven launches of a step become four,
// 38.1 -> 28.4 us for 512 x 1376 fp32 at r = 64, 38.5 -> 29.8 us for 1001 x 1365 bf16 at r = 96.  What is left is the
// host's (four launches and the caller's program around them; the kernels take 18 and 29 us).
// Both keep the arithmetic of the general kernel: the intermediate in fp32, cut into pieces for the second product.
// Used for r <= 128, where the intermediate of 64 rows fits the registers and LDS of a workgroup, and matrices whose
// launches would have 64 x 64 tiles anyway (pick_shape).

// acc += A B over one k-tile in LDS
template <int NSA, int NSB, int FM, int FN, typename OpA, typename OpB>
__device__ inline void multiply_tiles(f32x16 (&acc)[FM][FN], const unsigned short* sA, const unsigned short* sB, int a_row0,
                                      int b_row0, int a_pitch, int a_piece, int lane) {
#pragma unroll
    for (int kk = 0; kk < BK / 16; ++kk) {
        const int kofs = kk * 16 + (lane >> 5) * 8;
        bf16x8 fa[NSA][FM], fb[NSB][FN];
#pragma unroll
        for (int p = 0; p < NSA; ++p)
#pragma unroll
            for (int i = 0; i < FM; ++i)
                fa[p][i] = *(const bf16x8*)(sA + p * a_piece + (a_row0 + i * 32 + (lane & 31)) * a_pitch + kofs);
#pragma unroll
        for (int p = 0; p < NSB; ++p)
#pragma unroll
            for (int j = 0; j < FN; ++j)
                fb[p][j] = *(const bf16x8*)(sB + p * OpB::TILE + lds_at<false>(b_row0 + j * 32, lane & 31, kofs));
        constexpr int ORD = (NSA > NSB) ? NSA : NSB;           // smallest terms first
#pragma unroll
        for (int o = ORD - 1; o >= 0; --o)
#pragma unroll
            for (int pa = 0; pa < NSA; ++pa) {
                const int pb = o - pa;
                if (pb < 0 || pb >= NSB) continue;
#pragma unroll
                for (int i = 0; i < FM; ++i)
#pragma unroll
                    for (int j = 0; j < FN; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[pa][i], fb[pb][j], acc[i][j], 0, 0, 0);
            }
    }
}

// acc += A B over the operands' k range: two register stages, two LDS buffers (of NSA pieces of A and NSB of B), a
// barrier per k-tile.
template <int NSA, int NSB, int FM, int FN, typename OpA, typename OpB>
__device__ inline void product(f32x16 (&acc)[FM][FN], OpA& a, OpB& b, int klen, bool edge_a, bool edge_b, unsigned short* lds,
                               int wm, int wn, int lane) {
    constexpr int A_ELEMS = NSA * OpA::TILE, BUF = A_ELEMS + NSB * OpB::TILE;
    const int nt = (klen + BK - 1) / BK;
    typename OpA::Reg sa[2][OpA::NCH];
    typename OpB::Reg sb[2][OpB::NCH];
    const bool vectors = a.vector_ok() && b.vector_ok();
    auto fetch = [&](auto slot, int t) {
        constexpr int S = decltype(slot)::value;
        if (vectors) { a.load(sa[S], t); b.load(sb[S], t); }
        else { a.load_scalar(sa[S], t); b.load_scalar(sb[S], t); }
    };
    auto step = [&](auto slot, int t) {
        constexpr int S = decltype(slot)::value;
        unsigned short* d = lds + S * BUF;
        const bool partial = vectors && (t + 1) * BK > klen;
        a.template store<NSA>(sa[S], d, t, partial, edge_a && vectors);
        b.template store<NSB>(sb[S], d + A_ELEMS, t, partial, edge_b && vectors);
        __syncthreads();
        if (t + 2 < nt) fetch(slot, t + 2);
        multiply_tiles<NSA, NSB, FM, FN, OpA, OpB>(acc, d, d + A_ELEMS, wm * FM * 32, wn * FN * 32, lds_pitch<false>(), OpA::TILE, lane);
    };
    typedef std::integral_constant<int, 0> S0;
    typedef std::integral_constant<int, 1> S1;
    if (nt > 0) fetch(S0{}, 0);
    if (nt > 1) fetch(S1{}, 1);
    for (int t = 0; t < nt; t += 2) {
        step(S0{}, t);
        if (t + 1 < nt) step(S1{}, t + 1);
    }
}

template <int FM, int FN> __device__ inline void clear(f32x16 (&acc)[FM][FN]) {
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;
}

// x -> NS bf16 pieces at d, d + piece, ...
template <int NS> __device__ inline void put4(float (&x)[4], unsigned short* d, int piece) {
#pragma unroll
    for (int p = 0; p < NS; ++p) {
        bf16x4 h;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            h[j] = (__bf16)x[j];
            if (p + 1 < NS) x[j] -= (float)h[j];
        }
        *(bf16x4*)(d + p * piece) = h;
    }
}

// One partial core per workgroup: U_s^T (G_sc V_c) for 64 rows s and a range c of columns.  What G_sc V_c loses on its
// way into the second product stays where the ranges cancel each other (the general kernel cuts the finished sum into
// pieces), so it goes there in three pieces, as good as fp32, whatever the precision.  In as many as the other operands
// it cost up to 1 us less (1001 x 1365 bf16 r = 96 16.9 / 17.9), and an error of 0.6 where two halves of the columns cancel
// to 2^-8 (bf16 operands; now as with the general kernel).
template <bool G_BF16, int NSA, int NSB, int RP>
__global__ __launch_bounds__(NTHREADS, RP * NSB > 128 ? 1 : 2) void project_one_kernel(const ProjectOne q) {     // (LDS)
    constexpr int TM = 64, FN = RP / 64;
    typedef Operand<false, G_BF16, TM, false> OpG;
    typedef Operand<true, false, RP, false> OpV;
    constexpr int NSP = 3, FIRST = 2 * (NSA * OpG::TILE + NSB * OpV::TILE), HALF = (NSB + NSP) * OpV::TILE;
    __shared__ __attribute__((aligned(16))) unsigned short lds[FIRST > 2 * HALF ? FIRST : 2 * HALF];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wm = wave >> 1, wn = wave & 1;
    const int slab = blockIdx.x / q.chunks, chunk = blockIdx.x % q.chunks;
    const int row0 = slab * TM, rows = min(q.m - row0, TM);
    const int kbeg = chunk * q.kchunk, klen = min(q.n - kbeg, q.kchunk);
    const bool edge_r = q.r < RP;

    // the rows of U, behind the first product
    OpV u;
    u.init(q.U, q.r, q.r, 0, row0, rows, tid);
    typename OpV::Reg su[2][OpV::NCH];
    const bool vectors = u.vector_ok();
    auto fetch_u = [&](auto half) {
        constexpr int H = decltype(half)::value;
        if (vectors) u.load(su[H], H);
        else u.load_scalar(su[H], H);
    };
    fetch_u(std::integral_constant<int, 0>{});
    if (rows > BK) fetch_u(std::integral_constant<int, 1>{});

    f32x16 P[1][FN];
    clear(P);
    {
        OpG a; OpV b;
        a.init(q.G, q.ldg, q.m, row0, kbeg, klen, tid);
        b.init(q.V, q.r, q.r, 0, kbeg, klen, tid);
        product<NSA, NSB, 1, FN>(P, a, b, klen, row0 + TM > q.m, edge_r, lds, wm, wn, lane);
    }
    __syncthreads();
    // U_s and P, both with the slab's rows as the contraction: [32 rows][operand][piece][column][row]
    u.template store<NSB>(su[0], lds, 0, vectors && rows < BK, edge_r && vectors);
    if (rows > BK) u.template store<NSB>(su[1], lds + HALF, 1, vectors && rows < 2 * BK, edge_r && vectors);
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int e = 0; e < 16; e += 4) {
            float x[4] = {P[0][j][e], P[0][j][e + 1], P[0][j][e + 2], P[0][j][e + 3]};
            put4<NSP>(x, lds + wm * HALF + NSB * OpV::TILE + lds_at<false>((wn * FN + j) * 32, lane & 31, (e >> 2) * 8 + (lane >> 5) * 4),
                      OpV::TILE);
        }
    __syncthreads();
    f32x16 C[FN][FN];
    clear(C);
    for (int h = 0; h * BK < rows; ++h)
        multiply_tiles<NSB, NSP, FN, FN, OpV, OpV>(C, lds + h * HALF, lds + h * HALF + NSB * OpV::TILE, wm * FN * 32, wn * FN * 32,
                                                   lds_pitch<false>(), OpV::TILE, lane);
    TSR_GLOBAL float* out = (TSR_GLOBAL float*)q.part + (long long)blockIdx.x * q.r * q.r;
#pragma unroll
    for (int i = 0; i < FN; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int row = (wm * FN + i) * 32 + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3), col = (wn * FN + j) * 32 + (lane & 31);
                if (row < q.r && col < q.r) out[row * q.r + col] = C[i][j][e];
            }
}

// 64 rows of T = U D, kept as pieces in LDS, then W = beta W + alpha T V^T for a few 64 x 64 tiles of these rows.
template <int NS, int RP>
__global__ __launch_bounds__(NTHREADS, 2) void lift_one_kernel(const LiftOne q) {
    constexpr int TM = 64, FN = RP / 64, KT = RP / BK, TP = RP + 8;
    typedef Operand<false, false, TM, false> OpU;              // also the rows of V
    typedef Operand<true, false, RP, false> OpD;
    constexpr int T_ELEMS = NS * TM * TP, FIRST = 2 * NS * (OpU::TILE + OpD::TILE), SECOND = T_ELEMS + KT * NS * OpU::TILE;
    __shared__ __attribute__((aligned(16))) unsigned short lds[FIRST > SECOND ? FIRST : SECOND];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wm = wave >> 1, wn = wave & 1;
    const int slab = blockIdx.x / q.groups, group = blockIdx.x % q.groups;
    const int row0 = slab * TM, tiles = (q.n + 63) / 64, kt_used = (q.r + BK - 1) / BK;
    const int tile_end = min(tiles, (group + 1) * q.per_group);

    OpU v;
    typename OpU::Reg sv[KT][OpU::NCH];
    f32x16 old;
    const int rbase = row0 + wm * 32 + (lane >> 5) * 4, cbase = wn * 32 + (lane & 31);
    bool vectors = false;
    auto fetch = [&](int tile) {                               // rows of V and the tile of W, edges by clamped addresses
        v.init(q.V, q.r, q.n, tile * 64, 0, q.r, tid);
        vectors = v.vector_ok();
#pragma unroll
        for (int t = 0; t < KT; ++t) {
            if (t >= kt_used) continue;
            if (vectors) v.load(sv[t], t);
            else v.load_scalar(sv[t], t);
        }
        if (q.beta != 0.0f)
#pragma unroll
            for (int e = 0; e < 16; ++e)
                old[e] = __builtin_nontemporal_load((const TSR_GLOBAL float*)q.W + (long long)min(rbase + (e >> 2) * 8 + (e & 3), q.m - 1) * q.ldw +
                                                    min(tile * 64 + cbase, q.n - 1));
    };
    fetch(group * q.per_group);
    {
        f32x16 T[1][FN];
        clear(T);
        OpU a; OpD b;
        a.init(q.U, q.r, q.m, row0, 0, q.r, tid);
        b.init(q.D, q.r, q.r, 0, 0, q.r, tid);
        product<NS, NS, 1, FN>(T, a, b, q.r, row0 + TM > q.m, q.r < RP, lds, wm, wn, lane);
        __syncthreads();
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int row = wm * 32 + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3), col = (wn * FN + j) * 32 + (lane & 31);
                float x = (col < q.r) ? T[0][j][e] : 0.0f;
#pragma unroll
                for (int p = 0; p < NS; ++p) {
                    const __bf16 h = (__bf16)x;
                    lds[p * TM * TP + row * TP + col] = __builtin_bit_cast(unsigned short, h);
                    x -= (float)h;
                }
            }
    }
    unsigned short* sV = lds + T_ELEMS;
    for (int tile = group * q.per_group; tile < tile_end; ++tile) {
#pragma unroll
        for (int t = 0; t < KT; ++t)
            if (t < kt_used) v.template store<NS>(sv[t], sV + t * NS * OpU::TILE, t, vectors && (t + 1) * BK > q.r, false);
        const f32x16 w = old;
        __syncthreads();
        if (tile + 1 < tile_end) fetch(tile + 1);
        f32x16 acc[1][1];
        clear(acc);
        for (int t = 0; t < kt_used; ++t)
            multiply_tiles<NS, NS, 1, 1, OpU, OpU>(acc, lds + t * BK, sV + t * NS * OpU::TILE, wm * 32, wn * 32, TP, TM * TP, lane);
        const int col = tile * 64 + cbase;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int row = rbase + (e >> 2) * 8 + (e & 3);
            float x = q.alpha * acc[0][0][e];
            if (q.beta != 0.0f) x += q.beta * w[e];
            if (row < q.m && col < q.n) __builtin_nontemporal_store(x, (TSR_GLOBAL float*)q.W + (long long)row * q.ldw + col);
        }
        __syncthreads();
    }
}

hipError_t launch_project_one(const ProjectOne& q, int g_bf16, int split, int blocks, hipStream_t stream) {
    typedef void (*fn)(const ProjectOne);
    static const fn table[2][2][2] = {
        {{project_one_kernel<false, 1, 1, 64>, project_one_kernel<false, 1, 1, 128>},
         {project_one_kernel<false, 2, 2, 64>, project_one_kernel<false, 2, 2, 128>}},
        {{project_one_kernel<true, 1, 1, 64>, project_one_kernel<true, 1, 1, 128>},
         {project_one_kernel<true, 1, 2, 64>, project_one_kernel<true, 1, 2, 128>}}};
    hipLaunchKernelGGL(table[g_bf16 != 0][split != 0][q.r > 64], dim3(blocks), dim3(NTHREADS), 0, stream, q);
    return hipGetLastError();
}

hipError_t launch_lift_one(const LiftOne& q, int split, int blocks, hipStream_t stream) {
    typedef void (*fn)(const LiftOne);
    static const fn table[2][2] = {{lift_one_kernel<1, 64>, lift_one_kernel<1, 128>}, {lift_one_kernel<2, 64>, lift_one_kernel<2, 128>}};
    hipLaunchKernelGGL(table[split != 0][q.r > 64], dim3(blocks), dim3(NTHREADS), 0, stream, q);
    return hipGetLastError();
}

// ------------------------------------------------------------------ split-k reduction
// Four neighbouring elements per thread, the partials of all splits fetched eight at a time.
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const ReduceProblem* probs, const ReduceProblem single,
                                                            const float alpha, const float beta) {
    const ReduceProblem p = probs ? probs[blockIdx.y] : single;
    const TSR_GLOBAL float* part = (const TSR_GLOBAL float*)p.part;
    TSR_GLOBAL float* out = (TSR_GLOBAL float*)p.out;
    const long long total = (long long)p.M * p.N;
    const bool dense = p.ldc == p.N;
    const long long nv = total / 4;                           // whole vectors; the last elements one by one
    auto finish = [&](long long i, float s) {
        const long long o = dense ? i : (long long)((unsigned long long)i / (unsigned)p.N) * p.ldc + (long long)((unsigned long long)i % (unsigned)p.N);
        float v = alpha * s;
        if (beta != 0.0f) v += beta * out[o];
        out[o] = v;
    };
    const long long step = (long long)gridDim.x * blockDim.x;
    const long long me = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    for (long long q = me; q < nv; q += step) {
        // (the stride between partials is M x N: 16-byte loads at any element)
        const TSR_GLOBAL float* src = part + 4 * q;
        f32x4 s = {0.0f, 0.0f, 0.0f, 0.0f};
        int k = 0;
        for (; k + 8 <= p.splits; k += 8) {
            f32x4 x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) x[u] = *(const TSR_GLOBAL f32x4_u*)(src + (k + u) * p.stride);
#pragma unroll
            for (int u = 0; u < 8; ++u) s += x[u];
        }
        for (; k < p.splits; ++k) s += *(const TSR_GLOBAL f32x4_u*)(src + k * p.stride);
        if (dense) {
            f32x4 v = alpha * s;
            TSR_GLOBAL f32x4_u* o = (TSR_GLOBAL f32x4_u*)(out + 4 * q);
            if (beta != 0.0f) v += beta * (f32x4)*o;
            *o = v;
        } else {
#pragma unroll
            for (int u = 0; u < 4; ++u) finish(4 * q + u, s[u]);
        }
    }
    for (long long i = 4 * nv + me; i < total; i += step) {
        float s = 0.0f;
        for (int k = 0; k < p.splits; ++k) s += part[(long long)k * p.stride + i];
        finish(i, s);
    }
}

// The same for few outputs and many partials: sixteen vectors of outputs per workgroup, sixteen threads share the
// partials of each (neighbouring threads neighbouring vectors), their sums added in order.
__global__ __launch_bounds__(256) void splitk_reduce_wide_kernel(const ReduceProblem* probs, const ReduceProblem single,
                                                                 const float alpha, const float beta) {
    constexpr int G = 16;
    __shared__ f32x4 sums[G][G];
    const ReduceProblem p = probs ? probs[blockIdx.y] : single;
    const TSR_GLOBAL float* part = (const TSR_GLOBAL float*)p.part;
    TSR_GLOBAL float* out = (TSR_GLOBAL float*)p.out;
    const int x = threadIdx.x % G, g = threadIdx.x / G, total = p.M * p.N;
    const int i = 4 * (blockIdx.x * G + x);
    const int per = (p.splits + G - 1) / G, k0 = g * per, k1 = min(p.splits, k0 + per);
    const bool whole = i + 4 <= total;
    f32x4 s = {0.0f, 0.0f, 0.0f, 0.0f};
    auto at = [&](int k) {
        const TSR_GLOBAL float* q = part + k * p.stride + i;
        if (whole) return (f32x4)*(const TSR_GLOBAL f32x4_u*)q;
        f32x4 v = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int u = 0; u < 4; ++u) if (i + u < total) v[u] = q[u];
        return v;
    };
    int k = k0;
    for (; k + 8 <= k1; k += 8) {
        f32x4 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = at(k + u);
#pragma unroll
        for (int u = 0; u < 8; ++u) s += v[u];
    }
    for (; k < k1; ++k) s += at(k);
    sums[g][x] = s;
    __syncthreads();
    if (g != 0) return;
#pragma unroll
    for (int u = 1; u < G; ++u) s += sums[u][x];
    s = alpha * s;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        if (i + u >= total) continue;
        const long long o = (p.ldc == p.N) ? i + u : (long long)((i + u) / p.N) * p.ldc + (i + u) % p.N;
        out[o] = s[u] + (beta != 0.0f ? beta * out[o] : 0.0f);
    }
}

hipError_t launch_splitk_reduce(const ReduceProblem* probs_dev, const ReduceProblem* single, int count,
                                int max_elems, int max_splits, float alpha, float beta, hipStream_t stream) {
    if (count <= 0 || max_elems <= 0) return hipSuccess;
    int bx = (max_elems + 1023) / 1024;
    if (bx > 1024) bx = 1024;
    ReduceProblem s{};
    if (single) s = *single;
    // Threads that share the partials where there are many of them and too few outputs to fill the chip.  Device time behind
    // a kernel that writes the partials, us, one thread to all partials / shared: 5184 outputs of 8 partials 1.9 / 2.3, of 16
    // 2.3 / 2.3, of 28 3.8 / 2.7, of 128 8.3 / 3.4; 65536 of 16 3.5 / 4.0, of 28 5.8 / 5.4, of 128 8.5 / 7.9; 131072 of 16
    // 5.5 / 6.1, of 128 10.8 / 12.4 (the lines come in longer pieces where one thread has all partials).  Cores of the
    // 32000 x 2048 embedding and LM head, 256 partials, 15 -> 8.
    if (max_splits > 16 && (long long)bx * count <= 64) {
        hipLaunchKernelGGL(splitk_reduce_wide_kernel, dim3((max_elems + 63) / 64, count), dim3(256), 0, stream, probs_dev, s, alpha, beta);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(splitk_reduce_kernel, dim3(bx, count), dim3(256), 0, stream, probs_dev, s, alpha, beta);
    return hipGetLastError();
}

}  // namespace tsr
