// Batched block-Jacobi SVD kernels (FP64) for the truncation step.
//
// Each matrix is stored as nv row vectors of length len (W, row-major); Z (nv x
// nv, starts at I) accumulates the rotations.  An outer sweep forms the Gram
// matrix G = W W^T afresh (grouped GEMM), runs one cyclic two-sided
// block-Jacobi sweep on G, accumulating its rotations in Qt, and applies them,
// W <- Qt W and Z <- Qt Z (one grouped GEMM launch).  When a fresh G has |G_ij|
// <= tol sqrt(G_ii G_jj) everywhere the rows are orthogonal and their norms
// are the singular values.  Convergence is only ever judged on a fresh G, and
// Qt is a product of rotations orthogonal to working precision, so nothing of
// a sweep's updated G goes into the result.  (W = Z W0 in place of W <- Qt W
// saves a product but loses the small rows of a badly ordered graded block.)
//
// A sweep has np / 32 - 1 rounds (circle schedule over blocks of 32 rows, np =
// nv padded to a multiple of 64) and one launch more (jac_round_kernel): per
// pair of blocks one cyclic Jacobi sweep of the 64 x 64 sub-matrix of G in one
// workgroup, and beside it the previous round's G <- J^T G J and Qt <- J^T Qt
// on the FP64 matrix cores.  What bounds it is the chain of inner rotation
// rounds: a sweep takes about 2 nv of them whatever the block size, so the
// time goes down with the cost of one inner round and with the launches and
// loads around them.  Blocks of 32 rows have a quarter of the launches of
// blocks of 8 and need fewer sweeps.
// Matrices of at most 64 rows run whole in one workgroup (jac_small_kernel),
// except very long rows.
//
// Also here: the Householder QR that preconditions the iteration (panel and
// reflector-application kernels, below) and the copy / norm helpers.
#include "svd.hpp"

#include <algorithm>
#include <stdexcept>

namespace pdmrg {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef unsigned u2 __attribute__((ext_vector_type(2)));
typedef double d2 __attribute__((ext_vector_type(2)));

constexpr int J2 = 16;           // target rows of a reflector application
constexpr int JT = 256;          // its threads (4 waves)
constexpr int CH = 512;          // its columns staged in LDS at a time
constexpr int U = J2 * CH / JT;  // staged elements per thread and chunk
static_assert(J2 * CH % JT == 0 && CH % 16 == 0, "chunk must split evenly over the threads and 16-column steps");
constexpr unsigned kOut = 0x80000000u;   // buffer offset past every record

__device__ __forceinline__ d4 mfma_f64(double a, double b, d4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Raw buffer descriptor over the n doubles at p (p is the same in every lane).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rows_rsrc(const double *p, int64_t n) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    void *q = reinterpret_cast<void *>(((uint64_t)hi << 32) | lo);
    return __builtin_amdgcn_make_buffer_rsrc(q, 0, (int)(n * 8), 0x00020000);
}
__device__ __forceinline__ double bload(__amdgpu_buffer_rsrc_t r, unsigned off) {
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
}
__device__ __forceinline__ void bstore(__amdgpu_buffer_rsrc_t r, unsigned off, double v) {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, v), r, off, 0, 0);
}

// Rotation that zeroes a_pq of the symmetric 2 x 2 block (app, apq, aqq):
// column p becomes c col_p - s col_q, column q becomes s col_p + c col_q.  With
// d = a_qq - a_pp, h = sqrt(d^2 + 4 a_pq^2), y = 1 / h: the smaller angle has
// c^2 = (1 + |d| y) / 2, s = sign(d) a_pq y / c, t = s / c, so the chain holds
// two reciprocal square roots and no division.  d and 2 a_pq are first scaled
// by a power of two so the larger magnitude lies in [1/2, 1); then u = h^2
// lies in [1/4, 2] and c^2 in [1/2, 1], and hardware estimates with one
// third-order step each give full precision without range handling.  Skipped
// (c = 1, s = 0) when a_pq^2 <= 1e-32 |a_pp a_qq| (the relative rule that
// resolves the small eigenvalues of a graded Gram matrix).
__device__ __forceinline__ double rsqrt_full(double v) {
    const double y = __builtin_amdgcn_rsq(v);
    const double e = fma(-v * y, y, 1.0);              // y sqrt(v) = (1 - e)^(1/2)
    return fma(y * e, fma(e, 0.375, 0.5), y);
}
__device__ __forceinline__ void jacobi_angle(double app, double apq, double aqq, double &c, double &s, double &t,
                                             bool &skip) {
    const double d0 = aqq - app, b0 = 2.0 * apq;
    const int e = -__builtin_amdgcn_frexp_exp(fmax(fabs(d0), fabs(b0)));
    const double d = __builtin_amdgcn_ldexp(d0, e), b = __builtin_amdgcn_ldexp(b0, e);
    const double y = rsqrt_full(fma(d, d, b * b));
    const double c2 = fma(0.5 * fabs(d), y, 0.5);
    const double z = rsqrt_full(c2);
    const double h = copysign(0.5, d) * b * y;         // s c
    skip = apq == 0.0 || apq * apq <= 1e-32 * fabs(app * aqq);
    c = skip ? 1.0 : c2 * z;
    s = skip ? 0.0 : h * z;
    t = skip ? 0.0 : h * (z * z);
}

// ---------------------------------------------------------------------------
// One cyclic Jacobi sweep of a symmetric matrix of 2 P rows (P = 32, 16, 8) in
// one workgroup of 1 + NA + NQ waves.  Indices sit on 2 P positions, pair i =
// (t_i, b_i) = positions 2 i and 2 i + 1, and move after every round (t_0
// stays, b_0 -> t_1, t_i -> t_i+1, the last t -> the last b, b_i -> b_i-1), so
// 2 P - 1 rounds meet every pair once and end where they began.  Position t_i
// starts with row i, b_i with row P + i.
//   D wave (lanes 0 .. P - 1): the diagonal blocks.  Lane i computes pair i's
//     angle.  It takes the next round's a_pq from the block that holds it
//     before its rotation (the entry is rotated here as well), so that angles
//     and block rotations run side by side, one barrier a round;
//   A waves: a thread takes some of the P (P - 1) / 2 blocks (2 x 2) of pairs i
//     < j, rotates them from both sides and hands their entries to the blocks
//     they move to (fixed LDS addresses);
//   Q waves: lane = row of Q, P / NQ pairs of columns in registers; only the
//     columns that cross to another wave go through LDS.
// In round k the D wave computes rotation k while A and Q apply rotation k - 1.
// The round's length is the D wave's chain (LDS read, about 25 dependent FP64
// operations, LDS write, barrier) or, for P = 32, the LDS traffic of the A and
// the lane broadcasts of the Q waves: 0.45 us a round with 4 A and 8 Q waves,
// 0.30 us with the D wave alone; 0.48 with 3 and 8, 0.46 with 8 and 4.
template <int P>
struct EigCfg;
template <> struct EigCfg<32> { static constexpr int NA = 4, NQ = 8, INV2 = 16; };
template <> struct EigCfg<16> { static constexpr int NA = 2, NQ = 2, INV2 = 8; };
template <> struct EigCfg<8> { static constexpr int NA = 1, NQ = 1, INV2 = 4; };
constexpr int eig_threads(int p) { return p == 32 ? 64 * 13 : p == 16 ? 64 * 5 : 64 * 3; }
// Blocks (i, j) lie in P - 1 rows of P / 2 (the circle schedule on P pairs); the
// row stride is odd because the D wave reads blocks (i - 1, i + 1), one a row.
template <int P>
struct EigLds {
    static constexpr int kRow = P / 2 + 1, kTrash = (P - 1) * kRow, kEnt = kTrash + P / 2 + 1;
    double ex[2][4][kEnt];       // entries (2 x + y) of the off-diagonal blocks
    d2 cs[2][P];                 // rotations (c, s) of the pairs
    double dg[2][2 * P];         // diagonal by position
    double qx[2][EigCfg<P>::NQ][2][64];   // columns of Q leaving a wave: its last t, its first b
    int rank[64];                // rank of a row's eigenvalue, descending
    int any;
};

// LDS place of block (i, j), i < j, of the circle schedule on P pairs.
template <int P>
__device__ __forceinline__ int eig_block(int i, int j) {
    constexpr int M = P - 1;
    if (j == M) return EigLds<P>::kRow * i;
    const int r = (i + j) * EigCfg<P>::INV2 % M;
    const int d = (i - r + M) % M;
    return EigLds<P>::kRow * r + (d < P / 2 ? d : M - d);
}
template <int P>
__device__ __forceinline__ int eig_dest(int p) {
    if (p & 1) return p == 1 ? 2 : p - 2;
    return p == 0 ? 0 : p == 2 * P - 2 ? 2 * P - 1 : p + 2;
}
// LDS index [entry][block] of the entry at positions (p, q) of different pairs.
template <int P>
__device__ __forceinline__ int eig_slot(int p, int q) {
    const int lo = min(p >> 1, q >> 1), hi = max(p >> 1, q >> 1);
    const int x = (p >> 1) < (q >> 1) ? p & 1 : q & 1, y = (p >> 1) < (q >> 1) ? q & 1 : p & 1;
    return (2 * x + y) * EigLds<P>::kEnt + eig_block<P>(lo, hi);
}

// v of lane l, in scalar registers.
__device__ __forceinline__ double lane_value(double v, int l) {
    const u2 b = __builtin_bit_cast(u2, v);
    return __builtin_bit_cast(double, u2{(unsigned)__builtin_amdgcn_readlane((int)b.x, l),
                                         (unsigned)__builtin_amdgcn_readlane((int)b.y, l)});
}

// at(r, c): entry (r, c) of the symmetric matrix, r and c in 0 .. 2 P - 1.  Rows
// at and past n are absent (zero).  Returns true (uniformly) if a rotation was
// needed; then put(o, k, v) receives row o, column k of the rotation (new row
// o = sum_k v old row k; rows sorted by decreasing diagonal, absent ones in
// place) and put_g(r, c, v) every entry (r, c) of the rotated matrix.  Called
// by all eig_threads(P) threads of the workgroup.
template <int P, class At, class Put, class PutG>
__device__ __forceinline__ bool eig_sweep(EigLds<P> &L, int n, double tol, At at, Put put, PutG put_g) {
    using Lds = EigLds<P>;
    constexpr int NA = EigCfg<P>::NA, NQ = EigCfg<P>::NQ, NW = 1 + NA + NQ, R = 2 * P - 1;   // R rounds
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool isD = wave == 0, isA = !isD && wave <= NA;
    // A: the blocks of this thread
    constexpr int kBlk = (P * (P - 1) / 2 + 64 * NA - 1) / (64 * NA);
    int bi[kBlk], bj[kBlk], blk[kBlk], dst[kBlk][4];
    double a0[kBlk][4];
    if (isA) {
#pragma unroll
        for (int u = 0; u < kBlk; ++u) {
            const int b = tid - 64 + 64 * NA * u, r = b / (P / 2), l = b % (P / 2);
            const bool on = r < P - 1;
            const int p = l == 0 ? P - 1 : (r + l) % (P - 1), q = (r - l + P - 1) % (P - 1);
            bi[u] = on ? min(p, q) : 0;
            bj[u] = on ? max(p, q) : 1;
            blk[u] = on ? Lds::kRow * r + l : Lds::kTrash + l;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int dp = eig_dest<P>(2 * bi[u] + (e >> 1)), dq = eig_dest<P>(2 * bj[u] + (e & 1));
                // an entry that joins a diagonal block goes to an unused slot
                dst[u][e] = !on || (dp >> 1) == (dq >> 1) ? Lds::kTrash + l : eig_slot<P>(dp, dq);
                a0[u][e] = on ? at(bi[u] + P * (e >> 1), bj[u] + P * (e & 1)) : 0.0;
                L.ex[0][e][blk[u]] = a0[u][e];
            }
        }
    }
    // D: pair i of this lane (the lanes past P repeat it)
    const int di = lane % P;
    double app = 0, aqq = 0, apq = 0;
    if (isD) {
        app = at(di, di);
        aqq = at(P + di, P + di);
        apq = at(di, P + di);
        if (lane < P) {
            L.dg[0][2 * di] = app;
            L.dg[0][2 * di + 1] = aqq;
        }
        L.rank[lane] = lane < n ? 0 : lane;
        if (lane == 0) L.any = 0;
    }
    __syncthreads();
    // whether any relative off-diagonal exceeds tol
    bool big = false;
    auto rel = [&](double a, int p, int q) {
        const double dd = L.dg[0][p] * L.dg[0][q];
        big = big || (dd > 0.0 && a * a > tol * tol * dd);
    };
    if (isA)
#pragma unroll
        for (int u = 0; u < kBlk; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) rel(a0[u][e], 2 * bi[u] + (e >> 1), 2 * bj[u] + (e & 1));
    if (isD) rel(apq, 2 * di, 2 * di + 1);
    if (__ballot(big) && lane == 0) L.any = 1;
    __syncthreads();
    if (!L.any) return false;

    // Every role runs its own loop of the R + 1 iterations (one barrier each),
    // so no wave carries another role's registers through the loop.
    constexpr int NP = P / NQ;
    const int qw = wave - 1 - NA;
    double qt[NP], qb[NP];   // Q: columns of pairs NP qw .., lane = row
    if (isA) {
        double *e0 = &L.ex[0][0][0], *e1 = &L.ex[1][0][0];
        auto step = [&](const double *from, double *to, const d2 *cs) {
            double x[kBlk][4];
            d2 ri[kBlk], rj[kBlk];
#pragma unroll
            for (int u = 0; u < kBlk; ++u) {
                ri[u] = cs[bi[u]];
                rj[u] = cs[bj[u]];
#pragma unroll
                for (int e = 0; e < 4; ++e) x[u][e] = from[e * Lds::kEnt + blk[u]];
            }
#pragma unroll
            for (int u = 0; u < kBlk; ++u) {
                const double u00 = ri[u].x * x[u][0] - ri[u].y * x[u][2], u01 = ri[u].x * x[u][1] - ri[u].y * x[u][3];
                const double u10 = ri[u].y * x[u][0] + ri[u].x * x[u][2], u11 = ri[u].y * x[u][1] + ri[u].x * x[u][3];
                to[dst[u][0]] = rj[u].x * u00 - rj[u].y * u01;
                to[dst[u][1]] = rj[u].y * u00 + rj[u].x * u01;
                to[dst[u][2]] = rj[u].x * u10 - rj[u].y * u11;
                to[dst[u][3]] = rj[u].y * u10 + rj[u].x * u11;
            }
        };
        __syncthreads();
        for (int k = 1; k < R; k += 2) {
            step(e0, e1, L.cs[0]);
            __syncthreads();
            step(e1, e0, L.cs[1]);
            __syncthreads();
        }
        step(e0, e1, L.cs[0]);   // k = R: the final state, in ex[1]
        __syncthreads();
    } else if (isD) {
        // where a_pq of the next round stands before its rotation, and where
        // this pair's rotated diagonal and (zeroed) off-diagonal entry go
        const int st = di == 0 ? 0 : di == 1 ? 1 : 2 * di - 2, sb = di == P - 1 ? 2 * P - 2 : 2 * di + 3;
        const int sP = st >> 1, sQ = sb >> 1, sBlk = eig_block<P>(sP, sQ);
        const bool sx = st & 1, sy = sb & 1;
        const int dT = eig_dest<P>(2 * di), dB = eig_dest<P>(2 * di + 1), rslot = eig_slot<P>(dT, dB);
        double resid = 0.0;
        auto rotate = [&](int cur) {
            double c, s, t;
            bool skip;
            jacobi_angle(app, apq, aqq, c, s, t, skip);
            resid = skip ? apq : 0.0;
            if (lane < P) {
                L.cs[cur][di] = d2{c, s};
                L.dg[cur ^ 1][dT] = fma(-t, apq, app);
                L.dg[cur ^ 1][dB] = fma(t, apq, aqq);
            }
            __syncthreads();
        };
        auto fetch = [&](int cur) {
            const int prv = cur ^ 1;
            const double *e = &L.ex[prv][0][0];
            const double b00 = e[sBlk], b01 = e[Lds::kEnt + sBlk], b10 = e[2 * Lds::kEnt + sBlk],
                         b11 = e[3 * Lds::kEnt + sBlk];
            const d2 rp = L.cs[prv][sP], rq = L.cs[prv][sQ];
            app = L.dg[cur][2 * di];
            aqq = L.dg[cur][2 * di + 1];
            const double r0 = sx ? rp.y : rp.x, r1 = sx ? rp.x : -rp.y;
            const double q0 = sy ? rq.y : rq.x, q1 = sy ? rq.x : -rq.y;
            const double u0 = r0 * b00 + r1 * b10, u1 = r0 * b01 + r1 * b11;
            apq = q0 * u0 + q1 * u1;
            if (lane < P) (&L.ex[cur][0][0])[rslot] = resid;
        };
        __builtin_amdgcn_s_setprio(3);
        rotate(0);
        for (int k = 1; k < R; k += 2) {
            fetch(1);
            rotate(1);
            fetch(0);
            rotate(0);
        }
        fetch(1);   // k = R: the final diagonal blocks
        __builtin_amdgcn_s_setprio(0);
        __syncthreads();
    } else {
#pragma unroll
        for (int u = 0; u < NP; ++u) {
            qt[u] = lane == NP * qw + u ? 1.0 : 0.0;
            qb[u] = lane == P + NP * qw + u ? 1.0 : 0.0;
        }
        __syncthreads();
#pragma unroll 3
        for (int k = 1; k <= R; ++k) {
            const int cur = k & 1, prv = cur ^ 1;
            const d2 lr = L.cs[prv][NP * qw + (lane & (NP - 1))];
            if (k > 1) {   // the columns that crossed after rotation k - 2
                if (qw > 0) qt[0] = L.qx[prv][qw - 1][0][lane];
                if (qw < NQ - 1) qb[NP - 1] = L.qx[prv][qw + 1][1][lane];
            }
            double nt[NP], nb[NP];
#pragma unroll
            for (int u = 0; u < NP; ++u) {
                const double c = lane_value(lr.x, u), s = lane_value(lr.y, u);
                nt[u] = c * qt[u] - s * qb[u];
                nb[u] = s * qt[u] + c * qb[u];
            }
            L.qx[cur][qw][0][lane] = nt[NP - 1];
            L.qx[cur][qw][1][lane] = nb[0];
#pragma unroll
            for (int u = NP - 1; u > 0; --u) qt[u] = nt[u - 1];
            qt[0] = nt[0];                   // t_0 stays (other waves: replaced next round)
            if (qw == 0) qt[1] = nb[0];
#pragma unroll
            for (int u = 0; u < NP - 1; ++u) qb[u] = nb[u + 1];
            qb[NP - 1] = nt[NP - 1];         // last t -> last b (other waves: replaced next round)
            __syncthreads();
        }
    }
    // the last rotation wrote the final diagonal (positions as at the start) to dg[1]
    if (lane < n) {
        const double d = L.dg[1][2 * (lane % P) + lane / P];   // diagonal of row `lane`
        int rk = 0;
        for (int j = wave; j < n; j += NW) {
            const double dj = L.dg[1][2 * (j % P) + j / P];
            rk += (dj > d || (dj == d && j < lane)) ? 1 : 0;
        }
        atomicAdd(&L.rank[lane], rk);
    }
    const bool isQ = wave > NA;
    if (isQ) {   // the move after the last rotation
        if (qw > 0) qt[0] = L.qx[1][qw - 1][0][lane];
        if (qw < NQ - 1) qb[NP - 1] = L.qx[1][qw + 1][1][lane];
    }
    __syncthreads();
    if (isQ) {
        if (lane < 2 * P)
#pragma unroll
            for (int u = 0; u < NP; ++u) {
                put(L.rank[NP * qw + u], lane, qt[u]);
                put(L.rank[P + NP * qw + u], lane, qb[u]);
            }
    } else if (isA) {
#pragma unroll
        for (int u = 0; u < kBlk; ++u)
            if (blk[u] < Lds::kTrash)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int r = L.rank[bi[u] + P * (e >> 1)], c = L.rank[bj[u] + P * (e & 1)];
                    const double v = L.ex[1][e][blk[u]];
                    put_g(r, c, v);
                    put_g(c, r, v);
                }
    } else if (lane < P) {
        const int r = L.rank[di], c = L.rank[P + di];
        put_g(r, r, app);
        put_g(c, c, aqq);
        put_g(r, c, apq);
        put_g(c, r, apq);
    }
    return true;
}

constexpr int kEigThreads = eig_threads(32), kEigWaves = kEigThreads / 64;

// Blocks (of 32 rows) of pair l in round r of the circle schedule on nb (even) blocks.
__device__ __forceinline__ void jac_blocks(int nb, int r, int l, int &bi, int &bj) {
    const int p = l == 0 ? nb - 1 : (r + l) % (nb - 1), q = (r - l + nb - 1) % (nb - 1);
    bi = min(p, q);
    bj = max(p, q);
}

// Pair (of round r) that block x belongs to; hi: whether it is the larger block.
__device__ __forceinline__ int jac_pair_of(int nb, int r, int x, bool &hi) {
    const int d = x == nb - 1 ? 0 : (x - r + nb - 1) % (nb - 1);
    const int l = d < nb / 2 ? d : nb - 1 - d;
    int bi, bj;
    jac_blocks(nb, r, l, bi, bj);
    hi = x == bj;
    return l;
}

// A pair's 64 x 64 rotation is stored as operand fragments: per 16 x 16 tile
// (row tile, column tile) lane r + 16 g holds row r, columns 4 g .. 4 g + 3.
__device__ __forceinline__ int frag_at(int o, int k) {
    return ((o >> 4) * 4 + (k >> 4)) * 256 + ((o & 15) + 16 * ((k >> 2) & 3)) * 4 + (k & 3);
}

// Entry of G (blocks at and above the diagonal are kept) for a 16 x 16 x 16
// step: this lane's row x (0..15 of a 16-row slab), columns 4 g .. 4 g + 3.
__device__ __forceinline__ void load_g(const double *G, int64_t ld, int X, int x, int Y, int y, double (&a)[4]) {
    if (X <= Y) {
        const double *src = G + (int64_t)(32 * X + x) * ld + 32 * Y + y;
#pragma unroll
        for (int j = 0; j < 4; ++j) a[j] = src[j];
    } else {
        const double *src = G + (int64_t)(32 * Y + y) * ld + 32 * X + x;
#pragma unroll
        for (int j = 0; j < 4; ++j) a[j] = src[j * ld];
    }
}

// Launch k of a sweep (k = 0 .. number of rounds): the angles of round k run
// beside the updates of round k - 1, in one launch.  G goes from buffer (k - 1)
// & 1 to buffer k & 1; the rotations and the rotated 64 x 64 diagonal blocks
// (Gd) of round k are in halves k & 1 of Qr and Gd.
//   Workgroups 0 .. neig - 1, a pair of blocks (I, J) of round k each: the two
//   diagonal blocks are in Gd, the block between them is rotated here from the
//   old G, then one cyclic sweep (eig_sweep).
//   The others, a wave per 64 x 16 piece: G[p, q] <- J_p^T G[p, q] J_q (pairs
//   p <= q, from the old buffer to the new one; p = q: a copy of Gd) or Qt[p]
//   <- J_p^T Qt[p].  The middle product's accumulators (row 4 r + g, column
//   lane & 15) are the B operand of the second product as they are (its step
//   j takes k = 4 j + g), so a wave needs neither LDS nor a barrier.
// Neither fills the chip alone: the angles are a latency chain on one CU per
// pair, the updates are FP64 MFMA work for the rest.
__global__ __launch_bounds__(kEigThreads) void jac_round_kernel(const JacItem *__restrict__ items,
                                                                const JacTask *__restrict__ eig, int neig,
                                                                const JacTask *__restrict__ upd, int nupd, int k,
                                                                const int32_t *__restrict__ active) {
    __shared__ EigLds<32> L;
    __shared__ double T[64][34];     // old G between the pairs of I and J, times J's rotation
    __shared__ double B[32][33];     // the block between I and J
    const int tid = threadIdx.x, lane = tid & 63, r16 = lane & 15, g = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int cur = k & 1, prv = cur ^ 1;
    if ((int)blockIdx.x < neig) {
        const JacTask tk = eig[blockIdx.x];
        const JacItem it = items[tk.item];
        const int nb = it.np / 32, npair = nb / 2;
        if (!active[tk.item] || k >= nb - 1) return;
        int I, J;
        jac_blocks(nb, k, tk.a, I, J);
        const int n = min(max(it.nv - 32 * I, 0), 32) + min(max(it.nv - 32 * J, 0), 32);
        const double *gi = nullptr, *gj = nullptr;   // diagonal blocks in Gd (row stride 64)
        if (k > 0) {
            bool hi, hj;
            const int p = jac_pair_of(nb, k - 1, I, hi), q = jac_pair_of(nb, k - 1, J, hj);
            const double *Qp = it.Qr + ((int64_t)prv * npair + p) * 4096 + (hi ? 2048 : 0);
            const double *Qq = it.Qr + ((int64_t)prv * npair + q) * 4096 + (hj ? 2048 : 0);
            gi = it.Gd + ((int64_t)prv * npair + p) * 4096 + (hi ? 32 * 65 : 0);
            gj = it.Gd + ((int64_t)prv * npair + q) * 4096 + (hj ? 32 * 65 : 0);
            int pb[2], qb[2];
            jac_blocks(nb, k - 1, p, pb[0], pb[1]);
            jac_blocks(nb, k - 1, q, qb[0], qb[1]);
            if (w < 8) {   // T = G[p, q] Qq^T: rows 16 (w / 2), columns 16 (w % 2)
                const int mt = w >> 1, nt = w & 1;
                d4 acc = {0, 0, 0, 0};
                double a[4][4], b[4][4];
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) {
                    load_g(it.G[prv], it.np, pb[mt >> 1], 16 * (mt & 1) + r16, qb[ks >> 1], 16 * (ks & 1) + 4 * g, a[ks]);
#pragma unroll
                    for (int j = 0; j < 4; ++j) b[ks][j] = Qq[(nt * 4 + ks) * 256 + 4 * lane + j];
                }
#pragma unroll
                for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                    for (int j = 0; j < 4; ++j) acc = mfma_f64(a[ks][j], b[ks][j], acc);
#pragma unroll
                for (int r = 0; r < 4; ++r) T[16 * mt + 4 * r + g][16 * nt + r16] = acc[r];
            }
            double a[4][4];
            if (w < 4)
#pragma unroll
                for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                    for (int j = 0; j < 4; ++j) a[ks][j] = Qp[((w >> 1) * 4 + ks) * 256 + 4 * lane + j];
            __syncthreads();
            if (w < 4) {   // B = Qp T: rows 16 (w / 2), columns 16 (w % 2)
                d4 acc = {0, 0, 0, 0};
#pragma unroll
                for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        acc = mfma_f64(a[ks][j], T[16 * ks + 4 * g + j][16 * (w & 1) + r16], acc);
#pragma unroll
                for (int r = 0; r < 4; ++r) B[16 * (w >> 1) + 4 * r + g][16 * (w & 1) + r16] = acc[r];
            }
            __syncthreads();
        }
        auto at = [&](int r, int c) {
            const int lo = min(r, c), hi = max(r, c);
            if (k == 0) {
                const int gl = lo < 32 ? 32 * I + lo : 32 * J + lo - 32, gh = hi < 32 ? 32 * I + hi : 32 * J + hi - 32;
                return it.G[0][(int64_t)gl * it.np + gh];
            }
            if (hi < 32) return gi[64 * lo + hi];
            if (lo >= 32) return gj[64 * (lo - 32) + hi - 32];
            return B[lo][hi - 32];
        };
        double *Q = it.Qr + ((int64_t)cur * npair + tk.a) * 4096, *D = it.Gd + ((int64_t)cur * npair + tk.a) * 4096;
        auto put = [&](int o, int c, double v) { Q[frag_at(o, c)] = v; };
        auto put_g = [&](int r, int c, double v) { D[64 * r + c] = v; };
        if (!eig_sweep<32>(L, n, it.tol, at, put, put_g))
            for (int e = tid; e < 4096; e += kEigThreads) {
                put(e >> 6, e & 63, (e >> 6) == (e & 63) ? 1.0 : 0.0);
                put_g(e >> 6, e & 63, at(e >> 6, e & 63));
            }
        return;
    }
    // updates of round k - 1
    const int t = ((int)blockIdx.x - neig) * kEigWaves + w;
    if (k == 0 || t >= nupd) return;
    const JacTask tk = upd[t];
    const JacItem it = items[tk.item];
    const int nb = it.np / 32, npair = nb / 2, p = tk.a, nt = tk.c;
    if (!active[tk.item] || k > nb - 1) return;
    const int64_t ld = it.np;
    int pb[2], qb[2];
    jac_blocks(nb, k - 1, p, pb[0], pb[1]);
    const double *Qp = it.Qr + ((int64_t)prv * npair + p) * 4096;
    double b[4][4];   // B operand of the second product: rows 16 ks + 4 j + g, column lane & 15
    if (tk.b >= 0) {
        if (k == nb - 1) return;   // the next sweep starts from a fresh G
        const int q = tk.b;
        jac_blocks(nb, k - 1, q, qb[0], qb[1]);
        const int Y = qb[nt >> 1], yc = 16 * (nt & 1) + r16;
        if (p == q) {
            const double *D = it.Gd + ((int64_t)prv * npair + p) * 4096;
#pragma unroll
            for (int mt = 0; mt < 4; ++mt)
                if (pb[mt >> 1] <= Y)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int x = 16 * mt + 4 * r + g;
                        it.G[cur][(int64_t)(32 * pb[mt >> 1] + (x & 31)) * ld + 32 * Y + yc] = D[64 * x + 16 * nt + r16];
                    }
            return;
        }
        const double *Qq = it.Qr + ((int64_t)prv * npair + q) * 4096 + nt * 1024;
        d4 acc[4];
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) acc[mt] = d4{0, 0, 0, 0};
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            double f[4], a[4][4];
#pragma unroll
            for (int j = 0; j < 4; ++j) f[j] = Qq[ks * 256 + 4 * lane + j];
#pragma unroll
            for (int mt = 0; mt < 4; ++mt)
                load_g(it.G[prv], ld, pb[mt >> 1], 16 * (mt & 1) + r16, qb[ks >> 1], 16 * (ks & 1) + 4 * g, a[mt]);
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int mt = 0; mt < 4; ++mt) acc[mt] = mfma_f64(a[mt][j], f[j], acc[mt]);
        }
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
#pragma unroll
            for (int j = 0; j < 4; ++j) b[ks][j] = acc[ks][j];
    } else {
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                b[ks][j] = it.Qt[(int64_t)(32 * pb[ks >> 1] + 16 * (ks & 1) + 4 * j + g) * ld + 16 * nt + r16];
    }
    d4 acc[4];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) acc[mt] = d4{0, 0, 0, 0};
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
        double a[4][4];   // row r16 of tile mt, columns 16 ks + 4 j + g
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
#pragma unroll
            for (int j = 0; j < 4; ++j) a[mt][j] = Qp[(mt * 4 + ks) * 256 + (r16 + 16 * j) * 4 + g];
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int mt = 0; mt < 4; ++mt) acc[mt] = mfma_f64(a[mt][j], b[ks][j], acc[mt]);
    }
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int X = pb[mt >> 1], xr = 16 * (mt & 1) + 4 * r + g;
            if (tk.b < 0) {
                it.Qt[(int64_t)(32 * X + xr) * ld + 16 * nt + r16] = acc[mt][r];
                continue;
            }
            const int Y = qb[nt >> 1], yc = 16 * (nt & 1) + r16;
            if (X <= Y) it.G[cur][(int64_t)(32 * X + xr) * ld + 32 * Y + yc] = acc[mt][r];
            else it.G[cur][(int64_t)(32 * Y + yc) * ld + 32 * X + xr] = acc[mt][r];
        }
}

void launch_jac_round(const JacItem *items, const JacTask *eig, int neig, const JacTask *upd, int nupd, int k,
                      const int32_t *active, hipStream_t s) {
    const int grid = neig + (k > 0 ? (nupd + kEigWaves - 1) / kEigWaves : 0);
    if (grid > 0)
        hipLaunchKernelGGL(jac_round_kernel, dim3(grid), dim3(kEigThreads), 0, s, items, eig, neig, upd, nupd, k,
                           active);
}

// One workgroup per 64 x 64 block (row block <= column block) of a fresh G:
// largest |G_ij| / sqrt(G_ii G_jj) of every matrix (offmax, as the bits of a
// non-negative double), and Qt = I.
__global__ __launch_bounds__(256) void jac_begin_kernel(const JacItem *__restrict__ items,
                                                        const JacTask *__restrict__ tasks,
                                                        const int32_t *__restrict__ active,
                                                        unsigned long long *__restrict__ offmax) {
    __shared__ double d[2][64], f[2][64], red[4];   // norms^2 of the block's rows and columns, 1 / norm
    const JacTask tk = tasks[blockIdx.x];
    const JacItem it = items[tk.item];
    if (!active[tk.item]) return;
    const int tid = threadIdx.x;
    const int r0 = 64 * tk.a, c0 = 64 * tk.b;
    const double *G = it.G[0];
    double v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = G[(int64_t)(r0 + 4 * u + (tid >> 6)) * it.np + c0 + (tid & 63)];
    if (tid < 128) {   // 0: absent or zero
        const int r = (tid < 64 ? r0 : c0 - 64) + tid;
        const double g = r < it.nv ? G[(int64_t)r * it.np + r] : 0.0;
        d[tid >> 6][tid & 63] = g;
        f[tid >> 6][tid & 63] = g > 0.0 ? 1.0 / sqrt(g) : 0.0;
    }
    __syncthreads();
    double off = 0.0;
#pragma unroll
    for (int u = 0; u < 16; ++u) {
        const int i = 4 * u + (tid >> 6), j = tid & 63;
        // what eig_sweep would rotate (none where the product of the norms leaves
        // the range: rows that small or large count as orthogonal)
        const double dd = d[0][i] * d[1][j];
        if (r0 + i < c0 + j && dd > 0.0 && v[u] * v[u] > it.tol * it.tol * dd) off = fmax(off, fabs(v[u]) * f[0][i] * f[1][j]);
        it.Qt[(int64_t)(r0 + i) * it.np + c0 + j] = r0 + i == c0 + j ? 1.0 : 0.0;
        if (r0 != c0) it.Qt[(int64_t)(c0 + i) * it.np + r0 + j] = 0.0;
    }
#pragma unroll
    for (int w = 32; w > 0; w >>= 1) off = fmax(off, __shfl_xor(off, w));
    if ((tid & 63) == 0) red[tid >> 6] = off;
    __syncthreads();
    if (tid == 0) {
        off = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
        atomicMax(&offmax[tk.item], (unsigned long long)__double_as_longlong(off));
    }
}

void launch_jac_begin(const JacItem *items, const JacTask *tasks, int ntasks, const int32_t *active,
                      unsigned long long *offmax, hipStream_t s) {
    if (ntasks > 0) hipLaunchKernelGGL(jac_begin_kernel, dim3(ntasks), dim3(256), 0, s, items, tasks, active, offmax);
}

// A matrix of at most 2 P rows, whole iteration in one workgroup: Gram matrix
// (FP64 MFMA), one cyclic sweep of it, W <- J^T W and Z <- J^T Z, until the
// fresh Gram matrix meets the tolerance.  W and Z stay in global memory (the
// caches); no launch, no host step between sweeps.  What bounds it is the sweep
// of the Gram matrix on short rows and the latency of the passes over W on long
// ones, so both passes load several steps ahead: 48 x 1024 1290 -> 1050 us a call,
// 16 x 2048 894 -> 770.  Up to 16 rows the Gram matrix is one tile, a chain of MFMAs
// of one wave; from 1024 columns on all waves take a range of them, the next loads
// under way: 16 x 2048 770 -> 610, 8 x 4096 730 -> 510.
template <int P>
__global__ __launch_bounds__(eig_threads(P)) void jac_small_kernel(const JacSmall *__restrict__ items, int max_sweeps,
                                                                   int32_t *__restrict__ sweeps) {
    constexpr int kThreads = eig_threads(P), kWaves = kThreads / 64, kT = P / 8;   // kT: 16-row tiles
    // loads in flight, as registers allow: 16-wide steps of the Gram sums, tiles of columns of the update
    constexpr int kAhead = P == 8 ? 8 : 2, kCols = P == 8 ? 16 : P == 16 ? 4 : 1;
    __shared__ EigLds<P> L;
    __shared__ double Gs[2 * P][2 * P + 2];   // Gram matrix, then the rotation
    constexpr int kGw = P == 8 ? kWaves : 1;
    __shared__ double Gw[kGw][16][17];        // its sums over the waves' ranges
    const JacSmall it = items[blockIdx.x];
    const int tid = threadIdx.x, lane = tid & 63, r16 = lane & 15, g = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    for (int e = tid; e < it.nv * it.nv; e += kThreads) it.Z[e] = (e / it.nv == e % it.nv) ? 1.0 : 0.0;
    if (it.nv == 1) {   // nothing to rotate
        if (tid == 0) sweeps[blockIdx.x] = 0;
        return;
    }
    const int nt16 = (it.nv + 15) / 16;
    int done = -1;
    for (int sw = 0; sw < max_sweeps; ++sw) {
        __syncthreads();   // rows of W (and Z) are whole
        for (int e = tid; e < 4 * P * P; e += kThreads) Gs[e / (2 * P)][e % (2 * P)] = 0.0;
        __syncthreads();
        // tiles (ti <= tj) of the Gram matrix, one at a time per wave; the only tile
        // of up to 16 rows by all waves, a range of the columns each, if they are many
        const bool shared = P == 8 && it.len >= 1024;
        for (int t = w; t < (shared ? kWaves : nt16 * (nt16 + 1) / 2); t += kWaves) {
            int ti = 0, rest = shared ? 0 : t;
            while (rest >= nt16 - ti) { rest -= nt16 - ti; ++ti; }
            const int tj = ti + rest;
            const int steps = (it.len + 15) / 16;
            const int kend = shared ? min(it.len, 16 * (steps * (w + 1) / kWaves)) : it.len;
            const int ra = 16 * ti + r16, rb = 16 * tj + r16;
            const double *pa = it.W + (int64_t)min(ra, it.nv - 1) * it.len;
            const double *pb = it.W + (int64_t)min(rb, it.nv - 1) * it.len;
            d4 acc = {0, 0, 0, 0};
            const bool ia = ra < it.nv, ib = rb < it.nv;
            int k0 = shared ? 16 * (steps * w / kWaves) : 0;
            // whole runs of kAhead steps; P < 32: the next run's loads under way during the sums
            constexpr int kBuf = P == 32 ? 1 : 2;
            double a[kBuf][kAhead][4], b[kBuf][P == 8 ? 1 : kAhead][4];   // P = 8: one tile, b = a
            auto load = [&](int h, int k) {
#pragma unroll
                for (int u = 0; u < kAhead; ++u)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const double x = pa[k + 16 * u + 4 * g + j];
                        a[h][u][j] = ia ? x : 0.0;
                        if constexpr (P > 8) {
                            const double y = pb[k + 16 * u + 4 * g + j];
                            b[h][u][j] = ib ? y : 0.0;
                        }
                    }
            };
            auto mul = [&](int h) {
#pragma unroll
                for (int u = 0; u < kAhead; ++u)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        acc = mfma_f64(a[h][u][j], P == 8 ? a[h][u][j] : b[h][P == 8 ? 0 : u][j], acc);
            };
            const int runs = max(0, kend - k0) / (16 * kAhead);
            if constexpr (kBuf == 1)
                for (int i = 0; i < runs; ++i) {
                    load(0, k0);
                    mul(0);
                    k0 += 16 * kAhead;
                }
            if (kBuf == 2 && runs > 0) load(0, k0);
            for (int i = 0; kBuf == 2 && i < runs; i += 2) {
                if (i + 1 < runs) load(kBuf - 1, k0 + 16 * kAhead);
                mul(0);
                k0 += 16 * kAhead;
                if (i + 1 < runs) {
                    if (i + 2 < runs) load(0, k0 + 16 * kAhead);
                    mul(kBuf - 1);
                    k0 += 16 * kAhead;
                }
            }
            for (; k0 < kend; k0 += 16) {
                double a[4], b[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int k = k0 + 4 * g + j;
                    const bool in = k < it.len;
                    a[j] = in && ia ? pa[k] : 0.0;
                    b[j] = in && ib ? pb[k] : 0.0;
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) acc = mfma_f64(a[j], b[j], acc);
            }
            if (shared) {
#pragma unroll
                for (int r = 0; r < 4; ++r) Gw[w % kGw][4 * r + g][r16] = acc[r];
                continue;
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                Gs[16 * ti + 4 * r + g][16 * tj + r16] = acc[r];
                Gs[16 * tj + r16][16 * ti + 4 * r + g] = acc[r];
            }
        }
        __syncthreads();
        if (shared) {
            for (int e = tid; e < 256; e += kThreads) {
                double x = Gw[0][e / 16][e % 16];
                for (int q = 1; q < kWaves; ++q) x += Gw[q % kGw][e / 16][e % 16];
                Gs[e / 16][e % 16] = x;
            }
            __syncthreads();
        }
        auto at = [&](int r, int c) { return Gs[min(r, c)][max(r, c)]; };
        auto put = [&](int o, int k, double v) { Gs[o][k] = v; };
        if (!eig_sweep<P>(L, it.nv, it.tol, at, put, [](int, int, double) {})) {
            done = sw;
            break;
        }
        __syncthreads();
        // W <- J^T W, then Z: a wave takes up to kCols times 16 columns at a time
        const int cw = (it.len + 15) / 16, cz = (it.nv + 15) / 16;
        const int per = kCols == 1 ? 1 : min(kCols, (cw + cz + kWaves - 1) / kWaves);
        for (int t0 = w * per; t0 < cw + cz; t0 += kWaves * per) {
            double b[kCols][kT][4];
#pragma unroll
            for (int u = 0; u < kCols; ++u) {
                const int t = t0 + u;
                if (u >= per) break;
                const double *X = t < cw ? it.W : it.Z;
                const int len = t < cw ? it.len : it.nv, col = 16 * (t < cw ? t : t - cw) + r16;
#pragma unroll
                for (int ks = 0; ks < kT; ++ks)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int k = 16 * ks + 4 * g + j;
                        b[u][ks][j] = k < it.nv && t < cw + cz && col < len ? X[(int64_t)k * len + col] : 0.0;
                    }
            }
#pragma unroll
            for (int u = 0; u < kCols; ++u) {
                const int t = t0 + u;
                if (u >= per || t >= cw + cz) break;
                double *X = t < cw ? it.W : it.Z;
                const int len = t < cw ? it.len : it.nv, col = 16 * (t < cw ? t : t - cw) + r16;
                for (int ti = 0; ti < nt16; ++ti) {
                    d4 acc = {0, 0, 0, 0};
#pragma unroll
                    for (int ks = 0; ks < kT; ++ks)
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            acc = mfma_f64(Gs[16 * ti + r16][16 * ks + 4 * g + j], b[u][ks][j], acc);
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int o = 16 * ti + 4 * r + g;
                        if (o < it.nv && col < len) X[(int64_t)o * len + col] = acc[r];
                    }
                }
            }
        }
    }
    if (tid == 0) sweeps[blockIdx.x] = done;
}

// The narrowest instance that holds max_nv rows: for a dozen rows a sweep of
// the 64-row one costs 30 us, that of the 16-row one 6 us.
void launch_jac_small(const JacSmall *items, int nitems, int max_nv, int max_sweeps, int32_t *sweeps, hipStream_t s) {
    if (nitems <= 0) return;
    if (max_nv <= 16)
        hipLaunchKernelGGL(jac_small_kernel<8>, dim3(nitems), dim3(eig_threads(8)), 0, s, items, max_sweeps, sweeps);
    else if (max_nv <= 32)
        hipLaunchKernelGGL(jac_small_kernel<16>, dim3(nitems), dim3(eig_threads(16)), 0, s, items, max_sweeps, sweeps);
    else
        hipLaunchKernelGGL(jac_small_kernel<32>, dim3(nitems), dim3(eig_threads(32)), 0, s, items, max_sweeps, sweeps);
}

__global__ __launch_bounds__(256) void row_norm_kernel(const RowRef *rows, double *out) {
    __shared__ double sh[256];
    const RowRef r = rows[blockIdx.x];
    double acc = 0.0;
    for (int c = threadIdx.x; c < r.len; c += 256) acc += r.p[c] * r.p[c];
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[blockIdx.x] = sqrt(sh[0]);
}

void launch_row_norms(const RowRef *rows, int nrows, double *out, hipStream_t s) {
    if (nrows > 0) hipLaunchKernelGGL(row_norm_kernel, dim3(nrows), dim3(256), 0, s, rows, out);
}

__global__ __launch_bounds__(256) void copy_kernel(const CopyTask *tasks) {
    const CopyTask t = tasks[blockIdx.y];
    const int64_t n = (int64_t)t.rows * t.cols;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
        const int r = (int)(e / t.cols), c = (int)(e % t.cols);
        const int rs = t.ridx ? t.ridx[r] : r, cs = t.cidx ? t.cidx[c] : c;
        double v = t.trans ? t.src[(int64_t)cs * t.sld + rs] : t.src[(int64_t)rs * t.sld + cs];
        if (t.rscale) v *= t.rscale[r];
        if (t.cscale) v *= t.cscale[c];
        t.dst[(int64_t)r * t.dld + c] = v;
    }
}

void launch_copies(const CopyTask *tasks, int ntasks, int64_t max_elems, hipStream_t s) {
    if (ntasks <= 0 || max_elems <= 0) return;
    const int g = (int)std::min<int64_t>(256, (max_elems + 255) / 256);
    hipLaunchKernelGGL(copy_kernel, dim3(g, ntasks), dim3(256), 0, s, tasks);
}


// ---------------------------------------------------------------------------
// Householder QR preconditioning of the Jacobi iteration.
//
// Panel kernel: one workgroup of NT threads factors the 16 rows of a panel.
// Thread t holds positions j0 + t + NT u (u < UQ) of all 16 rows in
// registers.  Reflector j (pivot position p = j0 + j) needs one block
// reduction of 16 sums C_k = sum_{q > p} x_j[q] x_k[q] (C_j is the squared
// norm below the pivot) and the pivot-row entries E_k = x_k[p] (E_j is the
// pivot), which thread j publishes.  With beta = -sign(E_j) sqrt(E_j^2 + C_j),
// tau = (beta - E_j) / beta and v = x_j / (E_j - beta) below p (v_p = 1), the
// dot of v with row k is E_k + C_k / (E_j - beta): for later rows it gives
// their update, for earlier rows (which hold their reflectors there) the new
// column of T.  The sums are a reduce-scatter butterfly within each wave and
// a fixed-order sum over the waves, so every thread reads identical scalars
// and the result is reproducible.
template <int NT>
__device__ __forceinline__ void qr_sum16(double (&v)[16], double (*red)[16], double *res, int tid) {
    const int lane = tid & 63, wave = tid >> 6;
    double h8[8], h4[4], h2[2];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const bool up = lane & 16;
        h8[i] = (up ? v[8 + i] : v[i]) + __shfl_xor(up ? v[i] : v[8 + i], 16);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const bool up = lane & 8;
        h4[i] = (up ? h8[4 + i] : h8[i]) + __shfl_xor(up ? h8[i] : h8[4 + i], 8);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const bool up = lane & 4;
        h2[i] = (up ? h4[2 + i] : h4[i]) + __shfl_xor(up ? h4[i] : h4[2 + i], 4);
    }
    const bool up = lane & 2;
    double one = (up ? h2[1] : h2[0]) + __shfl_xor(up ? h2[0] : h2[1], 2);
    one += __shfl_xor(one, 1);
    one += __shfl_xor(one, 32);
    // lane bits 4..1 chose the halves: the lane holds value (lane >> 1) & 15
    if ((lane & 33) == 0) red[wave][(lane >> 1) & 15] = one;
    __syncthreads();
    if (tid < 16) {
        double a = red[0][tid];
#pragma unroll
        for (int w = 1; w < NT / 64; ++w) a += red[w][tid];
        res[tid] = a;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = res[i];
}

template <int NT, int UQ>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(1, 2))) void qr_panel_kernel(
    const QrPanel *tasks) {
    const QrPanel tk = tasks[blockIdx.x];
    const int nb = min(kQrPanel, tk.nv - tk.j0);
    const int tid = threadIdx.x;
    __shared__ double red[NT / 64][16];
    __shared__ double res[16];
    __shared__ double piv[2][kQrPanel];   // E of alternate steps: written before a step's first barrier
    __shared__ double Ts[kQrPanel][kQrPanel];
    if (tid < kQrPanel * kQrPanel) Ts[tid / kQrPanel][tid % kQrPanel] = 0.0;
    double x[kQrPanel][UQ];
#pragma unroll
    for (int r = 0; r < kQrPanel; ++r)
#pragma unroll
        for (int u = 0; u < UQ; ++u) {
            const int q = tk.j0 + tid + NT * u;
            x[r][u] = (r < nb && q < tk.len) ? tk.A[(int64_t)(tk.j0 + r) * tk.len + q] : 0.0;
        }
    // j runs as a loop; rows are picked and written back by selects, so every
    // register index is a constant
    for (int j = 0; j < nb; ++j) {   // nb is uniform over the workgroup
        const int p = tk.j0 + j;
        double xj[UQ];
#pragma unroll
        for (int u = 0; u < UQ; ++u) {
            double t = x[0][u];
#pragma unroll
            for (int r = 1; r < kQrPanel; ++r) t = r == j ? x[r][u] : t;
            const int q = tk.j0 + tid + NT * u;
            xj[u] = q > p ? t : 0.0;   // below the pivot only
        }
        double cs[kQrPanel];
#pragma unroll
        for (int k = 0; k < kQrPanel; ++k) {
            double t = 0.0;
#pragma unroll
            for (int u = 0; u < UQ; ++u) t = fma(xj[u], x[k][u], t);
            cs[k] = t;
        }
        double *E = piv[j & 1];
        if (tid == j)   // position p is thread j's u = 0
#pragma unroll
            for (int k = 0; k < kQrPanel; ++k) E[k] = x[k][0];
        qr_sum16<NT>(cs, red, res, tid);
        double sig = cs[0], alpha = E[0];
#pragma unroll
        for (int k = 1; k < kQrPanel; ++k) {
            sig = k == j ? cs[k] : sig;
            alpha = k == j ? E[k] : alpha;
        }
        double tau = 0.0, beta = alpha, inv = 0.0;
        if (sig > 0.0) {
            const double nrm = sqrt(fma(alpha, alpha, sig));
            beta = alpha >= 0.0 ? -nrm : nrm;
            tau = (beta - alpha) / beta;
            inv = 1.0 / (alpha - beta);
        }
        // reflector v: 0 before p, 1 at p, x * inv after; row j keeps beta at p
        double v[UQ];
#pragma unroll
        for (int u = 0; u < UQ; ++u) {
            const int q = tk.j0 + tid + NT * u;
            v[u] = q > p ? xj[u] * inv : (q == p ? 1.0 : 0.0);
            const bool keep = q < p;
#pragma unroll
            for (int r = 0; r < kQrPanel; ++r) x[r][u] = (r == j && !keep) ? (q == p ? beta : v[u]) : x[r][u];
        }
        // d_k = v . x_k (row k after the earlier steps)
        double d[kQrPanel];
#pragma unroll
        for (int k = 0; k < kQrPanel; ++k) d[k] = fma(cs[k], inv, E[k]);
#pragma unroll
        for (int k = 0; k < kQrPanel; ++k) {
            const double f = (k > j && k < nb) ? tau * d[k] : 0.0;
#pragma unroll
            for (int u = 0; u < UQ; ++u) x[k][u] = fma(-f, v[u], x[k][u]);
        }
        // T[0:j][j] = -tau T[0:j][0:j] (V[:, 0:j]^T v); T[j][j] = tau.  Thread i
        // only reads row i of T, which it wrote itself.
        if (tid < j) {
            double t = 0.0;
#pragma unroll
            for (int l = 0; l < kQrPanel; ++l)
                if (l >= tid && l < j) t = fma(Ts[tid][l], d[l], t);
            Ts[tid][j] = -tau * t;
        }
        if (tid == j) Ts[j][j] = tau;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kQrPanel; ++r)
#pragma unroll
        for (int u = 0; u < UQ; ++u) {
            const int q = tk.j0 + tid + NT * u;
            if (r < nb && q < tk.len) tk.A[(int64_t)(tk.j0 + r) * tk.len + q] = x[r][u];
        }
    if (tid < kQrPanel * kQrPanel) tk.T[tid] = Ts[tid / kQrPanel][tid % kQrPanel];
}

void launch_qr_panels(const QrPanel *tasks, int ntasks, int max_span, hipStream_t s) {
    if (ntasks <= 0) return;
    if (max_span <= 512)
        hipLaunchKernelGGL((qr_panel_kernel<256, 2>), dim3(ntasks), dim3(256), 0, s, tasks);
    else if (max_span <= 1024)
        hipLaunchKernelGGL((qr_panel_kernel<256, 4>), dim3(ntasks), dim3(256), 0, s, tasks);
    else if (max_span <= 2048)
        hipLaunchKernelGGL((qr_panel_kernel<512, 4>), dim3(ntasks), dim3(512), 0, s, tasks);
    else
        throw std::invalid_argument("qr panel: rows longer than the panel kernel holds");
}
static_assert(kQrMaxLen == 2048, "panel kernel reach");

// Apply kernel: one workgroup of 4 waves per (panel, group of 16 target rows).
// D = V Y^T over positions j0.. (FP64 MFMA, reflector rows masked to their
// support with the unit entry), C = T^T D or T D, then Y -= C^T V (FP64 MFMA),
// both through 512-position chunks staged in LDS.
__global__ __launch_bounds__(JT) void qr_apply_kernel(const QrApply *tasks) {
    const QrApply tk = tasks[blockIdx.x];
    __shared__ double vrows[J2][CH + 1];
    __shared__ double yrows[J2][CH + 1];
    __shared__ double Dp[4][J2][J2 + 1];
    __shared__ double Cs[J2][J2 + 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r16 = lane & 15, g = lane >> 4;
    const __amdgpu_buffer_rsrc_t rV = rows_rsrc(tk.V, (int64_t)tk.nb * tk.len);
    const __amdgpu_buffer_rsrc_t rY = rows_rsrc(tk.Y, (int64_t)tk.ntgt * tk.len);
    const int span = tk.len - tk.j0;
    const int nch = (span + CH - 1) / CH;
    auto stage = [&](int c0) {
        double a[U], b[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = u * JT + tid, r = e / CH, q = tk.j0 + c0 + e % CH;
            const bool in = q < tk.len;
            const unsigned ov = (r < tk.nb && in && q > tk.j0 + r) ? (unsigned)(((int64_t)r * tk.len + q) * 8) : kOut;
            const unsigned oy = (r < tk.ntgt && in) ? (unsigned)(((int64_t)r * tk.len + q) * 8) : kOut;
            a[u] = (r < tk.nb && q == tk.j0 + r) ? 1.0 : bload(rV, ov);
            b[u] = bload(rY, oy);
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = u * JT + tid;
            vrows[e / CH][e % CH] = a[u];
            yrows[e / CH][e % CH] = b[u];
        }
        __syncthreads();
    };
    {
        d4 acc = {0.0, 0.0, 0.0, 0.0};
        for (int ch = 0; ch < nch; ++ch) {
            const int c0 = ch * CH;
            stage(c0);
            const int w = min(CH, span - c0);
            for (int kk = wave * 16; kk < w; kk += 64) {
                double a[4], b[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    a[j] = vrows[r16][kk + 4 * g + j];
                    b[j] = yrows[r16][kk + 4 * g + j];
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) acc = mfma_f64(a[j], b[j], acc);
            }
        }
        // D[i][c] = v_i . y_c; register r of lane l: row 4 r + l / 16, column l % 16
#pragma unroll
        for (int r = 0; r < 4; ++r) Dp[wave][4 * r + g][r16] = acc[r];
    }
    __syncthreads();
    {
        const int ei = tid / J2, ej = tid % J2;
        double c = 0.0;
#pragma unroll
        for (int i = 0; i < J2; ++i) {
            const double t = tk.trans ? tk.T[i * J2 + ei] : tk.T[ei * J2 + i];
            const double dij = ((Dp[0][i][ej] + Dp[1][i][ej]) + Dp[2][i][ej]) + Dp[3][i][ej];
            c = fma(t, dij, c);
        }
        Cs[ei][ej] = c;   // coefficient of reflector ei in target row ej
    }
    __syncthreads();
    double qa[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) qa[j] = Cs[4 * j + g][r16];
    unsigned dbase[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int o = 4 * r + g;
        dbase[r] = o < tk.ntgt ? (unsigned)((int64_t)o * tk.len) : kOut;
    }
    // the last chunk is still staged: go backwards
    for (int i = 0; i < nch; ++i) {
        const int ch = nch - 1 - i;
        const int c0 = ch * CH;
        if (i > 0) stage(c0);
        const int w = min(CH, span - c0);
        for (int n0 = wave * 16; n0 < w; n0 += 64) {
            const int col = n0 + r16;
            double b[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) b[j] = vrows[4 * j + g][col];
            d4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int j = 0; j < 4; ++j) acc = mfma_f64(qa[j], b[j], acc);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int o = 4 * r + g;
                const unsigned offr =
                    (dbase[r] != kOut && col < w) ? (dbase[r] + tk.j0 + c0 + col) * 8u : kOut;
                bstore(rY, offr, yrows[o][col] - acc[r]);
            }
        }
        __syncthreads();   // before the next chunk overwrites the staged rows
    }
}

void launch_qr_apply(const QrApply *tasks, int ntasks, hipStream_t s) {
    if (ntasks > 0) hipLaunchKernelGGL(qr_apply_kernel, dim3(ntasks), dim3(JT), 0, s, tasks);
}

// R[i][j] = A[j][i] for j >= i (the factor's upper triangle as rows), else 0.
__global__ void qr_extract_r_kernel(const QrItem *items) {
    const QrItem it = items[blockIdx.y];
    const int64_t n = (int64_t)it.nv * it.nv;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
        const int i = (int)(e / it.nv), j = (int)(e % it.nv);
        it.R[(int64_t)i * it.ldr + j] = j >= i ? it.A[(int64_t)j * it.len + i] : 0.0;
    }
}

void launch_qr_extract_r(const QrItem *items, int nitems, int max_nv, hipStream_t s) {
    if (nitems <= 0 || max_nv <= 0) return;
    const int g = std::min(1024, (max_nv * max_nv + 255) / 256);
    hipLaunchKernelGGL(qr_extract_r_kernel, dim3(g, nitems), dim3(256), 0, s, items);
}

// Y[r][c] = Z[r][c] for c < nv, 0 after (Y: nv x len).
__global__ void qr_embed_z_kernel(const QrItem *items) {
    const QrItem it = items[blockIdx.y];
    const int64_t n = (int64_t)it.nv * it.len;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
        const int r = (int)(e / it.len), c = (int)(e % it.len);
        it.Y[e] = c < it.nv ? it.Z[(int64_t)r * it.ldz + c] : 0.0;
    }
}

void launch_qr_embed_z(const QrItem *items, int nitems, int64_t max_elems, hipStream_t s) {
    if (nitems <= 0 || max_elems <= 0) return;
    const int g = (int)std::min<int64_t>(1024, (max_elems + 255) / 256);
    hipLaunchKernelGGL(qr_embed_z_kernel, dim3(g, nitems), dim3(256), 0, s, items);
}

}  // namespace pdmrg
