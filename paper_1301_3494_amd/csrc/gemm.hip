// Grouped block-sparse GEMM on CDNA4 matrix cores (gfx950).
//
// One launch runs a list of output tiles drawn from many GEMM items (the U(1)
// sector blocks of one contraction, possibly of several bonds).  Each item is
// C (M x N) = sum over its K-segments of op(A) op(B); the segments let one
// output block accumulate products whose operands live in different places
// (e.g. the physical-index sum of an environment update).  An item may stack
// blocks with different output leading dimensions along M through a row
// offset table.
//
// Workgroup: 256 threads = 4 wave64.  FP64 / FP32 tiles are BM x BN with the
// waves on a WGM x WGN grid, each wave owning an (BM/WGM) x (BN/WGN) sub-tile
// of 16 x 16 MFMA blocks (v_mfma_f64_16x16x4 / v_mfma_f32_16x16x4).  FP64
// operands that stream from memory go straight into registers (gemm_r64).  BF16x3
// takes operands split once in memory (each 4-byte word a bf16 pair x = hi +
// lo, both rounded to nearest even) through the FP32 kernels (gemm_quad,
// gemm_dma) and accumulates lo*hi' + hi*lo' + hi*hi' with bf16 MFMAs in FP32.
//
// Operands are read with buffer loads: the descriptor of each segment spans
// its operand and an offset outside it returns zero, so ragged tile edges need
// no branches.  Global loads of the next K-step are issued before the MFMAs of
// the current one.  Workgroup b runs tiles[b]: the host places the tiles so
// that every XCD (b % 8) receives an even share of the work and the tiles
// that share an A panel share one XCD's L2.
#include "kernels.hpp"
#include "split.hpp"

#include <type_traits>

namespace pdmrg {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int NT = 256;

__device__ __forceinline__ d4 mfma16(double a, double b, d4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f4 mfma16(float a, float b, f4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

template <typename T> struct Acc;
template <> struct Acc<double> { using type = d4; };
template <> struct Acc<float> { using type = f4; };

// A pointer that is the same in every lane, held in scalar registers.
__device__ __forceinline__ void *uniform_ptr(const void *p) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return reinterpret_cast<void *>(((uint64_t)hi << 32) | lo);
}

// Raw buffer descriptor over [p, p + 2 GiB): an offset at or beyond kOutOfRange
// reads as zero.
constexpr unsigned kOutOfRange = 0x80000000u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t operand_rsrc(const void *p) {
    return __builtin_amdgcn_make_buffer_rsrc(uniform_ptr(p), 0, 0x7fffffff, 0x00020000);
}
__device__ __forceinline__ double buf_load(__amdgpu_buffer_rsrc_t r, unsigned off, double) {
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
}
__device__ __forceinline__ float buf_load(__amdgpu_buffer_rsrc_t r, unsigned off, float) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}

// Element offset of row r of an item's C.
__device__ __forceinline__ int64_t c_row(const GemmItem &it, const int64_t *__restrict__ rowoff, int r) {
    return it.rmap >= 0 ? rowoff[it.rmap + r] : (int64_t)r * it.ldc;
}

// 16-byte accesses to rows of any 4-byte alignment
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned w4u __attribute__((ext_vector_type(4), aligned(4)));

// Output of a tile of H_eff's stage 1 (EpiDev): its blocks that the W stage
// would only scale and copy go to T2 from here, and to T1 only if another sum
// reads them.  The W stage, at the rate of a copy, loses most of its traffic for
// a look-up a channel here.  W stage and stage 1: 8 x 4 cylinder, m = 1024, 30 ->
// 19 us and 77 -> 81; 24 x 8 FP32, m = 2000, 44 -> 19 and 101 -> 106; tri 12 x 6
// BF16x3, m = 3000, 126 -> 58 and 387 -> 409; 98 channels, m = 4000, 1.61 -> 0.54 ms
// and 5.30 -> 5.51.
// NC columns of a lane (those below N), its rows in ascending order.
template <int NC, typename TD>
struct EpiWriter {
    const int32_t *row;   // of the channel at hand: its first row, the next one's
    const EpiDst *dst;
    TD *out;
    int seg[NC], b[NC], start, end, nseg;
    EpiDst e[NC];
    // row0, dst0: those of the channel that holds the tile's first row
    __device__ __forceinline__ EpiWriter(void *out_, const int32_t *row0, const int32_t *col, const EpiDst *dst0, int nseg_,
                                         const int (&gn)[NC], int N)
        : row(row0), dst(dst0), out(static_cast<TD *>(out_)), nseg(nseg_) {
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            int s = 0;
            if (gn[j] < N)
                while (gn[j] >= col[s + 1]) ++s;
            seg[j] = s;
            b[j] = gn[j] - col[s];
        }
        fetch();
    }
    __device__ __forceinline__ void fetch() {
        start = row[0];
        end = row[1];
#pragma unroll
        for (int j = 0; j < NC; ++j) e[j] = dst[seg[j]];
    }
    __device__ __forceinline__ void seek(int gm) {
        if (gm < end) return;
        do {
            ++row;
            dst += nseg;
        } while (gm >= row[1]);
        fetch();
    }
    // v at row gm (after seek), column j
    template <typename T, typename TC>
    __device__ __forceinline__ void store(int gm, int j, T v, TC *c) const {
        if (e[j].keep) *c = (TC)v;
        if (e[j].off >= 0) {
            const T w = T(0) + (T)e[j].coef * v;   // as a sum of one term
            TD *o = out + e[j].off + (int64_t)(gm - start) * e[j].ld + b[j];
            if constexpr (std::is_same<TD, uint32_t>::value) *o = pack_split(w);
            else *o = (TD)w;
        }
    }
    // four neighbouring columns of one segment
    __device__ __forceinline__ void store4(int gm, const float (&v)[4], float *c) const {
        if (e[0].keep) *reinterpret_cast<f4u *>(c) = f4u{v[0], v[1], v[2], v[3]};
        if (e[0].off >= 0) {
            TD *o = out + e[0].off + (int64_t)(gm - start) * e[0].ld + b[0];
            float w[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) w[j] = 0.0f + (float)e[0].coef * v[j];
            if constexpr (std::is_same<TD, uint32_t>::value)
                *reinterpret_cast<w4u *>(o) = w4u{pack_split(w[0]), pack_split(w[1]), pack_split(w[2]), pack_split(w[3])};
            else
                *reinterpret_cast<f4u *>(o) = f4u{w[0], w[1], w[2], w[3]};
        }
    }
};

// ---------------------------------------------------------------- FP64 / FP32
// LDS tiles are M-major (A) / N-major (B) with the K index contiguous and an
// odd row stride (BK + 1 elements), so the global->LDS stores of either
// operand orientation and the MFMA operand reads (16 lanes = 16 rows, same k)
// spread over the banks.  Two LDS buffers: the next K-step's global loads are
// in flight during the current MFMAs and one barrier separates steps.
template <typename T> struct KStep;
template <> struct KStep<double> { static constexpr int BK = 16; };
template <> struct KStep<float> { static constexpr int BK = 32; };

// KDIV = 2 / 4: a half / quarter of the K step (and LDS) of KStep.  EPI: output
// through EpiWriter, in a kernel of its own so that plain lists keep their
// registers, and held to those of 6 waves a SIMD (4 without the bound: stage 1 of
// the 8 x 4 cylinder 95 us instead of 81).
template <typename T, typename TC, bool TA, bool TB, int BM, int BN, int WGM, int KDIV, bool EPI>
__global__ __launch_bounds__(NT, EPI && KDIV > 1 ? 6 : 1) void gemm_kmajor(Slots slots, const GemmItem *__restrict__ items,
                                                  const GemmSeg *__restrict__ segs,
                                                  const GemmTile *__restrict__ tiles,
                                                  const int64_t *__restrict__ rowoff, int ntiles, EpiDev epi) {
    constexpr int WGN = 4 / WGM;
    constexpr int BK = KStep<T>::BK / KDIV, LDK = BK + 1;
    constexpr int NLA = BM * BK / NT, NLB = BN * BK / NT;   // elements per thread and step
    constexpr int SM = BM / WGM, SN = BN / WGN;              // wave sub-tile
    constexpr int WBM = SM / 16, WBN = SN / 16;              // MFMA blocks per wave
    static_assert(NT % BK == 0 && NT % BM == 0 && NT % BN == 0 && WBM >= 1 && WBN >= 1, "tile shape");
    // the host has placed the tiles in launch order (idle tiles: item < 0)
    if ((int)blockIdx.x >= ntiles) return;
    const GemmTile tile = tiles[blockIdx.x];
    if (tile.item < 0) return;
    const GemmItem it = items[tile.item];
    __shared__ T As[2][BM][LDK];
    __shared__ T Bs[2][BN][LDK];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = (wave / WGN) * SM, wn = (wave % WGN) * SN;
    const int m0 = tile.m0, n0 = tile.n0;
    using V4 = typename Acc<T>::type;
    V4 acc[WBM][WBN];
#pragma unroll
    for (int i = 0; i < WBM; ++i)
#pragma unroll
        for (int j = 0; j < WBN; ++j) acc[i][j] = V4{0, 0, 0, 0};

    // coalesced thread -> element maps: consecutive threads walk the
    // contiguous global index of each operand
    //   A (M x K):  K contiguous (!TA): k = tid % BK, m = tid / BK + u * (NT / BK)
    //               M contiguous (TA):  m = tid % BM, k = tid / BM + u * (NT / BM)
    //   B (K x N):  N contiguous (!TB): n = tid % BN, k = tid / BN + u * (NT / BN)
    //               K contiguous (TB):  k = tid % BK, n = tid / BK + u * (NT / BK)
    auto a_idx = [&](int u, int &m, int &k) {
        if (TA) { m = tid % BM; k = tid / BM + u * (NT / BM); }
        else    { k = tid % BK; m = tid / BK + u * (NT / BK); }
    };
    auto b_idx = [&](int u, int &n, int &k) {
        if (TB) { k = tid % BK; n = tid / BK + u * (NT / BK); }
        else    { n = tid % BN; k = tid / BN + u * (NT / BN); }
    };
    T ra[NLA], rb[NLB];
    int K = 0, lda = 0, ldb = 0;
    __amdgpu_buffer_rsrc_t rA, rB;
    auto set_seg = [&](const GemmSeg &sg) {
        K = __builtin_amdgcn_readfirstlane(sg.K);
        lda = __builtin_amdgcn_readfirstlane(sg.lda);
        ldb = __builtin_amdgcn_readfirstlane(sg.ldb);
        rA = operand_rsrc(static_cast<const T *>(slots.p[sg.a_slot]) + sg.a_off);
        rB = operand_rsrc(static_cast<const T *>(slots.p[sg.b_slot]) + sg.b_off);
    };
    auto load = [&](int k0) {
#pragma unroll
        for (int u = 0; u < NLA; ++u) {
            int m, k;
            a_idx(u, m, k);
            const int gm = m0 + m, gk = k0 + k;
            const unsigned off = TA ? (unsigned)(gk * lda + gm) : (unsigned)(gm * lda + gk);
            ra[u] = buf_load(rA, (gm < it.M && gk < K) ? off * (unsigned)sizeof(T) : kOutOfRange, T());
        }
#pragma unroll
        for (int u = 0; u < NLB; ++u) {
            int n, k;
            b_idx(u, n, k);
            const int gn = n0 + n, gk = k0 + k;
            const unsigned off = TB ? (unsigned)(gn * ldb + gk) : (unsigned)(gk * ldb + gn);
            rb[u] = buf_load(rB, (gn < it.N && gk < K) ? off * (unsigned)sizeof(T) : kOutOfRange, T());
        }
    };
    auto store = [&](int buf) {
#pragma unroll
        for (int u = 0; u < NLA; ++u) {
            int m, k;
            a_idx(u, m, k);
            As[buf][m][k] = ra[u];
        }
#pragma unroll
        for (int u = 0; u < NLB; ++u) {
            int n, k;
            b_idx(u, n, k);
            Bs[buf][n][k] = rb[u];
        }
    };

    int sidx = 0, k0 = 0;
    while (sidx < it.nseg && segs[it.seg0 + sidx].K <= 0) ++sidx;
    int buf = 0;
    if (sidx < it.nseg) {
        set_seg(segs[it.seg0 + sidx]);
        load(0);
        store(0);
    }
    __syncthreads();
    while (sidx < it.nseg) {
        // advance to the next step and prefetch it
        k0 += BK;
        if (k0 >= K) {
            k0 = 0;
            ++sidx;
            while (sidx < it.nseg && segs[it.seg0 + sidx].K <= 0) ++sidx;
            if (sidx < it.nseg) set_seg(segs[it.seg0 + sidx]);
        }
        const bool more = sidx < it.nseg;
        if (more) load(k0);
#pragma unroll
        for (int kk = 0; kk < BK; kk += 4) {
            const int kr = kk + (lane >> 4), c = lane & 15;
            T a[WBM], b[WBN];
#pragma unroll
            for (int i = 0; i < WBM; ++i) a[i] = As[buf][wm + i * 16 + c][kr];
#pragma unroll
            for (int j = 0; j < WBN; ++j) b[j] = Bs[buf][wn + j * 16 + c][kr];
#pragma unroll
            for (int i = 0; i < WBM; ++i)
#pragma unroll
                for (int j = 0; j < WBN; ++j) acc[i][j] = mfma16(a[i], b[j], acc[i][j]);
        }
        if (more) store(buf ^ 1);
        __syncthreads();
        buf ^= 1;
    }
    // Result rows held by (lane, register r): v_mfma_f64_16x16x4 returns row
    // 4 r + lane/16, v_mfma_f32_16x16x4 row 4 (lane/16) + r; column lane % 16.
    constexpr bool kF64 = sizeof(T) == 8;
    TC *C = static_cast<TC *>(const_cast<void *>(slots.p[it.c_slot])) + it.c_off;
    if constexpr (EPI) {
        const EpiItem ei = epi.items[tile.item];
        int gn[WBN];
#pragma unroll
        for (int j = 0; j < WBN; ++j) gn[j] = n0 + wn + j * 16 + (lane & 15);
        EpiWriter<WBN, T> ew(const_cast<void *>(slots.p[epi.slot]), epi.row + ei.row0 + tile.chan, epi.col + ei.col0,
                             epi.dst + ei.dst0 + tile.chan * ei.nseg, ei.nseg, gn, it.N);
#pragma unroll
        for (int i = 0; i < WBM; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int gm = m0 + wm + i * 16 + (kF64 ? r * 4 + (lane >> 4) : (lane >> 4) * 4 + r);
                if (gm >= it.M) continue;
                ew.seek(gm);
#pragma unroll
                for (int j = 0; j < WBN; ++j)
                    if (gn[j] < it.N) ew.store(gm, j, acc[i][j][r], C + (int64_t)gm * it.ldc + gn[j]);
            }
        return;
    }
#pragma unroll
    for (int i = 0; i < WBM; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = kF64 ? r * 4 + (lane >> 4) : (lane >> 4) * 4 + r;
            const int gm = m0 + wm + i * 16 + row;
            if (gm >= it.M) continue;
            TC *Cr = C + c_row(it, rowoff, gm);
#pragma unroll
            for (int j = 0; j < WBN; ++j) {
                const int gn = n0 + wn + j * 16 + (lane & 15);
                if (gn < it.N) Cr[gn] = (TC)acc[i][j][r];
            }
        }
}

// ---------------------------------------------------------------- LDS DMA
// Non-transposed FP32 / FP64 operands (A: K contiguous, B: N contiguous) staged by
// buffer loads that write LDS directly (no register staging), NS stages deep:
// the loads of the next NS - 1 K-steps are in flight while the MFMAs of the
// current one run, and one barrier separates steps.  Each load instruction
// writes 64 consecutive dwords (lane i -> dword i), so the LDS layout follows
// from which element each lane fetches:
//   A stage: groups of 4 FP32 (2 FP64) rows x 16 k (64 dwords, one
//     instruction, whole 64-byte (128-byte) row pieces from global memory),
//     consecutive groups 68 dwords apart;
//   B stage: the 16 x BN tile row-major in 64-dword chunks (one instruction
//     each, whole row pieces), FP32 chunks 64 + 256 / BN dwords apart, FP64
//     chunks unpadded.
// Within a K-step, lane group g (lane / 16) of MFMA s (0..3) takes k = 4 g + s
// (the same permutation of k for A and B, so the sum is unchanged): a lane's
// four A values are adjacent (one 16-byte LDS read in FP32, two in FP64), and
// with the layouts above every LDS read of the MFMA operands touches each
// bank once per cycle (FP32 B reads serve 32 lanes a cycle, across k rows,
// hence the padding; FP64 B reads serve 16 lanes, one k row).
// The loads are written in inline assembly because the compiler, which tracks
// LDS written by its own direct loads, waits for all of them before any LDS
// read and so would drain the pipeline at every step; these loads have no
// register results, and the stage waits below are explicit.  A tile arrives
// as one FlatTile record (one scalar load): with several workgroups starting
// together on a CU, a chain of dependent descriptor loads (tile, item,
// segment) left the CU idle for microseconds at every tile start.
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef float f2v __attribute__((ext_vector_type(2)));

__device__ __forceinline__ u32x4 dma_rsrc(const void *p) {
    const uint64_t a = reinterpret_cast<uint64_t>(p);
    u32x4 r;
    r.x = __builtin_amdgcn_readfirstlane((uint32_t)a);
    r.y = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32)) & 0xffffu;
    r.z = 0x7fffffffu;   // 2 GiB range: offsets >= kOutOfRange read zero
    r.w = 0x00020000u;   // 32-bit data format
    return r;
}

#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
// LDS[lds + 4 lane] = dword at byte offset voff of the buffer (0 if out of range)
__device__ __forceinline__ void dma_dword(u32x4 rsrc, uint32_t lds, uint32_t voff) {
    asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dword %1, %2, 0 offen lds"
                 :: "s"(lds), "v"(voff), "s"(rsrc) : "memory", "m0");
}
#pragma clang diagnostic pop

template <int N> __device__ __forceinline__ void wait_vm() {
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}

// SPLIT (BF16x3): every 4-byte operand word holds a value as two bf16, the
// high part in its low half and the low part in its high half (x = hi + lo);
// the staging is the FP32 kernel's, and each K step of 16 issues three
// v_mfma_f32_16x16x16_bf16 (lo * hi', hi * lo', hi * hi', small terms first)
// in place of four v_mfma_f32_16x16x4_f32.
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
typedef short s4v __attribute__((ext_vector_type(4)));
typedef unsigned u2v __attribute__((ext_vector_type(2)));

__device__ __forceinline__ s4v split_hi(float w0, float w1, float w2, float w3) {
    const unsigned a = __builtin_bit_cast(unsigned, w0), b = __builtin_bit_cast(unsigned, w1);
    const unsigned c = __builtin_bit_cast(unsigned, w2), d = __builtin_bit_cast(unsigned, w3);
    return __builtin_bit_cast(s4v, u2v{(a & 0xffffu) | (b << 16), (c & 0xffffu) | (d << 16)});
}
__device__ __forceinline__ s4v split_lo(float w0, float w1, float w2, float w3) {
    const unsigned a = __builtin_bit_cast(unsigned, w0), b = __builtin_bit_cast(unsigned, w1);
    const unsigned c = __builtin_bit_cast(unsigned, w2), d = __builtin_bit_cast(unsigned, w3);
    return __builtin_bit_cast(s4v, u2v{(a >> 16) | (b & 0xffff0000u), (c >> 16) | (d & 0xffff0000u)});
}

template <typename T, typename TC, int BM, int BN, int WGM, int NS, bool SPLIT = false>
__global__ __launch_bounds__(NT) void gemm_dma(Slots slots, const FlatTile *__restrict__ tiles,
                                               const int64_t *__restrict__ rowoff, int ntiles, EpiDev epi) {
    constexpr int BK = 16;
    constexpr int EW = sizeof(T) / 4;                            // dwords per element
    constexpr int RG = 4 / EW;                                   // rows per A load group (64 dwords)
    constexpr int WGN = 4 / WGM;
    constexpr int SM = BM / WGM, SN = BN / WGN;
    constexpr int WBM = SM / 16, WBN = SN / 16;
    constexpr int AGS = 68, A_DW = (BM / RG) * AGS;              // A: groups of RG rows
    // B: 64-dword chunks of the row-major 16 x BN tile; FP32 reads (32 lanes a
    // cycle, four k rows) need the padding, FP64 reads (16 lanes) do not
    constexpr int PB = EW == 1 ? 256 / BN : 0, BCS = 64 + PB, B_DW = (BK * BN * EW / 64) * BCS;
    constexpr int ST_DW = A_DW + B_DW;                           // one stage, dwords
    constexpr int NA = BM / RG / 4, NB = BK * BN * EW / 256;     // loads per wave and step
    constexpr int NL = NA + NB;
    static_assert(NS >= 2 && NS <= 4 && WBM >= 1 && WBN >= 1 && BN <= 128 && NA >= 1 && NB >= 1 &&
                  (NS - 2) * NL <= 63, "shape");
    static_assert(A_DW % 4 == 0 && ST_DW % 4 == 0, "16-byte aligned A reads");
    using V4 = typename Acc<T>::type;
    __shared__ __attribute__((aligned(16))) float sm[NS * ST_DW];

    if ((int)blockIdx.x >= ntiles) return;
    const FlatTile ft = tiles[blockIdx.x];
    if (ft.M <= 0) return;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = (wave / WGN) * SM, wn = (wave % WGN) * SN;
    const int M = ft.M, N = ft.N, K = ft.K, m0 = ft.m0, n0 = ft.n0;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) float *)sm;
    const u32x4 rA = dma_rsrc(static_cast<const T *>(slots.p[ft.a_slot]) + ft.a_off);
    const u32x4 rB = dma_rsrc(static_cast<const T *>(slots.p[ft.b_slot]) + ft.b_off);
    const int nsteps = K > 0 ? (K + BK - 1) / BK : 0;

    // A load: lane -> row a_r of the group, element a_k of the 16, dword a_h of it
    const int a_r = lane / (16 * EW), a_k = (lane % (16 * EW)) / EW, a_h = lane % EW;
    // per-lane byte offsets of this lane's A rows and B columns (out of range: kOutOfRange)
    uint32_t arow[NA], bcol[NB];
#pragma unroll
    for (int u = 0; u < NA; ++u) {
        const int m = m0 + RG * (wave * NA + u) + a_r;
        arow[u] = m < M ? (uint32_t)m * (uint32_t)ft.lda * (uint32_t)sizeof(T) + 4u * a_h : kOutOfRange;
    }
#pragma unroll
    for (int v = 0; v < NB; ++v) {
        const int f = 64 * (wave * NB + v) + lane;                // dword of the B stage (unpadded)
        const int n = n0 + (f / EW) % BN;
        bcol[v] = n < N ? (uint32_t)n * (uint32_t)sizeof(T) + 4u * (f % EW) : kOutOfRange;
    }
    const uint32_t ldbb = (uint32_t)ft.ldb * (uint32_t)sizeof(T);

    V4 acc[WBM][WBN];
#pragma unroll
    for (int i = 0; i < WBM; ++i)
#pragma unroll
        for (int j = 0; j < WBN; ++j) acc[i][j] = V4{0, 0, 0, 0};

    // step `st` of the K loop into stage buffer st % NS
    auto issue = [&](int st) {
        const uint32_t sa = lds0 + (uint32_t)((st % NS) * ST_DW) * 4u, sb = sa + A_DW * 4u;
        const int k0 = st * BK;
        const int ka = k0 + a_k;
        const bool kav = ka < K;
#pragma unroll
        for (int u = 0; u < NA; ++u)
            dma_dword(rA, sa + (uint32_t)((wave * NA + u) * AGS) * 4u,
                      kav ? arow[u] + (uint32_t)ka * (uint32_t)sizeof(T) : kOutOfRange);
#pragma unroll
        for (int v = 0; v < NB; ++v) {
            const int x = wave * NB + v;                  // chunk of the B stage
            const int kb = k0 + (64 * x + lane) / EW / BN;
            dma_dword(rB, sb + (uint32_t)(x * BCS) * 4u, kb < K ? bcol[v] + (uint32_t)kb * ldbb : kOutOfRange);
        }
    };

    // per-lane LDS read offsets (dwords within a stage)
    const int c = lane & 15, g = lane >> 4;
    int aoff[WBM], boff[WBN][4];
#pragma unroll
    for (int i = 0; i < WBM; ++i) {
        const int r = wm + i * 16 + c;
        aoff[i] = (r / RG) * AGS + (r % RG) * 16 * EW + 4 * g * EW;
    }
#pragma unroll
    for (int j = 0; j < WBN; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            // k = 4 g + q: row-major dword of the 16 x BN tile, plus the padding of its chunk
            const int f = ((4 * g + q) * BN + wn + j * 16 + c) * EW;
            boff[j][q] = A_DW + f + (f >> 6) * PB;
        }

#pragma unroll
    for (int p = 0; p < NS - 1; ++p)
        if (p < nsteps) issue(p);
    for (int s = 0; s < nsteps; ++s) {
        // this wave's loads of step s are done once at most `newer` later steps remain in flight
        const int newer = min(nsteps - s - 1, NS - 2);
        if (NS >= 4 && newer >= 2) wait_vm<2 * NL>();
        else if (NS >= 3 && newer >= 1) wait_vm<NL>();
        else wait_vm<0>();
        __syncthreads();
        if (s + NS - 1 < nsteps) issue(s + NS - 1);
        const float *st = sm + (s % NS) * ST_DW;
        T a[WBM][4], b[WBN][4];
#pragma unroll
        for (int i = 0; i < WBM; ++i) {
            // the lane's four consecutive k of its row: EW 16-byte reads
            const f4 lo = *reinterpret_cast<const f4 *>(st + aoff[i]);
            if constexpr (EW == 1) {
                a[i][0] = lo.x; a[i][1] = lo.y; a[i][2] = lo.z; a[i][3] = lo.w;
            } else {
                const f4 hi = *reinterpret_cast<const f4 *>(st + aoff[i] + 4);
                a[i][0] = __builtin_bit_cast(double, f2v{lo.x, lo.y});
                a[i][1] = __builtin_bit_cast(double, f2v{lo.z, lo.w});
                a[i][2] = __builtin_bit_cast(double, f2v{hi.x, hi.y});
                a[i][3] = __builtin_bit_cast(double, f2v{hi.z, hi.w});
            }
        }
#pragma unroll
        for (int j = 0; j < WBN; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) b[j][q] = *reinterpret_cast<const T *>(st + boff[j][q]);
        if constexpr (SPLIT) {
            // a lane's four words are k = 4 g .. 4 g + 3 of its row (column):
            // exactly the four bf16 of one v_mfma_f32_16x16x16_bf16 operand
            s4v ah[WBM], al[WBM], bh[WBN], bl[WBN];
#pragma unroll
            for (int i = 0; i < WBM; ++i) {
                ah[i] = split_hi(a[i][0], a[i][1], a[i][2], a[i][3]);
                al[i] = split_lo(a[i][0], a[i][1], a[i][2], a[i][3]);
            }
#pragma unroll
            for (int j = 0; j < WBN; ++j) {
                bh[j] = split_hi(b[j][0], b[j][1], b[j][2], b[j][3]);
                bl[j] = split_lo(b[j][0], b[j][1], b[j][2], b[j][3]);
            }
#pragma unroll
            for (int i = 0; i < WBM; ++i)
#pragma unroll
                for (int j = 0; j < WBN; ++j) {
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(al[i], bh[j], acc[i][j], 0, 0, 0);
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(ah[i], bl[j], acc[i][j], 0, 0, 0);
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(ah[i], bh[j], acc[i][j], 0, 0, 0);
                }
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int i = 0; i < WBM; ++i)
#pragma unroll
                    for (int j = 0; j < WBN; ++j) acc[i][j] = mfma16(a[i][q], b[j][q], acc[i][j]);
        }
    }

    // result rows held by (lane, register r): v_mfma_f64_16x16x4 returns row
    // 4 r + lane/16, v_mfma_f32_16x16x4 and v_mfma_f32_16x16x16_bf16 row
    // 4 (lane/16) + r; column lane % 16
    TC *C = static_cast<TC *>(const_cast<void *>(slots.p[ft.c_slot])) + ft.c_off;
    if (epi.items) {
        using TD = typename std::conditional<SPLIT, uint32_t, T>::type;
        int gn[WBN];
#pragma unroll
        for (int j = 0; j < WBN; ++j) gn[j] = n0 + wn + j * 16 + c;
        EpiWriter<WBN, TD> ew(const_cast<void *>(slots.p[epi.slot]), epi.row + ft.erow, epi.col + ft.ecol,
                              epi.dst + ft.edst, ft.eseg, gn, N);
#pragma unroll
        for (int i = 0; i < WBM; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int gm = m0 + wm + i * 16 + (EW == 2 ? r * 4 + (lane >> 4) : (lane >> 4) * 4 + r);
                if (gm >= M) continue;
                ew.seek(gm);
#pragma unroll
                for (int j = 0; j < WBN; ++j)
                    if (gn[j] < N) ew.store(gm, j, acc[i][j][r], C + (int64_t)gm * ft.ldc + gn[j]);
            }
        return;
    }
#pragma unroll
    for (int i = 0; i < WBM; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = EW == 2 ? r * 4 + (lane >> 4) : (lane >> 4) * 4 + r;
            const int gm = m0 + wm + i * 16 + row;
            if (gm >= M) continue;
            TC *Cr = C + (ft.rmap >= 0 ? rowoff[ft.rmap + gm] : (int64_t)gm * ft.ldc);
#pragma unroll
            for (int j = 0; j < WBN; ++j) {
                const int gn = n0 + wn + j * 16 + c;
                if (gn < N) Cr[gn] = (TC)acc[i][j][r];
            }
        }
}

// ---------------------------------------------------------------- FP32 / BF16x3, quads
// Operands of 4-byte words moved 16 bytes a lane all the way: the LDS-DMA kernel
// above spends its vector slots on one-dword loads and reads B a word at a time
// (BF16x3, tri 12 x 6, m = 3000: matrix cores a third busy).  Four waves stacked
// along M, each 16 WBM rows by the tile's 64 columns:
//   A stage: rows of 16 k (64 bytes), chunk c (4 words) at c ^ (row / 4 % 4), so
//     that the 16 rows of an operand read spread over the banks;
//   B stage: rows of 64 columns; a lane reads 4 neighbouring columns of k = 4 g +
//     q, so MFMA column block j holds columns 4 x + j and one read serves four
//     blocks.
// k = 4 g + q in both operands, as in the LDS-DMA kernel.  KS = 2 stages two such
// steps for v_mfma_f32_16x16x32_bf16 (half the issue of the 16-deep one).
//
// A chunk of A that crosses the end of K is cut word by word; loads past the
// last column or row of an operand end within the kQuadPad bytes that the
// caller leaves behind it (those values are cut, or of columns not stored).
typedef unsigned w4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ w4 buf_quad(__amdgpu_buffer_rsrc_t r, unsigned off) {
    return __builtin_bit_cast(w4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
}
// the low (HI: the values' high parts) or high halves of four words
template <bool HI>
__device__ __forceinline__ u2v halves(unsigned a, unsigned b, unsigned c, unsigned d) {
    constexpr unsigned sel = HI ? 0x05040100u : 0x07060302u;
    return u2v{__builtin_amdgcn_perm(b, a, sel), __builtin_amdgcn_perm(d, c, sel)};
}

template <bool SPLIT, int WBM, int KS>
__global__ __launch_bounds__(NT) void gemm_quad(Slots slots, const FlatTile *__restrict__ tiles,
                                                const int64_t *__restrict__ rowoff, int ntiles, EpiDev epi) {
    constexpr int BM = 64 * WBM, BK = 16 * KS, WBN = 4;
    __shared__ w4 As[2][KS][BM * 4];
    __shared__ w4 Bs[2][KS][16 * 16];
    if ((int)blockIdx.x >= ntiles) return;
    const FlatTile ft = tiles[blockIdx.x];
    if (ft.M <= 0) return;
    const int tid = threadIdx.x, lane = tid & 63, r16 = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int M = ft.M, N = ft.N, K = ft.K, m0 = ft.m0, n0 = ft.n0;
    const __amdgpu_buffer_rsrc_t rA = operand_rsrc(static_cast<const float *>(slots.p[ft.a_slot]) + ft.a_off);
    const __amdgpu_buffer_rsrc_t rB = operand_rsrc(static_cast<const float *>(slots.p[ft.b_slot]) + ft.b_off);
    const int nsteps = K > 0 ? (K + BK - 1) / BK : 0;
    // this thread's chunks: A rows tid / 4 + 64 u, words 4 (tid % 4); B row tid / 16, columns 4 (tid % 16)
    const int ac = tid & 3, ar = tid >> 2, bc = tid & 15, bk = tid >> 4;
    unsigned aoff[WBM];
#pragma unroll
    for (int u = 0; u < WBM; ++u) {
        const int m = m0 + ar + 64 * u;
        aoff[u] = m < M ? ((unsigned)m * (unsigned)ft.lda + 4u * ac) * 4u : kOutOfRange;
    }
    const unsigned ldbb = (unsigned)ft.ldb * 4u;
    const unsigned boff = n0 + 4 * bc < N ? (unsigned)(n0 + 4 * bc) * 4u + (unsigned)bk * ldbb : kOutOfRange;
    w4 ra[KS][WBM], rb[KS];
    auto load = [&](int s) {
#pragma unroll
        for (int h = 0; h < KS; ++h) {
            const int k0 = s * BK + 16 * h, ka = k0 + 4 * ac;
#pragma unroll
            for (int u = 0; u < WBM; ++u) {
                ra[h][u] = buf_quad(rA, aoff[u] != kOutOfRange && ka < K ? aoff[u] + (unsigned)k0 * 4u : kOutOfRange);
                if (k0 + 16 > K)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (ka + q >= K) ra[h][u][q] = 0;
            }
            rb[h] = buf_quad(rB, boff != kOutOfRange && k0 + bk < K ? boff + (unsigned)k0 * ldbb : kOutOfRange);
        }
    };
    auto store = [&](int buf) {
#pragma unroll
        for (int h = 0; h < KS; ++h) {
#pragma unroll
            for (int u = 0; u < WBM; ++u) {
                const int r = ar + 64 * u;
                As[buf][h][4 * r + (ac ^ ((r >> 2) & 3))] = ra[h][u];
            }
            Bs[buf][h][tid] = rb[h];
        }
    };
    f4 acc[WBM][WBN];
#pragma unroll
    for (int i = 0; i < WBM; ++i)
#pragma unroll
        for (int j = 0; j < WBN; ++j) acc[i][j] = f4{0, 0, 0, 0};
    if (nsteps > 0) {
        load(0);
        store(0);
    }
    __syncthreads();
    for (int s = 0; s < nsteps; ++s) {
        const int buf = s & 1;
        if (s + 1 < nsteps) load(s + 1);
        w4 a[KS][WBM], b[KS][4];
#pragma unroll
        for (int h = 0; h < KS; ++h) {
#pragma unroll
            for (int i = 0; i < WBM; ++i) {
                const int r = wave * 16 * WBM + 16 * i + r16;
                a[h][i] = As[buf][h][4 * r + (g ^ ((r >> 2) & 3))];
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) b[h][q] = Bs[buf][h][(4 * g + q) * 16 + r16];
        }
        if constexpr (SPLIT) {
            using V = typename std::conditional<KS == 2, bf8, s4v>::type;
            auto pack = [](u2v x, u2v y) {
                if constexpr (KS == 2) return __builtin_bit_cast(bf8, w4{x.x, x.y, y.x, y.y});
                else return __builtin_bit_cast(s4v, x);
            };
            auto mfma = [](V x, V y, f4 c) {
                if constexpr (KS == 2) return __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, y, c, 0, 0, 0);
                else return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(x, y, c, 0, 0, 0);
            };
            V ah[WBM], al[WBM];
#pragma unroll
            for (int i = 0; i < WBM; ++i) {
                const w4 x = a[0][i], y = a[KS - 1][i];
                ah[i] = pack(halves<true>(x.x, x.y, x.z, x.w), halves<true>(y.x, y.y, y.z, y.w));
                al[i] = pack(halves<false>(x.x, x.y, x.z, x.w), halves<false>(y.x, y.y, y.z, y.w));
            }
#pragma unroll
            for (int j = 0; j < WBN; ++j) {
                const V bh = pack(halves<true>(b[0][0][j], b[0][1][j], b[0][2][j], b[0][3][j]),
                                  halves<true>(b[KS - 1][0][j], b[KS - 1][1][j], b[KS - 1][2][j], b[KS - 1][3][j]));
                const V bl = pack(halves<false>(b[0][0][j], b[0][1][j], b[0][2][j], b[0][3][j]),
                                  halves<false>(b[KS - 1][0][j], b[KS - 1][1][j], b[KS - 1][2][j], b[KS - 1][3][j]));
#pragma unroll
                for (int i = 0; i < WBM; ++i) acc[i][j] = mfma(al[i], bh, acc[i][j]);
#pragma unroll
                for (int i = 0; i < WBM; ++i) acc[i][j] = mfma(ah[i], bl, acc[i][j]);
#pragma unroll
                for (int i = 0; i < WBM; ++i) acc[i][j] = mfma(ah[i], bh, acc[i][j]);
            }
        } else {
#pragma unroll
            for (int h = 0; h < KS; ++h)
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int i = 0; i < WBM; ++i)
#pragma unroll
                        for (int j = 0; j < WBN; ++j)
                            acc[i][j] = mfma16(__builtin_bit_cast(float, (unsigned)a[h][i][q]),
                                               __builtin_bit_cast(float, (unsigned)b[h][q][j]), acc[i][j]);
        }
        if (s + 1 < nsteps) store(buf ^ 1);
        __syncthreads();
    }
    // register r of lane l: row 4 (l / 16) + r of the block, column 4 (l % 16) + j of the tile
    float *C = static_cast<float *>(const_cast<void *>(slots.p[ft.c_slot])) + ft.c_off;
    const int mw = m0 + wave * 16 * WBM + 4 * g, nw = n0 + 4 * r16;
    if (epi.items) {
        using TD = typename std::conditional<SPLIT, uint32_t, float>::type;
        int gn[WBN];
#pragma unroll
        for (int j = 0; j < WBN; ++j) gn[j] = nw + j;
        EpiWriter<WBN, TD> ew(const_cast<void *>(slots.p[epi.slot]), epi.row + ft.erow, epi.col + ft.ecol,
                              epi.dst + ft.edst, ft.eseg, gn, N);
        const bool quad = nw + 3 < N && ew.seg[0] == ew.seg[3];
#pragma unroll
        for (int i = 0; i < WBM; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int gm = mw + 16 * i + r;
                if (gm >= M) continue;
                ew.seek(gm);
                float *c = C + (int64_t)gm * ft.ldc + nw;
                const float v[4] = {acc[i][0][r], acc[i][1][r], acc[i][2][r], acc[i][3][r]};
                if (quad) {
                    ew.store4(gm, v, c);
                    continue;
                }
#pragma unroll
                for (int j = 0; j < WBN; ++j)
                    if (gn[j] < N) ew.store(gm, j, v[j], c + j);
            }
        return;
    }
#pragma unroll
    for (int i = 0; i < WBM; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int gm = mw + 16 * i + r;
            if (gm >= M) continue;
            float *c = C + (ft.rmap >= 0 ? rowoff[ft.rmap + gm] : (int64_t)gm * ft.ldc) + nw;
            if (nw + 3 < N) {
                *reinterpret_cast<f4u *>(c) = f4u{acc[i][0][r], acc[i][1][r], acc[i][2][r], acc[i][3][r]};
                continue;
            }
#pragma unroll
            for (int j = 0; j < WBN; ++j)
                if (nw + j < N) c[j] = acc[i][j][r];
        }
}

void launch_gemm_quad(bool split, TileShape shape, const Slots &slots, const FlatTile *tiles, const int64_t *rowoff,
                      const EpiDev &epi, int ntiles, hipStream_t s) {
    if (ntiles <= 0) return;
    const dim3 g(ntiles);
#define PD_QUAD(SP, WBM, KS) \
    hipLaunchKernelGGL((gemm_quad<SP, WBM, KS>), g, dim3(NT), 0, s, slots, tiles, rowoff, ntiles, epi)
    switch (shape) {
        case TileShape::T64x64_Q: if (split) PD_QUAD(true, 1, 1); else PD_QUAD(false, 1, 1); break;
        case TileShape::T128x64_Q: if (split) PD_QUAD(true, 2, 1); else PD_QUAD(false, 2, 1); break;
        case TileShape::T64x64_Q32: if (split) PD_QUAD(true, 1, 2); else PD_QUAD(false, 1, 2); break;
        case TileShape::T128x64_Q32: if (split) PD_QUAD(true, 2, 2); else PD_QUAD(false, 2, 2); break;
        default: break;
    }
#undef PD_QUAD
}

// ---------------------------------------------------------------- FP64, register-direct
// For operands that stream from memory.  Every wave computes a tile of 16 WM x
// 16 WN of its own from operands loaded straight into MFMA registers: no LDS,
// no barriers, so a wave never waits for another.  At the FP64 rate (2048 flops
// in 64 cycles) a 32 x 64 wave tile asks the L1 for 24 bytes a clock and CU,
// which it gives (64); the four waves of a workgroup take neighbouring tiles so
// that it holds what they share, and the tile of a workgroup can be 128 x 128,
// which halves the reads of the LDS kernel's 128 x 32.
//
// A K step is 8: MFMA j takes k = 2 g + j from lane group g in both operands.  A,
// with K contiguous in memory, is loaded 16 bytes a lane (k = 2 g, 2 g + 1 of
// row r16); B, with K strided, gives a lane columns 2 r16, 2 r16 + 1 of a pair
// of MFMA blocks, so the blocks of a pair hold alternate columns.  (Ascending k
// over the lane groups, as the staged kernel has it, costs two lane-row swaps a
// value here, 20 to 30 % of the time.)  Loads are NS - 1 steps ahead; offsets
// out of the operand read zero.  The end of a K not a multiple of 8 is loaded
// value by value (k past the end must not be read: it may hold anything).  In a
// pair that straddles an odd edge the load is moved one value back, so nothing
// past the operand is read.
//
// 42398 x 1564 x 397 (a stage 1 at m = 4000): 63 TFLOP/s with 64 x 64 a wave, 62
// with 32 x 64, 57 with 64 x 32, 48 with 32 x 32; the largest plain product of
// the vendor library on this card reaches 72.
typedef double d2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ d2 buf_load2(__amdgpu_buffer_rsrc_t r, unsigned off) {
    return __builtin_bit_cast(d2, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
}

// One operand of a wave: NB blocks of 16 rows (A: KC, K contiguous) or columns
// (B) from r0 on, n in all, leading dimension ld.
template <bool KC, int NB>
struct Frag64 {
    __amdgpu_buffer_rsrc_t rs;
    unsigned off[KC ? NB : NB / 2];   // of this lane's first value (k = 2 g)
    bool back[KC ? 1 : NB / 2];       // pair load moved one value back
    int r0, n, ld;
    // row of block i, MFMA row x
    static __device__ __forceinline__ int row(int i, int x) { return KC ? 16 * i + x : 32 * (i / 2) + 2 * x + (i & 1); }
    __device__ __forceinline__ void init(const double *p, int r0_, int n_, int ld_, int r16, int g) {
        rs = operand_rsrc(p);
        r0 = r0_;
        n = n_;
        ld = ld_;
        if constexpr (KC) {
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const int m = r0 + 16 * i + r16;
                off[i] = m < n ? (unsigned)(m * ld + 2 * g) * 8u : kOutOfRange;
            }
        } else {
#pragma unroll
            for (int i = 0; i < NB / 2; ++i) {
                const int m = r0 + 32 * i + 2 * r16;
                back[i] = m + 1 == n;
                off[i] = m < n ? (unsigned)(2 * g * ld + m - (back[i] ? 1 : 0)) * 8u : kOutOfRange;
            }
        }
    }
    // values of K step s: v[i][j] is block i at k = 8 s + 2 g + j
    __device__ __forceinline__ void load(int s, double (&v)[NB][2]) const {
        if constexpr (KC) {
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const d2 x = buf_load2(rs, off[i] == kOutOfRange ? kOutOfRange : off[i] + (unsigned)s * 64u);
                v[i][0] = x.x;
                v[i][1] = x.y;
            }
        } else {
            const unsigned o = (unsigned)s * 64u * (unsigned)ld;
#pragma unroll
            for (int i = 0; i < NB / 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const d2 x = buf_load2(rs, off[i] == kOutOfRange ? kOutOfRange : off[i] + o + (unsigned)(j * ld) * 8u);
                    v[2 * i][j] = back[i] ? x.y : x.x;
                    v[2 * i + 1][j] = x.y;   // past the edge if moved back: not stored
                }
        }
    }
    // values of k (k < K, else 0)
    __device__ __forceinline__ void load1(int k, int K, int r16, double (&v)[NB]) const {
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int m = r0 + row(i, r16);
            const unsigned o = KC ? (unsigned)(m * ld + k) : (unsigned)(k * ld + m);
            v[i] = buf_load(rs, (m < n && k < K) ? o * 8u : kOutOfRange, double());
        }
    }
};

// One wave's tile of WM x WN blocks at (m0, n0).
template <int WM, int WN, int NS>
__device__ __forceinline__ void r64_tile(const Slots &slots, const FlatTile &ft, const int64_t *__restrict__ rowoff,
                                         const EpiDev &epi, int m0, int n0, int r16, int g) {
    d4 acc[WM][WN];
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j) acc[i][j] = d4{0, 0, 0, 0};
    using FA = Frag64<true, WM>;
    using FB = Frag64<false, WN>;
    const int K = ft.K;
    FA fa;
    FB fb;
    fa.init(static_cast<const double *>(slots.p[ft.a_slot]) + ft.a_off, m0, ft.M, ft.lda, r16, g);
    fb.init(static_cast<const double *>(slots.p[ft.b_slot]) + ft.b_off, n0, ft.N, ft.ldb, r16, g);
    // a pair has no value to move back to in an operand of one column
    const int ns = ft.N == 1 ? 0 : K / 8;
    double va[NS][WM][2], vb[NS][WN][2];
    auto load = [&](int s, int st) {
        fa.load(s, va[st]);
        fb.load(s, vb[st]);
    };
    auto mul = [&](int st) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int i = 0; i < WM; ++i)
#pragma unroll
                for (int q = 0; q < WN; ++q) acc[i][q] = mfma16(va[st][i][j], vb[st][q][j], acc[i][q]);
    };
    const int kt = 8 * ns;
    double ta[2][WM], tb[2][WN];
    auto load_end = [&](int k) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
            if (k + 4 * h < K) {
                fa.load1(k + 4 * h + g, K, r16, ta[h]);
                fb.load1(k + 4 * h + g, K, r16, tb[h]);
            }
    };
    auto mul_end = [&](int k) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
            if (k + 4 * h < K)
#pragma unroll
                for (int i = 0; i < WM; ++i)
#pragma unroll
                    for (int q = 0; q < WN; ++q) acc[i][q] = mfma16(ta[h][i], tb[h][q], acc[i][q]);
    };
#pragma unroll
    for (int s = 0; s < NS - 1; ++s)
        if (s < ns) load(s, s);
    int s = 0;
    for (; s + 2 * NS - 1 <= ns; s += NS) {   // every load of the round is inside
#pragma unroll
        for (int u = 0; u < NS; ++u) {
            load(s + u + NS - 1, (u + NS - 1) % NS);
            mul(u);
        }
    }
    load_end(kt);   // in flight during the last steps
#pragma unroll
    for (int u = 0; u < 2 * NS - 1; ++u)
        if (s + u < ns) {
            if (s + u + NS - 1 < ns) load(s + u + NS - 1, (u + NS - 1) % NS);
            mul(u % NS);
        }
    mul_end(kt);
    for (int k = kt + 8; k < K; k += 8) {   // an operand of one column: all of K value by value
        load_end(k);
        mul_end(k);
    }
    // v_mfma_f64_16x16x4 result: register r of lane l is row 4 r + l / 16, column l % 16
    double *C = static_cast<double *>(const_cast<void *>(slots.p[ft.c_slot])) + ft.c_off;
    if (epi.items) {
        int gn[WN];
#pragma unroll
        for (int q = 0; q < WN; ++q) gn[q] = n0 + FB::row(q, r16);
        EpiWriter<WN, double> ew(const_cast<void *>(slots.p[epi.slot]), epi.row + ft.erow, epi.col + ft.ecol,
                                 epi.dst + ft.edst, ft.eseg, gn, ft.N);
#pragma unroll
        for (int i = 0; i < WM; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int gm = m0 + FA::row(i, 4 * r + g);
                if (gm >= ft.M) continue;
                ew.seek(gm);
#pragma unroll
                for (int q = 0; q < WN; ++q)
                    if (gn[q] < ft.N) ew.store(gm, q, acc[i][q][r], C + (int64_t)gm * ft.ldc + gn[q]);
            }
        return;
    }
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int gm = m0 + FA::row(i, 4 * r + g);
            if (gm >= ft.M) continue;
            double *Cr = C + (ft.rmap >= 0 ? rowoff[ft.rmap + gm] : (int64_t)gm * ft.ldc);
#pragma unroll
            for (int q = 0; q < WN; ++q) {
                const int gn = n0 + FB::row(q, r16);
                if (gn < ft.N) Cr[gn] = acc[i][q][r];
            }
        }
}

// A wave at the lower or right edge leaves out the blocks (by halves of its
// tile) that lie wholly outside.
template <int WM, int WN, int NS, int WPE>
__global__ __launch_bounds__(NT, WPE) void gemm_r64(Slots slots, const FlatTile *__restrict__ tiles,
                                                    const int64_t *__restrict__ rowoff, int ntiles, EpiDev epi) {
    if ((int)blockIdx.x >= ntiles) return;
    const FlatTile ft = tiles[blockIdx.x];
    const int lane = threadIdx.x & 63, r16 = lane & 15, g = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int m0 = ft.m0 + (w >> 1) * 16 * WM, n0 = ft.n0 + (w & 1) * 16 * WN;
    if (m0 >= ft.M || n0 >= ft.N) return;   // also an idle tile (M = 0)
    if constexpr (WN == 4)
        if (n0 + 32 >= ft.N) {
            r64_tile<WM, 2, NS>(slots, ft, rowoff, epi, m0, n0, r16, g);
            return;
        }
    if constexpr (WM == 4)
        if (m0 + 32 >= ft.M) {
            r64_tile<2, WN, NS>(slots, ft, rowoff, epi, m0, n0, r16, g);
            return;
        }
    r64_tile<WM, WN, NS>(slots, ft, rowoff, epi, m0, n0, r16, g);
}

template <int WM, int WN, int NS, int WPE>
static void dispatch_r64(dim3 g, hipStream_t s, const Slots &sl, const FlatTile *t, const int64_t *ro, const EpiDev &ep, int n) {
    hipLaunchKernelGGL((gemm_r64<WM, WN, NS, WPE>), g, dim3(NT), 0, s, sl, t, ro, n, ep);
}

void launch_gemm_r64(TileShape shape, const Slots &slots, const FlatTile *tiles, const int64_t *rowoff,
                     const EpiDev &epi, int ntiles, hipStream_t s) {
    if (ntiles <= 0) return;
    const dim3 g(ntiles);
    switch (shape) {
        case TileShape::T64x64_R: dispatch_r64<2, 2, 3, 4>(g, s, slots, tiles, rowoff, epi, ntiles); break;
        case TileShape::T128x64_R: dispatch_r64<4, 2, 2, 3>(g, s, slots, tiles, rowoff, epi, ntiles); break;
        case TileShape::T64x128_R: dispatch_r64<2, 4, 2, 3>(g, s, slots, tiles, rowoff, epi, ntiles); break;
        case TileShape::T128x128_R: dispatch_r64<4, 4, 2, 2>(g, s, slots, tiles, rowoff, epi, ntiles); break;
        default: break;
    }
}

struct GemmArgs {
    Slots sl;
    const GemmItem *it;
    const GemmSeg *sg;
    const GemmTile *tl;
    const int64_t *ro;
    EpiDev ep;
    int n;
};

template <typename T, typename TC, int BM, int BN, int WGM, int KDIV>
static void dispatch_shape(bool ta, bool tb, dim3 g, hipStream_t s, const GemmArgs &a) {
    if (a.ep.items)   // H_eff: not transposed
        hipLaunchKernelGGL((gemm_kmajor<T, TC, false, false, BM, BN, WGM, KDIV, true>), g, dim3(NT), 0, s, a.sl, a.it, a.sg, a.tl, a.ro, a.n, a.ep);
    else if (!ta && !tb)
        hipLaunchKernelGGL((gemm_kmajor<T, TC, false, false, BM, BN, WGM, KDIV, false>), g, dim3(NT), 0, s, a.sl, a.it, a.sg, a.tl, a.ro, a.n, a.ep);
    else if (ta && !tb)
        hipLaunchKernelGGL((gemm_kmajor<T, TC, true, false, BM, BN, WGM, KDIV, false>), g, dim3(NT), 0, s, a.sl, a.it, a.sg, a.tl, a.ro, a.n, a.ep);
    else if (!ta && tb)
        hipLaunchKernelGGL((gemm_kmajor<T, TC, false, true, BM, BN, WGM, KDIV, false>), g, dim3(NT), 0, s, a.sl, a.it, a.sg, a.tl, a.ro, a.n, a.ep);
    else
        hipLaunchKernelGGL((gemm_kmajor<T, TC, true, true, BM, BN, WGM, KDIV, false>), g, dim3(NT), 0, s, a.sl, a.it, a.sg, a.tl, a.ro, a.n, a.ep);
}

// Pipeline depth of the LDS-DMA kernel: two stages (loads one K step ahead)
// keep 8 FP32 workgroups of 64 x 64 resident per CU, which measured faster on
// the H_eff GEMMs than three or four stages at lower occupancy.
constexpr int kDmaStages = 2;
template <typename T, typename TC, int BM, int BN, int WGM, bool SPLIT>
static void dispatch_dma(dim3 g, hipStream_t s, const Slots &sl, const FlatTile *t, const int64_t *ro, const EpiDev &ep,
                         int n) {
    hipLaunchKernelGGL((gemm_dma<T, TC, BM, BN, WGM, kDmaStages, SPLIT>), g, dim3(NT), 0, s, sl, t, ro, n, ep);
}
template <typename T, typename TC, bool SPLIT = false>
static void dispatch_dma_shape(TileShape shape, dim3 g, hipStream_t s, const Slots &sl, const FlatTile *t,
                               const int64_t *ro, const EpiDev &ep, int n) {
    switch (shape) {
        case TileShape::T128x32_D: dispatch_dma<T, TC, 128, 32, 4, SPLIT>(g, s, sl, t, ro, ep, n); break;
        case TileShape::T64x64_D: dispatch_dma<T, TC, 64, 64, 2, SPLIT>(g, s, sl, t, ro, ep, n); break;
        case TileShape::T32x128_D: dispatch_dma<T, TC, 32, 128, 1, SPLIT>(g, s, sl, t, ro, ep, n); break;
        default: break;
    }
}

template <typename T, typename TC>
static void dispatch_kmajor(TileShape shape, bool ta, bool tb, dim3 g, hipStream_t s, const GemmArgs &a) {
    switch (shape) {
        case TileShape::T64x64: dispatch_shape<T, TC, 64, 64, 2, 1>(ta, tb, g, s, a); break;
        case TileShape::T128x32: dispatch_shape<T, TC, 128, 32, 4, 1>(ta, tb, g, s, a); break;
        case TileShape::T32x128: dispatch_shape<T, TC, 32, 128, 1, 1>(ta, tb, g, s, a); break;
        case TileShape::T128x128: dispatch_shape<T, TC, 128, 128, 2, 1>(ta, tb, g, s, a); break;
        case TileShape::T64x64_K16: dispatch_shape<T, TC, 64, 64, 2, 2>(ta, tb, g, s, a); break;
        case TileShape::T128x32_K16: dispatch_shape<T, TC, 128, 32, 4, 2>(ta, tb, g, s, a); break;
        // FP64 quarter-depth steps (BK = 4) would leave threads without an
        // element of a 32-wide tile; they run at half depth instead
        case TileShape::T64x64_K8: dispatch_shape<T, TC, 64, 64, 2, sizeof(T) == 8 ? 2 : 4>(ta, tb, g, s, a); break;
        case TileShape::T128x32_K8: dispatch_shape<T, TC, 128, 32, 4, sizeof(T) == 8 ? 2 : 4>(ta, tb, g, s, a); break;
        // LDS-DMA pipeline: FP32 non-transposed operands; otherwise the
        // half-depth kernel of the same tile
        // LDS-DMA shapes run through launch_gemm_flat; lists it cannot take
        // (FP64, transposed operands, several segments per item) run the
        // register-staged kernel of the same tile
        case TileShape::T128x32_D: dispatch_shape<T, TC, 128, 32, 4, 2>(ta, tb, g, s, a); break;
        case TileShape::T64x64_D: dispatch_shape<T, TC, 64, 64, 2, 2>(ta, tb, g, s, a); break;
        case TileShape::T32x128_D: dispatch_shape<T, TC, 32, 128, 1, 1>(ta, tb, g, s, a); break;
        default: break;   // launch_gemm_r64
    }
}

void launch_gemm_flat(GemmPrec prec, TileShape shape, bool c_is_f64, const Slots &slots, const FlatTile *tiles,
                      const int64_t *rowoff, const EpiDev &epi, int ntiles, hipStream_t s) {
    if (ntiles <= 0) return;
    const dim3 g(ntiles);
    if (prec == GemmPrec::F64) dispatch_dma_shape<double, double>(shape, g, s, slots, tiles, rowoff, epi, ntiles);
    else if (prec == GemmPrec::BF16X3 && c_is_f64)
        dispatch_dma_shape<float, double, true>(shape, g, s, slots, tiles, rowoff, epi, ntiles);
    else if (prec == GemmPrec::BF16X3) dispatch_dma_shape<float, float, true>(shape, g, s, slots, tiles, rowoff, epi, ntiles);
    else if (c_is_f64) dispatch_dma_shape<float, double>(shape, g, s, slots, tiles, rowoff, epi, ntiles);
    else dispatch_dma_shape<float, float>(shape, g, s, slots, tiles, rowoff, epi, ntiles);
}

void launch_gemm(GemmPrec prec, TileShape shape, bool ta, bool tb, bool c_is_f64, const Slots &slots,
                 const GemmItem *items, const GemmSeg *segs, const GemmTile *tiles, const int64_t *rowoff,
                 const EpiDev &epi, int ntiles, hipStream_t s) {
    if (ntiles <= 0) return;
    dim3 grid(ntiles);
    const GemmArgs a{slots, items, segs, tiles, rowoff, epi, ntiles};
    switch (prec) {
        case GemmPrec::F64:
            dispatch_kmajor<double, double>(shape, ta, tb, grid, s, a);
            break;
        case GemmPrec::F32:
            if (c_is_f64) dispatch_kmajor<float, double>(shape, ta, tb, grid, s, a);
            else dispatch_kmajor<float, float>(shape, ta, tb, grid, s, a);
            break;
        case GemmPrec::BF16X3:   // split operands: LDS-DMA lists only (launch_gemm_flat)
            break;
    }
}

}  // namespace pdmrg
