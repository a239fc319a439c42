// Device side of the skinny "gather rows -> MFMA GEMM -> scatter rows": row
// bookkeeping, output addressing and the small-M kernel body, shared by the
// GEMM kernels and the fused step kernel.  Internal to the library.
#pragma once

#include "common.hpp"
#include "gemm.hpp"

namespace ps {
namespace {

constexpr int kGemmBlock = 256;
constexpr int kSmallWaves = 4;    // gemm_small_kernel: waves per workgroup
constexpr int kSmallBlock = kSmallWaves * 64;

// Row bookkeeping --------------------------------------------------------------
// Refresh mode: sequence b owns rows [b*R, (b+1)*R), R = k_max + block_len:
// its first count_b rows are its stale positions, the last block_len rows
// its active block; rows in between (count_b < k_max) map to nothing.  A
// fixed stride costs no prefix over the counts, so a row's position is one
// load away.  Block-rows mode: row m is position block_start + m % block_len
// of sequence m / block_len.
__device__ __forceinline__ int gemm_rows_total(const GemmArgs& g) {
    return g.batch * (g.mode == kGemmRefresh ? g.k_max + g.block_len : g.block_len);
}

// Row m -> (sequence, position); b = -1 when the row maps to nothing.
__device__ __forceinline__ void map_row(const GemmArgs& g, int m, int& b, int& pos) {
    b = -1;
    pos = 0;
    if (m < 0 || m >= gemm_rows_total(g)) return;
    if (g.mode == kGemmBlockRows) {
        b = m / g.block_len;
        pos = g.block_start + (m - b * g.block_len);
        return;
    }
    const int R = g.k_max + g.block_len;
    const int sb = m / R;
    const int local = m - sb * R;
    if (local >= g.k_max) {
        b = sb;
        pos = g.block_start + (local - g.k_max);
        return;
    }
    int c = g.stale_count[sb];
    const int p = g.stale_idx[static_cast<size_t>(sb) * g.k_max + local];
    c = c < 0 ? 0 : (c > g.k_max ? g.k_max : c);
    if (local >= c || p < 0 || p >= g.seq) return;   // unused slot or out-of-range entry: refresh nothing
    b = sb;
    pos = p;
}

template <bool BF16>
__device__ __forceinline__ void store_elem(char* p, float v) {
    if constexpr (BF16) *reinterpret_cast<uint16_t*>(p) = static_cast<uint16_t>(f32_to_bf16_bits(v));
    else *reinterpret_cast<float*>(p) = v;
}

// Destination of output element (row with sequence b / position pos / row
// number m, column n).
template <bool BF16>
__device__ __forceinline__ char* out_ptr(const GemmArgs& g, int b, int pos, int m, int n) {
    constexpr size_t es = Elem<BF16>::kBytes;
    if (g.mode == kGemmBlockRows)
        return g.out0 + (static_cast<size_t>(m) * g.N + n) * es;
    const size_t row = static_cast<size_t>(b) * g.seq + pos;
    if (n < g.n0) return g.out0 + (row * g.n0 + n) * es;
    return g.out1 + (row * (g.N - g.n0) + (n - g.n0)) * es;
}
template <bool BF16>
__device__ __forceinline__ char* out_ptr(const QkvGemmArgs& g, int b, int pos, int m, int n) {
    constexpr size_t es = Elem<BF16>::kBytes;
    const size_t row = static_cast<size_t>(b) * g.seq + pos;
    if (n < g.n0) return g.out0 + (row * g.n0 + n) * es;
    if (n < g.n1) return g.out1 + (row * (g.n1 - g.n0) + (n - g.n0)) * es;
    return g.out2 + (static_cast<size_t>(m) * (g.N - g.n1) + (n - g.n1)) * es;
}

// 8 consecutive fp32 values -> destination (16-byte bf16 or 2x16-byte fp32 store).
template <bool BF16>
__device__ __forceinline__ void store8(char* dst, const float* v) {
    if constexpr (BF16) {
        st16(dst, make_uint4(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]),
                             pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7])));
    } else {
        st16(dst, make_uint4(__float_as_uint(v[0]), __float_as_uint(v[1]),
                             __float_as_uint(v[2]), __float_as_uint(v[3])));
        st16(dst + 16, make_uint4(__float_as_uint(v[4]), __float_as_uint(v[5]),
                                  __float_as_uint(v[6]), __float_as_uint(v[7])));
    }
}

// Weight row of output column n (nullptr past N).
__device__ __forceinline__ const char* weight_row(const GemmArgs& g, int n, int es) {
    if (n >= g.N) return nullptr;
    if (n < g.n0) return g.w0 + static_cast<size_t>(n) * g.K * es;
    return g.w1 + static_cast<size_t>(n - g.n0) * g.K * es;
}
__device__ __forceinline__ const char* weight_row(const QkvGemmArgs& g, int n, int es) {
    if (n >= g.N) return nullptr;
    if (n < g.n0) return g.w0 + static_cast<size_t>(n) * g.K * es;
    if (n >= g.n1) return g.w2 + static_cast<size_t>(n - g.n1) * g.K * es;
    return g.w1 + static_cast<size_t>(n - g.n0) * g.K * es;
}

// ---------------------------------------------------------------------------
// gemm_small_kernel: at most 16*MT rows, 16 columns per workgroup, the 4
// waves take super-steps w, w+4, w+8, ... of K and are summed in LDS.
// ---------------------------------------------------------------------------

template <bool BF16, int MT, class G>
__device__ __forceinline__ void small_body(const G& g, int bx, int by) {
    using T = Elem<BF16>;
    constexpr int ES = T::kBytes;
    constexpr int BM = MT * 16;
    __shared__ int rowb[BM], rowp[BM];
    __shared__ float red[kSmallWaves][BM][17];

    const int t = threadIdx.x;
    const int lane = t & 63;
    const int w = t >> 6;
    const int col0 = bx * 16;
    const int m0 = by * BM;
    const int kcol = (lane >> 4) * 16;   // lane group g reads bytes 16g + 64s: 64 contiguous bytes of a row per load
    const int nsteps = g.K / (256 / ES);
    // wave w: super-steps w, w+W, ...; the last one it owns is slast
    // (prefetches past it re-read slast and are ignored).
    constexpr int W = kSmallWaves;
    const int nmine = w < nsteps ? (nsteps - 1 - w) / W + 1 : 0;
    const int slast = w < nsteps ? w + W * (nmine - 1) : 0;

    // Weight row of column col0 + lane%16 (past N: row 0, never stored); its
    // first two super-steps are requested before the row bookkeeping.
    const char* brow = weight_row(g, col0 + (lane & 15), ES);
    if (!brow) brow = g.w0;
    auto load_b = [&](int step, uint4 (&rb)[4]) {
#pragma unroll
        for (int s = 0; s < 4; ++s) rb[s] = ld16(brow + step * 256 + 64 * s + kcol);
    };
    uint4 q0[4], q1[4], q2[4];
    load_b(min(w, slast), q0);
    load_b(min(w + W, slast), q1);

    if (m0 >= gemm_rows_total(g)) return;
    if (t < BM) {
        int b, pos;
        map_row(g, m0 + t, b, pos);
        rowb[t] = b;
        rowp[t] = pos;
    }
    __syncthreads();

    // Rows past the end read row 0 and are never stored.
    const char* arow[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const int r = mt * 16 + (lane & 15);
        const int b = rowb[r];
        arow[mt] = b >= 0 ? g.x + (static_cast<size_t>(b) * g.seq + rowp[r]) * g.K * ES : g.x;
    }
    auto load_a = [&](int step, uint4 (&ra)[MT][4]) {
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) ra[mt][s] = ld16(arow[mt] + step * 256 + 64 * s + kcol);
    };
    floatx4 acc[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[mt] = floatx4{0.f, 0.f, 0.f, 0.f};
    auto compute = [&](const uint4 (&ra)[MT][4], const uint4 (&rb)[4]) {
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) acc[mt] = Mma<BF16>::step(ra[mt][s], rb[s], acc[mt]);
    };

    uint4 a0[MT][4], a1[MT][4], a2[MT][4];
    load_a(min(w, slast), a0);
    load_a(min(w + W, slast), a1);
#define PS_SMALL_STEP(I, A_USE, B_USE, A_LOAD, B_LOAD)                      \
    {                                                                       \
        __builtin_amdgcn_sched_barrier(0);                                  \
        load_a(min(w + W * ((I) + 2), slast), A_LOAD);                      \
        load_b(min(w + W * ((I) + 2), slast), B_LOAD);                      \
        __builtin_amdgcn_sched_barrier(0);                                  \
        compute(A_USE, B_USE);                                              \
    }
    int ic = 0;
    for (; ic + 3 <= nmine; ic += 3) {
        PS_SMALL_STEP(ic, a0, q0, a2, q2)
        PS_SMALL_STEP(ic + 1, a1, q1, a0, q0)
        PS_SMALL_STEP(ic + 2, a2, q2, a1, q1)
    }
    if (ic < nmine) PS_SMALL_STEP(ic, a0, q0, a2, q2)
    if (ic + 1 < nmine) PS_SMALL_STEP(ic + 1, a1, q1, a0, q0)
#undef PS_SMALL_STEP

    // sum the waves in order: lane holds rows mt*16 + 4*(lane/16) + i, column lane%16
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int i = 0; i < 4; ++i) red[w][mt * 16 + 4 * (lane >> 4) + i][lane & 15] = acc[mt][i];
    __syncthreads();
    // thread -> (row r, 8 columns c)
    for (int idx = t; idx < BM * 2; idx += kSmallBlock) {
        const int r = idx >> 1, c = (idx & 1) * 8;
        const int b = rowb[r];
        const int n = col0 + c;
        if (b < 0 || n >= g.N) continue;
        float v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            float acc_j = red[0][r][c + j];
#pragma unroll
            for (int q = 1; q < kSmallWaves; ++q) acc_j += red[q][r][c + j];
            v[j] = acc_j;
        }
        store8<BF16>(out_ptr<BF16>(g, b, rowp[r], m0 + r, n), v);
    }
}

constexpr int kMaxSplit = 8;      // largest split-K factor of a plan

// ---------------------------------------------------------------------------
// dma_body (gemm_dma_kernel, and the fused step's Q projection): BM = 16*MT rows (one row tile) x 128 columns; wave w owns
// columns 32w..32w+31 as two 16-column tiles of v_mfma_f32_16x16x32_bf16.
// ---------------------------------------------------------------------------

constexpr int kDmaStage = 128;               // bytes of each row per stage
constexpr int kDmaMaxRowTiles = 10;          // 160 rows
// One 16-byte global -> LDS transfer per lane (the wave's lanes land
// contiguously from lds_base).  A plain device function, so the builtin never
// appears in a kernel template's host-side instantiation.
__device__ __forceinline__ void dma16(const void* src, void* lds_base) {
    __builtin_amdgcn_global_load_lds(src, (__attribute__((address_space(3))) void*)lds_base, 16, 0, 0);
}
// The same transfer marked non-temporal (cache policy nt): for weights that a
// single row tile reads once.
__device__ __forceinline__ void dma16_nt(const void* src, void* lds_base) {
    __builtin_amdgcn_global_load_lds(src, (__attribute__((address_space(3))) void*)lds_base, 16, 0, 2);
}

// s_waitcnt immediates (gfx9 encoding: vmcnt in bits 3:0 and 15:14, expcnt
// 6:4, lgkmcnt 11:8): wait until at most n vector-memory operations of this
// wave are outstanding / until its LDS reads are done.
constexpr int wait_vm(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8); }
constexpr int kWaitLgkm0 = 15 | (3 << 14) | (7 << 4);

// LDS offset of 16-byte chunk c of row r in a stage (rows of kDmaStage bytes).
__device__ __forceinline__ int dma_swz(int r, int c) { return r * kDmaStage + ((c ^ ((r >> 1) & 7)) << 4); }

// NS: LDS slots per operand (4: three stages in flight; 3: two, for a
// workgroup that must share its compute unit).  NTW: the plan has one row
// tile, so every weight byte is read once and its DMA is marked non-temporal
// (a compile-time choice: a branch inside the unrolled stage loop costs more
// than the hint saves).  REG: the operands go through registers instead of
// global -> LDS transfers (below); taken for row tiles of at most 64 rows,
// where it made the batch-1 Q projection 13.8 -> 13.3 us, while the 144- and
// 160-row refreshes ran 27.5 -> 31.1 and 25.4 -> 28.0 us with it.
template <bool BF16, int MT, int NST, int NS = 4, bool NTW = false, bool REG = (MT <= 4), class G>
__device__ __forceinline__ void dma_body(const G& g, int blk) {
    static_assert(NS == 3 || NS == 4, "three or four LDS slots");
    using T = Elem<BF16>;
    constexpr int ES = T::kBytes;
    constexpr int BM = MT * 16;
    constexpr int BN = 128;
    constexpr int ASZ = BM * kDmaStage, BSZ = BN * kDmaStage;
    constexpr int AG = BM / 8;                          // 8-row groups of A per stage (one DMA instruction each)
    constexpr int AIW = (AG + 3) / 4;                   // per wave (surplus ones repeat the last group)
    constexpr int NDMA = 4 + AIW;                       // DMA instructions per wave per stage
    static_assert(2 * NDMA <= 63, "outstanding DMA must fit the vmcnt counter");
    // one LDS object per slot and operand: the compiler can tell them apart
    __shared__ __align__(16) char sa0[ASZ], sa1[ASZ], sa2[REG ? 16 : ASZ], sa3[NS == 4 && !REG ? ASZ : 16];
    __shared__ __align__(16) char sb0[BSZ], sb1[BSZ], sb2[REG ? 16 : BSZ], sb3[NS == 4 && !REG ? BSZ : 16];
    __shared__ __align__(16) int rowb[BM];
    __shared__ int rowp[BM];

    const int tile = blk / g.ksplit;
    const int split = blk - tile * g.ksplit;
    const int col_tile = tile % g.col_tiles;
    const int m0 = (tile / g.col_tiles) * BM;           // one or two row tiles
    const int t = threadIdx.x;
    const int lane = t & 63;
    const int w = t >> 6;
    const int s0b = split * g.steps_per_split * 256;    // byte offset of the split in a row
    constexpr int nst_here = NST;                       // 128-byte stages of every split (the plan divides K evenly)

    // weights: wave w moves rows 32w + 8i + l/8 (i < 4) of the tile's 128
    // columns; lane l fills slot l%8 of its row
    const char* bsrc[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = 32 * w + 8 * i + (lane >> 3);
        const char* row = weight_row(g, col_tile * BN + r, ES);
        bsrc[i] = (row ? row : g.w0) + s0b + (((lane & 7) ^ ((r >> 1) & 7)) << 4);
    }
    auto issue_b = [&](int st, char* buf) {
        const int off = min(st, nst_here - 1) * kDmaStage;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if constexpr (NTW) dma16_nt(bsrc[i] + off, buf + (32 * w + 8 * i) * kDmaStage);
            else dma16(bsrc[i] + off, buf + (32 * w + 8 * i) * kDmaStage);
        }
    };
    // Row bookkeeping (one load per row); the first workgroup publishes the
    // map for the split-K reduction.
    int rb_ = -1, rp_ = 0;
    if (t < BM) map_row(g, m0 + t, rb_, rp_);
    if (t < BM) {
        rowb[t] = rb_;
        rowp[t] = rp_;
        if (g.ksplit > 1 && split == 0 && col_tile == 0 && m0 + t < g.m_max)
            *reinterpret_cast<int2*>(g.rowmap + 2 * (m0 + t)) = make_int2(rb_, rp_);
    }
    if (!__syncthreads_or(rb_ >= 0)) return;            // no row of this tile maps anywhere (uniform)
    // input rows: wave w moves groups w, w + 4, ... (8 rows each); rows that
    // map to nothing read row 0 and are never stored
    const char* asrc[AIW];
#pragma unroll
    for (int i = 0; i < AIW; ++i) {
        const int r = 8 * min(w + 4 * i, AG - 1) + (lane >> 3);
        const int b = rowb[r];
        const char* row = b >= 0 ? g.x + (static_cast<size_t>(b) * g.seq + rowp[r]) * g.K * ES : g.x;
        asrc[i] = row + s0b + (((lane & 7) ^ ((r >> 1) & 7)) << 4);
    }
    auto issue_a = [&](int st, char* buf) {
        const int off = min(st, nst_here - 1) * kDmaStage;
#pragma unroll
        for (int i = 0; i < AIW; ++i)
            dma16(asrc[i] + off, buf + 8 * min(w + 4 * i, AG - 1) * kDmaStage);
    };
    floatx4 acc[2][MT];
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int i = 0; i < MT; ++i) acc[c][i] = floatx4{0.f, 0.f, 0.f, 0.f};
    // a stage is two 64-byte pieces; lane l reads chunk 4p + l/16 of rows
    // 16mt + l%16 (A) and 32w + 16c + l%16 (B)
    auto compute = [&](const char* abuf, const char* bbuf) {
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int c = 4 * p + (lane >> 4);
            const uint4 bf0 = *reinterpret_cast<const uint4*>(bbuf + dma_swz(32 * w + (lane & 15), c));
            const uint4 bf1 = *reinterpret_cast<const uint4*>(bbuf + dma_swz(32 * w + 16 + (lane & 15), c));
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const uint4 af = *reinterpret_cast<const uint4*>(abuf + dma_swz(16 * mt + (lane & 15), c));
                acc[0][mt] = Mma<BF16>::step(af, bf0, acc[0][mt]);
                acc[1][mt] = Mma<BF16>::step(af, bf1, acc[1][mt]);
            }
        }
    };
    if constexpr (!REG) {
        issue_b(0, sb0);
        issue_a(0, sa0);
        issue_b(1, sb1);
        issue_a(1, sa1);
        if constexpr (NS == 4) {
            issue_b(2, sb2);
            issue_a(2, sa2);
        }

        // Stage s: wait for this wave's DMA of stage s and its own earlier LDS
        // reads; barrier (stage s is in LDS for every wave, and the slot of stage
        // s-1 is free); issue stage s+NS-1 into that slot; compute stage s.
        // Issue order (NS = 4) B0 A0 B1 A1 B2 A2 | B3 A3 | ...: the wait leaves
        // exactly the NS-2 newer stages outstanding.  Stages past the split
        // re-read its last stage, so every stage issues the same DMA count.
    #define PS_DMA_STEP(S, WAIT, AUSE, BUSE, ANEXT, BNEXT)                      \
        {                                                                       \
            __builtin_amdgcn_s_waitcnt(WAIT);                                   \
            __builtin_amdgcn_s_waitcnt(kWaitLgkm0);                             \
            __builtin_amdgcn_s_barrier();                                       \
            issue_b((S) + NS - 1, BNEXT);                                       \
            issue_a((S) + NS - 1, ANEXT);                                       \
            compute(AUSE, BUSE);                                                \
        }
        constexpr int WS = wait_vm((NS - 2) * NDMA);        // after stage s: stages s+1 .. s+NS-2
        char* const sa[4] = {sa0, sa1, sa2, sa3};
        char* const sb[4] = {sb0, sb1, sb2, sb3};
        // fully unrolled: every slot index is a constant and the compiler sees the
        // whole issue order (a loop would make it drain the DMA at the loop head)
    #pragma unroll
        for (int st = 0; st < NST; ++st)
            PS_DMA_STEP(st, WS, sa[st % NS], sb[st % NS], sa[(st + NS - 1) % NS], sb[(st + NS - 1) % NS])
    #undef PS_DMA_STEP
        __builtin_amdgcn_s_waitcnt(0);                      // the re-read tail DMA lands before the workgroup ends
    } else {
        // Register staging: each stage's chunks are loaded into registers P
        // stages ahead and written to the same LDS positions the DMA fills
        // (lane l of an instruction at base + 16 l), into two LDS slots.
        // Plain loads stream faster than global -> LDS transfers (a probe
        // with the batch-8 Q projection's addresses and no arithmetic: 14.4
        // against 18.4 us, 9.1 against 13.4 us when the data is in L2), but
        // the stores to LDS cost the large tiles more than that.  Iteration
        // s: compute slot s%2; wait for stage s+1's registers, write them to
        // slot (s+1)%2 (computed an iteration back), load stage s+1+P into
        // the freed set; barrier.  Stages past the split re-read its last
        // stage, so every iteration issues the same load count.
        constexpr int P = 3;
        static_assert(P * NDMA <= 63, "outstanding loads must fit the vmcnt counter");
        uint4 rs[P][NDMA];
        auto load_stage = [&](int st, uint4 (&r)[NDMA]) {
            const int off = min(st, nst_here - 1) * kDmaStage;
#pragma unroll
            for (int i = 0; i < 4; ++i) r[i] = NTW ? ld16_nt(bsrc[i] + off) : ld16(bsrc[i] + off);
#pragma unroll
            for (int i = 0; i < AIW; ++i) r[4 + i] = ld16(asrc[i] + off);
        };
        auto store_stage = [&](const uint4 (&r)[NDMA], char* abuf, char* bbuf) {
#pragma unroll
            for (int i = 0; i < 4; ++i) st16(bbuf + (32 * w + 8 * i) * kDmaStage + 16 * lane, r[i]);
#pragma unroll
            for (int i = 0; i < AIW; ++i)
                if (AG % 4 == 0 || w + 4 * i < AG)   // surplus instructions repeat the last group: no store
                    st16(abuf + 8 * (w + 4 * i) * kDmaStage + 16 * lane, r[4 + i]);
        };
#pragma unroll
        for (int j = 0; j < P; ++j) load_stage(j, rs[j]);
        __builtin_amdgcn_s_waitcnt(wait_vm((P - 1) * NDMA));
        store_stage(rs[0], sa0, sb0);
        load_stage(P, rs[0]);
        __syncthreads();
        constexpr int WR = wait_vm((P - 1) * NDMA);     // stages s+2 .. s+P stay in flight
#pragma unroll
        for (int st = 0; st < NST; ++st) {
            compute(st % 2 ? sa1 : sa0, st % 2 ? sb1 : sb0);
            if (st + 1 < NST) {
                __builtin_amdgcn_s_waitcnt(WR);
                store_stage(rs[(st + 1) % P], (st + 1) % 2 ? sa1 : sa0, (st + 1) % 2 ? sb1 : sb0);
                load_stage(st + 1 + P, rs[(st + 1) % P]);
            }
            __syncthreads();
        }
        __builtin_amdgcn_s_waitcnt(0);                  // the re-read tail loads land before the workgroup ends
    }

    // results straight from registers: register i of acc[c][mt] is row
    // 16mt + 4(l/16) + i, column 32w + 16c + l%16.  Split K (the usual case):
    // fp32 partials, the lane's four row flags read once per row tile.
    if (g.ksplit > 1) {
        float* part = g.ws + (static_cast<size_t>(split) * g.col_tiles + col_tile) * g.m_max * BN +
                      32 * w + (lane & 15);
        const bool c0 = col_tile * BN + 32 * w + (lane & 15) < g.N;
        const bool c1 = col_tile * BN + 32 * w + 16 + (lane & 15) < g.N;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const int r0 = 16 * mt + 4 * (lane >> 4);
            const int4 rb4 = *reinterpret_cast<const int4*>(&rowb[r0]);
            const int rv[4] = {rb4.x, rb4.y, rb4.z, rb4.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float* dst = part + static_cast<size_t>(m0 + r0 + i) * BN;
                if (rv[i] >= 0 && c0) dst[0] = acc[0][mt][i];
                if (rv[i] >= 0 && c1) dst[16] = acc[1][mt][i];
            }
        }
        return;
    }
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const int n = col_tile * BN + 32 * w + 16 * c + (lane & 15);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int r = 16 * mt + 4 * (lane >> 4) + i;
                const int b = rowb[r];
                if (b >= 0 && n < g.N) store_elem<BF16>(out_ptr<BF16>(g, b, rowp[r], m0 + r, n), acc[c][mt][i]);
            }
    }
}


// ---------------------------------------------------------------------------
// tile_body (gemm_tile_kernel, and the fused step's refresh): 64 to 256 rows x
// 128 to 256 columns of outputs per workgroup (the refresh of a whole batch,
// the dense rows of a stack).
//
// Eight waves, two per SIMD, in a 2 x 4 grid of blocks of MI x NJ tiles of
// v_mfma_f32_16x16x32_bf16; K in tiles of 64 (128 bytes of each row: whole
// cache lines), both operands by DMA into two LDS slots, one barrier per K
// tile.  What bounds it is the matrix pipe, and what that waits for:
//  - two waves per SIMD, so one wave's MFMAs run while the other waits for LDS
//    or the barrier, and the LDS fragment reads of eight waves reach twice the
//    rate of four;
//  - fragments are read one phase ahead of the MFMAs that use them (a phase is
//    a quarter of the wave's block, or a whole 32-k step for the smaller
//    blocks, whose registers hold two steps);
//  - the DMA instructions of a K tile are spread two per phase: issued in one
//    burst behind the barrier they fill the address unit's queue and the
//    waves' next MFMAs wait behind them (12288 x 8192 x 4096: 613 us in one
//    burst, 581 us spread).
// The 32x32x16 form measured 15% slower in the same loop, more barriers per K
// tile with finer slots 7-15% slower, 64-byte stages in four slots 7% slower.
// 256 x 256 tiles, 12288 x 8192 x 4096: 566 us, 1.46 PFLOP/s; a four-wave
// kernel of 32x32x16 tiles with 64-byte stages took 728 us, 1.13 PFLOP/s.
// Smaller tiles have three or four slots: with two, a K tile's DMA had to land
// within the short time of one K tile (128 x 128 tiles, 512 x 8192 x 4096: 52.7
// us with two slots and two workgroups per CU, 40.1 us with four slots).
// ---------------------------------------------------------------------------

constexpr int kTileStage = 128;                // bytes of each row per K tile (64 bf16)
constexpr int kTileGroupRows = 4;              // row tiles per band of the launch order
constexpr int kTileThreads = 512;              // eight waves, two per SIMD

// Workgroup blk -> (split, row tile, column tile).  Consecutive workgroups go
// to different XCDs, so the ids are first regrouped per XCD (XCD e takes a
// contiguous run of them, the first nb % 8 XCDs one more); each XCD then
// walks bands of kTileGroupRows row tiles column by column, which keeps the
// input rows and weight rows its compute units share in its own L2.  (The
// tile workgroups must be the first ones of their launch.)
// False for a workgroup past the last tile (fewer row tiles than launched for).
__device__ __forceinline__ bool tile_coords(const GemmArgs& g, int row_tiles, int bn, int blk, int& split, int& rt,
                                            int& ct) {
    const int ntc = (g.N + bn - 1) / bn;
    const int ntiles = row_tiles * ntc;
    const int nb = ntiles * g.ksplit;
    if (blk >= nb) return false;
    const int xcd = blk & 7;
    const int bid = xcd * (nb >> 3) + min(xcd, nb & 7) + (blk >> 3);
    split = bid / ntiles;
    const int tl = bid - split * ntiles;
    const int band = tl / (kTileGroupRows * ntc);
    const int rows_here = min(kTileGroupRows, row_tiles - band * kTileGroupRows);
    const int in = tl - band * kTileGroupRows * ntc;
    ct = in / rows_here;
    rt = band * kTileGroupRows + (in - ct * rows_here);
    return true;
}

// What a tile's rows are: the plan's (map_row) ...
template <class G>
struct PlanRows {
    const G& g;
    __device__ __forceinline__ int tiles(int) const { return g.row_tiles; }
    __device__ __forceinline__ void map(int m, int& b, int& pos) const { map_row(g, m, b, pos); }
};

// ... or packed: the lists' used entries alone (refresh mode without a block),
// one sequence after the other.
struct PackedRows {
    const GemmArgs& g;
    const int* first;      // [batch + 1] rows before each sequence's, and in all
    int total;
    __device__ __forceinline__ int tiles(int bm) const { return (total + bm - 1) / bm; }
    // b = -1 past the last row and for entries outside the sequence
    __device__ __forceinline__ void map(int m, int& b, int& pos) const {
        b = -1;
        pos = 0;
        if (m >= total) return;
        int lo = 0, hi = g.batch;                        // first[lo] <= m < first[hi]
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (first[mid] <= m) lo = mid;
            else hi = mid;
        }
        const int p = g.stale_idx[static_cast<size_t>(lo) * g.k_max + (m - first[lo])];
        if (p < 0 || p >= g.seq) return;
        b = lo;
        pos = p;
    }
};

// The running sum of the lists' counts into first[]; returns the total.  Every
// wave scans (one load, no barrier between), the first one stores.
__device__ __forceinline__ int packed_rows(const GemmArgs& g, int* first) {
    const int lane = threadIdx.x & 63;
    int total = 0;
    for (int b0 = 0; b0 < g.batch; b0 += kWave) {
        const int b = b0 + lane;
        const int c = b < g.batch ? min(max(g.stale_count[b], 0), g.k_max) : 0;
        const int incl = wave_incl_scan(c, lane);
        if (threadIdx.x < kWave && b < g.batch) first[b] = total + incl - c;
        total += __builtin_amdgcn_readlane(incl, kWave - 1);
    }
    if (threadIdx.x == 0) first[g.batch] = total;
    __syncthreads();
    return total;
}

// LDS slots per operand of a tile shape: as many as fit 150 KB, two to maxns.
constexpr int tile_slots(int mi, int nj, int maxns = 4) {
    const int slot = (32 * mi + 64 * nj) * kTileStage;
    return maxns >= 4 && 4 * slot <= 150 * 1024 ? 4 : maxns >= 3 && 3 * slot <= 150 * 1024 ? 3 : 2;
}

// A workgroup's LDS: the slots (separate objects, so the compiler can tell them
// apart) and its rows' sequences and positions.
struct TileLds {
    char *sa0, *sa1, *sa2, *sa3;
    char *sb0, *sb1, *sb2, *sb3;
    int *rowb, *rowp;
};

// The tile shapes (MI, NJ) that are instantiated.
#define PS_TILE_SHAPES(X) X(8, 4) X(8, 3) X(8, 2) X(6, 4) X(6, 3) X(6, 2) X(4, 4) X(4, 3) X(4, 2) \
    X(2, 4) X(2, 2)

// The pairs of a packed refresh: (MI, NJ) for full lists, (SMI, SNJ) for shorter
// ones, in three slots at most and together within the LDS of a CU.
#define PS_PACKED_PAIRS(X) X(6, 4, 6, 2) X(8, 2, 6, 2) X(8, 2, 4, 2) X(6, 2, 4, 2) X(4, 4, 4, 2)

// The shapes of the SwiGLU form (an even number of column tiles per wave).
#define PS_SWIGLU_SHAPES(X) X(8, 4) X(6, 4) X(4, 4) X(8, 2) X(6, 2) X(4, 2)

// MI x NJ: 16 x 16 MFMA tiles per wave (BM = 32 MI rows, BN = 64 NJ columns
// per workgroup).
//
// SWI: W is [2 F][K], gate rows over up rows, and the output is
// silu(gate) * up, [rows][F]: each wave's columns are NJ/2 tiles of gate
// features and the same features' NJ/2 tiles of up, so a lane holds both of a
// pair.  Unsplit, dense rows, F a multiple of 16.  gate and up are rounded to
// bf16 first, as the separate product stores them, and silu_mul is the separate
// pass's: the same bits as the unsplit product and that pass.
template <int MI, int NJ, bool SWI, int MAXNS, class G, class Rows>
__device__ __forceinline__ void tile_run(const G& g, const Rows& rows, const TileLds& lds, int blk) {
    static_assert(MI % 2 == 0 && MI >= 2 && MI <= 8 && NJ >= 2 && NJ <= 4, "64 to 256 rows, 128 to 256 columns");
    constexpr int ES = 2;                                // bf16 operands
    constexpr int BM = 32 * MI, BN = 64 * NJ;
    constexpr int AI = BM / 64, BI = BN / 64;            // DMA instructions per wave and K tile (8 rows each)
    constexpr int ND = AI + BI;
    constexpr int HA = MI / 2;                           // row tiles of a half block
    constexpr int HB0 = (NJ + 1) / 2, HB1 = NJ / 2;      // column tiles of its two halves
    constexpr bool kQuad = MI * NJ >= 24;                // the whole step's fragments twice would not fit
    constexpr int NS = tile_slots(MI, NJ, MAXNS);
    char* const sa0 = lds.sa0;
    char* const sa1 = lds.sa1;
    char* const sa2 = lds.sa2;
    char* const sa3 = lds.sa3;
    char* const sb0 = lds.sb0;
    char* const sb1 = lds.sb1;
    char* const sb2 = lds.sb2;
    char* const sb3 = lds.sb3;
    int* const rowb = lds.rowb;
    int* const rowp = lds.rowp;

    const int t = threadIdx.x;
    int split, rt, ct;
    if (!tile_coords(g, rows.tiles(BM), BN, blk, split, rt, ct)) return;
    const int lane = t & 63;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = w & 1, wn = w >> 1;
    const int m0 = rt * BM;
    const int n0 = ct * BN;
    // K tiles of this split: steps_per_split of them (an even number), the
    // last split what is left (even too: K is a multiple of 128)
    const int kt0 = split * g.steps_per_split;
    const int nkt = min(g.steps_per_split, g.K / 64 - kt0);
    const size_t k0b = static_cast<size_t>(kt0) * kTileStage;

    // Row bookkeeping: thread t < BM maps row m0 + t; the first workgroup of
    // each row tile publishes the map for the split-K reduction.
    int rb_ = -1, rp_ = 0;
    if (t < BM) {
        rows.map(m0 + t, rb_, rp_);
        rowb[t] = rb_;
        rowp[t] = rp_;
        if (g.ksplit > 1 && split == 0 && ct == 0 && m0 + t < g.m_max)
            *reinterpret_cast<int2*>(g.rowmap + 2 * (m0 + t)) = make_int2(rb_, rp_);
    }
    if (!__syncthreads_or(rb_ >= 0)) return;             // no row of this tile maps anywhere (uniform)

    // DMA sources: instruction i of wave w moves rows 8(w + 8i) .. +7 of a
    // slot; lane l fills chunk l%8 of row 8(w + 8i) + l/8, i.e. logical chunk
    // (l%8) ^ ((row/2)%8) (16-row fragment reads are conflict-free).  Rows
    // that map to nothing read row 0 of the input, columns past N weight row
    // 0; neither is stored.
    const char* asrc[AI];
    const char* bsrc[BI];
#pragma unroll
    for (int i = 0; i < AI; ++i) {
        const int r = 8 * (w + 8 * i) + (lane >> 3);
        const int b = rowb[r];
        const char* row = b >= 0 ? g.x + (static_cast<size_t>(b) * g.seq + rowp[r]) * g.K * ES : g.x;
        asrc[i] = row + k0b + (((lane & 7) ^ ((r >> 1) & 7)) << 4);
    }
#pragma unroll
    for (int i = 0; i < BI; ++i) {
        const int r = 8 * (w + 8 * i) + (lane >> 3);
        int n = n0 + r;
        if constexpr (SWI) {
            const int F = g.N / 2, c = r % (16 * NJ);    // column c of its wave: gate, then up
            const int f = (n0 + r - c) / 2 + c % (8 * NJ);
            n = f < F ? f + (c < 8 * NJ ? 0 : F) : g.N;
        }
        const char* row = weight_row(g, n, ES);
        bsrc[i] = (row ? row : g.w0) + k0b + (((lane & 7) ^ ((r >> 1) & 7)) << 4);
    }
    // DMA instructions d0 .. d0+n-1 of K tile kt (past the split: its last tile again)
    auto issue = [&](int d0, int n, int kt, char* abuf, char* bbuf) {
        const size_t off = static_cast<size_t>(min(kt, nkt - 1)) * kTileStage;
#pragma unroll
        for (int d = d0; d < d0 + n; ++d) {
            if (d < AI) dma16(asrc[d] + off, abuf + 8 * (w + 8 * d) * kTileStage);
            else if (d < ND) dma16(bsrc[d - AI] + off, bbuf + 8 * (w + 8 * (d - AI)) * kTileStage);
        }
    };

    // Fragment offsets: lane l reads row 16i + l%16 of its wave's block at
    // k-group l/16 of 32-k step s; the swizzle depends on l%16 only.
    const int fr = lane & 15, kg = lane >> 4;
    const int fsw = (fr >> 1) & 7;
    const int ao[2] = {(16 * MI * wm + fr) * kTileStage + ((kg ^ fsw) << 4),
                       (16 * MI * wm + fr) * kTileStage + (((4 + kg) ^ fsw) << 4)};
    const int bo[2] = {(16 * NJ * wn + fr) * kTileStage + ((kg ^ fsw) << 4),
                       (16 * NJ * wn + fr) * kTileStage + (((4 + kg) ^ fsw) << 4)};
    // n fragments of step s from row (column) tile i0 on
    auto read = [&](const char* buf, const int (&o)[2], int s, int i0, int n, uint4* f) {
#pragma unroll
        for (int i = 0; i < n; ++i)
            f[i] = *reinterpret_cast<const uint4*>(buf + o[s] + (i0 + i) * 16 * kTileStage);
    };

    // acc[i][j] holds the transposed tile: lane l has row l%16, columns
    // 4(l/16) .. +3
    floatx4 acc[MI][NJ];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    auto mma = [&](const uint4* fa, const uint4* fb, int i0, int ni, int j0, int nj) {
#pragma unroll
        for (int i = 0; i < ni; ++i)
#pragma unroll
            for (int j = 0; j < nj; ++j) acc[i0 + i][j0 + j] = mfma_bf16(fb[j], fa[i], acc[i0 + i][j0 + j]);
    };

    // The barrier of K tile T: this wave's reads of T are done and its DMA of
    // T+1 has landed, so T+1 may be read and T's slot takes T+NS.
#define PS_TILE_SYNC()                                                      \
    {                                                                       \
        __builtin_amdgcn_s_waitcnt(wait_vm((NS - 2) * ND) & kWaitLgkm0);    \
        __builtin_amdgcn_s_barrier();                                       \
        __builtin_amdgcn_sched_barrier(0);                                  \
    }
    issue(0, ND, 0, sa0, sb0);
    if constexpr (kQuad) {
        // Quarters of the block per phase, in the order A0B0 A0B1 A1B1 A1B0 |
        // A0B1 A0B0 A1B0 A1B1 over the two 32-k steps of a tile, so that each
        // phase needs one new half of fragments, read a phase ahead.
        uint4 a0[HA], a1[HA], b0[HB0], b1[HB0];
        issue(0, 4, 1, sa1, sb1);
        __builtin_amdgcn_s_waitcnt(wait_vm(4));
        __builtin_amdgcn_s_barrier();
        read(sa0, ao, 0, 0, HA, a0);
        read(sb0, bo, 0, 0, HB0, b0);
#define PS_TILE_PHASE(READ, DMA, FA, FB, I0, J0, JN)                        \
    {                                                                       \
        READ;                                                               \
        DMA;                                                                \
        mma(FA, FB, I0, HA, J0, JN);                                        \
        __builtin_amdgcn_sched_barrier(0);                                  \
    }
#define PS_TILE_STEP(T, AU, BU, AX, BX)                                                                       \
    {                                                                                                         \
        PS_TILE_PHASE(read(BU, bo, 0, HB0, HB1, b1), issue(4, 2, (T) + 1, AX, BX), a0, b0, 0, 0, HB0)         \
        PS_TILE_PHASE(read(AU, ao, 0, HA, HA, a1), issue(6, 2, (T) + 1, AX, BX), a0, b1, 0, HB0, HB1)         \
        PS_TILE_PHASE(read(AU, ao, 1, 0, HA, a0), , a1, b1, HA, HB0, HB1)                                     \
        PS_TILE_PHASE(read(BU, bo, 1, HB0, HB1, b1), , a1, b0, HA, 0, HB0)                                    \
        PS_TILE_PHASE(read(BU, bo, 1, 0, HB0, b0), , a0, b1, 0, HB0, HB1)                                     \
        PS_TILE_PHASE(read(AU, ao, 1, HA, HA, a1), , a0, b0, 0, 0, HB0)                                       \
        PS_TILE_SYNC()                                                                                        \
        PS_TILE_PHASE(read(AX, ao, 0, 0, HA, a0), issue(0, 2, (T) + 2, AU, BU), a1, b0, HA, 0, HB0)           \
        PS_TILE_PHASE(read(BX, bo, 0, 0, HB0, b0), issue(2, 2, (T) + 2, AU, BU), a1, b1, HA, HB0, HB1)        \
    }
        for (int kt = 0; kt < nkt; kt += 2) {
            PS_TILE_STEP(kt, sa0, sb0, sa1, sb1)
            PS_TILE_STEP(kt + 1, sa1, sb1, sa0, sb0)
        }
#undef PS_TILE_STEP
#undef PS_TILE_PHASE
    } else {
        // Whole 32-k steps, the next one's fragments read while this one's
        // MFMAs run.
        uint4 a[2][MI], b[2][NJ];
        issue(0, ND, 1, sa1, sb1);
        if constexpr (NS > 2) issue(0, ND, 2, sa2, sb2);
        if constexpr (NS > 3) issue(0, ND, 3, sa3, sb3);
        __builtin_amdgcn_s_waitcnt(wait_vm((NS - 1) * ND));
        __builtin_amdgcn_s_barrier();
        read(sa0, ao, 0, 0, MI, a[0]);
        read(sb0, bo, 0, 0, NJ, b[0]);
#define PS_TILE_STEP(T, AU, BU, AX, BX)                                     \
    {                                                                       \
        read(BU, bo, 1, 0, NJ, b[1]);                                       \
        read(AU, ao, 1, 0, MI, a[1]);                                       \
        mma(a[0], b[0], 0, MI, 0, NJ);                                      \
        __builtin_amdgcn_sched_barrier(0);                                  \
        PS_TILE_SYNC()                                                      \
        read(BX, bo, 0, 0, NJ, b[0]);                                       \
        read(AX, ao, 0, 0, MI, a[0]);                                       \
        issue(0, 2, (T) + NS, AU, BU);                                      \
        mma(a[1], b[1], 0, HA, 0, NJ);                                      \
        __builtin_amdgcn_sched_barrier(0);                                  \
        issue(2, ND - 2, (T) + NS, AU, BU);                                 \
        mma(a[1] + HA, b[1], HA, HA, 0, NJ);                                \
        __builtin_amdgcn_sched_barrier(0);                                  \
    }
        // (no exits inside the loop: with them the compiler copies the
        // accumulators at every step)
        static_assert(NS > 2, "the whole-step shapes have three or four slots");
        int kt = 0;
        for (; kt + NS <= nkt; kt += NS) {
            PS_TILE_STEP(kt, sa0, sb0, sa1, sb1)
            PS_TILE_STEP(kt + 1, sa1, sb1, sa2, sb2)
            if constexpr (NS == 3) {
                PS_TILE_STEP(kt + 2, sa2, sb2, sa0, sb0)
            } else {
                PS_TILE_STEP(kt + 2, sa2, sb2, sa3, sb3)
                PS_TILE_STEP(kt + 3, sa3, sb3, sa0, sb0)
            }
        }
        if (kt < nkt) {                                  // one or two steps are left (two of an even split in fours)
            PS_TILE_STEP(kt, sa0, sb0, sa1, sb1)
            if (NS == 4 || kt + 1 < nkt) PS_TILE_STEP(kt + 1, sa1, sb1, sa2, sb2)
        }
#undef PS_TILE_STEP
    }
#undef PS_TILE_SYNC
    __builtin_amdgcn_s_waitcnt(0);                       // every DMA (the re-read tail too) has landed
    __syncthreads();                                     // and every wave is done with the slots

    if constexpr (SWI) {
        constexpr int NP = NJ / 2;                       // pairs of column tiles
        constexpr int EP = 32 * NP + 16;                 // bytes of a staged row
        constexpr int ER = 16 * HA;
        constexpr int CPR = 2 * NP;                      // 16-byte chunks of a row
        char* ep = (w < 2 ? sa0 : w < 4 ? sa1 : w < 6 ? sb0 : sb1) + (w & 1) * ER * EP;
        const int F = g.N / 2, f0 = n0 / 2 + 16 * NP * wn;
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
            bool nan = false;
#pragma unroll
            for (int i = 0; i < HA; ++i)
#pragma unroll
                for (int j = 0; j < NP; ++j) {
                    const floatx4 gt = round_bf16(acc[HA * hh + i][j]), up = round_bf16(acc[HA * hh + i][j + NP]);
                    float v[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = silu_mul(gt[e], up[e]);
                    nan |= __builtin_isunordered(v[0], v[1]) || __builtin_isunordered(v[2], v[3]);
                    *reinterpret_cast<uint2*>(ep + (16 * i + fr) * EP + 32 * j + 8 * kg) =
                        make_uint2(cvt_pk_bf16(v[0], v[1]), cvt_pk_bf16(v[2], v[3]));
                }
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(nan) != 0, 0)) {
#pragma unroll
                for (int i = 0; i < HA; ++i)
#pragma unroll
                    for (int j = 0; j < NP; ++j)
                        quiet_bf16x4(reinterpret_cast<uint2*>(ep + (16 * i + fr) * EP + 32 * j + 8 * kg));
            }
            __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int q = 0; q < (ER * CPR + 63) / 64; ++q) {
                const int idx = 64 * q + lane;
                if (ER * CPR % 64 != 0 && idx >= ER * CPR) break;
                const int r = idx / CPR, c = (idx % CPR) * 8;
                const int lr = 16 * (MI * wm + HA * hh) + r;
                if (rowb[lr] >= 0 && f0 + c < F)
                    st16(g.out0 + (static_cast<size_t>(m0 + lr) * F + f0 + c) * 2, ld16(ep + r * EP + 2 * c));
            }
            __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
            __builtin_amdgcn_wave_barrier();
        }
        return;
    }
    const int cbase = n0 + 16 * NJ * wn;
    if (g.ksplit > 1) {
        // fp32 partials straight from registers: 64 contiguous bytes of 16 rows per store
        float* part = g.ws + static_cast<size_t>(split) * g.col_tiles * g.m_max * 128;
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            const int lr = 16 * (MI * wm + i) + fr;
            if (rowb[lr] < 0) continue;
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const int n = cbase + 16 * j + 4 * kg;
                if (n < g.N)
                    *reinterpret_cast<floatx4*>(part + (static_cast<size_t>(n >> 7) * g.m_max + m0 + lr) * 128 +
                                                (n & 127)) = acc[i][j];
            }
        }
        return;
    }
    // Outputs through LDS, half the wave's rows at a time in a region of its
    // own, then 8 consecutive columns of a row per lane.
    constexpr int EP = 32 * NJ + 16;                     // bytes of a staged row
    constexpr int ER = 16 * HA;                          // rows of a pass
    constexpr int CPR = 2 * NJ;                          // 16-byte chunks of a row
    static_assert(2 * ER * EP <= BM * kTileStage && 2 * ER * EP <= BN * kTileStage, "two waves' rows fit a slot");
    char* ep = (w < 2 ? sa0 : w < 4 ? sa1 : w < 6 ? sb0 : sb1) + (w & 1) * ER * EP;
    // NaNs become 0x7fc0, as from the other kernels: the rows are staged by
    // cvt_pk_bf16, looked through for NaNs while those LDS writes are under way,
    // and changed in LDS where the wave holds one.  (A branch every four values
    // made the batch-8 step 2.6 us of 215 slower.)
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
        bool nan = false;
#pragma unroll
        for (int i = 0; i < HA; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const floatx4 v = acc[HA * hh + i][j];
                *reinterpret_cast<uint2*>(ep + (16 * i + fr) * EP + 32 * j + 8 * kg) =
                    make_uint2(cvt_pk_bf16(v[0], v[1]), cvt_pk_bf16(v[2], v[3]));
            }
#pragma unroll
        for (int i = HA * hh; i < HA * (hh + 1); ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j)
                nan |= __builtin_isunordered(acc[i][j][0], acc[i][j][1]) ||
                       __builtin_isunordered(acc[i][j][2], acc[i][j][3]);
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(nan) != 0, 0)) {
#pragma unroll
            for (int i = 0; i < HA; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j)
                    quiet_bf16x4(reinterpret_cast<uint2*>(ep + (16 * i + fr) * EP + 32 * j + 8 * kg));
        }
        __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int q = 0; q < (ER * CPR + 63) / 64; ++q) {
            const int idx = 64 * q + lane;
            if (ER * CPR % 64 != 0 && idx >= ER * CPR) break;
            const int r = idx / CPR, c = (idx % CPR) * 8;
            const int lr = 16 * (MI * wm + HA * hh) + r;  // row within the tile
            const int b = rowb[lr];
            const int n = cbase + c;
            if (b >= 0 && n < g.N) st16(out_ptr<true>(g, b, rowp[lr], m0 + lr, n), ld16(ep + r * EP + 2 * c));
        }
        __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
        __builtin_amdgcn_wave_barrier();
    }
}

template <int MI, int NJ, bool SWI = false, class G>
__device__ __forceinline__ void tile_body(const G& g, int blk) {
    constexpr int A = 32 * MI * kTileStage, B = 64 * NJ * kTileStage, NS = tile_slots(MI, NJ);
    __shared__ __align__(16) char sa0[A], sa1[A], sa2[NS > 2 ? A : 16], sa3[NS > 3 ? A : 16];
    __shared__ __align__(16) char sb0[B], sb1[B], sb2[NS > 2 ? B : 16], sb3[NS > 3 ? B : 16];
    __shared__ int rowb[32 * MI], rowp[32 * MI];
    const TileLds lds{sa0, sa1, sa2, sa3, sb0, sb1, sb2, sb3, rowb, rowp};
    tile_run<MI, NJ, SWI, 4>(g, PlanRows<G>{g}, lds, blk);
}

// Packed rows in one of two tile shapes, in the same LDS: S* where the lists
// hold at most rows_small rows, else the larger one, whose grid is launched
// for full lists.  One launch, since the count is known on the device alone and
// a launch that returns at once takes 4.5 us: 16 lists of 96 entries, 8192 x
// 4096, half full 54.2 (two launches) to 51.9 us, 52% full 83.6 to 83.7, and 12
// lists 65% full 87.0 to 51.1.  Past the line the load of the counts and their
// sum, which the row map waits for, take 1 to 3 us more than unpacked rows.
template <int MI, int NJ, int SMI, int SNJ>
__device__ __forceinline__ void packed_body(const GemmArgs& g, int rows_small, int blk) {
    constexpr int A0 = 32 * MI * kTileStage, B0 = 64 * NJ * kTileStage, N0 = tile_slots(MI, NJ, 3);
    constexpr int A1 = 32 * SMI * kTileStage, B1 = 64 * SNJ * kTileStage, N1 = tile_slots(SMI, SNJ, 3);
    constexpr int A = A0 > A1 ? A0 : A1, B = B0 > B1 ? B0 : B1;
    constexpr int A2 = N0 > 2 ? (N1 > 2 ? A : A0) : N1 > 2 ? A1 : 16, B2 = N0 > 2 ? (N1 > 2 ? B : B0) : N1 > 2 ? B1 : 16;
    __shared__ __align__(16) char sa0[A], sa1[A], sa2[A2];
    __shared__ __align__(16) char sb0[B], sb1[B], sb2[B2];
    __shared__ int rowb[32 * (MI > SMI ? MI : SMI)], rowp[32 * (MI > SMI ? MI : SMI)];
    __shared__ int first[kMaxPacked + 1];
    const TileLds lds{sa0, sa1, sa2, sa2, sb0, sb1, sb2, sb2, rowb, rowp};
    const PackedRows rows{g, first, packed_rows(g, first)};
    if (rows.total <= rows_small) tile_run<SMI, SNJ, false, 3>(g, rows, lds, blk);
    else tile_run<MI, NJ, false, 3>(g, rows, lds, blk);
}

// Split-K reduction: thread = (column tile, row, 8 columns); sums the splits
// in order and stores the row through the published row map.  `id` counts the
// threads of the whole reduction (gemm_reduce_blocks workgroups of kGemmBlock).
template <bool BF16, class G>
__device__ __forceinline__ void reduce_body(const G& g, long id) {
    const long per_tile = static_cast<long>(g.m_max) * 16;
    const int ct = static_cast<int>(id / per_tile);
    if (ct >= g.col_tiles) return;
    const int rem = static_cast<int>(id - ct * per_tile);
    const int m = rem >> 4;
    const int c = (rem & 15) * 8;
    const size_t stride = static_cast<size_t>(g.col_tiles) * g.m_max * 128;   // one split
    const float* src = g.ws + (static_cast<size_t>(ct) * g.m_max + m) * 128 + c;
    float4 x[2 * kMaxSplit];
#pragma unroll
    for (int s = 0; s < kMaxSplit; ++s) {
        if (s < g.ksplit) {
            x[2 * s] = *reinterpret_cast<const float4*>(src + s * stride);
            x[2 * s + 1] = *reinterpret_cast<const float4*>(src + s * stride + 4);
        }
    }
    const int2 mp = *reinterpret_cast<const int2*>(g.rowmap + 2 * m);
    const int n = ct * 128 + c;
    if (mp.x < 0 || n >= g.N) return;
    float v[8] = {x[0].x, x[0].y, x[0].z, x[0].w, x[1].x, x[1].y, x[1].z, x[1].w};
#pragma unroll
    for (int s = 1; s < kMaxSplit; ++s) {
        if (s < g.ksplit) {
            v[0] += x[2 * s].x; v[1] += x[2 * s].y; v[2] += x[2 * s].z; v[3] += x[2 * s].w;
            v[4] += x[2 * s + 1].x; v[5] += x[2 * s + 1].y; v[6] += x[2 * s + 1].z; v[7] += x[2 * s + 1].w;
        }
    }
    store8<BF16>(out_ptr<BF16>(g, mp.x, mp.y, m, n), v);
}

}  // namespace
}  // namespace ps
