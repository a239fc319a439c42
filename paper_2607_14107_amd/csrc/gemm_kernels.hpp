// The products' kernels but the tile kernel, and the launch of a plan, for two
// weight matrices (GemmArgs, gemm.hip) or three (QkvGemmArgs, gemm_qkv.hip).
// Internal to the library.
#pragma once

#include "gemm_dev.hpp"
#include "host_common.hpp"

namespace ps {
namespace {

constexpr int kLda = 272;         // LDS row pitch (bytes) of the staged input rows

// ---------------------------------------------------------------------------
// gemm_rows_kernel: BM = 32*MT rows x 128 columns per workgroup; wave w owns
// columns 32w..32w+31 of all rows (lane l carries row/column l%32 and k-group
// l/32, 128 contiguous bytes per super-step).
// ---------------------------------------------------------------------------

template <int MT, class G>
__global__ __launch_bounds__(kGemmBlock) void gemm_rows_kernel(G g) {
    constexpr bool BF16 = false;
    using T = Elem<BF16>;
    constexpr int BM = MT * 32;
    constexpr int BN = 128;
    constexpr int RA = BM / 16;            // 16-byte chunks each thread stages per super-step
    constexpr int ES = T::kBytes;
    __shared__ __align__(16) char sa[2][BM * kLda];
    __shared__ int rowb[BM], rowp[BM];

    const int tile = blockIdx.x / g.ksplit;
    const int split = blockIdx.x - tile * g.ksplit;
    const int col_tile = tile % g.col_tiles;
    const int row_tile = tile / g.col_tiles;

    const int t = threadIdx.x;
    const int lane = t & 63;
    const int w = t >> 6;
    const int m0 = row_tile * BM;

    // The weight row this lane streams (column n of wave w; past N: row 0,
    // never stored), 128 contiguous bytes per super-step at k-group lane/32.
    // Its first two super-steps are requested before the row bookkeeping,
    // whose dependent loads (counts, prefix, stale indices) would otherwise
    // delay the weight stream.
    const int n = col_tile * BN + w * 32 + (lane & 31);
    const char* brow = weight_row(g, n, ES);
    if (!brow) brow = g.w0;
    brow += (lane >> 5) * 128;
    const int nsteps = g.K / (256 / ES);
    const int s0 = split * g.steps_per_split;
    const int s1 = min(nsteps, s0 + g.steps_per_split);
    const int slast = s1 - 1;
    auto load_b = [&](int step, uint4 (&rb)[8]) {
#pragma unroll
        for (int s = 0; s < 8; ++s) rb[s] = ld16(brow + step * 256 + 16 * s);
    };
    uint4 b0[8], b1[8], b2[8];
    load_b(s0, b0);
    load_b(min(s0 + 1, slast), b1);

    // Row bookkeeping: one load per row.  The first workgroup of each row
    // tile also publishes the map for the split-K reduction.
    int rb_ = -1, rp_ = 0;
    if (t < BM) map_row(g, m0 + t, rb_, rp_);
    if (t < BM) {
        rowb[t] = rb_;
        rowp[t] = rp_;
        if (g.ksplit > 1 && split == 0 && col_tile == 0 && m0 + t < g.m_max)
            *reinterpret_cast<int2*>(g.rowmap + 2 * (m0 + t)) = make_int2(rb_, rp_);
    }
    if (!__syncthreads_or(rb_ >= 0)) return;   // no row of this tile maps anywhere (uniform)

    // Rows that map to nothing read row 0 instead: their accumulators are
    // never stored, and every load stays unconditional (static wait counts).
    const char* arow[RA];
#pragma unroll
    for (int i = 0; i < RA; ++i) {
        const int r = (t >> 4) + 16 * i;
        const int b = rowb[r];
        arow[i] = b >= 0 ? g.x + (static_cast<size_t>(b) * g.seq + rowp[r]) * g.K * ES : g.x;
    }
    const int acol = (t & 15) * 16;

    floatx16 acc[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < 16; ++j) acc[i][j] = 0.f;

    auto load_a = [&](int step, uint4 (&ra)[RA]) {
#pragma unroll
        for (int i = 0; i < RA; ++i) ra[i] = ld16(arow[i] + step * 256 + acol);
    };
    auto store_a = [&](int buf, const uint4 (&ra)[RA]) {
#pragma unroll
        for (int i = 0; i < RA; ++i) st16(&sa[buf][((t >> 4) + 16 * i) * kLda + acol], ra[i]);
    };
    // The MT fragments of chunk s+1 are read from LDS while the MFMAs of
    // chunk s run (two register sets; the scheduling barriers keep that
    // order), so LDS latency is not exposed per MFMA.
    auto compute = [&](int buf, const uint4 (&rb)[8]) {
        const char* abase = &sa[buf][(lane & 31) * kLda + (lane >> 5) * 128];
        uint4 af[2][MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) af[0][mt] = *reinterpret_cast<const uint4*>(abase + mt * 32 * kLda);
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            __builtin_amdgcn_sched_barrier(0);
            if (s + 1 < 8) {
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    af[(s + 1) & 1][mt] = *reinterpret_cast<const uint4*>(abase + mt * 32 * kLda + 16 * (s + 1));
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) acc[mt] = Mma32<BF16>::step(af[s & 1][mt], rb[s], acc[mt]);
        }
        __builtin_amdgcn_sched_barrier(0);
    };

    // Software pipeline.  Issue order of the loads: ... B(s+1), A(s+1),
    // B(s+2), A(s+2) ...  Waiting for A(s+1) at the end of step s (to stage
    // it in LDS) therefore also covers B(s+1), which step s+1 needs, while
    // B(s+2) stays in flight: weights get two compute phases of latency
    // cover, the (L2-resident) input rows one.  (Two phases for the input
    // rows too, with a second register buffer, measured no faster.)
    // Prefetches past s1 - 1 re-read step s1 - 1 (cache hits, ignored) so
    // every iteration issues the same loads and the wait counts stay static.
    uint4 ra[RA];
    load_a(s0, ra);
    store_a(0, ra);                       // waits for A(s0) (and B(s0), B(s0+1))
    load_a(min(s0 + 1, slast), ra);
    __syncthreads();

    // step S: issue B(S+2) -> B_LOAD; compute with LDS[(S-s0)%2] and B_USE;
    // stage A(S+1) -> LDS[(S-s0+1)%2]; then issue A(S+2).
#define PS_GEMM_STEP(S, B_USE, B_LOAD)                                      \
    {                                                                       \
        const int s_ = (S);                                                 \
        __builtin_amdgcn_sched_barrier(0);                                  \
        load_b(min(s_ + 2, slast), B_LOAD);                                 \
        __builtin_amdgcn_sched_barrier(0);                                  \
        compute((s_ - s0) & 1, B_USE);                                      \
        if (s_ + 1 < s1) store_a((s_ - s0 + 1) & 1, ra);                    \
        __syncthreads();                                                    \
        load_a(min(s_ + 2, slast), ra);                                     \
    }
    int sc = s0;
    for (; sc + 3 <= s1; sc += 3) {      // single exit: buffers rotate b0 -> b1 -> b2
        PS_GEMM_STEP(sc, b0, b2)
        PS_GEMM_STEP(sc + 1, b1, b0)
        PS_GEMM_STEP(sc + 2, b2, b1)
    }
    if (sc < s1) PS_GEMM_STEP(sc, b0, b2)
    if (sc + 1 < s1) PS_GEMM_STEP(sc + 1, b1, b0)
#undef PS_GEMM_STEP

    // Epilogue, staged through LDS (the input staging buffers are free now):
    // register j of acc[mt] is row mt*32 + mfma32_row(lane, j) of column
    // 32w + lane%32; then each thread writes 8 consecutive columns of a row
    // (16-byte stores, 512 contiguous bytes per row of the tile).
    constexpr int EP = BN + 4;            // fp32 pitch of the staged tile
    static_assert(static_cast<size_t>(BM) * EP * 4 <= sizeof(sa), "epilogue tile must fit");
    float* ep = reinterpret_cast<float*>(&sa[0][0]);
    __syncthreads();                      // every wave is done reading sa
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int j = 0; j < 16; ++j)
            ep[(mt * 32 + mfma32_row(lane, j)) * EP + w * 32 + (lane & 31)] = acc[mt][j];
    __syncthreads();
    for (int idx = t; idx < BM * (BN / 8); idx += kGemmBlock) {
        const int r = idx / (BN / 8);
        const int c = (idx % (BN / 8)) * 8;
        const int b = rowb[r];
        const int nc = col_tile * BN + c;
        if (b < 0 || nc >= g.N) continue;
        const float* v = ep + r * EP + c;
        if (g.ksplit == 1) {
            store8<BF16>(out_ptr<BF16>(g, b, rowp[r], m0 + r, nc), v);
        } else {
            float* dst = g.ws + ((static_cast<size_t>(split) * g.col_tiles + col_tile) * g.m_max + (m0 + r)) * BN + c;
            *reinterpret_cast<float4*>(dst) = make_float4(v[0], v[1], v[2], v[3]);
            *reinterpret_cast<float4*>(dst + 4) = make_float4(v[4], v[5], v[6], v[7]);
        }
    }
}

// ---------------------------------------------------------------------------
// gemm_dma_kernel: the DMA-staged body of gemm_dev.hpp (dma_body).
// ---------------------------------------------------------------------------

template <int MT, int NST, bool NTW, class G>
__global__ __launch_bounds__(kGemmBlock) void gemm_dma_kernel(G g) {
    dma_body<true, MT, NST, 4, NTW>(g, blockIdx.x);
}

// Sum of the split-K partials, in split order (deterministic): thread ->
// (column tile, row, 8 columns) so that consecutive threads read consecutive
// 32-byte pieces of the contiguous partial tiles; the partial and row-map
// loads are independent, then one rounded 16-byte store.
template <bool BF16, class G>
__global__ __launch_bounds__(kGemmBlock) void gemm_reduce_kernel(G g) {
    reduce_body<BF16>(g, static_cast<long>(blockIdx.x) * kGemmBlock + threadIdx.x);
}

template <bool BF16, int MT, class G>
__global__ __launch_bounds__(kSmallBlock) void gemm_small_kernel(G g) {
    small_body<BF16, MT>(g, blockIdx.x, blockIdx.y);
}

template <class G>
bool dispatch_rows(const GemmPlan& p, const G& g, hipStream_t s) {
    const dim3 grid(p.grid), block(kGemmBlock);
    switch (p.mt) {   // 32-row tiles per workgroup
        case 1: hipLaunchKernelGGL((gemm_rows_kernel<1, G>), grid, block, 0, s, g); return true;
        case 2: hipLaunchKernelGGL((gemm_rows_kernel<2, G>), grid, block, 0, s, g); return true;
        case 3: hipLaunchKernelGGL((gemm_rows_kernel<3, G>), grid, block, 0, s, g); return true;
        case 4: hipLaunchKernelGGL((gemm_rows_kernel<4, G>), grid, block, 0, s, g); return true;
        case 5: hipLaunchKernelGGL((gemm_rows_kernel<5, G>), grid, block, 0, s, g); return true;
        case 6: hipLaunchKernelGGL((gemm_rows_kernel<6, G>), grid, block, 0, s, g); return true;
        case 7: hipLaunchKernelGGL((gemm_rows_kernel<7, G>), grid, block, 0, s, g); return true;
        case 8: hipLaunchKernelGGL((gemm_rows_kernel<8, G>), grid, block, 0, s, g); return true;
        default: return false;
    }
}

template <int MT, bool NTW, class G>
bool dispatch_dma_nst(const GemmPlan& p, const G& g, hipStream_t s) {
    const dim3 grid(p.grid), block(kGemmBlock);
    switch (2 * p.steps_per_split) {   // 128-byte stages per split
        case 8: hipLaunchKernelGGL((gemm_dma_kernel<MT, 8, NTW, G>), grid, block, 0, s, g); return true;
        case 16: hipLaunchKernelGGL((gemm_dma_kernel<MT, 16, NTW, G>), grid, block, 0, s, g); return true;
        default: break;
    }
    if constexpr (MT > 4) {            // 17..64 rows split K into 8 or 16 stages only
        switch (2 * p.steps_per_split) {
            case 10: hipLaunchKernelGGL((gemm_dma_kernel<MT, 10, NTW, G>), grid, block, 0, s, g); return true;
            case 12: hipLaunchKernelGGL((gemm_dma_kernel<MT, 12, NTW, G>), grid, block, 0, s, g); return true;
            case 14: hipLaunchKernelGGL((gemm_dma_kernel<MT, 14, NTW, G>), grid, block, 0, s, g); return true;
            default: break;
        }
    }
    return false;
}

// One row tile of 17..160 rows (it reads every weight byte once: non-temporal
// weight stream) or two of 81..128.
template <class G>
bool dispatch_dma(const GemmPlan& p, const G& g, hipStream_t s) {
    if (p.row_tiles == 1) {
        switch (p.mt) {   // 16-row tiles
            case 2: return dispatch_dma_nst<2, true>(p, g, s);
            case 3: return dispatch_dma_nst<3, true>(p, g, s);
            case 4: return dispatch_dma_nst<4, true>(p, g, s);
            case 5: return dispatch_dma_nst<5, true>(p, g, s);
            case 6: return dispatch_dma_nst<6, true>(p, g, s);
            case 7: return dispatch_dma_nst<7, true>(p, g, s);
            case 8: return dispatch_dma_nst<8, true>(p, g, s);
            case 9: return dispatch_dma_nst<9, true>(p, g, s);
            case 10: return dispatch_dma_nst<10, true>(p, g, s);
            default: return false;
        }
    }
    switch (p.mt) {
        case 6: return dispatch_dma_nst<6, false>(p, g, s);
        case 7: return dispatch_dma_nst<7, false>(p, g, s);
        case 8: return dispatch_dma_nst<8, false>(p, g, s);
        default: return false;
    }
}

template <bool BF16, class G>
bool dispatch_small(const GemmPlan& p, const G& g, hipStream_t s) {
    dim3 grid(p.col_tiles, p.row_tiles);
    switch (p.mt) {
        case 1: hipLaunchKernelGGL((gemm_small_kernel<BF16, 1, G>), grid, dim3(kSmallBlock), 0, s, g); return true;
        case 2: hipLaunchKernelGGL((gemm_small_kernel<BF16, 2, G>), grid, dim3(kSmallBlock), 0, s, g); return true;
        case 3: hipLaunchKernelGGL((gemm_small_kernel<BF16, 3, G>), grid, dim3(kSmallBlock), 0, s, g); return true;
        case 4: hipLaunchKernelGGL((gemm_small_kernel<BF16, 4, G>), grid, dim3(kSmallBlock), 0, s, g); return true;
        default: return false;
    }
}

// gemm_run for two or three weight matrices.
template <class G>
polestar_status run_plan(bool bf16, const GemmPlan& p, G g, hipStream_t stream, G* deferred) {
    gemm_finalize_args(p, g);
    bool ok;
    if (p.small) ok = bf16 ? dispatch_small<true>(p, g, stream) : dispatch_small<false>(p, g, stream);
    else if (p.tile) {
        ok = bf16 && p.steps_per_split % 2 == 0 && launch_tile(p, g, stream);
    } else if (p.dma) ok = bf16 && dispatch_dma(p, g, stream);
    else ok = !bf16 && dispatch_rows(p, g, stream);
    if (!ok) return POLESTAR_ERR_UNSUPPORTED;
    polestar_status st = launch_status();
    if (st != POLESTAR_OK || p.small || p.ksplit == 1) return st;
    if (deferred) {   // the caller launches the reduction (fused with other work)
        *deferred = g;
        return POLESTAR_OK;
    }
    const int blocks = gemm_reduce_blocks(p, g);
    if (bf16)
        hipLaunchKernelGGL((gemm_reduce_kernel<true, G>), dim3(blocks), dim3(kGemmBlock), 0, stream, g);
    else
        hipLaunchKernelGGL((gemm_reduce_kernel<false, G>), dim3(blocks), dim3(kGemmBlock), 0, stream, g);
    return launch_status();
}

}  // namespace
}  // namespace ps
