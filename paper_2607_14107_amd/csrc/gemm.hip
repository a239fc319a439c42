// Gather -> MFMA GEMM -> scatter, the core of the sparse K/V refresh
// (Sec. 4.1: re-project the stale rows and the active block; Corollary 1 of
// App. B: K = W_K h, V = W_V h) and of the Q projection of the active block.
//
// The rows are a few tens to a few thousand gathered ones, the [N][K] weight
// is read from HBM.  Four kernels (gemm_kernels.hpp, gemm_tile.hip), picked by
// gemm_plan:
//
// gemm_tile_kernel (bf16, more than 64 rows; tile_body in gemm_dev.hpp):
//   64 to 256 rows x 128 to 256 columns per workgroup, both operands by DMA.
//
// gemm_rows_kernel (fp32, more than 64 rows): a workgroup of 4 waves owns
//   BM = 32*MT rows and 128 columns; wave w computes all BM rows of columns
//   32w..32w+31 with v_mfma_f32_32x32x2_f32.  Per super-step of 256 bytes of
//   K:
//   - the gathered input rows are staged in LDS (16-byte coalesced loads,
//     272-byte row pitch: conflict-free MFMA reads) and shared by the waves;
//     a wave reads the fragments of the next chunk while the MFMAs of the
//     current one run;
//   - each wave streams its weight rows from HBM straight into registers,
//     128 contiguous bytes per lane, two super-steps ahead (triple buffer,
//     loop unrolled three times so the buffers rotate without copies).
//   A row's (sequence, position) is one load away (fixed stride of
//   k_max + block_len rows per sequence), so the first input rows follow
//   the weight prefetch closely.
//
// Where rows x columns do not fill the chip, K is split over workgroups; each
//   writes its fp32 partial tile to the workspace ([split][column
//   tile][row][128]), the row map goes next to it, and gemm_reduce_kernel
//   sums the partials in split order (deterministic) and scatters 16-byte
//   rows.
//
// gemm_dma_kernel (17 to 256 rows, e.g. the refresh of one sequence's stale
//   rows and block, or the Q projection of a batch's blocks): one of up to two
//   row tiles of up to 160 rows and 128 columns per workgroup, both operands
//   (bf16) brought into LDS by global_load_lds_dwordx4 (no VGPR staging, so the
//   weight loads never wait behind registers that MFMAs still read), in
//   stages of 128 bytes of each row; four LDS slots, three stages in flight,
//   one barrier per stage.  A stage's rows are XOR-swizzled in 16-byte chunks
//   (chunk c of row r at slot c ^ (r/2 % 8)) so that 16-row fragment reads
//   are conflict-free; the swizzle is applied to each lane's global address,
//   since a DMA instruction writes its lanes' data contiguously.  The waits
//   for the DMA are explicit s_waitcnt immediates (each wave issues the same
//   number of DMA instructions per stage), and each slot's LDS arrays are
//   separate objects so the compiler does not add waits of its own.
//   Measured on the batch-1 LLaDA-8B refresh (138 rows x 8192 x 4096): 21.5 us
//   for the split-K GEMM.
//
// gemm_small_kernel (at most 64 rows, e.g. the Q projection): a workgroup
//   owns all rows and 16 columns; its 4 waves take interleaved super-steps
//   of the full K with both operands loaded straight into registers and are
//   summed in LDS, so no partials leave the chip.  A load instruction covers
//   64 contiguous bytes of each of 16 rows.
//
// In all, A and B use the same lane -> k assignment, so k may be visited in
// any order.  All loads are unconditional (rows or columns past the end read
// row 0 and are never stored) so the compiler's wait counts stay static.
#include <algorithm>
#include <mutex>

#include "gemm_kernels.hpp"
#include "host_common.hpp"

namespace ps {

constexpr int kTargetWgs = 256;   // one workgroup per compute unit on MI355X

// Scratch of a split-K product: the partial tiles [ksplit][col_tiles][m_max][128]
// fp32 and the row map.
static size_t partial_bytes(int ksplit, long m_max, int N) {
    return align_up(static_cast<size_t>(ksplit) * ceil_div(N, 128) * m_max * 128 * sizeof(float), 256);
}
static size_t split_bytes(int ksplit, long m_max, int N) {
    if (ksplit == 1) return 0;
    return partial_bytes(ksplit, m_max, N) + align_up(static_cast<size_t>(m_max) * 2 * sizeof(int), 256);
}

// The split that the workspace sizes are quoted for.  The sizes are part of the
// interface (callers keep buffers of them, and a call with less is refused, as
// is one beyond polestar_refresh_kv_noalloc's array), so they follow this rule
// and not the kernels: a plan may split less than it, never more.  It prices
// 256- and 192-sided tiles at 3.9 GFLOP/ms per CU in rounds of 256 and the
// partials at 5 TB/s; fewer rows, narrow outputs and shapes too small for that
// count 128-column tiles of at most 160 or 256 rows.
static int quoted_split(bool bf16, long m_max, int N, int K) {
    const int nsteps = ceil_div(K, bf16 ? 128 : 64);
    const long col_tiles = ceil_div(N, 128);
    auto even_steps = [nsteps](int ks) { return nsteps % ks == 0 && nsteps / ks >= 4 && nsteps / ks <= 8; };
    if (m_max <= 64) {
        for (int ks = ceil_div(kTargetWgs, col_tiles); bf16 && m_max > 16 && ks <= kMaxSplit; ++ks)
            if (nsteps % ks == 0 && (nsteps / ks == 4 || nsteps / ks == 8)) return ks;
        return 1;
    }
    bool narrow = false;
    for (int ks = 1; ks <= kMaxSplit; ++ks) narrow |= even_steps(ks);
    narrow = narrow && bf16 && N <= 1024 && m_max <= 1280;
    if (bf16 && m_max > 160 && K % 64 == 0 && !narrow) {
        const int nstage = K / 32;
        int ksplit = 1, rows_tile = 256;
        long tiles = static_cast<long>(ceil_div(m_max, 256)) * ceil_div(N, 256);
        double best = 1e30;
        for (int rows = 256; rows >= 192; rows -= 64) {
            for (int cols = 256; cols >= 192; cols -= 64) {
                const long n = static_cast<long>(ceil_div(m_max, rows)) * ceil_div(N, cols);
                const double rate = (rows == 256 ? 1.0 : 0.95) * (cols == 256 ? 1.0 : 0.95);
                const double tile_us = static_cast<double>(rows) * cols * 2.0 * K / (3.9e6 * rate);
                for (int k = 1; k <= kMaxSplit; ++k) {
                    if (nstage % (4 * k) != 0 || nstage / k < 16) continue;
                    const double rounds = static_cast<double>((n * k + kTargetWgs - 1) / kTargetWgs);
                    const double cost = rounds * tile_us / k + (k > 1 ? 8.0 * k * m_max * N / 5e6 : 0.0);
                    if (cost < best) {
                        best = cost;
                        ksplit = k;
                        rows_tile = rows;
                        tiles = n;
                    }
                }
            }
        }
        if (tiles * ksplit >= kTargetWgs / 2 &&
            (ksplit <= 4 || nstage / ksplit >= 48 || ceil_div(m_max, rows_tile) >= 4))
            return ksplit;
    }
    if (bf16 && (m_max <= 320 || narrow)) {
        const long tiles = ceil_div(m_max, 160L) * col_tiles;
        long best = -1;
        int ksplit = 0;
        for (int ks = 1; ks <= kMaxSplit; ++ks) {
            if (!even_steps(ks)) continue;
            const long cost = (tiles * ks + kTargetWgs - 1) / kTargetWgs * (nsteps / ks);
            if (best < 0 || cost < best) {
                best = cost;
                ksplit = ks;
            }
        }
        if (ksplit > 0) return ksplit;
    }
    const long tiles = ceil_div(m_max, bf16 && (m_max <= 320 || narrow) ? 160L : 256L) * col_tiles;
    const int ks = std::min<long>(std::min(kMaxSplit, nsteps), tiles < kTargetWgs ? ceil_div(kTargetWgs, tiles) : 1);
    return ceil_div(nsteps, ceil_div(nsteps, ks));
}

// Estimated time (us) of the tile kernel with `tiles` tiles of 32 mi x 64 nj in
// ks splits of `steps` K tiles: ceil(tiles * ks / 256) rounds of one workgroup
// per CU, each a fixed cost (launch, row map, first DMA, stores) and its K
// tiles at the shape's time; a split run adds the reduction's launch and its
// fp32 partials written and read back (per MB).  The constants are a least
// squares fit to the times of every plan within a third of the best one, for
// 275 shapes of 65 to 4096 rows, 64 to 32768 columns and K 256 to 12288 (the
// layers' products and others over those ranges, weights not cached).  Over 943
// such shapes the plan that they choose is 0.7% slower than the fastest one in
// the geometric mean, 5% at the 95th percentile and 20% at most; each shape's
// time with every CU busy and partials at 0.32 us per MB: 1.5, 12 and 38%.
static double tile_kt(int mi, int nj) {
    switch (10 * mi + nj) {
        case 84: return 1.49;
        case 83: return 1.29;
        case 64: return 1.25;
        case 82: return 0.80;
        case 44: return 0.86;
        case 63: return 0.87;
        case 62: return 0.62;
        case 43: return 0.73;
        case 42: return 0.52;
        case 24: return 0.69;
        default: return 0.36;
    }
}
static double split_cost(int ks, long m_max, int N) {
    return ks > 1 ? 4.0 + 4.0 * ks * m_max * N * 0.4e-6 : 0.0;
}
static double rounds_cost(long workgroups, int steps, double kt) {
    return static_cast<double>((workgroups + kTargetWgs - 1) / kTargetWgs) * (steps * kt + 4.0);
}
static double tile_cost(int mi, int nj, long tiles, int ks, int steps, long m_max, int N) {
    return rounds_cost(tiles * ks, steps, tile_kt(mi, nj)) + split_cost(ks, m_max, N);
}

// The tile kernel's plan: the tile shape and split with the least estimated
// time among splits up to max_split, the larger tile and the smaller split on
// ties.  Every split runs an even number of K tiles and at least eight.
static void plan_tile(GemmPlan& p, long m_max, int N, int K, int max_split) {
    const int nkt = K / 64;                              // K tiles, an even number
    struct { int ks, steps; double cost; } split[kMaxSplit];   // the splits that K allows
    int nsplit = 0;
    for (int ks = 1; ks <= max_split; ++ks) {
        const int steps = 2 * ceil_div(nkt / 2, ks);
        if (ceil_div(nkt, steps) != ks || (ks > 1 && steps < 8)) continue;
        split[nsplit++] = {ks, steps, split_cost(ks, m_max, N)};
    }
    double best = 1e30;
    for (int mi = 8; mi >= 2; mi -= 2) {
        for (int nj = 4; nj >= 2; --nj) {
            if (mi == 2 && nj == 3) continue;            // not instantiated
            const long tiles = static_cast<long>(ceil_div(m_max, 32 * mi)) * ceil_div(N, 64 * nj);
            const double kt = tile_kt(mi, nj);
            for (int i = 0; i < nsplit; ++i) {
                const auto& s = split[i];
                if (s.ks > 1 && (tiles * (s.ks - 1) >= kTargetWgs ||   // already a full round
                                 s.cost >= best))
                    break;
                const double cost = rounds_cost(tiles * s.ks, s.steps, kt) + s.cost;
                if (cost < best) {
                    best = cost;
                    p.ksplit = s.ks;
                    p.tile_mi = mi;
                    p.tile_nj = nj;
                    p.steps_per_split = s.steps;
                }
            }
        }
    }
    p.tile = true;
    p.mt = 2 * p.tile_mi;
    p.col_tiles = ceil_div(N, 128);                      // of the partials
    p.row_tiles = ceil_div(m_max, 32 * p.tile_mi);
    p.grid = static_cast<int>(static_cast<long>(p.row_tiles) * ceil_div(N, 64 * p.tile_nj) * p.ksplit);
}

// The DMA kernel's plan for 65 to 256 rows: row tiles of at most 160 rows, K
// split evenly into 8 to 16 stages of 128 bytes per row; the split with the
// fewest stages in one round of one workgroup per CU.  False when no split
// does.
static bool plan_dma(GemmPlan& p, long m_max, int N, int K, int max_split) {
    const int nsteps = K / 128;
    const int row_tiles = ceil_div(m_max, 16L * kDmaMaxRowTiles), col_tiles = ceil_div(N, 128);
    for (int ks = max_split; ks >= 1; --ks) {
        if (nsteps % ks != 0 || nsteps / ks < 4 || nsteps / ks > 8) continue;
        if (static_cast<long>(row_tiles) * col_tiles * ks > kTargetWgs) continue;
        p.dma = true;
        p.ksplit = ks;
        p.steps_per_split = nsteps / ks;
        p.row_tiles = row_tiles;
        p.col_tiles = col_tiles;
        p.mt = ceil_div(ceil_div(m_max, row_tiles), 16);
        p.grid = row_tiles * col_tiles * ks;
        return true;
    }
    return false;
}

GemmPlan gemm_plan(bool bf16, long m_max, int N, int K) {
    GemmPlan p{};
    const int ks = bf16 ? 128 : 64;
    const int nsteps = ceil_div(K, ks);
    if (m_max <= 0) m_max = 1;
    const int quoted = quoted_split(bf16, m_max, N, K);
    p.ws_bytes = split_bytes(quoted, m_max, N);
    if (!gemm_k_ok(bf16, K)) return p;   // only its size is asked for
    // 17..64 rows (bf16): the DMA kernel with split-K partials streams each
    // weight once with its A rows shared through LDS, where the small kernel
    // re-reads the rows once per 16 columns (the 32-row LLaDA-8B block
    // projection: 12.4 against 13.7 us with the reduce, 64 rows 13.6 against
    // 21.0);
    if (m_max <= 64 && bf16 && m_max > 16) {
        const int col_tiles = ceil_div(N, 128);
        for (int ks = ceil_div(kTargetWgs, col_tiles); ks <= kMaxSplit; ++ks) {
            if (nsteps % ks == 0 && (nsteps / ks == 4 || nsteps / ks == 8)) {
                p.dma = true;
                p.row_tiles = 1;
                p.col_tiles = col_tiles;
                p.ksplit = ks;
                p.steps_per_split = nsteps / ks;
                p.mt = ceil_div(m_max, 16);
                p.grid = col_tiles * ks;
                return p;
            }
        }
    }
    // others, or when K does not split into 8 or 16 stages, the small kernel
    // (their quoted workspace is none, so nothing else could split K)
    if (m_max <= 64) {
        p.small = true;
        p.mt = ceil_div(m_max, 16);
        p.row_tiles = 1;
        p.col_tiles = ceil_div(N, 16);
        p.ksplit = 1;
        p.steps_per_split = nsteps;
        p.grid = p.col_tiles;
        return p;
    }
    // bf16 above that: the tile kernel, but for two ranges that the DMA kernel
    // runs in one round:
    // - one row tile of 65 to 160 rows whose weights are a round's worth of its
    //   longest splits (60 MB and K >= 4096, or 56 MB up to 96 rows); it marks
    //   their stream non-temporal.  Against the tile kernel on weights that are
    //   not cached, 66 / 96 / 138 / 160 rows: 8192 x 4096 0.82 0.83 0.84 0.88 of
    //   its time, 7680 x 4096 0.82 0.88 0.92 0.96, 4480 x 7168 0.85 0.93 0.95
    //   0.95, 3840 x 8192 0.80 0.83 0.87 0.89, 5376 x 6144 0.85 0.97 0.98 1.0,
    //   8192 x 3584 0.85 0.91 0.98 1.08 (128 rows 0.92 to 1.13, 3584: 1.28); less
    //   than that, 6144 x 4096 0.99 1.05 1.10 1.09, 5632 x 5120 0.99 1.06 1.09
    //   1.05, 3072 x 8192 0.97 1.06 1.07 1.06; shorter K, 10880 x 3072 0.86 0.99
    //   1.18 1.13, 16384 x 2048 1.08 1.13 1.10 1.12, 32768 x 1024 0.83 0.90 0.98
    //   1.04.  The kernels behind it also find more of theirs in the caches (a
    //   batch-1 LLaDA-8B step 57.5 against 61.8 us);
    // - 161 to 256 rows of K >= 1536 in two row tiles (4096 x 4096: 176 rows
    //   20.3 against 24.2 us, 224 rows 22.7 / 25.5, 256 rows 27.2 / 26.1; with
    //   K = 1024 and below the tile kernel is 10-45% faster; for narrower weights
    //   it is by itself up to 30% faster at longer K too, but the fused step
    //   takes these Q projections into its select launch from the DMA kernel).
    if (bf16) {
        const long weights = static_cast<long>(N) * K;
        const bool dma_rows = m_max <= 96    ? m_max > 64 && weights >= 28L << 20
                              : m_max <= 160 ? K >= 4096 && weights >= 30L << 20
                                             : m_max <= 256 && K >= 1536;
        if (!(dma_rows && plan_dma(p, m_max, N, K, quoted))) plan_tile(p, m_max, N, K, quoted);
        return p;
    }
    // fp32: the row kernel, 256-row tiles of 128 columns, K split to fill one
    // round of workgroups
    p.col_tiles = ceil_div(N, 128);
    p.row_tiles = ceil_div(m_max, 256);
    const long tiles = static_cast<long>(p.row_tiles) * p.col_tiles;
    int ksplit = 1;
    if (tiles < kTargetWgs) ksplit = ceil_div(kTargetWgs, tiles);
    if (ksplit > kMaxSplit) ksplit = kMaxSplit;
    if (ksplit > nsteps) ksplit = nsteps;
    p.steps_per_split = ceil_div(nsteps, ksplit);
    p.ksplit = ceil_div(nsteps, p.steps_per_split);
    p.mt = ceil_div(m_max, 32L * p.row_tiles);
    p.grid = static_cast<int>(static_cast<long>(p.row_tiles) * p.col_tiles * p.ksplit);
    return p;
}

GemmArgs refresh_gemm_args(int batch, int seq, int d, int kvd, const void* h_cur, const int32_t* stale_idx,
                           const int32_t* stale_count, int k_max, int block_start, int block_len,
                           const void* w_k, const void* w_v, void* k_cache, void* v_cache, void* workspace) {
    GemmArgs g{};
    g.x = static_cast<const char*>(h_cur);
    g.w0 = static_cast<const char*>(w_k);
    g.w1 = static_cast<const char*>(w_v);
    g.n0 = kvd;
    g.N = 2 * kvd;
    g.K = d;
    g.mode = kGemmRefresh;
    g.batch = batch;
    g.seq = seq;
    g.stale_idx = k_max > 0 ? stale_idx : nullptr;
    g.stale_count = k_max > 0 ? stale_count : nullptr;
    g.k_max = k_max;
    g.block_start = block_start;
    g.block_len = block_len;
    g.out0 = static_cast<char*>(k_cache);
    g.out1 = static_cast<char*>(v_cache);
    g.ws = static_cast<float*>(workspace);
    g.m_max = batch * (k_max + block_len);
    return g;
}

void gemm_finalize_args(const GemmPlan& p, GemmArgs& g) {
    g.rowmap = p.ksplit > 1 ? reinterpret_cast<int*>(reinterpret_cast<char*>(g.ws) + partial_bytes(p.ksplit, g.m_max, g.N))
                            : nullptr;
    g.ksplit = p.ksplit;
    g.steps_per_split = p.steps_per_split;
    g.row_tiles = p.row_tiles;
    g.col_tiles = p.col_tiles;
}

int gemm_reduce_blocks(const GemmPlan& p, const GemmArgs& g) {
    if (p.small || p.ksplit == 1) return 0;
    return ceil_div(static_cast<long>(p.col_tiles) * g.m_max * 16, kGemmBlock);
}

// Estimated time of a tile plan for m rows.
static double plan_cost(const GemmPlan& p, long m, int N) {
    const long tiles = static_cast<long>(ceil_div(m, 32 * p.tile_mi)) * ceil_div(N, 64 * p.tile_nj);
    return tile_cost(p.tile_mi, p.tile_nj, tiles, p.ksplit, p.steps_per_split, m, N);
}

// The SwiGLU form's plan, false where two calls are faster (or the only way).
// It runs unsplit, in the cheapest tile shape that pairs gate and up columns,
// when its estimate and its longer epilogue (expf and a division per pair: 5.5
// us for a round of 256 x 256 tiles, by the pairs of a lane for smaller ones)
// are no more above the product's own plan than the separate pass costs (3.5 us
// and 6 bytes per feature at 5 TB/s).  Both ways measured on 236 shapes of 65 to
// 4000 rows: the choice is 0.4% off the faster one in the geometric mean, 15% at
// most; two calls always 7%, one launch wherever there is one 4%.  4096 channels
// to 2 x 12288, 1024 rows: 171.8 us in one launch against 192.6 in two; 512 rows
// 94.2 against 90.5 (192 tiles of 256 x 256, or 256 of 256 x 192 and the pass).
static bool swiglu_plan(const GemmPlan& plan, long m_max, int N, int K, GemmPlan& p) {
    if (!plan.tile || N % 32 != 0) return false;
    p = plan;
    p.ksplit = 1;
    p.steps_per_split = K / 64;
    const int nkt = K / 64;
    double best = 1e30;
#define PS_CASE(MI, NJ)                                                                                          \
    {                                                                                                            \
        const long tiles = static_cast<long>(ceil_div(m_max, 32 * MI)) * ceil_div(N, 64 * NJ);                   \
        const double rounds = static_cast<double>((tiles + kTargetWgs - 1) / kTargetWgs);                        \
        const double cost = tile_cost(MI, NJ, tiles, 1, nkt, m_max, N) + rounds * (5.5 / 32) * (MI * NJ);        \
        if (cost < best) {                                                                                       \
            best = cost;                                                                                         \
            p.tile_mi = MI;                                                                                      \
            p.tile_nj = NJ;                                                                                      \
            p.row_tiles = ceil_div(m_max, 32 * MI);                                                              \
            p.grid = static_cast<int>(tiles);                                                                    \
        }                                                                                                        \
    }
    PS_SWIGLU_SHAPES(PS_CASE)
#undef PS_CASE
    return best <= plan_cost(plan, m_max, N) + 3.5 + 3.0 * m_max * N / 5e6;
}

bool gemm_run_swiglu(const GemmPlan& plan, GemmArgs g, hipStream_t stream) {
    GemmPlan p;
    if (!swiglu_plan(plan, g.m_max, g.N, g.K, p)) return false;
    gemm_finalize_args(p, g);
    return launch_tile_swiglu(p, g, stream);
}

polestar_status gemm_run(bool bf16, const GemmPlan& p, GemmArgs g, hipStream_t stream, GemmArgs* deferred) {
    return run_plan(bf16, p, g, stream, deferred);
}

// The packed form of a refresh whose unpacked plan is `plan`, false where it has
// none: its larger shape must be no slower than the plan's (2%: lists may be
// full), and half-full lists, the usual packet (the members of half the
// clusters), must gain more than the 2 us that the running sum of the counts
// takes.  rows_small goes on past half as far as the smaller shape's estimate is
// below the larger one's.  8192 x 4096 weights, lists of 96 entries, unpacked
// and packed, with uneven counts: 16 lists 45% full 83.7 and 48.4 us, 50% 84.9 /
// 51.9, 52% (the first past the line) 81.9 / 83.7, 65% 82.3 / 83.4, 80% 84.6 /
// 85.0, 100% 86.7 / 90.2; 12 lists 50% 78.3 / 49.5, 65% 80.6 / 51.1, 80% 81.0 /
// 83.3, 100% 85.8 / 86.6; 8 lists 50% 44.3 / 43.9, 100% 51.6 / 52.8.  In a
// denoising loop (16 sequences, 6 layers of 2048 channels, half of 8 clusters
// refreshed) the lists were 0.21 to 0.73 full, 0.49 in the median, and at most
// half in 54 to 61% of the packets.
static bool packed_plan(const GemmPlan& plan, long m_max, int N, int K, PackedPlan& q) {
    const int nkt = K / 64;
    const double now = plan_cost(plan, m_max, N);
    double best = now - 2.0;
    auto cost = [&](int mi, int nj, long row_tiles) {
        return tile_cost(mi, nj, row_tiles * ceil_div(N, 64 * nj), 1, nkt, m_max, N);
    };
#define PS_CASE(MI, NJ, SMI, SNJ)                                                                                     \
    {                                                                                                                 \
        const long full_tiles = ceil_div(m_max, 32 * MI), half_tiles = ceil_div(ceil_div(m_max, 2), 32 * SMI);        \
        const double full = cost(MI, NJ, full_tiles), half = cost(SMI, SNJ, half_tiles);                              \
        if (full <= 1.02 * now && half < best) {                                                                      \
            best = half;                                                                                              \
            long rt = half_tiles;                                                                                     \
            while (rt * 32 * SMI < m_max && cost(SMI, SNJ, rt + 1) < full) ++rt;                                      \
            const long grid = std::max(full_tiles * ceil_div(N, 64 * NJ), rt * ceil_div(N, 64 * SNJ));                \
            q = {MI, NJ, SMI, SNJ, static_cast<int>(rt * 32 * SMI), static_cast<int>(grid)};                          \
        }                                                                                                             \
    }
    PS_PACKED_PAIRS(PS_CASE)
#undef PS_CASE
    return best < now - 2.0;
}

polestar_status gemm_run_refresh(bool bf16, const GemmPlan& p, GemmArgs g, hipStream_t stream) {
    PackedPlan q;
    if (!bf16 || !p.tile || p.ksplit > 1 || g.block_len > 0 || g.k_max == 0 || g.batch > kMaxPacked ||
        !packed_plan(p, g.m_max, g.N, g.K, q))
        return gemm_run(bf16, p, g, stream);
    gemm_finalize_args(p, g);
    if (!launch_packed(q, g, stream)) return POLESTAR_ERR_UNSUPPORTED;
    return launch_status();
}

}  // namespace ps

// What a product of m rows runs as, for tests that name the kernels they are
// about (host only, not in the public headers).  out: kernel (0 small, 1 DMA, 2
// tile, 3 rows), the tile kernel's rows and columns of a workgroup, splits of K.
static void plan_info(const ps::GemmPlan& p, int* out) {
    out[0] = p.small ? 0 : p.dma ? 1 : p.tile ? 2 : 3;
    out[1] = p.tile ? 32 * p.tile_mi : 0;
    out[2] = p.tile ? 64 * p.tile_nj : 0;
    out[3] = p.ksplit;
}

extern "C" void ps_gemm_plan_info(int bf16, long m, int N, int K, int* out) {
    plan_info(ps::gemm_plan(bf16 != 0, m, N, K), out);
}

// The packed refresh of that product: rows and columns of the larger and the
// smaller tile, the rows up to which the smaller one runs; 0 where the rows
// are not packed.
extern "C" int ps_packed_plan_info(long m, int N, int K, int* out) {
    const ps::GemmPlan p = ps::gemm_plan(true, m, N, K);
    ps::PackedPlan q;
    if (!p.tile || p.ksplit > 1 || !ps::packed_plan(p, m, N, K, q)) return 0;
    const int v[5] = {32 * q.mi, 64 * q.nj, 32 * q.small_mi, 64 * q.small_nj, q.rows_small};
    std::copy(v, v + 5, out);
    return 1;
}

// The same for the one-launch SwiGLU product of N = 2 ffn columns; 0 where
// polestar_linear_swiglu makes two calls.
extern "C" int ps_swiglu_plan_info(long m, int N, int K, int* out) {
    ps::GemmPlan p;
    if (!ps::swiglu_plan(ps::gemm_plan(true, m, N, K), m, N, K, p)) return 0;
    plan_info(p, out);
    return 1;
}

extern "C" size_t polestar_refresh_kv_workspace_size(polestar_dtype dtype, int batch, int d,
                                                     int n_kv_heads, int head_dim, int k_max,
                                                     int block_len) {
    using namespace ps;
    if (!dtype_ok(dtype) || batch <= 0 || d <= 0 || n_kv_heads <= 0 || head_dim <= 0 ||
        k_max < 0 || block_len < 0)
        return 0;
    const long m_max = static_cast<long>(batch) * (k_max + block_len);
    const int N = 2 * n_kv_heads * head_dim;
    return gemm_plan(dtype == POLESTAR_BF16, m_max, N, d).ws_bytes;
}

extern "C" polestar_status polestar_refresh_kv(polestar_dtype dtype, int batch, int seq, int d,
                                               int n_kv_heads, int head_dim, const void* h_cur,
                                               const int32_t* stale_idx,
                                               const int32_t* stale_count, int k_max,
                                               int block_start, int block_len, const void* w_k,
                                               const void* w_v, void* k_cache, void* v_cache,
                                               void* workspace, size_t workspace_bytes,
                                               hipStream_t stream) {
    using namespace ps;
    if (!dtype_ok(dtype) || batch <= 0 || seq <= 0 || d <= 0 || n_kv_heads <= 0 ||
        head_dim <= 0 || k_max < 0 || k_max > seq || block_start < 0 || block_len < 0 ||
        block_start > seq - block_len || !h_cur || !w_k || !w_v || !k_cache || !v_cache ||
        (k_max > 0 && (!stale_idx || !stale_count)))
        return POLESTAR_ERR_INVALID_ARGUMENT;
    if ((head_dim != 64 && head_dim != 128) || !gemm_k_ok(dtype == POLESTAR_BF16, d) ||
        !aligned16(h_cur) || !aligned16(w_k) || !aligned16(w_v) || !aligned16(k_cache) ||
        !aligned16(v_cache) || !aligned16(workspace))
        return POLESTAR_ERR_UNSUPPORTED;
    if (batch > 65536) return POLESTAR_ERR_UNSUPPORTED;
    const long m_max = static_cast<long>(batch) * (k_max + block_len);
    if (m_max == 0) return POLESTAR_OK;
    if (m_max > 0x7fffffffL / 4) return POLESTAR_ERR_UNSUPPORTED;
    const bool bf16 = dtype == POLESTAR_BF16;
    const int kvd = n_kv_heads * head_dim;
    const GemmPlan p = gemm_plan(bf16, m_max, 2 * kvd, d);
    if (workspace_bytes < p.ws_bytes || (p.ws_bytes > 0 && !workspace)) return POLESTAR_ERR_WORKSPACE;
    const GemmArgs g = refresh_gemm_args(batch, seq, d, kvd, h_cur, stale_idx, stale_count, k_max, block_start,
                                         block_len, w_k, w_v, k_cache, v_cache, workspace);
    return gemm_run_refresh(bf16, p, g, stream);
}

// ---------------------------------------------------------------------------
// polestar_refresh_kv_noalloc: polestar_refresh_kv with its split-K partials
// and row map in a file-scope device array instead of a caller workspace.
// Each device holds its own copy of the array; its address on a device is
// looked up once (hipGetSymbolAddress, with that device current) and kept,
// since the array's name in host code is only a host-side stand-in.  The
// kernels need no initialised scratch (every partial that the reduction
// reads is written first in the same call), so nothing is cleared.
// ---------------------------------------------------------------------------

namespace ps {
namespace {
constexpr size_t kScratchBytes = size_t{64} << 20;
constexpr int kMaxDevices = 64;
}  // namespace
}  // namespace ps

static __device__ __align__(256) char scratch[ps::kScratchBytes];

namespace ps {
namespace {

std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// The current device's copy of the array, or nullptr if its address cannot
// be obtained (status in *st).
void* device_scratch(polestar_status* st) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
        *st = dev >= kMaxDevices ? POLESTAR_ERR_UNSUPPORTED : POLESTAR_ERR_LAUNCH;
        return nullptr;
    }
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
            *st = POLESTAR_ERR_LAUNCH;
            return nullptr;
        }
        g_scratch_ptr[dev] = p;
    }
    return g_scratch_ptr[dev];
}

}  // namespace
}  // namespace ps

extern "C" size_t polestar_refresh_kv_noalloc_max_bytes(void) { return ps::kScratchBytes; }

extern "C" polestar_status polestar_refresh_kv_noalloc(polestar_dtype dtype, int batch, int seq, int d,
                                                       int n_kv_heads, int head_dim, const void* h_cur,
                                                       const int32_t* stale_idx,
                                                       const int32_t* stale_count, int k_max,
                                                       int block_start, int block_len, const void* w_k,
                                                       const void* w_v, void* k_cache, void* v_cache,
                                                       hipStream_t stream) {
    using namespace ps;
    // The same validation as polestar_refresh_kv, before the scratch lookup.
    if (!dtype_ok(dtype) || batch <= 0 || seq <= 0 || d <= 0 || n_kv_heads <= 0 ||
        head_dim <= 0 || k_max < 0 || k_max > seq || block_start < 0 || block_len < 0 ||
        block_start > seq - block_len || !h_cur || !w_k || !w_v || !k_cache || !v_cache ||
        (k_max > 0 && (!stale_idx || !stale_count)))
        return POLESTAR_ERR_INVALID_ARGUMENT;
    if ((head_dim != 64 && head_dim != 128) || !gemm_k_ok(dtype == POLESTAR_BF16, d) ||
        !aligned16(h_cur) || !aligned16(w_k) || !aligned16(w_v) || !aligned16(k_cache) ||
        !aligned16(v_cache))
        return POLESTAR_ERR_UNSUPPORTED;
    if (batch > 65536) return POLESTAR_ERR_UNSUPPORTED;
    const long m_max = static_cast<long>(batch) * (k_max + block_len);
    if (m_max == 0) return POLESTAR_OK;
    if (m_max > 0x7fffffffL / 4) return POLESTAR_ERR_UNSUPPORTED;
    const bool bf16 = dtype == POLESTAR_BF16;
    const int kvd = n_kv_heads * head_dim;
    const GemmPlan p = gemm_plan(bf16, m_max, 2 * kvd, d);
    if (p.ws_bytes > kScratchBytes) return POLESTAR_ERR_WORKSPACE;
    void* ws = nullptr;
    if (p.ws_bytes > 0) {
        polestar_status st = POLESTAR_OK;
        ws = device_scratch(&st);
        if (!ws) return st;
    }
    const GemmArgs g = refresh_gemm_args(batch, seq, d, kvd, h_cur, stale_idx, stale_count, k_max, block_start,
                                         block_len, w_k, w_v, k_cache, v_cache, ws);
    return gemm_run_refresh(bf16, p, g, stream);
}
