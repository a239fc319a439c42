// The tile kernel (tile_body of gemm_dev.hpp) and its launches.  In a file of
// their own: the kernels are large, and with them in the code objects of the
// small kernels that a layer step launches between them (gemm.hip, step.hip)
// the batch-1 LLaDA-8B step ran 0.4 us slower on cold caches (57.9 against 57.5
// us per step).
#include "gemm_dev.hpp"
#include "host_common.hpp"

namespace ps {
namespace {

template <int MI, int NJ, class G>
__global__ __launch_bounds__(kTileThreads) void gemm_tile_kernel(G g) {
    tile_body<MI, NJ>(g, blockIdx.x);
}

template <int MI, int NJ>
__global__ __launch_bounds__(kTileThreads) void gemm_swiglu_kernel(GemmArgs g) {
    tile_body<MI, NJ, true>(g, blockIdx.x);
}

template <int MI, int NJ, int SMI, int SNJ>
__global__ __launch_bounds__(kTileThreads) void gemm_packed_kernel(GemmArgs g, int rows_small) {
    packed_body<MI, NJ, SMI, SNJ>(g, rows_small, blockIdx.x);
}

// refresh on the tile kernel, unsplit | Q split-K reduce: the tile
// workgroups come first (tile_body's XCD-aware order counts from id 0), the
// reduction's after them, on compute units the tiles leave free or as a short
// tail, so the Q reduce needs no launch of its own (bf16 only, as the tile
// kernel).
struct TileQArgs {
    GemmArgs r;    // refresh (n_tile workgroups, first)
    GemmArgs q;    // Q projection
    int n_tile;
};

static_assert(kTileThreads % kGemmBlock == 0, "a workgroup of the reduce role takes whole reduce blocks");

template <int MI, int NJ>
__global__ __launch_bounds__(kTileThreads) void tile_qred_kernel(TileQArgs k) {
    if (static_cast<int>(blockIdx.x) < k.n_tile) {
        tile_body<MI, NJ>(k.r, blockIdx.x);
        return;
    }
    reduce_body<true>(k.q, static_cast<long>(blockIdx.x - k.n_tile) * kTileThreads + threadIdx.x);
}

template <class G>
bool launch_tile_of(const GemmPlan& p, const G& g, hipStream_t stream) {
    const dim3 grid(p.grid), block(kTileThreads);
    switch (10 * p.tile_mi + p.tile_nj) {
#define PS_CASE(MI, NJ) \
        case 10 * MI + NJ: hipLaunchKernelGGL((gemm_tile_kernel<MI, NJ, G>), grid, block, 0, stream, g); return true;
        PS_TILE_SHAPES(PS_CASE)
#undef PS_CASE
        default: return false;
    }
}

}  // namespace

bool launch_tile(const GemmPlan& p, const GemmArgs& g, hipStream_t stream) { return launch_tile_of(p, g, stream); }
bool launch_tile(const GemmPlan& p, const QkvGemmArgs& g, hipStream_t stream) { return launch_tile_of(p, g, stream); }

bool launch_tile_swiglu(const GemmPlan& p, const GemmArgs& g, hipStream_t stream) {
    const dim3 grid(p.grid), block(kTileThreads);
    switch (10 * p.tile_mi + p.tile_nj) {
#define PS_CASE(MI, NJ) \
        case 10 * MI + NJ: hipLaunchKernelGGL((gemm_swiglu_kernel<MI, NJ>), grid, block, 0, stream, g); return true;
        PS_SWIGLU_SHAPES(PS_CASE)
#undef PS_CASE
        default: return false;
    }
}

bool launch_packed(const PackedPlan& p, const GemmArgs& g, hipStream_t stream) {
    const dim3 grid(p.grid), block(kTileThreads);
    switch (1000 * p.mi + 100 * p.nj + 10 * p.small_mi + p.small_nj) {
#define PS_CASE(MI, NJ, SMI, SNJ)                                                                             \
        case 1000 * MI + 100 * NJ + 10 * SMI + SNJ:                                                           \
            hipLaunchKernelGGL((gemm_packed_kernel<MI, NJ, SMI, SNJ>), grid, block, 0, stream, g, p.rows_small); \
            return true;
        PS_PACKED_PAIRS(PS_CASE)
#undef PS_CASE
        default: return false;
    }
}

bool launch_tile_qred(const GemmPlan& p, const GemmArgs& g, const GemmArgs& q, int n_qred, hipStream_t stream) {
    TileQArgs k{};
    k.r = g;
    k.q = q;
    k.n_tile = p.grid;
    const dim3 grid(p.grid + ceil_div(n_qred, kTileThreads / kGemmBlock)), block(kTileThreads);
    switch (10 * p.tile_mi + p.tile_nj) {
#define PS_CASE(MI, NJ) \
        case 10 * MI + NJ: hipLaunchKernelGGL((tile_qred_kernel<MI, NJ>), grid, block, 0, stream, k); return true;
        PS_TILE_SHAPES(PS_CASE)
#undef PS_CASE
        default: return false;
    }
}

}  // namespace ps
