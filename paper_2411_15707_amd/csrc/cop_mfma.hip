// Prepared weights on the matrix cores, host side: the staging of the shares into byte planes, the
// limits of the path and the dispatch of a call to its kernel (cop_mfma_kernel.hpp; few rows:
// cop_thin.hip).
#include "cop_mfma_common.hpp"
#include <atomic>

namespace nimbus {

// ---------------------------------------------------------------------------
// per call: X -> DX signed byte planes in A-operand tile order
// ---------------------------------------------------------------------------
// (blockIdx.y: the problem, when the shares of several calls are staged in one launch)
template <int NB>
struct StagePtrs {
    const uint64_t *X[NB];
    uint32_t *xd[NB];
};

// One thread = four consecutive k of one row: one 32-bit word in each plane.
struct StageItem {
    uint32_t word, lane, tile;      // which 4 of the lane's 16 k-slots; rt * KB + kb
    int row, k0;
};

__device__ __forceinline__ StageItem stage_item(uint32_t gid, uint32_t KB)
{
    StageItem it;
    it.word = gid & 3u;
    it.lane = (gid >> 2) & 63u;
    it.tile = gid >> 8;
    it.row = (int)(it.tile / KB) * kTile + (int)(it.lane & 31u);
    it.k0 = (int)(it.tile % KB) * kTile + (int)(it.lane >> 5) * 16 + (int)it.word * 4;
    return it;
}

// (flipping bit 7 of a byte turns it into the two's complement digit byte - 128; what lies past
// the row or past k has zero digits)
template <int DX>
__device__ __forceinline__ void store_planes(uint32_t *__restrict__ xd, const StageItem &it, const uint32_t (&x)[4])
{
    uint32_t w[4];
    transpose4(x[0], x[1], x[2], x[3], w);
#pragma unroll
    for (int d = 0; d < DX; ++d) xd[(((size_t)it.tile * DX + d) * 64u + it.lane) * 4u + it.word] = w[d];
}

template <int DX, int NB>
__global__ __launch_bounds__(256) void x_planes_kernel(
    const StagePtrs<NB> sp, int m, int k, int KB, uint32_t total, uint32_t offx)
{
    const uint64_t *__restrict__ const X = sp.X[blockIdx.y];
    const uint32_t gid = blockIdx.x * 256u + threadIdx.x;
    if (gid >= total) return;
    const StageItem it = stage_item(gid, (uint32_t)KB);
    uint32_t x[4];
#pragma unroll
    for (int b = 0; b < 4; ++b)
        x[b] = it.row < m && it.k0 + b < k ? (uint32_t)X[(size_t)it.row * k + it.k0 + b] ^ offx : 0u;
    store_planes<DX>(sp.xd[blockIdx.y], it, x);
}

// Shares of more than 32 bits: the planes of the lower halves, four, and behind all of them the DH
// planes of the upper halves, from one reading of the shares.  What bounds it is the launch, for many
// shares the bytes; as a launch for each half (us a staging call, 64-bit shares) 128 x 768 6.1 -> 4.0,
// 512 x 4096 9.5 -> 5.1, 2048 x 8192 67.3 -> 39.8.
template <int DH>
__global__ __launch_bounds__(256) void x_planes_wide_kernel(
    const uint64_t *__restrict__ X, uint32_t *__restrict__ xd, int m, int k, int KB, uint32_t total,
    uint32_t offx_lo, uint32_t offx_hi)
{
    const uint32_t gid = blockIdx.x * 256u + threadIdx.x;
    if (gid >= total) return;
    const StageItem it = stage_item(gid, (uint32_t)KB);
    uint32_t lo[4], hi[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const bool there = it.row < m && it.k0 + b < k;
        const uint64_t x = there ? X[(size_t)it.row * k + it.k0 + b] : 0u;
        lo[b] = there ? (uint32_t)x ^ offx_lo : 0u;
        hi[b] = there ? (uint32_t)(x >> 32) ^ offx_hi : 0u;
    }
    store_planes<4>(xd, it, lo);
    store_planes<DH>(xd + (size_t)total * 4u, it, hi);
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
// (asked once per device)
int compute_units()
{
    if (launch_log && launch_log->compute_units > 0) return launch_log->compute_units;
    static std::atomic<int> cached[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    int n = cached[dev].load(std::memory_order_relaxed);
    if (n == 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1)
            n = 256;
        cached[dev].store(n, std::memory_order_relaxed);
    }
    return n;
}

TileBlocks tile_blocks(const Problem &p, int count)
{
    // Row blocks of 64 rows where all of those find a compute unit of their own: half as many products
    // per workgroup (810 sizes of 65 to 512 rows, k from 64 to 480: 1.28 times as fast on average as blocks
    // of 128 rows, none slower; 100 x 400 x 4096 15.9 us with those, 11.4 with 64, 128 x 480 x 8192 17.7
    // and 13.4).  With a second round of workgroups the larger blocks were ahead (100 x 768 x 12288).
    uint32_t cus = (uint32_t)compute_units();
    if (cus >= 8) cus &= ~7u;
    if (p.m > 64 && (uint64_t)(p.C / 64u) * (uint64_t)((p.m + 63) / 64) * (uint32_t)count <= cus)
        return {(p.m + 63) / 64, 2};
    // Else of 128 rows at most, and of even size: 130 rows are 96 and 34, not 128 and 2 (a workgroup walks
    // tiles that lie a multiple of eight apart, so that with two or four row blocks it has the same one
    // in all of them; 130 x 200 x 16384 27.4 us with 128 and 2, 24.7 with 96 and 34).
    const int row_blocks = (p.m + 127) / 128, row_tiles = (p.m + kTile - 1) / kTile;
    return {row_blocks, (row_tiles + row_blocks - 1) / row_blocks};
}

bool mfma_supported(const Problem &p)
{
    const int DX = planes_x(p.x_bits), DQ = planes_q(p.q_bits_max);
    if (DX < 2 || DX > 4 || DQ < 7 || DQ > 8) return false;
    const long long pairs = DX < DQ ? DX : DQ;
    // |D_d| < 2^30 (zero padding of k adds nothing)
    if ((long long)p.k * pairs * 16384ll >= (1ll << 30)) return false;
    // one workgroup per 128 x 64 output tile in a one-dimensional grid
    const uint64_t workgroups = (uint64_t)(p.C / (2 * kTile)) * (uint64_t)((p.m + 127) / 128);
    if (workgroups >= (1ull << 31)) return false;
    // the value reduced in the epilogue is below (2^(sh+1) + 2^33 + 1) * q (the second
    // 2^32 q: the previous pass of a wide share); the floating-point quotient needs it
    // below 2^47 * q
    return bias_shift(p) + 2 <= 47;
}

template <int DX>
static hipError_t stage_impl(const Problem &p, int count, const uint64_t *const *X, void *const *workspace,
                             hipStream_t stream)
{
    const int KB = kblocks(p.k);
    const int RT = (p.m + kTile - 1) / kTile;
    const uint32_t xtotal = (uint32_t)RT * KB * 256;
    auto go = [&](auto nb_c) {
        constexpr int NB = decltype(nb_c)::value;
        StagePtrs<NB> sp{};
        for (int i = 0; i < count; ++i) {
            sp.X[i] = X[i];
            sp.xd[i] = (uint32_t *)workspace[i];
        }
        return launch(x_planes_kernel<DX, NB>, dim3((xtotal + 255) / 256, (uint32_t)count), dim3(256), stream,
                      sp, p.m, p.k, KB, xtotal, share_offset(p.x_bits, DX));
    };
    return count == 1 ? go(std::integral_constant<int, 1>{}) : go(std::integral_constant<int, kMaxBatch>{});
}

template <int DH>
static hipError_t stage_wide_impl(const Problem &p, const uint64_t *X, void *workspace, hipStream_t stream)
{
    const int KB = kblocks(p.k);
    const int RT = (p.m + kTile - 1) / kTile;
    const uint32_t xtotal = (uint32_t)RT * KB * 256;
    return launch(x_planes_wide_kernel<DH>, dim3((xtotal + 255) / 256), dim3(256), stream, X, (uint32_t *)workspace,
                  p.m, p.k, KB, xtotal, share_offset(32, 4), share_offset(p.x_bits - 32, DH));
}

// (of more than 32 bits: both halves, one behind the other)
hipError_t launch_stage_shares(const Problem &p, const uint64_t *X, void *workspace, hipStream_t stream)
{
    if (p.x_bits <= 32) return launch_stage_shares_batch(p, 1, &X, &workspace, stream);
    switch (planes_x(p.x_bits - 32)) {
    case 2: return stage_wide_impl<2>(p, X, workspace, stream);
    case 3: return stage_wide_impl<3>(p, X, workspace, stream);
    default: return stage_wide_impl<4>(p, X, workspace, stream);
    }
}

// the shares (up to 32 bits) of count calls of the same shape in one launch
hipError_t launch_stage_shares_batch(const Problem &p, int count, const uint64_t *const *X,
                                     void *const *workspace, hipStream_t stream)
{
    if (count < 1 || count > kMaxBatch) return hipErrorInvalidValue;
    switch (planes_x(p.x_bits)) {
    case 2: return stage_impl<2>(p, count, X, workspace, stream);
    case 3: return stage_impl<3>(p, count, X, workspace, stream);
    default: return stage_impl<4>(p, count, X, workspace, stream);
    }
}

// the launches of the tile kernel (cop_mfma_x*.hip: one pair of plane counts each)
template <int DX, int DQ>
hipError_t mfma_impl(const Problem &p, int count, const void *const *staged,
                     const void *const *prepared, const uint64_t *const *masks,
                     const uint64_t *prev, uint64_t *const *outs, hipStream_t stream);

hipError_t launch_cop_mfma(const Problem &p, const void *staged, const void *prepared,
                           const uint64_t *mask, const uint64_t *prev, uint64_t *out,
                           hipStream_t stream)
{
    return launch_cop_mfma_batch(p, 1, &staged, &prepared, &mask, prev, &out, stream);
}

hipError_t launch_cop_mfma_batch(const Problem &p, int count, const void *const *staged,
                                 const void *const *prepared, const uint64_t *const *masks,
                                 const uint64_t *prev, uint64_t *const *outs, hipStream_t stream)
{
    if (count < 1 || count > kMaxBatch) return hipErrorInvalidValue;
    // few rows: a kernel of their own (cop_thin.hip, with both sides measured)
    if (thin_applies(p, count)) return launch_cop_thin(p, count, nullptr, 0, staged, prepared, masks, prev, outs, stream);
    const int DX = planes_x(p.x_bits), DQ = planes_q(p.q_bits_max);
#define NIMBUS_CASE(dx, dq) \
    if (DX == dx && DQ == dq) \
        return mfma_impl<dx, dq>(p, count, staged, prepared, masks, prev, outs, stream);
    NIMBUS_CASE(2, 7)
    NIMBUS_CASE(3, 7)
    NIMBUS_CASE(4, 7)
    NIMBUS_CASE(2, 8)
    NIMBUS_CASE(3, 8)
    NIMBUS_CASE(4, 8)
#undef NIMBUS_CASE
    return hipErrorInvalidValue;
}

}  // namespace nimbus
