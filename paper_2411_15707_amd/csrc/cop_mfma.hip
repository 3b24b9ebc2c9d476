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

template <int DX, int NB>
__global__ __launch_bounds__(256) void x_planes_kernel(
    const StagePtrs<NB> sp, int m, int k, int KB, uint32_t total, uint32_t offx, int half_shift)
{
    const uint64_t *__restrict__ const X = sp.X[blockIdx.y];
    uint32_t *__restrict__ const xd = sp.xd[blockIdx.y];
    // one thread = four consecutive k of one row: one 32-bit word in each of the DX planes
    const uint32_t gid = blockIdx.x * 256u + threadIdx.x;
    if (gid >= total) return;
    const uint32_t word = gid & 3u;                 // which 4 of the lane's 16 k-slots
    const uint32_t lane = (gid >> 2) & 63u;
    const uint32_t tile = gid >> 8;                 // rt * KB + kb
    const uint32_t kb = tile % (uint32_t)KB;
    const uint32_t rt = tile / (uint32_t)KB;
    const int row = (int)rt * kTile + (int)(lane & 31u);
    const int kbase = (int)kb * kTile + (int)(lane >> 5) * 16 + (int)word * 4;

    uint32_t w[DX];
#pragma unroll
    for (int d = 0; d < DX; ++d) w[d] = 0;
    if (row < m) {
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int i = kbase + b;
            if (i < k) {
                // flipping bit 7 of a byte turns it into the two's complement digit byte - 128
                // (half_shift = 32 selects the upper half of a share wider than 32 bits)
                const uint32_t x = (uint32_t)(X[(size_t)row * k + i] >> half_shift) ^ offx;
#pragma unroll
                for (int d = 0; d < DX; ++d) w[d] |= ((x >> (8 * d)) & 0xffu) << (8 * b);
            }
        }
    }
#pragma unroll
    for (int d = 0; d < DX; ++d)
        xd[(((size_t)tile * DX + d) * 64u + lane) * 4u + word] = w[d];
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
static hipError_t stage_impl(const Problem &p, int count, const uint64_t *const *X, int half_shift,
                             void *const *workspace, hipStream_t stream)
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
                      sp, p.m, p.k, KB, xtotal, share_offset(p.x_bits, DX), half_shift);
    };
    return count == 1 ? go(std::integral_constant<int, 1>{}) : go(std::integral_constant<int, kMaxBatch>{});
}

// p.x_bits (<= 32) is the width of the half that is staged; half_shift is 0 or 32
hipError_t launch_stage_shares(const Problem &p, const uint64_t *X, int half_shift,
                               void *workspace, hipStream_t stream)
{
    return launch_stage_shares_batch(p, 1, &X, half_shift, &workspace, stream);
}

// the shares of count calls of the same shape in one launch
hipError_t launch_stage_shares_batch(const Problem &p, int count, const uint64_t *const *X,
                                     int half_shift, void *const *workspace, hipStream_t stream)
{
    if (count < 1 || count > kMaxBatch) return hipErrorInvalidValue;
    switch (planes_x(p.x_bits)) {
    case 2: return stage_impl<2>(p, count, X, half_shift, workspace, stream);
    case 3: return stage_impl<3>(p, count, X, half_shift, workspace, stream);
    default: return stage_impl<4>(p, count, X, half_shift, workspace, stream);
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
