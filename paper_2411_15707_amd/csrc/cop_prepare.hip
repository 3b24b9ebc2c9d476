// Setup phase of the prepared weights, gfx950: canonical ctW -> signed byte planes of the
// centred residues in matrix-core operand order, and the column sums (nimbus_cop_prepare; the
// layout is described at nimbus_cop_prepare in include/nimbus_cop.h and used by cop_mfma_kernel.hpp).
#include "cop_mfma_common.hpp"

namespace nimbus {

// One workgroup = COLS columns over all of k, a 32-column tile or half of one: wave w re-lays the
// k-blocks w, w + WAVES, ... (pairs of them with half a tile, so that every lane has sixteen loads in
// flight) and adds up the words on the way, so that ctW is read once (the sums used to be a kernel of
// their own with one thread per column: 64 workgroups and another pass over ctW, five sixths of the
// time for the 768 x 16384 residues of a BERT-base up-projection).
// Lane l holds column l % COLS and sixteen k-slots of a block, the upper ones where l / COLS is odd: a
// load brings 256 contiguous bytes of two rows (128 of four), a store a whole 1 KB operand tile (two
// halves).  Bound by HBM: 8 bytes in and DQ bytes out per residue, 5.1-5.4 TB/s of both together where
// there are 256 column tiles or more (a copy of 1 GiB reaches 5.2): 35.5 us for those 768 x 16384
// residues, 312.6 in two kernels.  With fewer tiles, by the compute units that have one.
template <int DQ, int WAVES, int COLS>
__global__ __launch_bounds__(WAVES * 64) void prepare_kernel(
    const uint64_t *__restrict__ ctW, int k, uint32_t C, int log_n, int L, LimbTable limbs, int KB,
    uint4 *__restrict__ planes, uint64_t *__restrict__ colsum)
{
    __shared__ uint64_t part[WAVES][64][2];
    const uint32_t lane = threadIdx.x & 63u;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    constexpr int SPAN = kTile / COLS;              // k-blocks that a wave takes at a time
    const uint32_t col = blockIdx.x * COLS + lane % COLS, ct = blockIdx.x / SPAN;
    const int half_block = (int)(lane / COLS) & 1, step = (int)(lane / COLS) >> 1;
    // (the 32 columns of a tile lie in one limb: N >= 32)
    const Limb &P = limbs.limb[((ct * kTile) >> log_n) % (uint32_t)L];
    const uint64_t q = P.q, half = (q - 1) >> 1;
    uint64_t bias = 0;                              // 0x80 in each of the DQ low bytes
#pragma unroll
    for (int d = 0; d < DQ; ++d) bias |= (uint64_t)0x80 << (8 * d);

    // sums of the lower and of the upper halves of the words: k < 2^24 of 32 bits each
    uint64_t sum_lo = 0, sum_hi = 0;
    for (int kb0 = wave * SPAN; kb0 < KB; kb0 += WAVES * SPAN) {
        const int kb = kb0 + step, i0 = kb * kTile + half_block * 16;
        const uint64_t *const p = ctW + (size_t)i0 * C + col;
        uint64_t c[16];
        if ((kb0 + SPAN) * kTile <= k) {
#pragma unroll
            for (int b = 0; b < 16; ++b) c[b] = __builtin_nontemporal_load(p + (size_t)b * C);
        } else {                                    // rows past k count as zero
#pragma unroll
            for (int b = 0; b < 16; ++b) c[b] = i0 + b < k ? p[(size_t)b * C] : 0;
        }
        uint32_t w[8][4];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            uint64_t v[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint64_t x = c[4 * g + j];
                sum_lo += (uint32_t)x;
                sum_hi += x >> 32;
                // c' + bias has the unsigned bytes digit + 128; flipping bit 7 gives the digits
                v[j] = ((x > half ? x - q : x) + bias) ^ bias;
            }
            uint32_t t[4];
            transpose4((uint32_t)v[0], (uint32_t)v[1], (uint32_t)v[2], (uint32_t)v[3], t);
#pragma unroll
            for (int d = 0; d < 4; ++d) w[d][g] = t[d];
            transpose4((uint32_t)(v[0] >> 32), (uint32_t)(v[1] >> 32), (uint32_t)(v[2] >> 32),
                       (uint32_t)(v[3] >> 32), t);
#pragma unroll
            for (int d = 0; d < 4; ++d) w[4 + d][g] = t[d];
        }
        if (kb >= KB) continue;
        uint4 *const out =
            planes + ((size_t)ct * KB + kb) * DQ * 64u + (half_block * kTile + col % kTile);
#pragma unroll
        for (int d = 0; d < DQ; ++d) {
            const v4i r = {(int)w[d][0], (int)w[d][1], (int)w[d][2], (int)w[d][3]};
            __builtin_nontemporal_store(r, (v4i *)(out + d * 64));
        }
    }

    part[wave][lane][0] = sum_lo;
    part[wave][lane][1] = sum_hi;
    __syncthreads();
    if (threadIdx.x < COLS) {
        uint64_t lows = 0, highs = 0;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
#pragma unroll
            for (int g = 0; g < 64; g += COLS) {
                lows += part[w][lane + g][0];
                highs += part[w][lane + g][1];
            }
        }
        uint64_t lo = lows, hi = 0;                 // lows + 2^32 highs in 128 bits
        add128(hi, lo, highs >> 32, highs << 32);
        colsum[col] = barrett128(hi, lo, P);      // k * q < 2^(b+63)
    }
}

template <int DQ>
static hipError_t prepare_impl(const Problem &p, const uint64_t *ctW, void *prepared, hipStream_t stream)
{
    const int KB = kblocks(p.k);
    const uint32_t CT = (uint32_t)(p.C / kTile);
    uint64_t *const colsum = (uint64_t *)((char *)prepared + (size_t)CT * KB * DQ * kTileBytes);
    int log_n = 0;
    while ((1 << log_n) < p.N) ++log_n;
    auto go = [&](auto waves_c, auto cols_c) {
        constexpr int WAVES = decltype(waves_c)::value, COLS = decltype(cols_c)::value;
        return launch(prepare_kernel<DQ, WAVES, COLS>, dim3(CT * (kTile / COLS)), dim3(WAVES * 64),
                      stream, ctW, p.k, (uint32_t)p.C, log_n, p.L, p.limbs, KB, (uint4 *)prepared, colsum);
    };
    constexpr std::integral_constant<int, 16> k16;
    constexpr std::integral_constant<int, 8> k8;
    constexpr std::integral_constant<int, 4> k4;
    constexpr std::integral_constant<int, 1> k1;
    constexpr std::integral_constant<int, kTile / 2> half;
    constexpr std::integral_constant<int, kTile> whole;
    // (Tiles are counted for 256 compute units, whatever the device has.)
    // Up to 128 tiles leave half of the compute units without one: half a tile to a workgroup, from
    // five k-blocks on (us, whole tiles and halves: 160 x 2048 residues 5.4 and 4.8, 768 x 2048 11.8
    // and 9.9, 3072 x 2048 39.8 and 28.2, 3072 x 4096 45.1 and 39.9; two tiles on some units of the
    // chip and one on others are no gain, 768 x 6144 16.3 and 20.2, nor two on each, 768 x 8192 19.7
    // and 22.9, where the shorter rows of a load count).
    if (CT <= 128 && KB >= 5) return KB > 16 ? go(k16, half) : KB > 8 ? go(k8, half) : go(k4, half);
    // Sixteen waves per tile where every wave has a k-block: more loads in flight per compute unit
    // (768 x 16384 residues 35.8 us with 16 waves, 36.6 with 4; 3072 x 16384 of 59 bits 151.7 and
    // 160.3).  With fewer k-blocks most of them would only meet at the barrier (100 x 65536: 23.8
    // and 20.8 us).
    if (KB >= 16) return go(k16, whole);
    // Eight to fifteen k-blocks: eight waves (262 x 8192 9.5 us with 4 waves, 7.8 with 8, 8.6 with 16;
    // 262 x 16384 15.4, 14.5, 15.2), and sixteen where a compute unit has four tiles to take in turn
    // (480 x 32768 45.0, 44.7, 43.7; 352 x 98304 98.8, 96.7, 93.4).  Five to seven: eight where each
    // unit has one tile (160 x 8192 6.4 us with 4 waves, 5.5 with 8; 160 x 12288 8.3 and 8.6).
    if (KB >= 8) return CT < 1024 ? go(k8, whole) : go(k16, whole);
    if (KB >= 5 && CT <= 256) return go(k8, whole);
    // Fewer rows than a k-block has: one wave, so that the compute unit's waves all have tiles of their
    // own (1 x 2^20 residues 58.4 us with 4 waves, 44.1 with 1; 20 x 2^20 87.6 and 60.4).  A whole
    // k-block has sixteen loads in flight per lane as it is (32 x 2^20: 85.2 and 90.4).  A launch has
    // fewer than 2^32 threads, so from 2^24 column tiles on it is one wave too.
    if (p.k < kTile || CT >= (1u << 24)) return go(k1, whole);
    return go(k4, whole);
}

hipError_t launch_prepare(const Problem &p, const uint64_t *ctW, void *prepared, hipStream_t stream)
{
    if (planes_q(p.q_bits_max) == 7) return prepare_impl<7>(p, ctW, prepared, stream);
    return prepare_impl<8>(p, ctW, prepared, stream);
}

}  // namespace nimbus
