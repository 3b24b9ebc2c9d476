// Setup phase of the prepared weights, gfx950: canonical ctW -> signed byte planes of the
// centred residues in matrix-core operand order, and the column sums (nimbus_cop_prepare; the
// layout is described at nimbus_cop_prepare in include/nimbus_cop.h and used by cop_mfma_kernel.hpp).
#include "cop_mfma_common.hpp"

namespace nimbus {

// One workgroup = one 32-column tile over all of k: wave w re-lays the k-blocks w, w + WAVES, ...
// and adds up the words on the way, so that ctW is read once (the sums used to be a kernel of their
// own with one thread per column: 64 workgroups and another pass over ctW, five sixths of the time
// for the 768 x 16384 residues of a BERT-base up-projection).
// Lane l holds column l % 32 and the 16 k-slots (l / 32) * 16 .. +15 of a block: a load brings 256
// contiguous bytes of two rows, a store a whole 1 KB operand tile.  Bound by HBM: 8 bytes in and
// DQ bytes out per residue, 5.1-5.4 TB/s of both together where there are 256 column tiles or more
// (a copy of 1 GiB reaches 5.2): 35.5 us for those 768 x 16384 residues, 312.6 in two kernels.
template <int DQ, int WAVES>
__global__ __launch_bounds__(WAVES * 64) void prepare_kernel(
    const uint64_t *__restrict__ ctW, int k, uint32_t C, int log_n, int L, LimbTable limbs, int KB,
    uint4 *__restrict__ planes, uint64_t *__restrict__ colsum)
{
    __shared__ uint64_t part[WAVES][64][2];
    const uint32_t lane = threadIdx.x & 63u;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t ct = blockIdx.x;
    // (the 32 columns of a tile lie in one limb: N >= 32)
    const Limb &P = limbs.limb[((ct * kTile) >> log_n) % (uint32_t)L];
    const uint64_t q = P.q, half = (q - 1) >> 1;
    uint64_t bias = 0;                              // 0x80 in each of the DQ low bytes
#pragma unroll
    for (int d = 0; d < DQ; ++d) bias |= (uint64_t)0x80 << (8 * d);

    // sums of the lower and of the upper halves of the words: k < 2^24 of 32 bits each
    uint64_t sum_lo = 0, sum_hi = 0;
    for (int kb = wave; kb < KB; kb += WAVES) {
        const int i0 = kb * kTile + (int)(lane >> 5) * 16;
        const uint64_t *const p = ctW + (size_t)i0 * C + (ct * kTile + (lane & 31u));
        uint64_t c[16];
        if ((kb + 1) * kTile <= k) {
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
        uint4 *const out = planes + ((size_t)ct * KB + kb) * DQ * 64u + lane;
#pragma unroll
        for (int d = 0; d < DQ; ++d) {
            const v4i r = {(int)w[d][0], (int)w[d][1], (int)w[d][2], (int)w[d][3]};
            __builtin_nontemporal_store(r, (v4i *)(out + d * 64));
        }
    }

    part[wave][lane][0] = sum_lo;
    part[wave][lane][1] = sum_hi;
    __syncthreads();
    if (threadIdx.x < 32u) {
        uint64_t lows = 0, highs = 0;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            lows += part[w][lane][0] + part[w][lane + 32][0];
            highs += part[w][lane][1] + part[w][lane + 32][1];
        }
        uint64_t lo = lows, hi = 0;                 // lows + 2^32 highs in 128 bits
        add128(hi, lo, highs >> 32, highs << 32);
        colsum[ct * kTile + lane] = barrett128(hi, lo, P);      // k * q < 2^(b+63)
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
    auto go = [&](auto waves_c) {
        constexpr int WAVES = decltype(waves_c)::value;
        return launch(prepare_kernel<DQ, WAVES>, dim3(CT), dim3(WAVES * 64), stream, ctW, p.k,
                      (uint32_t)p.C, log_n, p.L, p.limbs, KB, (uint4 *)prepared, colsum);
    };
    // Sixteen waves per tile where every wave has a k-block: more loads in flight per compute unit
    // (768 x 16384 residues 35.8 us with 16 waves, 36.6 with 4; 3072 x 16384 of 59 bits 151.7 and
    // 160.3).  With fewer k-blocks most of them would only meet at the barrier (100 x 65536: 23.8
    // and 20.8 us).
    if (KB >= 16) return go(std::integral_constant<int, 16>{});
    // Fewer rows than a k-block has: one wave, so that the compute unit's waves all have tiles of their
    // own (1 x 2^20 residues 58.4 us with 4 waves, 44.1 with 1; 20 x 2^20 87.6 and 60.4).  A whole
    // k-block has sixteen loads in flight per lane as it is (32 x 2^20: 85.2 and 90.4).  A launch has
    // fewer than 2^32 threads, so from 2^24 column tiles on it is one wave too.
    if (p.k < kTile || CT >= (1u << 24)) return go(std::integral_constant<int, 1>{});
    return go(std::integral_constant<int, 4>{});
}

hipError_t launch_prepare(const Problem &p, const uint64_t *ctW, void *prepared, hipStream_t stream)
{
    if (planes_q(p.q_bits_max) == 7) return prepare_impl<7>(p, ctW, prepared, stream);
    return prepare_impl<8>(p, ctW, prepared, stream);
}

}  // namespace nimbus
