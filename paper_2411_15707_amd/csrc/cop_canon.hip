// Matrix-core (int8 MFMA) kernel for the COP accumulation on the CANONICAL layout, gfx950:
// nimbus_cop_matmul without any setup pass.  Same contraction and same reduction as the kernel
// for prepared weights (cop_mfma_kernel.hpp; Algorithm 1 step 2 + step 4 of the paper), but both
// operands arrive as 64-bit words and are split into signed byte planes inside the loop, 64 k a
// stage, one stage ahead of the products:
//
//   ciphertext words  ctW[k][C]: a 64 x 64 tile per stage comes straight into registers, eight
//       consecutive k of one column per thread (a wave reads whole rows of 64 columns), asked
//       for a stage before they are recoded into signed bytes (digits of the residue c itself:
//       unlike the setup pass of the other kernel it does not centre first where it need
//       not, which would cost five vector instructions a word), transposed and written as one
//       8-byte word into each of the DQ operand tiles;
//   shares  X[m][k]: a 128 x 64 tile per stage from L2, two items of eight consecutive k of one
//       row per thread, one 8-byte word into each of the DX planes.
//
// The operand tiles in LDS (two buffers) have the register order of v_mfma_i32_16x16x64_i8; wave w owns
// 16 columns and half of the 16-row tiles, its operands rotate, and there is one barrier per
// stage, all as in the kernel for prepared weights.  The column sums S that the share offset OFFX
// needs (x = x' + OFFX) are gathered on the way: every thread adds up the words it converts,
// the partial sums meet in LDS after the loop.
//
// What bounds it: the conversion's vector instructions (about 124 per thread and stage) next to
// the products; with few stages the fetch of code that runs once (asking for the second stage's words
// together with the first's changes nothing).  Against the kernel of cop_canon32.hip (32 k a stage, raw words
// through LDS, 4-byte writes): 128 x 768 x 16384, 20-bit shares, 46.9 us -> 41.8; half as many LDS writes
// and barriers, no words through LDS on the way in, and few rows pay for their own 16-row tiles only (1 x
// 768 x 16384 1.4 times as fast).  Where that kernel is the faster one it runs: stages_of_32().
#include "cop_canon.hpp"

namespace nimbus {


typedef int v2i __attribute__((ext_vector_type(2)));

template <int OFF>
__device__ __forceinline__ void lds_write_b64(uint32_t addr, uint32_t lo, uint32_t hi)
{
    const uint64_t v = (uint64_t)hi << 32 | lo;
    asm volatile("ds_write_b64 %0, %1 offset:%2" ::"v"(addr), "v"(v), "n"(OFF) : "memory");
}

// FULL: m is a multiple of 128.  SHARED: several row blocks per column tile (m > 128); they
// start at the same k and load the ciphertext without the streaming hint, so that the
// tile is found in the L2 of their XCD by all but the first.
// CENTRE: the ciphertext digits are those of the centred residue (c or c - q) instead of the
// residue itself.  Needed when a residue can exceed what DQ signed digits express,
// 127 (256^DQ - 1) / 255 (moduli within half a percent of 2^(8 DQ - 1)); costs five vector
// instructions a word.
template <int DX, int DQ, bool FULL, bool SHARED, bool CENTRE>
__global__ __launch_bounds__(512, 1) void cop_canon_kernel(const CanonArgs ca)
{
    const MfmaArgs &a = ca.e;
    constexpr int ND = DX + DQ - 1;
    // operand tiles of one stage, 16 rows (or columns) x 64 k of one plane in 1 KB: 8 DX of the
    // shares, 4 DQ of the ciphertext, twice
    constexpr int A_BYTES = 8 * DX * kTileBytes, B_BYTES = 4 * DQ * kTileBytes, STAGE = A_BYTES + B_BYTES;
    static_assert(2 * STAGE <= 160 * 1024, "LDS");
    static_assert(64 * 8 * 16 <= STAGE, "the column sums reuse the operand tiles");
    __shared__ __attribute__((aligned(1024))) unsigned char lds[2 * STAGE];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // 0..7
    const int wh = wave >> 2, wc = wave & 3;        // 16-row tiles wh, wh + 2, ...; 16-column group

    // workgroup -> (64-column tile, row block), as in the kernel for prepared weights
    uint32_t ct2, rb;
    {
        const uint32_t id = blockIdx.x;
        const uint32_t RB = (uint32_t)a.RB;
        const uint32_t CT2a = (a.CT >> 1) & ~7u;
        if (!SHARED) {
            rb = 0;
            ct2 = id;
        } else if (id < CT2a * RB) {
            const uint32_t xcd = id & 7u, slot = id >> 3;
            rb = slot % RB;
            ct2 = (slot / RB) * 8u + xcd;
        } else {
            const uint32_t t = id - CT2a * RB;
            rb = t % RB;
            ct2 = CT2a + t / RB;
        }
    }
    const int block_rows = FULL ? 128 : (int)a.block_tiles * kTile;
    const int row_first = (int)rb * block_rows;
    const int row_end = FULL || row_first + block_rows < a.m ? row_first + block_rows : a.m;
    const int S = (a.KB + 1) >> 1;                  // stages of 64 k
    const uint32_t K = (uint32_t)ca.k, C = a.C;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(NIMBUS_AS3 void *)&lds[0];

    // stage s is the 64 k from 64 ((s + s_start) mod S) on (column tiles start at different k)
    uint32_t s_start = ct2 % (uint32_t)S;
    auto next_stage = [&](uint32_t s) -> uint32_t { return s + 1 == (uint32_t)S ? 0u : s + 1; };

    // ---- ciphertext: wave w converts the k 8 w .. 8 w + 7 of the stage, lane l column l ----
    // Rows past k read as zero, from an offset that lies behind the end of every descriptor (ctW is a
    // multiple of 512 bytes and smaller than 4 GB), and a zero word recodes to zero digits.
    constexpr uint32_t kPastEnd = 0xfffffe00u;
    const uint64_t ct_first = (uint64_t)ct2 * 64u * 8u;
    const __amdgpu_buffer_rsrc_t rsrc_ct = __builtin_amdgcn_make_buffer_rsrc(
        (void *)((const unsigned char *)ca.ctW + ct_first), 0,
        (uint32_t)((uint64_t)K * C * 8u - ct_first), 0x00027000);
    const uint32_t row_bytes = C * 8u;
    // its place in the operand tiles (slot j 16 + column % 16 of the tile, half of the 16 bytes);
    // plane b follows at b KB.  Share tiles rotate the rows of a k-quarter j by 4 j, so that the
    // eight lanes of a row (below) write to different banks; so do these.
    const uint32_t cv_j = (uint32_t)wave >> 1;
    const uint32_t cv_out = lds0 + A_BYTES + ((uint32_t)lane >> 4) * (DQ * kTileBytes) +
                            (cv_j * 16u + (((uint32_t)lane + 4u * cv_j) & 15u)) * 16u + ((uint32_t)wave & 1u) * 8u;
    uint64_t cv_q = 0;                              // modulus of the lane's column (N >= 32)
    if constexpr (CENTRE) {
        const uint32_t blk = (ct2 * 64u + (uint32_t)(lane & 32)) >> a.log_n;
        const uint32_t l = a.L == 1 ? 0u : blk - (uint32_t)a.L * __umulhi(blk, a.l_magic);
        cv_q = a.q[l];
    }
    const uint64_t cv_half = (cv_q - 1) >> 1;
    uint64_t bias = 0;                              // 0x80 in each of the DQ low bytes
#pragma unroll
    for (int d = 0; d < DQ; ++d) bias |= (uint64_t)0x80 << (8 * d);
    // sums of the lower and of the upper halves of the words this thread converts (one
    // 32 x 32 + 64-bit multiply-add by one each: k / 8 words of 32 bits cannot overflow 64)
    uint64_t sum_lo = 0, sum_hi = 0;

    // ---- shares: item i of a thread is eight k of row 16 w + 8 i + l / 8, octet l % 8 ----
    const uint64_t x_first = (uint64_t)row_first * K * 8u;
    const uint64_t x_left = (uint64_t)a.m * K * 8u - x_first;
    const __amdgpu_buffer_rsrc_t rsrc_x = __builtin_amdgcn_make_buffer_rsrc(
        (void *)((const unsigned char *)ca.X + x_first), 0,
        x_left > 0xffffffffull ? 0xffffffffu : (uint32_t)x_left, 0x00027000);
    uint32_t x_off[2], x_out[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const uint32_t r = 16u * (uint32_t)wave + 8u * (uint32_t)i + ((uint32_t)lane >> 3), o = (uint32_t)lane & 7u;
        x_off[i] = r * K * 8u + o * 64u;
        x_out[i] = lds0 + (r >> 4) * (DX * kTileBytes) + ((o >> 1) * 16u + ((r + 4u * (o >> 1)) & 15u)) * 16u + (o & 1u) * 8u;
    }

    v2i cw[8];                                      // raw words of the stage after the one at hand
    auto load_ct = [&](uint32_t s) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const uint32_t row = s * 64u + (uint32_t)wave * 8u + (uint32_t)i;
            cw[i] = __builtin_amdgcn_raw_buffer_load_b64(
                rsrc_ct, (row < K ? row * row_bytes : kPastEnd) + (uint32_t)lane * 8u, 0, SHARED ? 0 : 2);
        }
    };
    auto load_x = [&](v4i (&x)[4], int i, uint32_t s) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
            x[u] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_x, x_off[i] + s * 512u + (uint32_t)u * 16u, 0, 0);
    };
    // words 4 h .. 4 h + 3: the sums, and the signed base-256 digits of the residue (centred first where
    // it has to be): c' + 0x80..80 has the bytes digit + 128, and flipping bit 7 of each gives
    // the digits as signed bytes
    auto ct_recode = [&](int h) {
#pragma unroll
        for (int i = 4 * h; i < 4 * h + 4; ++i) {
            const uint64_t c = (uint64_t)(uint32_t)cw[i].y << 32 | (uint32_t)cw[i].x;
            asm("v_mad_u64_u32 %0, vcc, %1, 1, %0" : "+v"(sum_lo) : "v"((uint32_t)c) : "vcc");
            asm("v_mad_u64_u32 %0, vcc, %1, 1, %0" : "+v"(sum_hi) : "v"((uint32_t)(c >> 32)) : "vcc");
            const uint64_t cc = CENTRE && c > cv_half ? c - cv_q : c;  // two's complement of c'
            const uint64_t d = (cc + bias) ^ bias;
            cw[i] = v2i{(int)(uint32_t)d, (int)(uint32_t)(d >> 32)};
        }
    };
    auto ct_write = [&](auto half_c, uint32_t buf) {     // planes 0-3, or 4 .. DQ-1
        constexpr int half = decltype(half_c)::value;
        const uint32_t at = cv_out + buf;
        uint32_t lo[4], hi[4];
        transpose4((uint32_t)cw[0][half], (uint32_t)cw[1][half], (uint32_t)cw[2][half], (uint32_t)cw[3][half], lo);
        transpose4((uint32_t)cw[4][half], (uint32_t)cw[5][half], (uint32_t)cw[6][half], (uint32_t)cw[7][half], hi);
        static_for<0, half ? DQ - 4 : 4>([&](auto d_c) {
            constexpr int d = decltype(d_c)::value;
            lds_write_b64<(4 * half + d) * kTileBytes>(at, lo[d], hi[d]);
        });
    };
    auto x_write = [&](const v4i (&x)[4], int i, uint32_t buf) {
        const uint32_t at = x_out[i] + buf;
        uint32_t lo[4], hi[4];
        // flipping bit 7 of the shifted bytes turns them into the digits byte - 128
        transpose4((uint32_t)x[0].x ^ a.offx, (uint32_t)x[0].z ^ a.offx, (uint32_t)x[1].x ^ a.offx,
                   (uint32_t)x[1].z ^ a.offx, lo);
        transpose4((uint32_t)x[2].x ^ a.offx, (uint32_t)x[2].z ^ a.offx, (uint32_t)x[3].x ^ a.offx,
                   (uint32_t)x[3].z ^ a.offx, hi);
        static_for<0, DX>([&](auto d_c) {
            constexpr int d = decltype(d_c)::value;
            lds_write_b64<d * kTileBytes>(at, lo[d], hi[d]);
        });
    };

    // ---- operands out of LDS: 16-row tile t is rows 16 t .. of the block, this wave has wh + 2 i ----
    const uint32_t slot = ((uint32_t)lane & 48u) + (((uint32_t)lane + 4u * ((uint32_t)lane >> 4)) & 15u);
    const uint32_t laneA = lds0 + (uint32_t)(wh * DX) * kTileBytes + slot * 16u;
    const uint32_t laneB = lds0 + A_BYTES + (uint32_t)(wc * DQ) * kTileBytes + slot * 16u;

    // the stages for a wave of NT 16-row tiles, then its part of the epilogue
    auto pass = [&](auto nt_c) {
        constexpr int NT = decltype(nt_c)::value, NA = NT > 0 ? NT : 1;
        constexpr int NG = NT * DX;                 // groups of DQ products, one share operand each
        // Both items of the shares a stage ahead where the registers allow it, else the second is asked
        // for when the first is converted (128 x 768 x 16384, 20-bit shares: 41.8 us and 45.1; with
        // spills 36 bytes a thread cost a tenth).
        constexpr bool BOTH = ND * NT * 4 + DQ * 4 <= (FULL && !CENTRE ? 176 : 160);
        v4i xw[BOTH ? 2 : 1][4];
        uint32_t s_load = s_start;                  // next stage to ask for
        load_x(xw[0], 0, s_load);
        if constexpr (BOTH) load_x(xw[1], 1, s_load);
        load_ct(s_load);
        v4i acc[ND][NA];
#pragma unroll
        for (int d = 0; d < ND; ++d)
#pragma unroll
            for (int i = 0; i < NT; ++i) {
                acc[d][i] = v4i{0, 0, 0, 0};
                tie(acc[d][i]);
            }
        // stage 0 converted, stage 1 asked for
        x_write(xw[0], 0, 0);
        if constexpr (!BOTH) load_x(xw[0], 1, s_load);
        s_load = next_stage(s_load);
        if constexpr (BOTH) {
            x_write(xw[1], 1, 0);
            if (S > 1) {
                load_x(xw[0], 0, s_load);
                load_x(xw[1], 1, s_load);
            }
        }
        ct_recode(0);
        ct_recode(1);
        ct_write(std::integral_constant<int, 0>{}, 0);
        ct_write(std::integral_constant<int, 1>{}, 0);
        if constexpr (!BOTH) {
            x_write(xw[0], 1, 0);
            if (S > 1) load_x(xw[0], 0, s_load);
        }
        if (S > 1) load_ct(s_load);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        v4i xa[2], xb[DQ];
        uint32_t rd = 0;                            // buffer that is read next
        auto read_a = [&](auto g_c) {
            constexpr int g = decltype(g_c)::value;
            xa[g & 1] = lds_read_b128<(g / DX * 2 * DX + g % DX) * kTileBytes>(laneA + rd);
        };
        auto read_b = [&](auto d_c) {
            xb[decltype(d_c)::value] = lds_read_b128<decltype(d_c)::value * kTileBytes>(laneB + rd);
        };
        if constexpr (NT > 0) {
            read_a(std::integral_constant<int, 0>{});
            static_for<0, DQ>([&](auto d_c) { read_b(d_c); });
        }
        for (int s = 0; s < S; ++s) {
            const uint32_t nb = rd ? 0u : (uint32_t)STAGE;
            // conversion of stage s + 1, in pieces between the products; what it frees asks for stage s + 2
            const bool more = s + 1 < S, ask = s + 2 < S;
            auto piece = [&](auto n_c) {
                constexpr int n = decltype(n_c)::value;
                if (!more) return;
                if constexpr (n == 0) {
                    x_write(xw[0], 0, nb);
                    if constexpr (!BOTH) load_x(xw[0], 1, s_load);
                    s_load = next_stage(s_load);
                    if (BOTH && ask) load_x(xw[0], 0, s_load);
                } else if constexpr (n == (BOTH ? 1 : 5)) {
                    x_write(xw[BOTH], 1, nb);
                    if (ask) load_x(xw[BOTH], BOTH, s_load);
                } else if constexpr (n == (BOTH ? 2 : 1)) {
                    ct_recode(0);
                } else if constexpr (n == (BOTH ? 3 : 2)) {
                    ct_recode(1);
                } else if constexpr (n == (BOTH ? 4 : 3)) {
                    ct_write(std::integral_constant<int, 0>{}, nb);
                } else if constexpr (n == (BOTH ? 5 : 4)) {
                    ct_write(std::integral_constant<int, 1>{}, nb);
                }
                if constexpr (n == 5)
                    if (ask) load_ct(s_load);
            };
            constexpr int PIECES = 6;
            auto meet = [&]() {
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                rd = nb;
            };
            if constexpr (NT == 0) {
                static_for<0, PIECES>([&](auto n_c) { piece(n_c); });
                meet();
            } else {
                constexpr int SPAN = (NG - 1) * DQ;
                static_for<0, NG>([&](auto g_c) {
                    constexpr int g = decltype(g_c)::value, i = g / DX, dx = g % DX;
                    if constexpr (g == NG - 1) meet();
                    if constexpr (g + 1 < NG) read_a(std::integral_constant<int, g + 1>{});
                    else xa[(g + 1) & 1] = lds_read_b128<0>(laneA + rd);
                    static_for<0, DQ>([&](auto d_c) {
                        constexpr int dq = decltype(d_c)::value, pos = g * DQ + dq;
                        if constexpr (g == 0) wait_lds<DQ - dq>(xb[dq]);
                        else if constexpr (dq == 0 && g < NG - 1) wait_lds<1>(xa[g & 1]);
                        tie(xa[g & 1]);
                        tie(xb[dq]);
                        acc[dx + dq][i] =
                            __builtin_amdgcn_mfma_i32_16x16x64_i8(xa[g & 1], xb[dq], acc[dx + dq][i], 0, 0, 0);
                        tie(acc[dx + dq][i]);
                        static_for<0, PIECES>([&](auto n_c) {
                            if constexpr (decltype(n_c)::value * SPAN / PIECES == pos) piece(n_c);
                        });
                        if constexpr (g == NG - 1) read_b(d_c);
                    });
                });
                if constexpr (NG % 2 == 1) {        // an odd number of groups: the next stage starts from set 0
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                    tie(xa[1]);
                    xa[0] = xa[1];
                }
            }
        }
        // (the last stage has read operands ahead: nothing may copy or reuse their registers before they are back)
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        if constexpr (NT > 0) {
            tie(xa[NG & 1]);
            static_for<0, DQ>([&](auto d_c) { tie(xb[decltype(d_c)::value]); });
        }
        __builtin_amdgcn_s_barrier();
        {
            const uint32_t at = lds0 + ((uint32_t)lane * 8u + (uint32_t)wave) * 16u;
            asm volatile("ds_write_b64 %0, %1\n\tds_write_b64 %0, %2 offset:8"
                         ::"v"(at), "v"(sum_lo), "v"(sum_hi) : "memory");
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        if constexpr (NT > 0) {
            uint32_t limb;
            {
                const uint32_t blk = (ct2 * 64u + (uint32_t)wc * 16u) >> a.log_n;
                limb = a.L == 1 ? 0u : blk - (uint32_t)a.L * __umulhi(blk, a.l_magic);
                limb = __builtin_amdgcn_readfirstlane(limb);
            }
            // column sums: the eight waves' parts meet in LDS (over the operand tiles)
            uint64_t colsum_S;
            {
                const uint32_t at = lds0 + ((uint32_t)(wc * 16 + (lane & 15)) * 8u) * 16u;
                uint64_t lows = 0, highs = 0;       // each below 2^32 k
                static_for<0, 8>([&](auto g_c) {
                    constexpr int g = decltype(g_c)::value;
                    uint64_t plo, phi;
                    asm volatile("ds_read_b64 %0, %2 offset:%3\n\tds_read_b64 %1, %2 offset:%4\n\t"
                                 "s_waitcnt lgkmcnt(0)"
                                 : "=&v"(plo), "=&v"(phi) : "v"(at), "n"(g * 16), "n"(g * 16 + 8) : "memory");
                    lows += plo;
                    highs += phi;
                });
                uint64_t lo = lows, hi = 0;         // lows + 2^32 highs in 128 bits
                add128(hi, lo, highs >> 32, highs << 32);
                colsum_S = barrett128(hi, lo, ca.limbs.limb[limb]);      // k * q < 2^(b+63)
            }
            constexpr int NE = 4 * NT;
            const int row0 = row_first + 16 * wh + 4 * (lane >> 4);
            const uint32_t col = ct2 * 64u + (uint32_t)wc * 16u + (uint32_t)(lane & 15);
            auto roff = [](int r) -> int { return 32 * (r >> 2) + (r & 3); };
            cop_finish<ND, NE, FULL>(
                [&](int d, int r) -> int32_t { return acc[d][r >> 2][r & 3]; }, roff,
                [&](uint64_t (&w)[NE]) {
#pragma unroll
                    for (int r = 0; r < NE; ++r) w[r] = 0;
                    if (!a.mask) return;
                    const uint64_t *const mask0 = a.mask + ((size_t)row0 * C + col);
#pragma unroll
                    for (int r = 0; r < NE; ++r)
                        if (FULL || row0 + roff(r) < row_end)
                            w[r] = __builtin_nontemporal_load(&mask0[(size_t)roff(r) * C]);
                },
                a, nullptr, a.out, limb, colsum_S, row0, col, row_end);
        }
    };
    if constexpr (FULL) {
        pass(std::integral_constant<int, 4>{});
    } else {
        const int nt = ((row_end - row_first + 15) / 16 + 1 - wh) >> 1;
        switch (nt) {
        case 3:
        case 4: pass(std::integral_constant<int, 4>{}); break;
        case 2: pass(std::integral_constant<int, 2>{}); break;
        case 1: pass(std::integral_constant<int, 1>{}); break;
        default: pass(std::integral_constant<int, 0>{});
        }
    }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
// DQ signed digits express the values up to 127 (256^DQ - 1) / 255: is there a limb whose
// residues can be larger?
static bool needs_centring(const Problem &p, int DQ)
{
    uint64_t top = 0;
    for (int d = 0; d < DQ; ++d) top = top * 256u + 127u;
    for (int l = 0; l < p.L; ++l)
        if (p.limbs.limb[l].q - 1 > top) return true;
    return false;
}

bool canon_supported(const Problem &p)
{
    if (p.x_bits > 32 || !mfma_supported(p)) return false;
    // where the digits stand for the residues themselves, not the centred ones, the sums are
    // twice as large and the multiple of q that makes them non-negative is one bit longer; the
    // value reduced in the epilogue must stay below 2^47 q all the same
    if (!needs_centring(p, planes_q(p.q_bits_max)) && bias_shift(p) + 3 > 47) return false;
    // four share planes times eight ciphertext planes: eleven accumulator tiles and the
    // conversion's registers do not fit one wave
    if (planes_x(p.x_bits) == 4 && planes_q(p.q_bits_max) == 8) return false;
    // 32-bit offsets inside the buffer descriptors: the whole of ctW, and the 128 rows of X of
    // a row block
    if ((uint64_t)p.k * p.C * 8u >= (1ull << 32)) return false;
    if ((uint64_t)p.k * 8u * 128u >= (1ull << 32)) return false;
    return true;
}

static CanonArgs canon_args(const Problem &p, int DX, int DQ, const uint64_t *X, const uint64_t *ctW,
                            const uint64_t *mask, uint64_t *out)
{
    CanonArgs ca{};
    fill_common_args(p, DX, mask, nullptr, out, &ca.e, needs_centring(p, DQ) ? 0 : 1);
    ca.X = X;
    ca.ctW = ctW;
    ca.k = p.k;
    ca.limbs = p.limbs;
    return ca;
}

// Which kernel: that of cop_canon32.hip (32 k a stage) or this one (us, there and here).
//   three share and eight ciphertext planes: there (20-bit shares, moduli of 62 bits, 128 x 768 x 16384 50.3
//       and 54.4, 100 x 1500 x 8192 78.8 and 97.3: the accumulators leave too few registers here);
//   four share planes and centred digits, m a multiple of 128: there (32-bit shares, moduli just below
//       2^55, 128 x 160 x 8192 17.5 and 20.1, 128 x 928 x 2048 54.5 and 58.9; 512 x 416 x 8192 even, 256 x
//       1504 x 4096 here by 1 %: this kernel spills four registers);
//   more than 96 rows in a row block and one, three or five k-blocks, without row tests seven too:
//       there (20-bit shares, 128 x 95 x 8192 13.6 and 15.3, 128 x 160 x 8192 16.1 and 17.2): the last stage is
//       half empty, and a second one costs the fetch of the whole loop's code;
//   else here (128 x 60 x 8192 11.9 and 11.0, 300 x 220 x 8192 35.4 and 34.0, 70 x 95 x 8192 13.0 and 11.9).
// Over 2559 sizes of 40 to 512 rows the choice is 0.4 % off the better one on average and 10 % at worst (191
// x 1502 x 4096, 32-bit shares, centred); this kernel everywhere would be 1.2 % and 16 % off.
static bool stages_of_32(const Problem &p, int DX, int DQ, bool centre, int block_rows)
{
    const int KB = kblocks(p.k);
    if (DX == 3 && DQ == 8) return true;
    if (DX == 4 && centre && p.m % 128 == 0) return true;
    return block_rows > 96 && KB % 2 == 1 && (p.m % 128 == 0 ? KB <= 7 : KB <= 5);
}

template <int DX, int DQ>
static hipError_t canon_impl(const Problem &p, const uint64_t *X, const uint64_t *ctW,
                             const uint64_t *mask, uint64_t *out, hipStream_t stream)
{
    const bool centre = needs_centring(p, DQ);
    CanonArgs ca = canon_args(p, DX, DQ, X, ctW, mask, out);
    const dim3 grid((ca.e.CT / 2) * (uint32_t)ca.e.RB);
    const bool full = p.m % 128 == 0, shared = ca.e.RB > 1;
    ca.e.block_tiles = (uint32_t)(((p.m + kTile - 1) / kTile + ca.e.RB - 1) / ca.e.RB);     // row blocks of even size
    const int block_rows = (int)ca.e.block_tiles * kTile < p.m ? (int)ca.e.block_tiles * kTile : p.m;
    if (stages_of_32(p, DX, DQ, centre, block_rows)) return launch_cop_canon32<DX, DQ>(p, ca, centre, stream);
    if constexpr (DX == 3 && DQ == 8) {
        return hipErrorInvalidValue;
    } else {
        auto go = [&](auto full_c, auto shared_c, auto centre_c) {
            return launch(cop_canon_kernel<DX, DQ, decltype(full_c)::value, decltype(shared_c)::value,
                                           decltype(centre_c)::value>,
                          grid, dim3(512), stream, ca);
        };
        using T = std::true_type;
        using F = std::false_type;
        if constexpr (DX == 4) {                    // (centred and without row tests: cop_canon32.hip)
            if (centre) return shared ? go(F{}, T{}, T{}) : go(F{}, F{}, T{});
        } else if constexpr (DQ == 7) {             // (eight digits express every q < 2^62)
            if (centre) {
                if (full) return shared ? go(T{}, T{}, T{}) : go(T{}, F{}, T{});
                return shared ? go(F{}, T{}, T{}) : go(F{}, F{}, T{});
            }
        }
        if (full) return shared ? go(T{}, T{}, F{}) : go(T{}, F{}, F{});
        return shared ? go(F{}, T{}, F{}) : go(F{}, F{}, F{});
    }
}

hipError_t launch_cop_canon(const Problem &p, const uint64_t *X, const uint64_t *ctW,
                            const uint64_t *mask, uint64_t *out, hipStream_t stream)
{
    const int DX = planes_x(p.x_bits), DQ = planes_q(p.q_bits_max);
#define NIMBUS_CASE(dx, dq) \
    if (DX == dx && DQ == dq) return canon_impl<dx, dq>(p, X, ctW, mask, out, stream);
    NIMBUS_CASE(2, 7)
    NIMBUS_CASE(3, 7)
    NIMBUS_CASE(4, 7)
    NIMBUS_CASE(2, 8)
    NIMBUS_CASE(3, 8)
#undef NIMBUS_CASE
    return hipErrorInvalidValue;
}

}  // namespace nimbus
