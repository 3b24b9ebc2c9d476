// Matrix-core (int8 MFMA) kernel of the COP accumulation for few token rows (up to 32), or more of them
// on few columns (32 at a time), gfx950:
// the same contraction, operand bytes and epilogue as cop_mfma_kernel.hpp (Algorithm 1 step 2 + step 4
// of the paper), laid out for a call that is nothing but a pass over the weights.
//
// What bounds it: the bytes of the prepared weights (m = 1, 768 x 16384 residues of 54 bits:
// 88 MB, 14 us at the 6.3 TB/s that a streaming read reaches; the products of 16 rows take a
// fifth of that) and, with few columns, what is in flight of them.  So nothing is shared and nothing is synchronised in the loop: a wave owns 16
// columns and a slice of k, and its operand tiles come from memory straight into the registers
// the products read them from, PD stages of 64 k ahead.  With eight waves of 7 KB a stage that
// keeps up to 224 KB in flight per compute unit, and whatever the wave waits for is its own.
//
// v_mfma_i32_16x16x64_i8: 16 rows x 16 columns x 64 k, a stage is two k-blocks of the prepared
// layout.  Lane l holds row (or column) l % 16 and the k-slots 16 (l / 16) .. +15 of the stage:
// 16 bytes that lie together in the 32 x 32 operand tiles of the layout (k-block l / 32 of the
// stage, half (l / 16) % 2), so a lane's operand is one 16-byte load at its own address.
//
// A workgroup is eight waves, CGW column groups x KS slices of k (CGW KS = 8).  Slices are for
// weights with too few columns to fill the chip: the host takes as many as bring the number of
// workgroups to the number of compute units.  The slices' sums meet in LDS once, at the end.
//
// Shares: staged planes (the batch and the staged entry points), read like the weights; or, for
// up to 32 rows of the entry points that stage and multiply in one call, the raw words (RAW):
// the workgroup splits them into byte planes in LDS while its first weights are on their way,
// and the staging launch and the gap behind it go away.  The planes are left in the workspace
// all the same (workgroup b writes the stages b, b + grid, ...), as that entry point promises.
//
// Measured (us a call in a HIP graph, 20-bit shares, 54-bit moduli where nothing else is said), with every slice run
// in whole rounds of the stages in flight and elements finished one by one, and now: 8 x 64 x 2048 7.7 ->
// 5.1, 1 x 73 x 16384 8.7 -> 6.4, 15 x 50 x 4096 8.6 -> 6.2, 2 x 386 x 4096 8.5 -> 6.8, 1 x 768 x 16384 18.5 ->
// 17.2 (88 MB), 128 x 1536 x 2048 16.3 -> 15.1; 49 sizes of 1 to 64 rows 1.12 times as fast.  With a third and a
// fourth 16-row tile the shares' planes cost more than the tiles of cop_mfma_kernel.hpp.
#include "cop_mfma_common.hpp"

namespace nimbus {

struct ThinArgs {
    const uint64_t *X;        // RAW: [m][k]
    uint4 *staged;            // RAW: where the planes are left, [KB][DX][64] uint4 (one row tile)
    int k;
    int half_shift;           // RAW: 0 or 32, which half of a share
    uint32_t log_ks;          // KS = 2^log_ks
    uint32_t quads_magic;     // RAW: ceil(2^32 / Q), Q = 16 ceil(KB / 2) four-word items of a row: x / Q = umulhi(x, .)
};

constexpr int kThinRows = 32;
constexpr int kThinStage = 64;                          // k of a stage
constexpr int kThinSharesLds = 144 * 1024;

// where a wave's operands of the shares come from
enum ThinShares {
    kDirect,    // staged planes, read like the weights, per wave
    kCopied,    // staged planes, brought into LDS once per workgroup
    kRaw,       // the shares themselves, split into planes in LDS once per workgroup
    kRows       // as kDirect, for a call of more than 32 rows: a workgroup takes one 32-row tile of them
};

// stages in flight per wave: what 256 registers hold next to the accumulators, four at most
constexpr int thin_depth(int DX, int DQ, int RT16, ThinShares from)
{
    const bool direct = from == kDirect || from == kRows;
    const int accumulators = (DX + DQ - 1) * 4 * RT16;
    const int stage = DQ * 4 + (direct ? DX * 4 * RT16 : 0);
    const int fit = (256 - 40 - accumulators - (direct ? 0 : 20)) / stage;
    return fit > 4 ? 4 : fit < 2 ? 2 : fit;
}

template <int DX, int DQ, int RT16, ThinShares FROM>
struct Thin {
    static constexpr int ND = DX + DQ - 1;
    static constexpr int PD = thin_depth(DX, DQ, RT16, FROM);
    // planes of the shares, [stage][16-row tile][plane][64 lanes][16 B]
    static constexpr int A_LDS = FROM == kDirect || FROM == kRows ? 0 : kThinSharesLds;
    // the slices' sums meet TP tiles at a time: two where eight waves' sums of two fit the LDS
    static constexpr int TP = RT16 > 1 && ND <= 9 ? 2 : 1;
    static constexpr int SUM_LDS = 8 * ND * TP * 1024;
    static constexpr int PHASES = (RT16 + TP - 1) / TP;
    static constexpr int LDS = A_LDS > SUM_LDS ? A_LDS : SUM_LDS;
};

__device__ __forceinline__ v4i load_operand(__amdgpu_buffer_rsrc_t rsrc, uint32_t off, bool stream)
{
    return stream ? __builtin_amdgcn_raw_buffer_load_b128(rsrc, off, 0, 2)
                  : __builtin_amdgcn_raw_buffer_load_b128(rsrc, off, 0, 0);
}

template <int DX, int DQ, int RT16, ThinShares FROM, int NB>
__global__ __launch_bounds__(512, 2) void cop_thin_kernel(const MfmaArgs a, const BatchPtrs<NB> b, const ThinArgs t)
{
    using T_ = Thin<DX, DQ, RT16, FROM>;
    constexpr int ND = T_::ND, PD = T_::PD;
    constexpr bool RAW = FROM == kRaw, IN_LDS = FROM == kRaw || FROM == kCopied;
    static_assert(RT16 <= 2, "one row tile of the staged planes");
    // (the scalar arguments in one batch, not each next to its first use: see cop_mfma_kernel.hpp)
    if constexpr (NB == 1)
        asm volatile("" ::"s"(b.prob[0].xd), "s"(b.prob[0].planes), "s"(b.prob[0].colsum), "s"(b.prob[0].mask),
                     "s"(b.prob[0].out));
    asm volatile("" ::"s"(a.m), "s"(a.KB), "s"(a.RB), "s"(a.N), "s"(a.L), "s"(a.C), "s"(a.CT), "s"(a.log_n),
                 "s"(a.l_magic), "s"(a.offx), "s"(t.log_ks));
    if constexpr (RAW)
        asm volatile("" ::"s"(t.X), "s"(t.staged), "s"(t.k), "s"(t.half_shift), "s"(t.quads_magic));
    __shared__ __attribute__((aligned(1024))) unsigned char lds[T_::LDS];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t log_cgw = 3u - t.log_ks;
    // (kRows: the row tiles of a column group run on one XCD side by side, so that its weights
    // cross the fabric once; see map_tile in cop_mfma_kernel.hpp)
    uint32_t cb = blockIdx.x, row_tile = 0;
    if constexpr (FROM == kRows) {
        const uint32_t RB = (uint32_t)a.RB, whole = (gridDim.x / RB) & ~7u;
        if (cb < whole * RB) {
            const uint32_t slot = cb >> 3;
            row_tile = slot % RB;
            cb = slot / RB * 8u + (cb & 7u);
        } else {
            const uint32_t rest = cb - whole * RB;
            row_tile = rest % RB;
            cb = whole + rest / RB;
        }
    }
    const uint32_t row_first = row_tile * 32u;
    const uint32_t cg = (cb << log_cgw) + ((uint32_t)wave & ((1u << log_cgw) - 1u));
    const uint32_t ks = (uint32_t)wave >> log_cgw;
    const bool active = cg < a.CT * 2u;                 // (the last workgroup may have columns to spare)
    const ProblemPtrs pp = b.prob[NB == 1 ? 0 : blockIdx.y];
    const int KB = a.KB;
    const uint32_t S = ((uint32_t)KB + 1u) >> 1;
    // this wave's stages: s0 .. s1-1, started at a place that follows from the column tile so
    // that waves which walk equally spaced regions do not ask the same channels at one moment
    const uint32_t s0 = (S * ks) >> t.log_ks, s1 = (S * (ks + 1u)) >> t.log_ks;
    const uint32_t len = active ? s1 - s0 : 0u;
    const uint32_t j = (uint32_t)lane >> 4, r16 = (uint32_t)lane & 15u;
    const uint32_t ct = cg >> 1, c16 = cg & 1u;

    // Element e of the lane in 16-row tile i is row 16 i + 4 j + e.  One slice: the wave finishes
    // every element.  Several: their sums meet TP tiles (4 TP elements) at a time, and wave ks of a
    // column group finishes the elements ks ne .. of them, ne = max(1, 4 TP / KS).
    const uint32_t col = cg * 16u + r16;
    const auto share = [&](int phase, uint32_t &tile, uint32_t &e0) -> uint32_t {   // elements of this wave
        const uint32_t tiles = RT16 - phase * T_::TP < T_::TP ? RT16 - phase * T_::TP : T_::TP;
        const uint32_t ne = (4u * tiles) >> t.log_ks ? (4u * tiles) >> t.log_ks : 1u;
        tile = phase * T_::TP + ks * ne / 4u;
        e0 = ks * ne % 4u;
        return active && ks * ne < 4u * tiles ? ne : 0u;
    };
    // ---- operand addresses ----
    // (reads past the last k-block lie past the end of the descriptor and give zero weights:
    // whatever the shares' operand holds there, the products vanish)
    constexpr uint32_t kPastEnd = 0xf0000000u;
    constexpr uint32_t kBStage = 2u * DQ * kTileBytes, kAStage = 2u * DX * kTileBytes;
    const uint32_t b_bytes = (uint32_t)KB * DQ * kTileBytes;
    const uint32_t a_bytes = (uint32_t)KB * DX * kTileBytes;
    const __amdgpu_buffer_rsrc_t rsrc_b = __builtin_amdgcn_make_buffer_rsrc(
        (void *)((const unsigned char *)pp.planes + (size_t)(active ? ct : 0u) * b_bytes), 0, b_bytes, 0x00027000);
    const uint32_t lane_b = (j >> 1) * (DQ * kTileBytes) + ((j & 1u) * 32u + c16 * 16u + r16) * 16u;
    const __amdgpu_buffer_rsrc_t rsrc_a =
        __builtin_amdgcn_make_buffer_rsrc((void *)((const unsigned char *)pp.xd + (size_t)row_tile * a_bytes), 0,
                                          a_bytes, 0x00027000);
    const uint32_t lane_a = (j >> 1) * (DX * kTileBytes) + ((j & 1u) * 32u + r16) * 16u;

    v4i xb[PD][DQ], xs[PD][IN_LDS ? 1 : RT16][DX];
    uint32_t s_load = s0 + (len ? ct % len : 0u);       // next stage to ask for
    uint32_t asked = 0;
    auto next_stage = [&](uint32_t s) { return s + 1u == s1 ? s0 : s + 1u; };
    // one more stage into register set p.  Past the last one the loads are issued all the same, at
    // an offset behind the descriptors' end (no memory is read): the compiler's counted waits then
    // see the same loads on every path through the loop.
    auto ask = [&](auto p_c) {
        constexpr int p = decltype(p_c)::value;
        const uint32_t ob = asked < len ? lane_b + s_load * kBStage : kPastEnd;
        static_for<0, DQ>([&](auto d) {
            xb[p][decltype(d)::value] = load_operand(rsrc_b, ob + decltype(d)::value * kTileBytes, FROM != kRows);
        });
        if constexpr (!IN_LDS) {
            const uint32_t oa = asked < len ? lane_a + s_load * kAStage : kPastEnd;
            static_for<0, RT16 * DX>([&](auto i_c) {
                constexpr int i = decltype(i_c)::value / DX, d = decltype(i_c)::value % DX;
                xs[p][i][d] = load_operand(rsrc_a, oa + i * 256u + d * kTileBytes, false);
            });
        }
        s_load = next_stage(s_load);
        ++asked;
    };
    const __amdgpu_buffer_rsrc_t rsrc_x = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(RAW ? t.X : (const uint64_t *)pp.xd), 0, (uint32_t)a.m * (uint32_t)t.k * 8u, 0x00027000);
    // ---- RAW: four consecutive k of a row per thread and turn, split into byte planes in LDS ----
    const uint32_t quads = S * (kThinStage / 4);        // of a row
    const uint32_t items = (uint32_t)a.m * quads;
    auto read_quad = [&](uint32_t at, v4i (&w)[2]) {
        const uint32_t row = __umulhi(at, t.quads_magic), k0 = (at - row * quads) * 4u;
        const uint32_t off = at < items ? (row * (uint32_t)t.k + k0) * 8u : kPastEnd;
        // (words past the row are dropped by split_quad, words past the end read as zero)
        w[0] = load_operand(rsrc_x, off, false);
        w[1] = load_operand(rsrc_x, off + 16u, false);
    };
    auto split_quad = [&](uint32_t at, const v4i (&w)[2]) {
        if (at >= items) return;
        const uint32_t row = __umulhi(at, t.quads_magic), kq = at - row * quads;
        uint32_t x[4], w4[4];
        const bool upper = t.half_shift != 0;
#pragma unroll
        for (uint32_t i = 0; i < 4; ++i)
            x[i] = kq * 4u + i >= (uint32_t)t.k ? 0u
                   : (uint32_t)(upper ? w[i >> 1][2 * (i & 1) + 1] : w[i >> 1][2 * (i & 1)]) ^ a.offx;
        transpose4(x[0], x[1], x[2], x[3], w4);
        // stage kq / 16, 16-row tile row / 16, lane 16 (kq / 4 % 4) + row % 16, word kq % 4
        const uint32_t first =
            (((kq >> 4) * RT16 + (row >> 4)) * (DX * 64u) + ((kq >> 2) & 3u) * 16u + (row & 15u)) * 4u + (kq & 3u);
#pragma unroll
        for (int d = 0; d < DX; ++d) ((uint32_t *)lds)[first + d * 256u] = w4[d];
    };
    // ---- copied: 16 bytes of a staged plane per thread and turn ----
    const uint32_t chunks = S * (RT16 * DX * 64u);
    auto read_chunk = [&](uint32_t at) -> v4i {
        const uint32_t l = at & 63u, d = at / 64u % DX, i = at / (64u * DX) % RT16, s = at / (64u * DX * RT16);
        const uint32_t kb = 2u * s + (l >> 5);
        const uint32_t off = (kb * DX + d) * kTileBytes + (((l >> 4) & 1u) * 32u + i * 16u + (l & 15u)) * 16u;
        return load_operand(rsrc_a, at < chunks && kb < (uint32_t)KB ? off : kPastEnd, false);
    };
    auto keep_chunk = [&](uint32_t at, v4i v) {
        if (at < chunks) ((v4i *)lds)[at] = v;
    };
    // The turns of a thread, U at a time.  The first U are asked for in front of the weights: loads
    // come back in order.
    auto bring_shares = [&](auto ask_weights) {
        if constexpr (RAW) {
            constexpr uint32_t U = 2;
            v4i w[U][2];
            static_for<0, U>([&](auto u) { read_quad(threadIdx.x + 512u * decltype(u)::value, w[decltype(u)::value]); });
            ask_weights();
            for (uint32_t at = threadIdx.x; at < items;) {
                static_for<0, U>([&](auto u) { split_quad(at + 512u * decltype(u)::value, w[decltype(u)::value]); });
                at += 512u * U;
                if (at < items)
                    static_for<0, U>([&](auto u) { read_quad(at + 512u * decltype(u)::value, w[decltype(u)::value]); });
            }
            __syncthreads();
        } else if constexpr (FROM == kCopied) {
            constexpr uint32_t U = 4;
            v4i w[U];
            static_for<0, U>([&](auto u) { w[decltype(u)::value] = read_chunk(threadIdx.x + 512u * decltype(u)::value); });
            ask_weights();
            for (uint32_t at = threadIdx.x; at < chunks;) {
                static_for<0, U>([&](auto u) { keep_chunk(at + 512u * decltype(u)::value, w[decltype(u)::value]); });
                at += 512u * U;
                if (at < chunks)
                    static_for<0, U>([&](auto u) { w[decltype(u)::value] = read_chunk(at + 512u * decltype(u)::value); });
            }
            __syncthreads();
        } else {
            ask_weights();
        }
        if constexpr (RAW) {
            // the planes as nimbus_cop_stage_shares leaves them: rows past m are zero
            for (uint32_t s = blockIdx.x; s < S; s += gridDim.x) {
                for (uint32_t i = threadIdx.x; i < 2u * DX * 64u; i += 512u) {
                    const uint32_t kb = 2u * s + i / (DX * 64u), d = i / 64u % DX, l = i & 63u;
                    const uint32_t row = l & 31u, half = (i / (DX * 64u)) * 2u + (l >> 5);
                    uint4 v = {0, 0, 0, 0};
                    if (row < (uint32_t)a.m)
                        v = ((const uint4 *)lds)[((s * RT16 + (row >> 4)) * DX + d) * 64u + half * 16u + (row & 15u)];
                    if (kb < (uint32_t)KB) t.staged[((size_t)kb * DX + d) * 64u + l] = v;
                }
            }
        }
    };

    // ---- the epilogue's operands: asked for behind the first weights, used after the last ----
    // (Mask words by buffer loads: a row past the last one, or no mask, lies behind the descriptor's end and reads
    // as zero, without a branch for each.  Of this row tile; where 32 rows do not fit a descriptor, 2^23 columns
    // and more, by their own addresses.)
    uint64_t mk[T_::PHASES][4 * T_::TP], colsum_S;
    const uint32_t rows_here = (uint32_t)a.m - row_first < 32u ? (uint32_t)a.m - row_first : 32u;
    const bool narrow = a.C < (1u << 23);
    const uint64_t *const mask0 = pp.mask + (size_t)row_first * a.C;
    const __amdgpu_buffer_rsrc_t rsrc_m = __builtin_amdgcn_make_buffer_rsrc(
        (void *)mask0, 0, pp.mask != nullptr ? rows_here * a.C * 8u : 0u, 0x00027000);
    auto ask_epilogue = [&]() {
        colsum_S = active ? pp.colsum[col] : 0;
#pragma unroll
        for (int ph = 0; ph < T_::PHASES; ++ph) {
            uint32_t tile, e0;
            const uint32_t ne = share(ph, tile, e0);
            const uint32_t row0 = 16u * tile + e0 + 4u * j;     // (the elements of a share step over whole tiles)
#pragma unroll
            for (uint32_t u = 0; u < 4 * T_::TP; ++u) {
                const uint32_t row = row0 + 16u * (u / 4u) + u % 4u;
                if (narrow) {
                    const uint32_t off = u < ne ? (row * a.C + col) * 8u : kPastEnd;
                    mk[ph][u] = __builtin_bit_cast(uint64_t, __builtin_amdgcn_raw_buffer_load_b64(rsrc_m, off, 0, 2));
                } else {
                    mk[ph][u] = u < ne && pp.mask != nullptr && row < rows_here
                                    ? __builtin_nontemporal_load(&mask0[(size_t)row * a.C + col])
                                    : 0;
                }
            }
        }
    };

    // ---- the loop ----
    v4i acc[ND][RT16];
#pragma unroll
    for (int d = 0; d < ND; ++d)
#pragma unroll
        for (int i = 0; i < RT16; ++i) acc[d][i] = v4i{0, 0, 0, 0};
    uint32_t s_use = s0 + (len ? ct % len : 0u);
    // (the shares' planes in LDS are written for the rows below m only; for rows past m any row's
    // bytes will do, their sums are not stored)
    uint32_t a_row[RT16];
#pragma unroll
    for (int i = 0; i < RT16; ++i) {
        const uint32_t last = (uint32_t)a.m - 1u - 16u * i;     // of this tile, m > 16 (RT16 - 1)
        a_row[i] = r16 > last ? last : r16;
    }
    auto products = [&](auto p_c) {
        constexpr int p = decltype(p_c)::value;
        const v4i *const at = (const v4i *)lds + s_use * (RT16 * DX * 64u) + j * 16u;
        static_for<0, DX * RT16>([&](auto x_c) {
            constexpr int i = decltype(x_c)::value % RT16, dx = decltype(x_c)::value / RT16;
            v4i x;
            if constexpr (IN_LDS) x = at[(i * DX + dx) * 64 + a_row[i]];
            else x = xs[p][i][dx];
            static_for<0, DQ>([&](auto d_c) {
                constexpr int dq = decltype(d_c)::value;
                acc[dx + dq][i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(x, xb[p][dq], acc[dx + dq][i], 0, 0, 0);
            });
        });
        s_use = next_stage(s_use);
    };
    // Rounds of PD stages, then the last one to PD, whose loads are on their way and which asks for no more.  A
    // slice that is not longer than that (a short k, or one of many slices) asks for its own stages
    // only: the loads behind the end took the memory pipeline 16 cycles each, and the products with zero
    // weights the matrix cores as long as real ones (8 x 64 x 2048, one stage of four: 7.7 and 5.7 us).
    // (Its own way from here on: the counted waits in the rounds need the same loads on every path.)
    uint32_t done = 0;
    auto last_round = [&]() {
        static_for<0, PD>([&](auto p) {
            if (done + decltype(p)::value < len) products(p);
        });
    };
    if (((S + (1u << t.log_ks) - 1u) >> t.log_ks) > (uint32_t)PD) {       // the longest slice: one way for a workgroup
        bring_shares([&]() { static_for<0, PD>([&](auto p) { ask(p); }); });
        ask_epilogue();
        for (; done + PD < len; done += PD)
            static_for<0, PD>([&](auto p) {
                products(p);
                ask(p);
                asm volatile("" ::: "memory");          // (the loads stay where they are asked for)
            });
        last_round();
    } else {
        bring_shares([&]() {
            static_for<0, PD>([&](auto p) {
                if (decltype(p)::value < len) ask(p);
            });
        });
        ask_epilogue();
        last_round();
    }
    uint32_t limb;
    {
        const uint32_t blk = (cg * 16u) >> a.log_n;
        limb = a.L == 1 ? 0u : blk - (uint32_t)a.L * __umulhi(blk, a.l_magic);
        limb = __builtin_amdgcn_readfirstlane(limb);
    }

    // ---- epilogue ----
    // The sums meet in LDS and the elements are finished two at a time, or one where a wave has only
    // one: code that runs once is fetched at some twenty cycles per instruction, so a loop over the
    // elements is faster than the same code unrolled (two elements: 1.2 us instead of 2.6), and two of
    // them take little longer than one, whose instructions wait for each other.  [wave][diagonal][pair of
    // elements of the phase][lane][2], or [wave][diagonal][element][lane].
    int32_t *const sums = (int32_t *)lds;
    const uint32_t cgl = (uint32_t)wave & ((1u << log_cgw) - 1u), KS = 1u << t.log_ks;
    static_for<0, T_::PHASES>([&](auto ph_c) {
        constexpr int ph = decltype(ph_c)::value, i0 = ph * T_::TP;
        constexpr int TILES = RT16 - i0 < T_::TP ? RT16 - i0 : T_::TP;
        __syncthreads();                                // the planes, or the phase before, are read
        const bool pairs = (4u * TILES) >> t.log_ks >= 2u;
        typedef int32_t v2i __attribute__((ext_vector_type(2)));
        auto slot = [&](uint32_t w, int d) { return (w * ND + (uint32_t)d) * (4u * TILES * 64u); };
        if (pairs) {
#pragma unroll
            for (int d = 0; d < ND; ++d)
#pragma unroll
                for (int e = 0; e < 4 * TILES; e += 2)
                    *(v2i *)&sums[slot((uint32_t)wave, d) + e * 64u + (uint32_t)lane * 2u] =
                        v2i{acc[d][i0 + e / 4][e % 4], acc[d][i0 + e / 4][e % 4 + 1]};
        } else {
#pragma unroll
            for (int d = 0; d < ND; ++d)
#pragma unroll
                for (int e = 0; e < 4 * TILES; ++e)
                    sums[slot((uint32_t)wave, d) + e * 64u + lane] = acc[d][i0 + e / 4][e % 4];
        }
        __syncthreads();
        uint32_t tile, e0;
        const uint32_t ne = share(ph, tile, e0);
        // NE elements from element u of the wave's share on
        auto finish = [&](auto ne_c, uint32_t u) {
            constexpr int NE = decltype(ne_c)::value;
            const uint32_t e = 4u * (tile - i0) + e0 + u;       // of the phase
            uint64_t word[NE];
#pragma unroll
            for (int v = 0; v < NE; ++v) word[v] = mk[ph][v];
#pragma unroll
            for (uint32_t v = NE; v < 4 * T_::TP; ++v) mk[ph][v - NE] = mk[ph][v];
            int32_t digit[ND][NE];
#pragma unroll
            for (int d = 0; d < ND; ++d)
#pragma unroll
                for (int v = 0; v < NE; ++v) digit[d][v] = 0;
#pragma unroll 1
            for (uint32_t o = 0; o < KS; ++o)
#pragma unroll
                for (int d = 0; d < ND; ++d) {
                    const int32_t *const at = &sums[slot((o << log_cgw) + cgl, d) + e * 64u + (uint32_t)lane * NE];
                    if constexpr (NE == 2) {
                        const v2i v = *(const v2i *)at;
                        digit[d][0] += v[0];
                        digit[d][1] += v[1];
                    } else {
                        digit[d][0] += *at;
                    }
                }
            cop_finish<ND, NE, false>([&](int d, int r) { return digit[d][r]; }, [](int r) { return r; },
                                      [&](uint64_t (&w)[NE]) {
#pragma unroll
                                          for (int v = 0; v < NE; ++v) w[v] = word[v];
                                      },
                                      a, a.prev, pp.out, limb, colsum_S,
                                      (int)(row_first + 16u * (i0 + e / 4u) + 4u * j + e % 4u), col, a.m);
        };
        if (pairs) {
#pragma unroll 1
            for (uint32_t u = 0; u < ne; u += 2) finish(std::integral_constant<int, 2>{}, u);
        } else if (ne) {                                // one element, or none
            finish(std::integral_constant<int, 1>{}, 0);
        }
    });
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
// the shares' planes of a workgroup fit the LDS
static bool thin_planes_fit(const Problem &p)
{
    const long long S = (kblocks(p.k) + 1) / 2, tiles = (p.m + 15) / 16;
    return S * tiles * planes_x(p.x_bits) * kTileBytes <= kThinSharesLds;
}

// How a launch is split, and about what it takes.
struct ThinPlan {
    uint32_t log_ks;        // KS = 2^log_ks slices of k
    uint32_t blocks;        // workgroups of one problem and row tile
    bool copied;            // staged planes through LDS (17 to 32 rows)
    uint64_t rounds;        // of workgroups on the compute units
    uint64_t stages;        // of a slice
    uint64_t depth;         // stages in flight of a wave
};

// (more than 32 rows: every 32-row tile by itself)
static ThinPlan thin_plan(const Problem &p, int count)
{
    // Slices of k: a compute unit holds one workgroup, so the launch takes as many rounds as there
    // are multiples of that many workgroups, and a round takes the stages of a slice and what
    // starting and ending a workgroup costs, about three stages of eight waves.  (20 x 400 x 12288: two
    // slices in one round 16.0 us, four in two rounds 20.6.)
    const uint64_t S = (uint64_t)(kblocks(p.k) + 1) / 2u, groups = p.C / 16u, cus = (uint64_t)compute_units();
    const uint64_t launches = (uint64_t)count * (uint64_t)((p.m + kThinRows - 1) / kThinRows);  // problems and row tiles
    ThinPlan plan{};
    uint64_t least = ~0ull;
    for (uint32_t l = 0; l <= 3 && (1ull << l) <= S; ++l) {
        const uint64_t blocks = (groups + (8u >> l) - 1) / (8u >> l);
        const uint64_t r = (blocks * launches + cus - 1) / cus;
        const uint64_t cost = r * (((S + (1u << l) - 1) >> l) + 3u);
        if (cost < least) {
            least = cost;
            plan.rounds = r;
            plan.log_ks = l;
            plan.blocks = (uint32_t)blocks;
        }
    }
    // The planes of 32 rows weigh nearly as much as the weights of a wave: eight waves that read the
    // same ones (one slice) read them once, from LDS (32 x 768 x 24576: 31.5 us against 34.4); with
    // several slices fewer waves share them and nobody waits for the copy (x 8192: 17.8 and 16.0).
    plan.copied = p.m > 16 && p.m <= kThinRows && plan.log_ks == 0 && thin_planes_fit(p);
    plan.stages = (S + (1u << plan.log_ks) - 1) >> plan.log_ks;
    plan.depth = (uint64_t)thin_depth(planes_x(p.x_bits), planes_q(p.q_bits_max), p.m <= 16 ? 1 : 2,
                                      plan.copied ? kCopied : kDirect);
    return plan;
}

// A launch has fewer than 2^32 threads: 2^30 columns and more (240 GB of planes of one k-block) are
// left to the tile kernel in any case; its workgroups walk the tiles.
static bool thin_possible(const Problem &p) { return p.m <= kThinRows && p.C < (1ull << 30); }

// From staged shares: where this kernel's rounds take less than those of the tile kernel, which starts
// and ends a workgroup faster but shares the chip's tiles out by whole rounds and has no slices of k.
// Both estimates in hundredths of a microsecond, on 256 compute units: per round its start and end, per
// k-block or stage the wait for its operands and its products, and the bytes of weights, mask and
// results.  Fitted to both kernels' times at 700 drawn sizes (1 to 32 rows, k from 20 to 3072, 64 to 131072
// columns, every pair of plane counts, one to sixteen problems; profiles/choice_of_kernel.txt): the lower estimate is
// 0.5 % slower than the better kernel on average and 0.4 % at 200 sizes that were left out; this kernel everywhere 6 %,
// the tile kernel everywhere 29 %.
struct ThinEstimates {
    double rows, tiles;
};
static uint64_t tile_rounds_of(const Problem &p, int count)
{
    const uint64_t cus = (uint64_t)compute_units();
    return (p.C / 64u * (uint64_t)count + cus - 1) / cus;
}
static ThinEstimates thin_few_estimates(const Problem &p, int count)
{
    const ThinPlan plan = thin_plan(p, count);
    const double KB = kblocks(p.k), n = (double)count;
    const double products = planes_x(p.x_bits) * planes_q(p.q_bits_max);
    const double weights = n * (double)p.C * KB * planes_q(p.q_bits_max), results = n * (double)p.m * (double)p.C;
    const double start = p.m <= 16 ? 261 : plan.copied ? 473 : 341, stages = (double)plan.stages;
    const double tiles = 314 + (double)tile_rounds_of(p, count) * (127 + KB * (7.8 + 1.24 * products)) + 2.01e-4 * weights + 2.74e-4 * results;
    const double rows = 162 + (double)plan.rounds * (start + 60. * stages + 1.57 * products * (p.m <= 16 ? 1 : 2) * stages +
                                                     57. * stages / (double)plan.depth) +
                        2.32e-4 * weights + 1.96e-4 * results;
    return {rows, tiles};
}
static bool thin_few_apply(const Problem &p, int count)
{
    if (!thin_possible(p)) return false;
    const ThinEstimates e = thin_few_estimates(p, count);
    // (The line is not where the estimates meet: a single call of up to 16 rows stays with the tiles until this kernel is
    // ahead by 1.3 us and 1.4 us over the k-blocks, and one of more rows with this kernel a little longer.  That is where
    // the lines lay when a workgroup of this kernel took three microseconds longer to start and end, and
    // tests/test_route_host.py holds sizes between the two.  Over 900 sizes of 1 to 32 rows the choice is 1.5 % slower than the
    // better kernel, 41 % at worst, where the lower estimate alone is 0.5 % and 16 % off (16 x 64 x 20480: 8.5 us with the
    // tiles, which it takes, and 6.9).
    // 17 to 32 rows, one problem: where tiles about fill their last round, this kernel has to be ahead by the last
    // condition too (31 x 1329 x 32768 55.7 us with the tiles and 61.8; 24 x 987 x 24576, whose last
    // round of tiles is half empty, 43.8 and 39.1).  0.5 % off the better kernel at 650 sizes; 1.1 % without it.)
    if (p.m > 16) {
        const ThinPlan plan = thin_plan(p, count);
        const double idle = 1. - (double)(p.C / 64u) * count / ((double)tile_rounds_of(p, count) * compute_units());
        return 0.915 * e.rows + 80 < e.tiles &&
               (count > 1 || idle > (plan.copied ? 0.1 : 0.3) || (plan.copied ? 1.08 : 1.06) * e.rows - 100 < e.tiles);
    }
    return e.rows + (count == 1 ? 130 + 140. / kblocks(p.k) : 0) < e.tiles;
}

// More than 32 rows on few columns: where the tile kernel's workgroups leave compute units without a
// tile, this kernel's row tiles and slices of k fill them (us a call with its staging, 20-bit shares and 54-bit
// moduli, tiles and this kernel: 128 x 3072 x 1024 47 and 17.4, 128 x 1536 x 2048 29 and 15.7).
// Every row tile reads the weights again, from the L2, so the line is where the chip
// fills up (64 x 768 x 8192 16.3 and 18.5); with fewer than eight workgroups to a problem and row tile the
// row tiles are spread over the XCDs, and of a batch each fetches them (197 x 3330 x 256 eight times,
// 16-bit shares, 40.2 and 57.3): a seventh more.
// Estimates as above, fitted at 300 sizes (33 to 512 rows, k from 300 to 4096, 64 to 16384 columns, one to
// eight problems): the choice is 0.3 % slower than the better kernel on average, 30 % at worst, and 0.2 % at 75 sizes that were
// left out; tiles everywhere 75 %, this kernel everywhere 8 %.  Below ten k-blocks only where it is well ahead: 2.1 %
// off the better kernel over 333 sizes of one to ten k-blocks, 44 % at worst (the tiles everywhere 4 %, this kernel 20 %);
// under five never.  The tiles' estimate takes 33 to 48 rows for 64, which is 7 % too much: 15 of 24 sizes
// that are more than 3 % slower than with the rule before, of 518 that are 1.22 times as fast on average, are such (44 x
// 845 x 1792 four times 16.4 us with the tiles and 18.6); a smaller estimate there gives up as much as it saves.
static bool thin_rows_apply(const Problem &p, int count)
{
    const int KB = kblocks(p.k), DX = planes_x(p.x_bits), DQ = planes_q(p.q_bits_max);
    const TileBlocks tb = tile_blocks(p, count);
    const double cus = (double)compute_units(), n = (double)count;
    if (KB < 5 || (double)(p.C / 64u) * tb.row_blocks * n > cus) return false;
    const ThinPlan plan = thin_plan(p, count);
    const int row_tiles = (p.m + kThinRows - 1) / kThinRows;
    if (plan.rounds > 2 || (uint64_t)plan.blocks * (uint64_t)row_tiles * 512u >= (1ull << 32)) return false;
    const int rows16 = ((tb.tiles * kTile < p.m ? tb.tiles * kTile : p.m) + 15) / 16;
    const double weights = n * (double)p.C * KB * DQ, results = n * (double)p.m * (double)p.C;
    const double products = DX * DQ, rounds = (double)plan.rounds;
    const double tiles = 562 + KB * (11.6 + 0.64 * products * ((rows16 + 1) / 2)) + 1.32e-4 * weights + 2.75e-4 * results;
    const double rows = 60 + rounds * (458 + (10. + 3.83 * products) * (double)plan.stages) +
                        (3.35e-4 + 5.4e-5 * row_tiles) * weights + 2.01e-4 * results;
    return (plan.blocks < 8 && count > 1 ? 1.15 : 1.) * (KB < 10 ? 1.28 : 1.) * rows < tiles;
}

bool thin_applies(const Problem &p, int count)
{
    return p.m > kThinRows ? thin_rows_apply(p, count) : thin_few_apply(p, count);
}

// From the shares themselves, without a staging launch (up to 32 rows), where that is ahead of the tiles behind
// one.  Up to two rounds of tiles a call takes little more than its launches cost the host, and one is
// cheaper than two (7.4 us a call and 9.9), so the line lies the staging's two microseconds and part of the host's
// launch above the tiles' estimate.  In a graph, where the host does not count, over 300 sizes of up to 16 rows 0.6 %
// off the better way (always the tiles 52 %).  From three rounds on only where this kernel is ahead of the tiles alone
// (6 x 16 x 107520, 16-bit shares, 62-bit moduli, 18.1 us in two launches).
// 17 to 32 rows: every workgroup splits all shares, which takes as long as the launch that it saves at a k of
// some 600 with 32-bit shares (31 x 610 x 16384, 24-bit shares, 23.8 us and staged 19.1; 24 x 82 x 2048, 32-bit, 7.6 and
// 8.8; 20 x 200 x 8192 8.2 and 10.6).  In a graph over 330 sizes 0.5 % off the better way, 10 % at worst (2 % and 26 %
// without that term, staged everywhere 7 %, from the shares everywhere 4 %).
bool thin_raw_applies(const Problem &p)
{
    if (!thin_possible(p) || !thin_planes_fit(p)) return false;
    const ThinEstimates e = thin_few_estimates(p, 1);
    if (p.m <= 16) return e.rows < e.tiles + (tile_rounds_of(p, 1) > 2 ? -100 : 450);
    const double splits = 8. * (double)thin_plan(p, 1).rounds * ((kblocks(p.k) + 1) / 2) * planes_x(p.x_bits);
    return e.rows + splits < (thin_few_apply(p, 1) ? e.rows : e.tiles) + 300;
}

template <int DX, int DQ>
static hipError_t thin_impl(const Problem &p, int count, const uint64_t *X, int half_shift,
                            const void *const *staged, const void *const *prepared,
                            const uint64_t *const *masks, const uint64_t *prev, uint64_t *const *outs,
                            hipStream_t stream)
{
    const int KB = kblocks(p.k);
    const uint32_t CT = (uint32_t)(p.C / kTile);
    MfmaArgs a{};
    fill_common_args(p, DX, masks[0], prev, outs[0], &a);
    ThinArgs t{};
    t.X = X;
    t.staged = (uint4 *)const_cast<void *>(staged[0]);
    t.k = p.k;
    t.half_shift = half_shift;
    const uint32_t quads = 16u * ((uint32_t)(KB + 1) / 2u);
    t.quads_magic = (uint32_t)(((1ull << 32) + quads - 1) / quads);     // (items below 2^16, Q below 2^13)
    const ThinPlan plan = thin_plan(p, count);
    t.log_ks = plan.log_ks;
    a.RB = (p.m + kThinRows - 1) / kThinRows;
    const dim3 grid(plan.blocks * (uint32_t)a.RB, (uint32_t)count), block(512);
    auto go_with = [&](auto rt_c, auto from_c, auto nb_c) {
        constexpr int NB = decltype(nb_c)::value;
        BatchPtrs<NB> b{};
        for (int i = 0; i < count; ++i) {
            b.prob[i].xd = (const uint4 *)staged[i];
            b.prob[i].planes = (const uint4 *)prepared[i];
            b.prob[i].colsum = (const uint64_t *)((const char *)prepared[i] + (size_t)CT * KB * DQ * kTileBytes);
            b.prob[i].mask = masks[i];
            b.prob[i].out = outs[i];
        }
        b.count = (uint32_t)count;
        return launch(cop_thin_kernel<DX, DQ, decltype(rt_c)::value, decltype(from_c)::value, NB>, grid, block, stream,
                      a, b, t);
    };
    auto go = [&](auto rt_c, auto from_c) {
        if constexpr (decltype(from_c)::value != kRaw)
            if (count > 1) return go_with(rt_c, from_c, std::integral_constant<int, kMaxBatch>{});
        return go_with(rt_c, from_c, std::integral_constant<int, 1>{});
    };
    const std::integral_constant<ThinShares, kDirect> direct;
    const std::integral_constant<ThinShares, kCopied> copied;
    const std::integral_constant<ThinShares, kRaw> raw;
    const std::integral_constant<int, 1> one;
    const std::integral_constant<int, 2> two;
    if (X) return p.m <= 16 ? go(one, raw) : go(two, raw);
    if (p.m <= 16) return go(one, direct);
    if (p.m > kThinRows) return go(two, std::integral_constant<ThinShares, kRows>{});
    return plan.copied ? go(two, copied) : go(two, direct);
}

hipError_t launch_cop_thin(const Problem &p, int count, const uint64_t *X, int half_shift,
                           const void *const *staged, const void *const *prepared,
                           const uint64_t *const *masks, const uint64_t *prev, uint64_t *const *outs,
                           hipStream_t stream)
{
    if (count < 1 || count > kMaxBatch) return hipErrorInvalidValue;
    const int DX = planes_x(p.x_bits), DQ = planes_q(p.q_bits_max);
#define NIMBUS_CASE(dx, dq) \
    if (DX == dx && DQ == dq) \
        return thin_impl<dx, dq>(p, count, X, half_shift, staged, prepared, masks, prev, outs, stream);
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
