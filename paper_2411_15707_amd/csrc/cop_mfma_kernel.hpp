// Matrix-core (int8 MFMA) kernel of the COP accumulation on prepared weights, gfx950: the kernel and
// the launch that picks its instance.  Included by the translation units that instantiate it, one per
// pair of plane counts (side by side they compile in a sixth of the time).
//
// The contraction out = X * ctW (Algorithm 1 step 2 of the paper) is an exact
// integer matrix product with a 2^x_bits-bounded left operand and a q-bounded
// right operand.  Both are split into signed bytes so that the products run on
// v_mfma_i32_16x16x64_i8:
//
//   x  = x' + OFFX,  x' = sum_{a<DX} dx_a 256^a,  dx_a = byte_a(x) - 128 for the bytes that
//                    can reach 128 (8a + 8 <= x_bits), dx_a = byte_a(x) for the others (the
//                    top byte of a 20-bit share is a digit in [0, 15]: small operands keep
//                    the multipliers quieter, and the kernel's speed is set by power);
//                    OFFX = sum of 128 * 256^a over the shifted bytes   (no carries needed)
//   c' = c or c - q  (centred, |c'| <= (q-1)/2),  c' = sum_{b<DQ} dq_b 256^b,
//                    dq_b in [-128, 127]  (carry-propagating recode, done once
//                    per weight matrix by nimbus_cop_prepare)
//
//   sum_i x_i c_i  =  sum_i x'_i c'_i  +  OFFX * S   (mod q),   S = sum_i c_i mod q
//   sum_i x'_i c'_i = sum_d 256^d D_d,   D_d = sum_{a+b=d} sum_i dx_a(i) dq_b(i)
//
// Each D_d is one int32 MFMA accumulator (all byte pairs of one diagonal d
// accumulate into the same tile).  |dx dq| <= 2^14, at most min(DX,DQ) pairs per
// diagonal, so |D_d| <= k * min(DX,DQ) * 2^14, which the host keeps below 2^30.
// The epilogue forms V = sum_d D_d 256^d + (q << sh) + OFFX*S + mask, where the
// multiple of q makes the total non-negative, and reduces V once.
//
// Operand tiles are 32 x 32 bytes stored in the register order of the MFMA: the
// 16 bytes of lane l belong to row (or column) l % 32 and to k-slots
// (l / 32) * 16 .. +15 of the tile.  The A and B operands of the instruction
// use the same lane/byte -> k mapping, so any fixed assignment of k-slots to
// actual k indices gives the same sum as long as both sides share it.
#pragma once
#include "cop_mfma_common.hpp"

namespace nimbus {

// The pipeline.  A workgroup of eight waves (two per SIMD) owns 128 token rows x 64
// coefficient columns.  Wave w owns 16 columns, group w % 4, and of every 32-row tile the
// rows of half w / 4: up to four 16 x 16 output tiles, DX+DQ-1 int32 accumulators each.  The
// two waves of a SIMD share its columns and split the rows, so that every SIMD has the same
// products to do whatever the number of rows: a call of 77 rows costs five 16-row tiles on each.
//
// v_mfma_i32_16x16x64_i8: a step of the loop is 64 values of k, two k-blocks of the operand
// layout.  Lane l holds row (or column) l % 16 and the k-slots 16 (l / 16) .. +15 of the step: 16
// bytes that lie together in a 32 x 32 operand tile (k-block l / 32 of the step, half
// (l / 16) % 2), so that an operand is one ds_read_b128 from wherever its tile is.
//
// A stage is one k-block: 4*DX operand tiles of X (12 KB for DX = 3) and 2*DQ operand tiles of
// ciphertext planes (14 KB for DQ = 7), each in an LDS ring of its own.  Both are filled by
// direct-to-LDS loads of whole tiles (64 lanes x 16 B; the texture address unit spends the
// same time on narrower loads); nothing passes through registers on the way in.  Wave w < 4
// loads the DX planes of row tile w, waves 4 and 5 the two halves of the planes of the first
// column tile, waves 6 and 7 those of the second (one wave of each kind per SIMD, at most four
// loads per wave and stage).  A load is a buffer load: descriptor with the workgroup's base, the
// lane's 16 bytes, and one wave-uniform offset that is carried from stage to stage, so
// issuing it costs no vector arithmetic.  A wave knows how many loads it issues per stage, so
// "stage s has landed" is a wait on the number of its younger loads, then the barrier.
//
// Inside a wave the operands rotate.  A step's products run in groups of DQ: row tile by row
// tile, share plane by share plane, each group one share operand times the DQ ciphertext operands
// of the step.  Share operands are read AHEAD groups before their own, and during the last group
// every ciphertext operand is refilled from the next step right behind its last use.  One barrier
// per step stands in front of the first read of the next step; it makes that step's stages
// visible and frees the slots of this one, whose operands every wave has in registers by then.
// The loads of the stages LEAD ahead go out, spread over the products, in front of it.  LDS reads
// come back in order, so every wait is a count of younger reads.
//
// Measured against the kernel before (v_mfma_i32_32x32x32_i8, a wave per 32 x 32 output tile, a barrier
// per k-block, whole 32-row tiles on waves of two SIMDs each; us a call, both on one card): 128 x 768 x
// 16384 35.7 -> 32.7 (33.7 -> 33.4 on the card with the smallest difference), 128 x 3072 x 16384 with
// packing 122.1 -> 112.2, 512 x 1024 x 49152 with packing 481.8 -> 458.2, 128 x 768 x 32768 of 64-bit
// shares 186.3 -> 177.8, four problems of 77 x 1001 x 16384 177.3 -> 137.8; 628 sizes of 33 to 512
// rows 1.09 times as fast on average.  The instruction takes half the accumulator traffic per
// product, a step one barrier instead of two, and the 77 rows five tiles on every SIMD instead
// of eight on two of them.  Slower, by up to a twentieth: a few k-blocks of an odd number (200 x 98304,
// 256 rows 154 and 162: the last one costs more than half a step).
//
// What the loop is bound by (measured).  Its duration follows the operand values: the
// chip lowers its clock under the combined matrix-core and memory load (1.5 to 1.8 GHz
// here against the 2.4 GHz of the data sheet).  Fewer cycles do not translate one to one: the
// chip answers a denser loop with a lower clock.  What the schedule has to respect: enough
// bytes in flight per CU (a streaming read reaches 3.9 TB/s chip-wide with 8 KB in flight per CU,
// 6.5 with 16 KB, 7.0 from 32 KB on, direct-to-LDS and register loads alike), the
// ciphertext loads spread over the step, and instruction issue (all eight waves run
// in lockstep between barriers, so every scalar instruction costs: ring offsets carried
// and wrapped instead of recomputed, and the wait for "at most n loads pending", an
// immediate of the instruction, done by a compare chain over the two or three counts
// that can occur).

template <int DX, int DQ>
struct Pipe {
    static constexpr int ND = DX + DQ - 1;
    static constexpr int A_BYTES = 4 * DX * kTileBytes;     // of a stage
    static constexpr int B_BYTES = 2 * DQ * kTileBytes;
    // Slots of the rings: the two stages of the step at hand and those on their way.  Stages
    // 0 .. LEAD-1 are issued up front, step t issues 2t + LEAD and 2t + LEAD + 1.  The ciphertext
    // (HBM) is two whole steps ahead; the shares (L2) as far as the LDS has room, one step at least.
    static constexpr int RING_B = 6;
    static constexpr int FIT_A = (160 * 1024 - RING_B * B_BYTES) / A_BYTES;
    static constexpr int RING_A = FIT_A > 6 ? 6 : FIT_A;
    static constexpr int LEAD_A = RING_A - 2, LEAD_B = RING_B - 2;
    static_assert(LEAD_A >= 2 && LEAD_A <= LEAD_B, "a step's stages are issued in the step before at the latest");
    static constexpr int LDS_BYTES = RING_A * A_BYTES + RING_B * B_BYTES;
    // load slots per wave and stage: a row tile's DX planes, or half of a column tile's DQ
    static constexpr int MAXU = 4;
    static constexpr int PH = (DQ + 1) / 2;         // planes of a column tile on its first wave
    static_assert(DX <= MAXU && PH <= MAXU, "four load slots per wave and stage");
    // share operands in registers: the group's own and AHEAD groups' (a divisor of the groups of a
    // step, so that the sets fall in place again with the next one)
    static constexpr int SETS = DX == 3 ? 3 : (DX == 4 && DQ == 7 ? 4 : 2);
    static constexpr int AHEAD = SETS - 1;
    static_assert(DX % SETS == 0, "operand sets");
};

// FULL: m is a multiple of 128, so every wave has its four 16-row tiles: the code for waves with
// fewer and the row tests around the loads and stores of the epilogue (a compare, an exec
// update and a branch each) are left out.
//
// The wave's mask words are asked for when the loop has no stage left to ask for, or one, about two steps
// before its end, into registers that the operands leave free, instead of when the loop is over:
// the 16 B per output that mask and result move would otherwise all fall into the last microseconds of
// a tile, where they are the only traffic and every workgroup asks at once.  MASKAHEAD: in the instances
// without row tests, given a mask and at most nine accumulators per output.  With row tests it is
// decided at run time, where the registers hold them: at most nine accumulators, or three 16-row tiles.
// Before, only without row tests and for 14 k-blocks and more of an even number (us, 20-bit shares, 54-bit
// moduli: 64 x 125 x 32768 19.2 -> 17.0, 256 x 95 x 98304 119.0 -> 109.1, 512 x 190 x 16384 51.7 -> 43.4, 400 x
// 160 x 98304, 16-bit shares, 222.8 -> 209.4; 1000 sizes of up to 415 k 5 % faster on average).
//
// SHARED: the launch has several row blocks per column tile (m > 128).  They run on one XCD
// at the same time, start at the same k-block and load without the streaming hint, so the
// ciphertext tile comes over the fabric once and the other row blocks find it in the L2.
template <int DX, int DQ, bool FULL, bool MASKAHEAD, bool SHARED, int NB>
__global__ __launch_bounds__(512, 1) void cop_mfma_kernel(const MfmaArgs a, const BatchPtrs<NB> b)
{
    using P_ = Pipe<DX, DQ>;
    // Every scalar argument the setup needs, asked for in one batch: left to the compiler the
    // loads sit next to their first uses, and the setup waits for the constant cache once
    // per group of them instead of once.
    asm volatile("" ::"s"(b.prob[0].xd), "s"(b.prob[0].planes), "s"(b.prob[0].colsum),
                 "s"(b.prob[0].mask), "s"(b.prob[0].out), "s"(a.m), "s"(a.KB), "s"(a.RB),
                 "s"(a.L), "s"(a.CT), "s"(a.kb_magic), "s"(a.log_n), "s"(a.l_magic));
    constexpr int ND = P_::ND, MAXU = P_::MAXU, PH = P_::PH;
    constexpr int SETS = P_::SETS, AHEAD = P_::AHEAD;
    static_assert(!MASKAHEAD || (FULL && ND <= 9), "mask words ahead: full row blocks, and they must fit");
    __shared__ __attribute__((aligned(1024))) unsigned char lds[P_::LDS_BYTES];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // 0..7
    const int wh = wave >> 2, wc = wave & 3;        // half of the 32-row tiles, 16-column group

    // tile id -> (64-column tile, row block).  A workgroup takes the tiles blockIdx.x,
    // blockIdx.x + gridDim.x, ... (the host launches one workgroup per compute unit when there
    // are more tiles than that).  Workgroups are dealt round-robin to the 8 XCDs, and with a
    // grid that is a multiple of 8 so are the tile ids; the RB row blocks that share a column
    // tile are kept on one XCD and adjacent in that order so that tile is fetched from HBM
    // once.  (The column tiles past the last multiple of 8, if any, are not worth the trouble.)
    // (the pointers of a single call are asked for with the first batch of scalar loads: an
    // indexed load would sit on the path to the first loads of the launch)
    const bool single = NB == 1 || b.count == 1;
    // (a launch may hold several problems of the same shape: tile ids run through the first
    // problem's tiles, then the second's, ...; p is the problem)
    auto map_tile = [&](uint32_t id, uint32_t &p, uint32_t &ct2, uint32_t &rb) {
        p = 0;
        if (!single) {
            while (id >= b.tiles_each) {            // at most kMaxBatch - 1 rounds, scalar
                id -= b.tiles_each;
                ++p;
            }
        }
        const uint32_t RB = (uint32_t)a.RB;
        const uint32_t CT2a = (a.CT >> 1) & ~7u;
        if (!SHARED) {                              // one row block: no division
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
    };
    const uint32_t block_tiles = FULL ? 4u : a.block_tiles;         // row tiles of a row block
    const int KB = a.KB;
    // ---- this wave's share of the loads of one stage (sources at k-block 0) ----
    // Waves 0-3 (the first wave of each SIMD) load the X tiles, from L2: wave w the DX planes
    // of row tile w of the row block (a wave without a row tile loads nothing).  Waves 4-7 (the
    // second of each SIMD) load the ciphertext tiles, from HBM:
    // waves 4 and 5 the planes of the first column tile (planes 0-3 and 4 .. DQ-1), waves 6
    // and 7 those of the second.  A load's source is the wave's buffer descriptor (base of
    // the tile's X or ciphertext region), the lane's 16 bytes, and a wave-uniform
    // offset: the operand tile's place at k-block 0 plus the carried k-block offset.  (A row
    // tile or column tile of planes spans KB * D KiB < 2^23 bytes.  Everything up to the first
    // loads is scalar work on the critical path of the launch: no divisions, and whatever the
    // loads do not need comes after them.)
    const uint32_t a_tile_bytes = (uint32_t)KB * DX * kTileBytes;     // one row tile, all k-blocks
    const uint32_t b_tile_bytes = (uint32_t)KB * DQ * kTileBytes;     // one column tile
    const bool loads_x = wave < 4;
    const uint32_t lane16 = (uint32_t)lane * 16u;
    const uint32_t src_step = (uint32_t)(loads_x ? DX : DQ) * kTileBytes;   // per k-block
    const uint32_t src_end = (uint32_t)KB * src_step;
    const uint32_t slot_step = loads_x ? P_::A_BYTES : P_::B_BYTES;
    const uint32_t slot_end = loads_x ? P_::RING_A * P_::A_BYTES : P_::RING_B * P_::B_BYTES;
    const int lead = loads_x ? P_::LEAD_A : P_::LEAD_B;
    uint32_t dst0;                                  // the first operand tile's byte offset in slot 0 of the LDS
    int n_loads;                                    // loads per stage
    if (loads_x) {
        dst0 = (uint32_t)wave * DX * kTileBytes;
        n_loads = DX;
    } else {
        const uint32_t c = (uint32_t)(wave >> 1) & 1u, hi = (uint32_t)wave & 1u;
        dst0 = (uint32_t)(P_::RING_A * P_::A_BYTES) + (c * DQ + hi * PH) * kTileBytes;
        n_loads = hi ? DQ - PH : PH;
    }
    // Issue side of a tile: descriptor, the first operand tile's offset at k-block 0, and the
    // wave-uniform state for the next stage to issue (byte offset of its k-block in the
    // source, byte offset of its slot in the ring; carried and wrapped, never recomputed).
    // Stage s of a tile is k-block (s + k_start) mod KB: the sum over k does not care about
    // the order, and workgroups that walk their (equally spaced) ciphertext regions in
    // lockstep would otherwise ask the same memory channels for data at the same moment.
    // The start depends on the column tile alone: row blocks that share a column tile walk
    // it together.
    __amdgpu_buffer_rsrc_t rsrc;
    uint32_t toff0;                                 // the first operand tile's byte offset at k-block 0
    uint32_t src_off, slot_off;
    int row_first = 0, row_end = 0, nt = 4;         // rows of the block, 16-row tiles of this wave: half wh of the 32-row tiles
    auto begin_tile = [&](uint32_t p, uint32_t ct2, uint32_t rb) {
        row_first = (int)(rb * block_tiles) * kTile;
        if constexpr (!FULL) {
            row_end = row_first + (int)block_tiles * kTile < a.m ? row_first + (int)block_tiles * kTile : a.m;
            nt = ((row_end - row_first + 15) / 16 + 1 - wh) >> 1;
        }
        const uint4 *xd_p = b.prob[0].xd, *planes_p = b.prob[0].planes;
        if (!single) {
            xd_p = b.prob[p].xd;
            planes_p = b.prob[p].planes;
        }
        const unsigned char *const a_base =
            (const unsigned char *)xd_p + (size_t)rb * block_tiles * a_tile_bytes;
        const unsigned char *const b_base =
            (const unsigned char *)planes_p + (size_t)ct2 * 2u * b_tile_bytes;
        rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(loads_x ? a_base : b_base), 0, 0xffffffff,
                                                 0x00027000);
        if (loads_x) {
            toff0 = (uint32_t)wave * a_tile_bytes;
            if constexpr (!FULL) {                  // does the row tile exist?
                n_loads = row_first + wave * kTile < row_end ? DX : 0;
            }
        } else {
            const uint32_t c = (uint32_t)(wave >> 1) & 1u, hi = (uint32_t)wave & 1u;
            toff0 = c * b_tile_bytes + hi * (PH * kTileBytes);
        }
        n_loads = __builtin_amdgcn_readfirstlane(n_loads);
        uint32_t k_start = ct2 - __umulhi(ct2, a.kb_magic) * (uint32_t)KB;   // ct2 mod KB
        if (k_start >= (uint32_t)KB) k_start -= (uint32_t)KB;
        src_off = k_start * src_step;
        slot_off = 0;
    };
    auto bump = [](uint32_t v, uint32_t step, uint32_t end) -> uint32_t {
        v += step;
        return v == end ? 0u : v;
    };
    // load u of the stage at the carried offsets
    auto issue_one = [&](auto u_c) {
        constexpr uint32_t u = decltype(u_c)::value;
        dma_tile<!SHARED>(rsrc, lane16, toff0 + u * kTileBytes + src_off, lds + (dst0 + u * kTileBytes + slot_off));
    };
    auto next_issue = [&]() {
        src_off = bump(src_off, src_step, src_end);
        slot_off = bump(slot_off, slot_step, slot_end);
    };
    auto issue_first_stages = [&](auto between) {
        static_for<0, P_::LEAD_B>([&](auto st_c) {
            constexpr int st = decltype(st_c)::value;
            if (st < lead && st < KB) {
                static_for<0, MAXU>([&](auto u_c) {
                    if (decltype(u_c)::value < n_loads) issue_one(u_c);
                });
                next_issue();
            }
            between(st_c);
        });
    };

    uint32_t tile = blockIdx.x, prob, ct2, rb;
    map_tile(tile, prob, ct2, rb);
    begin_tile(prob, ct2, rb);

    // One pass per tile, for a wave of NT 16-row tiles (none: the wave's loads and the barriers).  The
    // first stages of a tile other than the first are in flight when its pass begins: they
    // were issued in front of the epilogue of the tile before it.  Returns whether there is another.
    auto pass = [&](auto nt_c, bool first) -> bool {
    constexpr int NT = decltype(nt_c)::value, NA = NT > 0 ? NT : 1;
    v4i acc[ND][NA];
    auto clear = [&](int d) {
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            acc[d][i] = v4i{0, 0, 0, 0};
            tie(acc[d][i]);
        }
    };
    if (first) {
        // ---- up front: the first stages of the first tile ----
        // The accumulators are cleared between the stages: the memory pipeline takes the first
        // loads of a launch slowly (nothing is translated or cached yet), and the moves fill
        // the time the wave would spend waiting for it to accept the next one.
        issue_first_stages([&](auto st_c) {
#pragma unroll
            for (int d = decltype(st_c)::value; d < ND; d += P_::LEAD_B) clear(d);
        });
    } else {
#pragma unroll
        for (int d = 0; d < ND; ++d) clear(d);
    }
    __builtin_amdgcn_sched_barrier(0);
    // ---- what the first loads did not need ----
    // The column's ciphertext sum is needed after the loop; asked for now it costs two
    // registers, not a round trip to memory at the end.  An ordinary load: the compiler places
    // the wait for it at its first use, and the statements below that clobber memory keep the
    // load itself up here.  (One more load ahead of the loop's counted waits only makes them
    // wait for it too; it is the oldest but the first stages by then.)
    const uint64_t *colsum_p = b.prob[0].colsum;
    const uint64_t *mask_p = b.prob[0].mask;
    uint64_t *out_p = b.prob[0].out;
    if (!single) {
        colsum_p = b.prob[prob].colsum;
        mask_p = b.prob[prob].mask;
        out_p = b.prob[prob].out;
    }
    const uint64_t colsum_S = colsum_p[ct2 * 64u + (uint32_t)wc * 16u + (uint32_t)(lane & 15)];
    asm volatile("" ::: "memory");
    // The limb of this wave's 16 columns (they lie in one (polynomial, limb) block of N >= 32
    // columns), worked out here with a shift and a multiply-high: after the loop it would sit
    // on the path to the first loads of the epilogue.
    uint32_t limb;
    {
        const uint32_t blk = (ct2 * 64u + (uint32_t)wc * 16u) >> a.log_n;
        limb = a.L == 1 ? 0u : blk - (uint32_t)a.L * __umulhi(blk, a.l_magic);
        limb = __builtin_amdgcn_readfirstlane(limb);
        asm volatile("" : "+s"(limb));
    }

    // Operands come out of LDS through explicit ds_read_b128 instructions: reads the
    // compiler can see would each be made to wait for every direct-to-LDS load in flight.
    // Lanes 0-31 read the first stage of a step, lanes 32-63 the second.
    const uint32_t lds0 = (uint32_t)(uintptr_t)(NIMBUS_AS3 void *)&lds[0];
    const uint32_t in_tile = (((uint32_t)lane >> 4) & 1u) * 512u + ((uint32_t)lane & 15u) * 16u;
    const uint32_t laneA = lds0 + (uint32_t)wh * 256u + in_tile;
    const uint32_t laneB = lds0 + (uint32_t)(P_::RING_A * P_::A_BYTES) +
                           (uint32_t)((wc >> 1) * DQ) * kTileBytes + (uint32_t)(wc & 1) * 256u + in_tile;
    // ring offsets of the step that is read next, per lane
    uint32_t rdA = ((uint32_t)lane >> 5) * P_::A_BYTES, rdB = ((uint32_t)lane >> 5) * P_::B_BYTES;
    auto next_read = [&]() {
        // (below the ring's end the difference wraps around and the minimum is the sum itself)
        rdA += 2u * P_::A_BYTES;
        rdB += 2u * P_::B_BYTES;
        const uint32_t wA = rdA - P_::RING_A * P_::A_BYTES, wB = rdB - P_::RING_B * P_::B_BYTES;
        rdA = rdA < wA ? rdA : wA;
        rdB = rdB < wB ? rdB : wB;
    };
    v4i xa[SETS], xb[DQ];
    // share operand of group g (16-row tile g / DX, plane g % DX), ciphertext operand of plane d, of
    // the step at (rdA, rdB)
    auto read_a = [&](auto g_c, auto set_c) {
        constexpr int g = decltype(g_c)::value;
        xa[decltype(set_c)::value] = lds_read_b128<g * kTileBytes>(laneA + rdA);
    };
    auto read_b = [&](auto d_c) {
        xb[decltype(d_c)::value] = lds_read_b128<decltype(d_c)::value * kTileBytes>(laneB + rdB);
    };

    // At the barrier of step t the stages 2t + 2 and 2t + 3 have to have landed, and the loads of
    // the stages behind them that have been issued are younger (no stage 2t + 2: nothing to wait for).
    auto younger = [&](int t) -> int {
        if (2 * t + 2 >= KB) return 63;
        const int issued = KB < 2 * t + lead + 2 ? KB : 2 * t + lead + 2;
        return issued > 2 * t + 4 ? (issued - (2 * t + 4)) * n_loads : 0;
    };
    const int steady_pending = (lead - 2) * n_loads;
    auto wait_steady = [&]() {
        constexpr int WA = (P_::LEAD_A - 2) * DX, WB = P_::LEAD_B - 2;
        constexpr int least = WA < WB * (DQ - PH) ? WA : WB * (DQ - PH);
        constexpr int most = WA < WB * (DQ - PH) ? WB * (DQ - PH) : WA;
        wait_vmem_of<WB * PH, most, least>(steady_pending);
    };
    asm volatile("" ::: "memory");
    {
        // Stages 0 and 1 are there before the loop; the younger loads are those up to stage lead - 1.
        // Loads and stores complete in the order they were issued: behind a tile without row tests
        // the stores of its epilogue, of which every wave has as many as elements, may be pending too.
        // (Waiting for them cost every tile but the first the way of its last store to memory.)
        const int st = (KB < lead ? KB : lead) - 2;
        wait_vmem_n((st > 0 ? st * n_loads : 0) + (FULL && !first ? 4 * NT : 0));
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    }
    // the lane's mask words, where they are asked for ahead: MASKAHEAD, and with row tests where the
    // registers hold them
    constexpr bool MASKREGS = MASKAHEAD || (!FULL && NT > 0 && (ND <= 9 || NT < 4));
    uint64_t mk[4 * NA];
    // (128 rows of the mask in one descriptor)
    const bool ahead = MASKAHEAD || (MASKREGS && mask_p != nullptr && a.C < (1u << 22));
    if constexpr (MASKREGS && !MASKAHEAD) {
#pragma unroll
        for (int r = 0; r < 4 * NT; ++r) mk[r] = 0;
    }
    const uint32_t col = ct2 * 64u + (uint32_t)wc * 16u + (uint32_t)(lane & 15);
    const int row0 = row_first + 16 * wh + 4 * (lane >> 4);
    auto roff = [](int r) -> int { return 32 * (r >> 2) + (r & 3); };

    // the step in front of which they were asked for; its wait need not cover them where every stage that
    // it needs is older (where the shares are less far ahead than the ciphertext some are asked for in it)
    int mask_step = -1;
    constexpr int MASKLOADS = MASKREGS && P_::LEAD_A == P_::LEAD_B ? 4 * NT : 0;
    auto ask_mask = [&]() {
        if constexpr (MASKAHEAD) {
            const uint64_t *const mask0 = mask_p + ((size_t)row0 * a.C + col);
#pragma unroll
            for (int r = 0; r < 4 * NT; ++r) mk[r] = __builtin_nontemporal_load(&mask0[(size_t)roff(r) * a.C]);
        } else if constexpr (MASKREGS) {
            // (a load for every row, there or not: the wait of the step counts them)
            const __amdgpu_buffer_rsrc_t rsrc_m = __builtin_amdgcn_make_buffer_rsrc(
                (void *)(mask_p + (size_t)row_first * a.C), 0, (uint32_t)(row_end - row_first) * a.C * 8u, 0x00027000);
            uint32_t at = ((uint32_t)(row0 - row_first) * a.C + col) * 8u;
#pragma unroll
            for (int r = 0; r < 4 * NT; ++r) {
                mk[r] = __builtin_bit_cast(uint64_t, __builtin_amdgcn_raw_buffer_load_b64(rsrc_m, at, 0, 2));
                at += (r % 4 == 3 ? 29u : 1u) * 8u * a.C;
                asm volatile("" : "+v"(at));
            }
        }
        asm volatile("" ::: "memory");
    };

    // Step t.  STEADY: every stage up to 2t + LEAD_B + 1 exists.
    auto step = [&](int t, auto steady_c) {
        constexpr bool STEADY = decltype(steady_c)::value;
        constexpr int NG = NT * DX, NBAR = NG - AHEAD;      // groups; the barrier stands in front of group NBAR
        // the loads of two stages, over the first quarter of the products in front of the barrier (the
        // kernel on 128 x 3072 x 16384 104.3 us, spread over all of them 107.3, with the first few
        // 105.6); over the first half or third where the shares are less far ahead
        constexpr int NITEMS = 2 * MAXU, SPAN = NBAR * DQ / (P_::LEAD_A == P_::LEAD_B ? 4 : P_::LEAD_B - P_::LEAD_A + 1);
        int issue_n[2] = {n_loads, n_loads};
        if constexpr (!STEADY) {
            if (2 * t + lead >= KB) issue_n[0] = 0;
            if (2 * t + lead + 1 >= KB) issue_n[1] = 0;
        }
        static_for<0, NG>([&](auto g_c) {
            constexpr int g = decltype(g_c)::value;
            constexpr int i = g / DX, dx = g % DX;
            if constexpr (g == NBAR) {
                // every operand of this step is in registers but the ciphertext's last group reads on
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                if constexpr (STEADY) wait_steady();
                else wait_vmem_n(younger(t) + (MASKLOADS && younger(t) < 63 - 16 && t == mask_step ? MASKLOADS : 0));
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                next_read();
            }
            read_a(std::integral_constant<int, (g + AHEAD) % NG>{}, std::integral_constant<int, (g + AHEAD) % SETS>{});
            static_for<0, DQ>([&](auto d_c) {
                constexpr int dq = decltype(d_c)::value, pos = g * DQ + dq;
                // first group: the reads younger than ciphertext operand dq are those behind it and
                // the share operand just asked for
                if constexpr (g == 0) wait_lds<DQ - dq>(xb[dq]);
                else if constexpr (dq == 0 && g < NBAR) wait_lds<AHEAD>(xa[g % SETS]);
                tie(xa[g % SETS]);
                tie(xb[dq]);
                acc[dx + dq][i] =
                    __builtin_amdgcn_mfma_i32_16x16x64_i8(xa[g % SETS], xb[dq], acc[dx + dq][i], 0, 0, 0);
                tie(acc[dx + dq][i]);
                static_for<0, NITEMS>([&](auto j_c) {
                    constexpr int j = decltype(j_c)::value, u = j % MAXU;
                    if constexpr (j * SPAN / NITEMS == pos) {
                        if (u < issue_n[j / MAXU]) issue_one(std::integral_constant<int, u>{});
                        if constexpr (u == MAXU - 1) next_issue();
                    }
                });
                // (the last step reads a stale slot: valid LDS, never used)
                if constexpr (g == NG - 1) read_b(d_c);
            });
        });
        asm volatile("" ::: "memory");
    };
    // The last stage where their number is odd: one k-block, half of what the instruction takes.  Its
    // other half takes the next share plane of the same k-block against the ciphertext plane
    // before, two products of one diagonal: lanes 0-31 hold the planes dx and d, lanes 32-63 dx + 1
    // and d - 1 (none for d = 0, for lanes 0-31 none for d = DQ, and none beyond the last share plane).
    // 15 products instead of 21 for <3, 7>, 16 instead of 28 for <4, 7>.
    // (What the upper lanes find in front of the first ciphertext plane and behind the last share
    // plane is some other operand tile, and set to zero.)  Nothing is read ahead of it, and its reads
    // end behind the last barrier: the next tile's loads wait for one more.
    auto last_stage = [&]() {
        constexpr int NP = (DX + 1) / 2;            // pairs of share planes
        int lane_l = lane;                          // (opaque: see the epilogue)
        asm volatile("" : "+v"(lane_l));
        const uint32_t upper = (uint32_t)lane_l >> 5;
        const int lower_only = upper ? 0 : -1;
        rdA = __builtin_amdgcn_readfirstlane(rdA) + upper * kTileBytes;
        rdB = __builtin_amdgcn_readfirstlane(rdB);
        v4i xe = lds_read_b128<(DQ - 1) * kTileBytes>(laneB + rdB);
        rdB -= upper * kTileBytes;
        static_for<0, DQ>([&](auto d_c) { read_b(d_c); });
        auto read_pair = [&](auto n_c) {            // pair n % NP of 16-row tile n / NP, into operand set n % 2
            constexpr int n = decltype(n_c)::value;
            read_a(std::integral_constant<int, n / NP * DX + n % NP * 2>{}, std::integral_constant<int, n & 1>{});
        };
        read_pair(std::integral_constant<int, 0>{});
        static_for<0, NT * NP>([&](auto n_c) {
            constexpr int n = decltype(n_c)::value, i = n / NP, dx = n % NP * 2;
            constexpr bool two = dx + 1 < DX;
            if constexpr (n + 1 < NT * NP) read_pair(std::integral_constant<int, n + 1>{});
            if constexpr (n == 0) {
                wait_lds<(NT * NP > 1)>(xe);
                static_for<0, DQ>([&](auto d_c) { tie(xb[decltype(d_c)::value]); });
                xb[0] &= lower_only;
                xe &= ~lower_only;
            }
            wait_lds<(n + 1 < NT * NP)>(xa[n & 1]);
            if constexpr (!two) xa[n & 1] &= lower_only;
            auto product = [&](int d, v4i &y) {
                tie(y);
                acc[dx + d][i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(xa[n & 1], y, acc[dx + d][i], 0, 0, 0);
                tie(acc[dx + d][i]);
            };
#pragma unroll
            for (int d = 0; d < DQ; ++d) product(d, xb[d]);
            if constexpr (two) product(DQ, xe);
            tie(xa[n & 1]);
        });
    };
    if constexpr (NT > 0) {
        static_for<0, AHEAD>([&](auto g_c) { read_a(g_c, g_c); });
        static_for<0, DQ>([&](auto d_c) { read_b(d_c); });
        int t = 0;
        for (; 2 * t + P_::LEAD_B + 1 < KB; ++t) step(t, std::true_type{});
        if (ahead) {
            mask_step = t;
            ask_mask();
        }
        for (; 2 * t + 1 < KB; ++t) step(t, std::false_type{});
        // the last step has read operands of a step that does not exist; nothing may copy or reuse those
        // registers before the reads are back
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        static_for<0, AHEAD>([&](auto s_c) { tie(xa[decltype(s_c)::value]); });
        static_for<0, DQ>([&](auto d_c) { tie(xb[decltype(d_c)::value]); });
        if (KB & 1) last_stage();
    } else {
        for (int t = 0; 2 * t + 1 < KB; ++t) {
            static_for<0, 2>([&](auto h_c) {
                if (2 * t + lead + decltype(h_c)::value < KB)
                    static_for<0, MAXU>([&](auto u_c) {
                        if (decltype(u_c)::value < n_loads) issue_one(u_c);
                    });
                next_issue();
            });
            wait_vmem_n(younger(t));
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
        }
    }
    const bool more = tile + gridDim.x < a.tiles;
    if ((KB & 1) && more) {                         // (the last stage's reads: see last_stage)
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    }

    // ---- the next tile's first stages, issued in front of this tile's epilogue ----
    // Every wave has the last stages in registers once all have passed the last barrier (its
    // reads are waited for in front of it): the rings are free, and the loads have the whole
    // epilogue, which uses neither the rings nor the memory pipeline much, to land.
    const int row_first_e = row_first, row_end_e = row_end;
    const uint32_t ct2_e = ct2, limb_e = limb;
    if (more) {
        tile += gridDim.x;
        map_tile(tile, prob, ct2, rb);
        begin_tile(prob, ct2, rb);
        issue_first_stages([](auto) {});
    }
    asm volatile("" ::: "memory");

    // ---- epilogue: rebuild, add the constant and the mask, reduce, store ----
    // (the lane number goes through an opaque copy: what the epilogue derives from it would
    // otherwise be computed once in front of all tiles and held in registers through the loop)
    int lane_e = lane;
    asm volatile("" : "+v"(lane_e));
    if constexpr (NT > 0) {
        constexpr int NE = 4 * NT;
        const int row_e = row_first_e + 16 * wh + 4 * (lane_e >> 4);
        const uint32_t col_e = ct2_e * 64u + (uint32_t)wc * 16u + (uint32_t)(lane_e & 15);
        // element r of the lane is row 32 (r / 4) + r % 4 behind row_e
        cop_finish<ND, NE, FULL>(
            [&](int d, int r) -> int32_t { return acc[d][r >> 2][r & 3]; }, roff,
            [&](uint64_t (&w)[NE]) {
#pragma unroll
                for (int r = 0; r < NE; ++r) {
                    if constexpr (MASKREGS) w[r] = mk[r];
                    else w[r] = 0;
                }
                if (ahead || !mask_p) return;
                const uint64_t *const mask0 = mask_p + ((size_t)row_e * a.C + col_e);
#pragma unroll
                for (int r = 0; r < NE; ++r)
                    if (FULL || row_e + roff(r) < row_end_e)
                        w[r] = __builtin_nontemporal_load(&mask0[(size_t)roff(r) * a.C]);
            },
            a, a.prev, out_p, limb_e, colsum_S, row_e, col_e, row_end_e);
    }
    return more;
    };

    for (bool first = true, more = true; more; first = false) {
        if constexpr (FULL) {
            more = pass(std::integral_constant<int, 4>{}, first);
        } else {
            switch (nt) {
            case 4: more = pass(std::integral_constant<int, 4>{}, first); break;
            case 3: more = pass(std::integral_constant<int, 3>{}, first); break;
            case 2: more = pass(std::integral_constant<int, 2>{}, first); break;
            case 1: more = pass(std::integral_constant<int, 1>{}, first); break;
            default: more = pass(std::integral_constant<int, 0>{}, first);
            }
        }
    }
}

// count problems of the same shape in one launch (count = 1: the ordinary call); the masks are
// all there or all null; prev only with count = 1
template <int DX, int DQ>
hipError_t mfma_impl(const Problem &p, int count, const void *const *staged,
                            const void *const *prepared, const uint64_t *const *masks,
                            const uint64_t *prev, uint64_t *const *outs, hipStream_t stream)
{
    const int KB = kblocks(p.k);
    const uint32_t CT = (uint32_t)(p.C / kTile);
    const uint64_t *const mask = masks[0];

    MfmaArgs a{};
    fill_common_args(p, DX, mask, prev, outs[0], &a);
    // One workgroup per compute unit at most (a compute unit holds one at a time anyway);
    // each walks the tiles id, id + grid, ...  A grid that is a multiple of 8 keeps a tile id's
    // XCD the same on every pass.
    uint32_t cus = (uint32_t)compute_units();
    if (cus >= 8) cus &= ~7u;
    const TileBlocks tb = tile_blocks(p, count);
    a.block_tiles = (uint32_t)tb.tiles;
    a.RB = tb.row_blocks;
    a.tiles = (CT / 2u) * (uint32_t)a.RB;
    const uint32_t tiles_each = a.tiles;
    a.tiles *= (uint32_t)count;
    const dim3 grid(a.tiles < cus ? a.tiles : cus);
    using P_ = Pipe<DX, DQ>;
    constexpr bool kCanMaskAhead = P_::ND <= 9;
    const bool full = p.m % 128 == 0 && a.block_tiles == 4;
    // mask words ahead: see the kernel
    const bool mask_ahead = kCanMaskAhead && mask != nullptr && full;
    auto launch_with = [&](auto full_c, auto maskahead_c, auto shared_c, auto nb_c) {
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
        b.tiles_each = tiles_each;
        return nimbus::launch(cop_mfma_kernel<DX, DQ, decltype(full_c)::value, decltype(maskahead_c)::value,
                                              decltype(shared_c)::value, NB>,
                              grid, dim3(512), stream, a, b);
    };
    auto launch = [&](auto full_c, auto maskahead_c, auto shared_c) {
        return count == 1 ? launch_with(full_c, maskahead_c, shared_c, std::integral_constant<int, 1>{})
                          : launch_with(full_c, maskahead_c, shared_c, std::integral_constant<int, kMaxBatch>{});
    };
    using T = std::true_type;
    using F = std::false_type;
    if constexpr (kCanMaskAhead) {
        if (mask_ahead) return a.RB > 1 ? launch(T{}, T{}, T{}) : launch(T{}, T{}, F{});
    }
    if (a.RB > 1) return full ? launch(T{}, F{}, T{}) : launch(F{}, F{}, T{});
    return full ? launch(T{}, F{}, F{}) : launch(F{}, F{}, F{});
}

}  // namespace nimbus
