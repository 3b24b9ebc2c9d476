// The product by the secret for rings of 2^10 to 2^13 coefficients and moduli from 2^34 to 2^59: a
// transform that stops two stages early.  (Other rings and moduli:
// rlwe_poly_kernel; at 2^14 coefficients, 16 to a thread of 1024, this kernel's registers spill: decryption 10 %
// faster, encryption up to 8 % slower.)
//
// All stages but the last two leave N/4 blocks of four coefficients, block B a residue modulo
// X^4 - zeta_B (zeta_B = the root of the block's parent, negated for odd B).  The product by the
// transformed secret is made there, as polynomials of four coefficients: with b the secret's block
//   c_0 = a_0 b_0 + a_1 zb_3 + a_2 zb_2 + a_3 zb_1,   c_1 = a_0 b_1 + a_1 b_0 + a_2 zb_3 + a_3 zb_2,  ...
// from the seven constants b_0 .. b_3 and zb_i = zeta b_i; the four products of a coefficient share one
// multiplication of their quotients' sum by the modulus.  A coefficient costs 4 products instead of 1 and
// two stages fewer each way: about the same instructions (39 against 47), but 7 constants for four coefficients
// in the middle where the full transform reads 4 + 2 x 3, and those are what the kernel
// waited for: vector loads complete in order, so constants asked for behind the coefficients' loads
// and stores in HBM wait for those.  For the same reason the constants of the other rounds come from
// where they do not queue there: through the scalar cache where they are the same for a wave, from the
// LDS where the round's fit (copied in at the start), and by vector loads a round ahead elsewhere.
//
// us a call before (full transform) and now: 768 rows of 4096 coefficients, two limbs, encrypted
// 83.0 -> 64.1; phases of 128 x 4096 x 2 13.35 -> 13.20, 300 x 4096 x 2 31.4 -> 26.3, 300 x 8192 x 2 70.2 ->
// 61.0, 8 x 8192 20.0 -> 18.0, 1000 x 4096 x 2 84.0 -> 70.6; rings of 1024 are even (one polynomial encrypted 5.5 -> 5.6,
// 2000 20.8 -> 20.3).  Bound by vector instructions in large batches: 252 a coefficient and 87 % of the SIMDs' issue cycles for
// 4096 phases of 4096 coefficients, 284 and 73 % encrypted (133 registers, three waves a SIMD instead of four); some 200 of them
// are butterflies and block products.  With one polynomial to a compute unit, 265 and 36 %, by the rounds' LDS trips between
// them.  (profiles/rlwe_product_kernel_config3_server_side.txt)
#pragma once
#include "rlwe_kernels.hpp"

namespace nimbus {

inline bool product_kernel_applies(const RlweArgs &a, int L, int logN)
{
    return logN >= kProductMinLogN && logN <= kProductMaxLogN && lazy_kind(a, L) != kNever;
}

// Stages per round by ring degree and batch size (the last two of a ring included: they count as
// stages of the round in the middle, whose threads hold whole blocks of four), at most three
// kinds of a ring.  The lines are those of 256 compute units, whatever the device has.
// Up to one polynomial per compute unit, many waves to a polynomial; more, fewer rounds; from
// 1024 polynomials on a compute unit has several workgroups at a time and few registers a thread
// matter less than few rounds.  us, 2 / 3 / 4 stages: 4096 coefficients, 256 polynomials 13.0 / 13.2 / 15.5,
// 600 30.5 / 25.7 / 27.5, 1536 (encrypted) 77.8 / 66.3 / 64.6; 2048, 256 polynomials 8.5 / 8.7 / 12.5, 2000 37.1 /
// 35.0 / 40.3; 1024, 3000 polynomials 25 / 27 / 28.
constexpr int product_kinds(int logN) { return logN == 12 ? 3 : logN == 11 ? 2 : 1; }
__host__ __device__ constexpr int product_stages(int logN, int kind)
{
    return logN == 13 ? 3 : 2 + kind;
}
constexpr int product_kind(int logN, size_t polys)
{
    const int kind = polys <= 256 ? 0 : polys < 1024 ? 1 : 2;
    return kind < product_kinds(logN) ? kind : product_kinds(logN) - 1;
}
// The rounds: `maxs` stages each, the first takes what is left.  (Whole rounds at the end have the fewest
// constants to load, and follow each other without a workgroup barrier: 8192 coefficients
// as 1 + 3 + 3 + 3 + 3 stages, not 3 + 3 + 3 + 2 + 2.)
__host__ __device__ constexpr int product_rounds(int logN, int maxs) { return (logN + maxs - 1) / maxs; }
__host__ __device__ constexpr int product_round_start(int logN, int maxs, int round)
{
    return round == 0 ? 0 : logN - (product_rounds(logN, maxs) - round) * maxs;
}

// The 9 N entries of a limb for this kernel.  The first quarter, in the natural order: the N/4 forward and
// (at N) inverse powers that the stages 0 .. log N - 3 use, and the secret's transform without the
// last two stages, times 4/N.  Then a set for each kind: forward powers, inverse powers, block
// constants.  The powers are in the order of power_slot() for its rounds; constant e of block k
// of middle group g sits at  ((7 k + e) << (log N - S)) + g,  S the stages of the middle.
__host__ __device__ constexpr int product_secret_at(int N) { return 5 * N / 4; }
__host__ __device__ constexpr int product_set_at(int N, int kind) { return (kind + 1) * (9 * N / 4); }
__host__ __device__ constexpr int product_inverse_at(int N) { return N / 4; }
__host__ __device__ constexpr int product_blocks_at(int N) { return N / 2; }    // 7 N / 4 entries

template <int LOGN, int MAXS, int IDX>
struct ProductRound {
    static constexpr int F = product_rounds(LOGN, MAXS), TOTAL = 2 * F - 1;
    static constexpr int J = IDX < F ? IDX : 2 * F - 2 - IDX;       // forward round
    static constexpr int P0 = product_round_start(LOGN, MAXS, J);
    static constexpr int S = product_round_start(LOGN, MAXS, J + 1) - P0;
    static constexpr int R = 1 << S, LT = LOGN - P0 - S, NT = threads_for(LOGN, MAXS);
    static constexpr int G = (1 << LOGN) >> S, GP = G / NT;          // groups, groups of a thread
    static_assert(G % NT == 0 && GP >= 1 && S <= 4 && NT >= 64, "whole groups per thread");
    static constexpr bool MIDDLE = IDX == F - 1, INVERSE = IDX > F - 1, LAST = IDX == TOTAL - 1;
    static constexpr int STAGES = MIDDLE ? S - 2 : S;
    // Where the constants come from.  One block per wave: through the scalar cache.  At most 256 of them
    // (from stage P0 on, in the order of the set): in the LDS.  The inverse powers of a round are the
    // negated forward ones in reverse order, so one copy serves both ways.
    static constexpr bool UNIFORM = P0 == 0 || LT >= 6;
    static constexpr int LDS_FIRST = 1 << P0, LDS_END = 1 << (P0 + S);
    static constexpr bool IN_LDS = !UNIFORM && !MIDDLE && LDS_END <= 256;
    static constexpr bool BY_VECTOR = !UNIFORM && !IN_LDS;
    // by vector loads: a round ahead where the registers hold them, with the middle's first block
    static constexpr int POWERS = (1 << STAGES) - 1;
    static constexpr bool AHEAD = BY_VECTOR && GP * POWERS <= 8;
    static constexpr bool BLOCK_AHEAD = MIDDLE && MAXS < 4;

    // bounds in multiples of q, as in RoundOf; the middle leaves sums of four products
    static constexpr int stages_of(int idx)
    {
        const int j = idx < F ? idx : 2 * F - 2 - idx;
        return product_round_start(LOGN, MAXS, j + 1) - product_round_start(LOGN, MAXS, j) - (idx == F - 1 ? 2 : 0);
    }
    static constexpr unsigned tout_of(int idx, int lazy)
    {
        return idx + 1 < TOTAL ? lazy_units(lazy) >> stages_of(idx + 1) : kFoldUnits;
    }
    static constexpr unsigned bin_of(int idx, int lazy)
    {
        unsigned b = 4 * product_units(lazy);
        for (int i = F - 1; i < idx; ++i)
            b = inverse_round_out(stages_of(i), b, tout_of(i, lazy), product_units(lazy));
        return b;
    }
};

// entries [first, end) of the set that the rounds in the LDS use (they follow each other)
template <int LOGN, int MAXS, int IDX = 0>
constexpr int lds_entries_first()
{
    using Me = ProductRound<LOGN, MAXS, IDX>;
    if constexpr (Me::IN_LDS) return Me::LDS_FIRST;
    else if constexpr (IDX + 1 < Me::F) return lds_entries_first<LOGN, MAXS, IDX + 1>();
    else return 0;
}
template <int LOGN, int MAXS, int IDX = 0>
constexpr int lds_entries_end()
{
    using Me = ProductRound<LOGN, MAXS, IDX>;
    const int here = Me::IN_LDS ? Me::LDS_END : 0;
    if constexpr (IDX + 1 < Me::F) {
        const int later = lds_entries_end<LOGN, MAXS, IDX + 1>();
        return later > here ? later : here;
    } else {
        return here;
    }
}

template <int GP, int POWERS, bool BLOCK>
struct VectorTable {
    Twiddle e[GP][POWERS > 0 ? POWERS : 1];
    Twiddle block[BLOCK ? 7 : 1];
};
struct NoVectorTable {};

// the constants of block k of the middle's group g
template <typename Rd, int LOGN>
__device__ __forceinline__ void load_block(const Twiddle *__restrict__ set, int g, int k, Twiddle (&b)[7])
{
#pragma unroll
    for (int e = 0; e < 7; ++e) b[e] = set[product_blocks_at(1 << LOGN) + (k * 7 + e) * Rd::G + g];
}
// the powers of a thread's groups in round Rd (`table`: forward or inverse), and what goes with them
template <typename Rd, int LOGN, bool BLOCK>
__device__ __forceinline__ auto load_powers(const Twiddle *__restrict__ set, const Twiddle *__restrict__ table, int tid)
{
    VectorTable<Rd::GP, Rd::POWERS, BLOCK> t;
#pragma unroll
    for (int j = 0; j < Rd::GP; ++j) {
        const Group<LOGN, Rd::P0, Rd::S> grp(tid + j * Rd::NT);
#pragma unroll
        for (int st = 0; st < Rd::STAGES; ++st)
#pragma unroll
            for (int i = 0; i < (1 << st); ++i)
                t.e[j][(1 << st) - 1 + i] = table[grp.template entry<true>(st, i)];
    }
    if constexpr (BLOCK) load_block<Rd, LOGN>(set, tid, 0, t.block);
    return t;
}

// floor(x w' / 2^64) or at most 2 less (see mul_loose())
template <int LAZY>
__device__ __forceinline__ uint64_t quotient_of(uint64_t x, uint64_t ws)
{
    const uint32_t x0 = (uint32_t)x, x1 = (uint32_t)(x >> 32);
    const uint32_t w0 = (uint32_t)ws, w1 = (uint32_t)(ws >> 32);
    return LAZY == kLoose ? (uint64_t)x1 * w1 + __umulhi(x0, w1) + __umulhi(x1, w0) : __umul64hi(x, ws);
}
template <int LAZY>
__device__ __forceinline__ uint64_t product_of(uint64_t x, const Twiddle &t, uint64_t nq)
{
    return x * t.w + quotient_of<LAZY>(x, t.ws) * nq;
}

// the first STAGES forward stages of a group of 2^S coefficients; F(st, j): table entry
template <int S, int STAGES, int LAZY, typename Fwd>
__device__ __forceinline__ void forward_stages(uint64_t (&x)[1 << S], const Mod &md, Fwd F)
{
    constexpr int R = 1 << S;
#pragma unroll
    for (int st = 0; st < STAGES; ++st) {
        const int half = R >> (st + 1);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (r & half) continue;
            const uint64_t u = x[r], v = product_of<LAZY>(x[r + half], F(st, r >> (S - st)), md.nq);
            x[r] = u + v;
            x[r + half] = u + product_units(LAZY) * md.q - v;
        }
    }
}

// the same stages backwards.  BIN, TOUT: see group_butterflies().  NEGATED: I(st, j) hands out the
// negatives of the entries, which the order of the difference makes up for.
template <int S, int STAGES, int LAZY, unsigned BIN, unsigned TOUT, bool NEGATED, typename Inv>
__device__ __forceinline__ void inverse_stages(uint64_t (&x)[1 << S], const Mod &md, Inv I)
{
    constexpr int R = 1 << S;
    static_assert((BIN << STAGES) <= lazy_units(LAZY), "inverse round overflows");
    unsigned b[R];              // folded away: every index below is a constant after unrolling
#pragma unroll
    for (int r = 0; r < R; ++r) b[r] = BIN;
#pragma unroll
    for (int st = STAGES - 1; st >= 0; --st) {
        const int half = R >> (st + 1);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (r & half) continue;
            const uint64_t u = x[r], v = x[r + half];
            x[r] = u + v;
            const uint64_t d = NEGATED ? v + b[r] * md.q - u : u + b[r + half] * md.q - v;
            x[r + half] = product_of<LAZY>(d, I(st, r >> (S - st)), md.nq);
            b[r] += b[r + half];
            b[r + half] = product_units(LAZY);
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (b[r] > TOUT) x[r] = fold(x[r], md);
}

// a(X) b(X) modulo X^4 - zeta, b = (b_0, b_1, b_2, b_3, zb_1, zb_2, zb_3).  Quotients and products are
// summed modulo 2^64: what is left, the sum of four results of product_of(), fits.
template <int LAZY>
__device__ __forceinline__ void block_product(uint64_t *a, const Twiddle (&b)[7], const Mod &md)
{
    uint64_t c[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        uint64_t h = 0, p = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const Twiddle &t = b[i <= k ? k - i : 7 + k - i];
            h += quotient_of<LAZY>(a[i], t.ws);
            p += a[i] * t.w;
        }
        c[k] = p + h * md.nq;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) a[k] = c[k];
}

// what separates round IDX from the next one: nothing but the order of a wave's own LDS accesses
// where both keep every wave inside its own coefficients (see wave_local_after())
template <int LOGN, int MAXS, int IDX>
__device__ __forceinline__ void between_product_rounds()
{
    using Me = ProductRound<LOGN, MAXS, IDX>;
    using Next = ProductRound<LOGN, MAXS, IDX + 1>;
    if constexpr (Me::S == Next::S && Me::LT <= 6 && Next::LT <= 6) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
        __syncthreads();
    }
}

// Round IDX and all behind it.  `mine`: the round's powers where they come by vector loads; the next
// round's are asked for in front of this one's arithmetic.  `ask_addend` runs in front of one of the last
// rounds, behind the last wait for a vector load.  xio: the thread's coefficients tid + i NT (group tid + j NT
// of the first and the last round: i = j + r GP), brought and taken away.
template <int LOGN, int MAXS, int LAZY, int IDX, typename Table, typename Hook>
__device__ __forceinline__ void product_rounds_from(uint64_t *lds, const Twiddle *lds_powers,
                                                    const Twiddle *__restrict__ set, const Mod &md, int tid,
                                                    const Table &mine, Hook ask_addend, uint64_t *xio)
{
    using Me = ProductRound<LOGN, MAXS, IDX>;
    using Grp = Group<LOGN, Me::P0, Me::S>;
    constexpr int S = Me::S, R = Me::R, GP = Me::GP, N = 1 << LOGN, P0 = Me::P0;
    constexpr unsigned BIN = IDX < Me::F - 1 ? 0 : Me::bin_of(IDX, LAZY), TOUT = Me::tout_of(IDX, LAZY);
    constexpr int ASK = Me::TOTAL - (MAXS == 4 ? 1 : 2);
    static_assert(ASK >= Me::F, "behind the middle");
    const Twiddle *const fwd = set, *const inv = set + product_inverse_at(N);
    uint64_t x[GP][R];
    int base[GP], i0[GP];
#pragma unroll
    for (int j = 0; j < GP; ++j) {
        const Grp grp(tid + j * Me::NT);
        base[j] = pad(grp.base);
        i0[j] = P0 == 0 ? 0 : Me::UNIFORM ? __builtin_amdgcn_readfirstlane(grp.i0) : grp.i0;
    }
    // (a group's coefficients are a padded step apart: below LT + S = 4 they share one block of 16)
    auto slot = [&](int j, int r) { return base[j] + Grp::padded_step(r); };
#pragma unroll
    for (int j = 0; j < GP; ++j)
#pragma unroll
        for (int r = 0; r < R; ++r) x[j][r] = IDX == 0 ? xio[j + r * GP] : lds[slot(j, r)];

    auto ask_next = [&]() {
        if constexpr (Me::LAST) {
            return NoVectorTable{};
        } else {
            using Next = ProductRound<LOGN, MAXS, IDX + 1>;
            if constexpr (Next::AHEAD)
                return load_powers<Next, LOGN, Next::BLOCK_AHEAD>(set, Next::INVERSE ? inv : fwd, tid);
            else
                return NoVectorTable{};
        }
    };
    const auto &powers = [&]() -> decltype(auto) {
        if constexpr (Me::BY_VECTOR && !Me::AHEAD)
            return load_powers<Me, LOGN, Me::BLOCK_AHEAD>(set, Me::INVERSE ? inv : fwd, tid);
        else
            return (mine);
    }();
    // entry j of stage st of the thread's group g (see Group::entry())
    auto power = [&](int g, int st, int j) -> Twiddle {
        if constexpr (Me::UNIFORM) {
            typedef const __attribute__((address_space(4))) Twiddle *Uniform;
            const Uniform at = (Uniform)(Me::INVERSE ? inv : fwd) + ((1 << (P0 + st)) + (j << P0) + i0[g]);
            return Twiddle{at->w, at->ws};
        } else if constexpr (Me::IN_LDS) {
            constexpr int first = lds_entries_first<LOGN, MAXS>();
            const int e = Me::INVERSE ? (((1 << st) - 1 - j) << P0) + ((1 << P0) - 1 - i0[g]) : (j << P0) + i0[g];
            return lds_powers[(1 << (P0 + st)) + e - first];
        } else {
            return powers.e[g][(1 << st) - 1 + j];
        }
    };
    auto finish = [&](const auto &next) {
        if constexpr (Me::LAST) {
#pragma unroll
            for (int j = 0; j < GP; ++j)
#pragma unroll
                for (int r = 0; r < R; ++r) xio[j + r * GP] = x[j][r];
        } else {
#pragma unroll
            for (int j = 0; j < GP; ++j)
#pragma unroll
                for (int r = 0; r < R; ++r) lds[slot(j, r)] = x[j][r];
            between_product_rounds<LOGN, MAXS, IDX>();
            product_rounds_from<LOGN, MAXS, LAZY, IDX + 1>(lds, lds_powers, set, md, tid, next, ask_addend, xio);
        }
    };
    // (the scheduling barriers keep what is asked for ahead in front of the arithmetic)
    if constexpr (Me::MIDDLE) {
        constexpr int BLOCKS = R / 4;
        const auto inverse = load_powers<Me, LOGN, false>(set, inv, tid);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < GP; ++j)
            forward_stages<S, Me::STAGES, LAZY>(x[j], md, [&](int st, int i) { return powers.e[j][(1 << st) - 1 + i]; });
#pragma unroll
        for (int j = 0; j < GP; ++j)
#pragma unroll
            for (int k = 0; k < BLOCKS; ++k) {
                Twiddle b[7];
                if constexpr (Me::BLOCK_AHEAD) {
                    if (j == 0 && k == 0) {
#pragma unroll
                        for (int e = 0; e < 7; ++e) b[e] = powers.block[e];
                    } else {
                        load_block<Me, LOGN>(set, tid + j * Me::NT, k, b);
                    }
                } else {
                    load_block<Me, LOGN>(set, tid + j * Me::NT, k, b);
                }
                __builtin_amdgcn_sched_barrier(0);
                block_product<LAZY>(&x[j][k * 4], b, md);
                __builtin_amdgcn_sched_barrier(0);
            }
        const auto next = ask_next();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < GP; ++j)
            inverse_stages<S, Me::STAGES, LAZY, BIN, TOUT, false>(
                x[j], md, [&](int st, int i) { return inverse.e[j][(1 << st) - 1 + i]; });
        finish(next);
    } else {
        const auto next = ask_next();
        if constexpr (IDX == ASK) ask_addend();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < GP; ++j) {
            auto entry = [&](int st, int i) { return power(j, st, i); };
            if constexpr (Me::INVERSE) inverse_stages<S, S, LAZY, BIN, TOUT, Me::IN_LDS>(x[j], md, entry);
            else forward_stages<S, S, LAZY>(x[j], md, entry);
        }
        finish(next);
    }
}

// One workgroup per (ciphertext, limb), as rlwe_poly_kernel; LAZY is kLoose or kTight.
template <int LOGN, int MAXS, bool ENCRYPT, int LAZY>
__global__ __launch_bounds__(threads_for(LOGN, MAXS)) void rlwe_product_kernel(PolyArgs a)
{
    constexpr int N = 1 << LOGN, NT = threads_for(LOGN, MAXS), IT = N / NT;
    constexpr int FIRST = lds_entries_first<LOGN, MAXS>(), IN_LDS = lds_entries_end<LOGN, MAXS>() - FIRST;
    __shared__ uint64_t lds[padded_size(N)];
    __shared__ Twiddle lds_powers[IN_LDS > 0 ? IN_LDS : 1];
    const int tid = threadIdx.x;
    const uint32_t row = blockIdx.x / (uint32_t)a.L, l = blockIdx.x % (uint32_t)a.L;
    const RlweLimb &P = a.limbs.limb[l];
    const uint64_t q = P.red.q;
    const Mod md = make_mod(P);
    const Twiddle *const set = a.tables + (size_t)l * limb_table_entries(N) + product_set_at(N, a.set);
    // thread `tid` has the coefficients tid + i NT on the way in and on the way out
    const uint64_t *const in = ENCRYPT ? a.src + ((size_t)row * a.L + l) * N
                                       : a.src + (((size_t)row * 2 + 1) * a.L + l) * N;
    uint64_t *const out = ENCRYPT ? a.dst + (((size_t)row * 2 + 0) * a.L + l) * N
                                  : a.dst + ((size_t)row * a.L + l) * N;
    uint64_t *const c1 = a.dst + (((size_t)row * 2 + 1) * a.L + l) * N;
    // (visible to all behind the barrier that ends the first round)
    for (int i = tid; i < IN_LDS; i += NT) lds_powers[i] = set[FIRST + i];
    uint64_t x[IT], addend[IT];
    int err[IT];
#pragma unroll
    for (int i = 0; i < IT; ++i) x[i] = in[tid + i * NT];
    if constexpr (ENCRYPT) {
#pragma unroll
        for (int i = 0; i < IT; ++i) c1[tid + i * NT] = x[i];
    }
    auto ask_addend = [&]() {
#pragma unroll
        for (int i = 0; i < IT; ++i) {
            if constexpr (ENCRYPT) {
                addend[i] = encrypt_weight(a, row, (uint32_t)(tid + i * NT), N);
                err[i] = a.e[(size_t)row * N + tid + i * NT];
            } else {
                addend[i] = a.src[(((size_t)row * 2 + 0) * a.L + l) * N + tid + i * NT];
            }
        }
    };
    product_rounds_from<LOGN, MAXS, LAZY, 0>(lds, lds_powers, set, md, tid, NoVectorTable{}, ask_addend, x);
#pragma unroll
    for (int i = 0; i < IT; ++i) {
        const uint64_t as = cond_sub(x[i], md.nq);                          // [0, 2q) -> [0, q)
        if constexpr (ENCRYPT) out[tid + i * NT] = finish_encrypt(as, addend[i], err[i], P, md);
        else out[tid + i * NT] = finish_phase(as, addend[i], q);
    }
}

template <bool ENCRYPT, int LAZY>
static hipError_t launch_product_with(PolyArgs a, int logN, size_t polys, hipStream_t stream)
{
    const int kind = product_kind(logN, polys);
    a.set = kind;
    auto go = [&](auto logn_c) {
        constexpr int LOGN = decltype(logn_c)::value;
        auto with = [&](auto kind_c) {
            constexpr int MAXS = product_stages(LOGN, decltype(kind_c)::value);
            return launch(rlwe_product_kernel<LOGN, MAXS, ENCRYPT, LAZY>, dim3((unsigned)polys),
                          dim3(threads_for(LOGN, MAXS)), stream, a);
        };
        if constexpr (product_kinds(LOGN) > 2)
            if (kind == 2) return with(std::integral_constant<int, 2>{});
        if constexpr (product_kinds(LOGN) > 1)
            if (kind == 1) return with(std::integral_constant<int, 1>{});
        return with(std::integral_constant<int, 0>{});
    };
    switch (logN) {
    case 10: return go(std::integral_constant<int, 10>{});
    case 11: return go(std::integral_constant<int, 11>{});
    case 12: return go(std::integral_constant<int, 12>{});
    case 13: return go(std::integral_constant<int, 13>{});
    default: return hipErrorInvalidValue;
    }
}

// the product by the secret and what follows it, for every ring and modulus
template <bool ENCRYPT>
static hipError_t launch_product(const PolyArgs &a, int logN, size_t polys, hipStream_t stream)
{
    if (!product_kernel_applies(a.limbs, a.L, logN)) return launch_poly<ENCRYPT>(a, logN, polys, stream);
    if (lazy_kind(a.limbs, a.L) == kLoose) return launch_product_with<ENCRYPT, kLoose>(a, logN, polys, stream);
    return launch_product_with<ENCRYPT, kTight>(a, logN, polys, stream);
}

}  // namespace nimbus
