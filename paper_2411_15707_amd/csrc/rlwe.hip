// Server side of the Nimbus linear layer on gfx950: negacyclic number-theoretic transform
// per RNS limb, and on top of it the setup-phase encryption of the weight rows (Algorithm 1
// step 1 with the row-wise encoding of Section 3.2, Eq. (2)) and the decryption + decoding
// of returned ciphertexts (Algorithm 1 step 5; Enc / Dec of Appendix B.1).
// Declarations and the contract of every entry point: include/nimbus_rlwe.h.
//
// One workgroup transforms one polynomial of one limb entirely inside the LDS:
//   load -> forward rounds -> pointwise product with the transformed secret -> inverse
//   rounds -> (add c0 | assemble c0) -> store,
// so a product c1 * s costs one read of c1 and one write of the result in HBM.  (A ring of
// 2^15 coefficients does not fit: two workgroups per polynomial take one half each, with
// the first forward stage done on the way in and the last inverse stage in a pass of its
// own; see Part below.)
//
// Transform (the usual in-place pair for X^N + 1, psi a primitive 2N-th root of unity):
//   forward:  stages m = 1, 2, 4, ..., N/2 blocks; in block i of a stage every pair
//             (j, j + t), t = N / 2m, becomes (u + w v, u - w v) with w = psi^brv(m + i);
//             natural order in, bit-reversed order out;
//   inverse:  the same stages backwards, (u, v) -> (u + v, (u - v) w^-1); the factor 1/N
//             is folded into the table of the transformed secret.
// A round keeps 2^S coefficients of a thread in registers for S <= 4 consecutive stages;
// between rounds the coefficients go through the LDS.  The last forward round, the
// pointwise product and the first inverse round work on the same coefficients of the same
// thread and are one round.  The first round takes its coefficients straight from the
// coalesced loads and the last one hands its own to the stores (one group per thread: the
// same coefficients), and rounds that keep every wave inside its own coefficients follow
// each other without a workgroup barrier.
//
// Arithmetic: a product by a table constant w uses its companion w' = floor(w 2^64 / q):
//   x w - floor(x w' / 2^64) q  lies in [0, 2q) for every 64-bit x.
// Moduli below 2^62: values kept lazily in [0, 4q) (forward) and [0, 2q) (inverse) by one
// conditional subtraction per butterfly.  Moduli from 2^34 to 2^58 (every parameter set of
// the benchmark configurations): no conditional subtractions, bounds tracked at compile time
// instead, and a cheaper quotient estimate; see group_butterflies.
//
// Rings of 2^10 to 2^13 coefficients with moduli from 2^34 to 2^59 take another kernel, whose transform
// stops two stages early: rlwe_product.hpp.
//
// Tables: the constants of a transform are read once per polynomial from the second-level
// cache; they are stored again, for each kind of batch, in the order in which the threads of the
// product kernels read them (neighbouring lanes, neighbouring entries; see power_slot()).
#include "rlwe_product.hpp"

namespace nimbus {

__device__ uint64_t powmod(uint64_t base, uint32_t e, const Limb &P)
{
    uint64_t r = 1;
    while (e) {
        if (e & 1u) r = mulmod(r, base, P);
        base = mulmod(base, base, P);
        e >>= 1;
    }
    return r;
}

// floor(w * 2^64 / q) for w < q < 2^62: schoolbook binary division
__device__ uint64_t companion(uint64_t w, uint64_t q)
{
    uint64_t r = w, quo = 0;
    for (int i = 0; i < 64; ++i) {
        r <<= 1;
        quo <<= 1;
        if (r >= q) {
            r -= q;
            quo |= 1u;
        }
    }
    return quo;
}

// ---------------------------------------------------------------------------
// setup: powers of psi in bit-reversed order, forward and inverse, with companions
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void rlwe_powers_kernel(RlweArgs a, int logN, int L,
                                                          Twiddle *__restrict__ tables)
{
    const uint32_t N = 1u << logN;
    const uint32_t gid = blockIdx.x * 256u + threadIdx.x;
    if (gid >= N * (uint32_t)L) return;
    const uint32_t l = gid >> logN, i = gid & (N - 1u);
    const RlweLimb &P = a.limb[l];
    const uint32_t e = __brev(i) >> (32 - logN);
    Twiddle *const t = tables + (size_t)l * limb_table_entries((int)N);
    const uint64_t f = powmod(P.psi, e, P.red), g = powmod(P.psi_inv, e, P.red);
    t[i] = Twiddle{f, companion(f, P.red.q)};
    t[N + i] = Twiddle{g, companion(g, P.red.q)};
}

// ---------------------------------------------------------------------------
// setup: transform of the secret, times 1/N, with companions
// one workgroup per limb
// ---------------------------------------------------------------------------
// (SKIP: the last stages that are left out, with the factor 2^SKIP / N; see rlwe_product.hpp)
template <int LOGN, int PRE, int SKIP>
__global__ __launch_bounds__(threads_for(LOGN - PRE, 4)) void rlwe_secret_kernel(
    RlweArgs a, const int8_t *__restrict__ s, Twiddle *__restrict__ tables)
{
    constexpr int N = 1 << LOGN, NP = N >> PRE, NT = threads_for(LOGN - PRE, 4);
    __shared__ uint64_t lds[padded_size(NP)];
    const int tid = threadIdx.x, l = blockIdx.x >> PRE, h = blockIdx.x & ((1 << PRE) - 1);
    const RlweLimb &P = a.limb[l];
    const uint64_t q = P.red.q;
    const Mod md = make_mod(P);
    Twiddle *const t = tables + (size_t)l * limb_table_entries(N);
    auto lifted = [&](int c) -> uint64_t {
        const int v = s[c];
        return v < 0 ? q - (uint64_t)(-v) : (uint64_t)v;
    };
    if constexpr (PRE == 0) {
        for (int c = tid; c < N; c += NT) lds[pad(c)] = lifted(c);
    } else {
        const Twiddle w0 = t[1];                            // stage 0 has one block: entry 1
        for (int c = tid; c < NP; c += NT)
            lds[pad(c)] = enter_part<PRE>(lifted(c), lifted(c + NP), w0, md, h);
    }
    __syncthreads();
    forward_only<LOGN, PRE, 4, PRE, NT, LOGN - SKIP>(lds, t, md, tid, h);
    for (int c = tid; c < NP; c += NT) {
        uint64_t v = lds[pad(c)];               // [0, 4q)
        v = v >= 2 * q ? v - 2 * q : v;
        v = v >= q ? v - q : v;
        v = mulmod(v, P.n_inv, P.red);
        if constexpr (SKIP > 0) v = mulmod(v, 1u << SKIP, P.red);
        t[(SKIP > 0 ? product_secret_at(N) : 2 * N) + h * NP + c] = Twiddle{v, companion(v, q)};
    }
}

// setup: set 0 of every limb copied into the order of the product kernels with `maxs` stages
// per round (see power_slot()); one thread per entry
__global__ __launch_bounds__(256) void rlwe_table_set_kernel(Twiddle *__restrict__ tables, int logN, int L,
                                                             int pre, int maxs, int set)
{
    const uint32_t N = 1u << logN;
    const uint32_t gid = blockIdx.x * 256u + threadIdx.x;
    if (gid >= N * (uint32_t)L) return;
    const uint32_t l = gid >> logN, e = gid & (N - 1u);
    const Twiddle *const from = tables + (size_t)l * limb_table_entries((int)N);
    Twiddle *const to = tables + (size_t)l * limb_table_entries((int)N) + (size_t)set * set_entries((int)N);
    const int p = power_slot(logN, pre, maxs, (int)e);
    to[p] = from[e];
    to[N + p] = from[N + e];
    to[2 * N + secret_slot(logN, pre, maxs, (int)e)] = from[2 * N + e];
}

// setup: the sets of rlwe_product_kernel, blockIdx.y the kind of batch (see rlwe_product.hpp); one thread per
// coefficient of the secret's transform, the first N/4 for a power each way too.  Bound by its launch: with one for
// each kind the setup of 4096 coefficients took 60.2 us (three kinds, two limbs), now 52.3; of 2048 (two) 55.0 and 50.5.
__global__ __launch_bounds__(256) void rlwe_product_set_kernel(RlweArgs a, Twiddle *__restrict__ tables, int logN, int L)
{
    const int N = 1 << logN, kind = (int)blockIdx.y, maxs = product_stages(logN, kind);
    const uint32_t gid = blockIdx.x * 256u + threadIdx.x;
    if (gid >= (uint32_t)N * (uint32_t)L) return;
    const uint32_t l = gid >> logN;
    const int c = (int)(gid & (uint32_t)(N - 1));
    const Twiddle *const from = tables + (size_t)l * limb_table_entries(N);
    Twiddle *const to = tables + (size_t)l * limb_table_entries(N) + product_set_at(N, kind);
    int round = 0;                                      // the round whose stages hold the power's
    if (c < N / 4) {
        int slot = c;
        if (c > 0) {
            int s = 0;
            while ((2 << s) <= c) ++s;                  // stage of entry c: 2^s <= c < 2^(s+1)
            while (product_round_start(logN, maxs, round + 1) <= s) ++round;
            const int p0 = product_round_start(logN, maxs, round), st = s - p0, b = c - (1 << s);
            slot = (1 << s) + ((b & ((1 << st) - 1)) << p0) + (b >> st);
        }
        to[slot] = from[c];
        to[product_inverse_at(N) + slot] = from[N + c];
    }
    while (product_round_start(logN, maxs, round + 1) < logN) ++round;
    const int S = logN - product_round_start(logN, maxs, round);
    const int block = c >> 2, i = c & 3, k = block & ((1 << (S - 2)) - 1), group = c >> S, groups = N >> S;
    Twiddle *const at = to + product_blocks_at(N) + (size_t)k * 7 * groups + group;
    const Twiddle b = from[product_secret_at(N) + c];
    at[i * groups] = b;
    if (i == 0) return;
    // zeta: the parent block's power (stage log N - 3: N/8 blocks), for an odd block its negative
    const Limb &P = a.limb[l].red;
    const uint64_t root = from[N / 8 + (block >> 1)].w;
    const uint64_t w = mulmod(b.w, block & 1 ? P.q - root : root, P);
    at[(3 + i) * groups] = Twiddle{w, companion(w, P.q)};
}

// ---------------------------------------------------------------------------
// decoding: CRT of the limb phases, then rounding division by Delta
// ---------------------------------------------------------------------------
// Up to four limbs, Q < 2^248.  Mixed-radix form of the Chinese remainder theorem:
//   phi = a_0 + q_0 (a_1 + q_1 (a_2 + q_2 a_3)),
//   a_j = ( ... ((phi_j - a_0) q_0^-1 - a_1) q_1^-1 - ... - a_{j-1}) q_{j-1}^-1  mod q_j.
// The products by the constants q_i^-1 take any 64-bit factor and leave a value below 2 q_j
// (mul_lazy), so nothing is reduced on the way: with c_ij the multiple of q_j from q_i up to q_i + q_j,
// phi_j + c_ij - a_i < 2 q_j + q_i + q_j < 2^64.  One conditional subtraction makes the digit
// canonical.
//
// The quotient (phi + Delta/2) / Delta, below 2^33, is formed in double precision: the digits
// and moduli, sums, products and the reciprocal round fewer than sixteen times, so the estimate, below
// 2^33, is off by less than 2^33 16 2^-53 = 2^-16.  Only where its fraction lies within 2^-14 of an
// integer (never for a ciphertext that decrypts with noise to spare) is it settled with integers
// of L words.
//
// Bound by HBM: (L + 1) 8 bytes a coefficient.  256 x 8192 coefficients of three limbs: 12.6 us; 26.5 with
// a reduction of a 128-bit value per step and four-word integers throughout.
struct DecodeArgs {
    const uint64_t *phi;    // [T][L][N]
    uint64_t *m_hat;        // [T][N]
    int logN;
    uint64_t total;         // T * N
    uint64_t q[kMaxLimbs];
    Twiddle inv[kMaxLimbs][kMaxLimbs];      // inv[i][j] = q_i^-1 mod q_j for i < j
    uint64_t above[kMaxLimbs][kMaxLimbs];   // c_ij
    uint64_t delta[kMaxLimbs], half[kMaxLimbs];     // Delta and floor(Delta / 2), least significant word first
    double q_d[kMaxLimbs], half_d, delta_inv;       // rounded; delta_inv = 1 / Delta
    uint64_t t_mask;
};

template <int W>
struct Wide {
    uint64_t w[W];
};

template <int W>
__device__ __forceinline__ Wide<W> wide_mul_add(const Wide<W> &a, uint64_t m, uint64_t add)    // a m + add
{
    Wide<W> r;
    u128 carry = add;
#pragma unroll
    for (int i = 0; i < W; ++i) {
        const u128 p = (u128)a.w[i] * m + carry;
        r.w[i] = (uint64_t)p;
        carry = p >> 64;
    }
    return r;
}

template <int W>
__device__ __forceinline__ Wide<W> wide_add(const Wide<W> &a, const Wide<W> &b)
{
    Wide<W> r;
    u128 carry = 0;
#pragma unroll
    for (int i = 0; i < W; ++i) {
        const u128 t = (u128)a.w[i] + b.w[i] + carry;
        r.w[i] = (uint64_t)t;
        carry = t >> 64;
    }
    return r;
}

// a - b modulo 2^(64 W) and whether it borrowed (a < b)
template <int W>
__device__ __forceinline__ bool wide_sub(const Wide<W> &a, const Wide<W> &b, Wide<W> &r)
{
    uint64_t borrow = 0;
#pragma unroll
    for (int i = 0; i < W; ++i) {
        const u128 t = (u128)a.w[i] - b.w[i] - borrow;
        r.w[i] = (uint64_t)t;
        borrow = (uint64_t)(t >> 64) & 1u;
    }
    return borrow != 0;
}

// floor((phi + half) / Delta) from an estimate within one of it, for the phase with these digits
template <int L>
__device__ __forceinline__ uint64_t settle_quotient(const DecodeArgs &a, const uint64_t (&digit)[L], uint64_t est)
{
    Wide<L> num = {}, delta, half;
    num.w[0] = digit[L - 1];
#pragma unroll
    for (int j = L - 2; j >= 0; --j) num = wide_mul_add<L>(num, a.q[j], digit[j]);
#pragma unroll
    for (int i = 0; i < L; ++i) {
        delta.w[i] = a.delta[i];
        half.w[i] = a.half[i];
    }
    num = wide_add<L>(num, half);               // < 1.5 Q: fits
    const Wide<L> prod = wide_mul_add<L>(delta, est, 0);    // about num
    Wide<L> rem, over;
    if (wide_sub<L>(num, prod, rem)) {          // one too many
        est -= 1;
        rem = wide_add<L>(rem, delta);          // wraps back to num - est Delta
    }
    return wide_sub<L>(rem, delta, over) ? est : est + 1;   // one too few
}

template <int L>
__global__ __launch_bounds__(256) void rlwe_decode_kernel(const DecodeArgs a)
{
    const uint64_t gid = (uint64_t)blockIdx.x * 256u + threadIdx.x;
    if (gid >= a.total) return;
    const uint64_t N = 1ull << a.logN;
    const uint64_t row = gid >> a.logN, c = gid & (N - 1);
    const uint64_t *const ph = a.phi + row * (uint64_t)L * N + c;
    uint64_t digit[L];
#pragma unroll
    for (int j = 0; j < L; ++j) digit[j] = ph[(uint64_t)j * N];
#pragma unroll
    for (int j = 1; j < L; ++j) {
        const uint64_t nq = negated(a.q[j]);
        uint64_t v = digit[j];
#pragma unroll
        for (int i = 0; i < j; ++i) v = mul_lazy(v + (a.above[i][j] - digit[i]), a.inv[i][j], nq);
        digit[j] = cond_sub(v, nq);             // below 2 q_j -> below q_j
    }
    double num = (double)digit[L - 1];
#pragma unroll
    for (int j = L - 2; j >= 0; --j) num = fma(num, a.q_d[j], (double)digit[j]);
    const double quo = (num + a.half_d) * a.delta_inv;
    const double whole = floor(quo), frac = quo - whole;
    uint64_t est = (uint64_t)whole;
    if (frac < 0x1p-14 || frac > 1.0 - 0x1p-14) est = settle_quotient<L>(a, digit, est);
    a.m_hat[gid] = est & a.t_mask;
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
static uint64_t h_mulmod(uint64_t a, uint64_t b, uint64_t q) { return (uint64_t)((u128)a * b % q); }

static uint64_t h_powmod(uint64_t base, uint64_t e, uint64_t q)
{
    uint64_t r = 1 % q;
    base %= q;
    while (e) {
        if (e & 1) r = h_mulmod(r, base, q);
        base = h_mulmod(base, base, q);
        e >>= 1;
    }
    return r;
}

// inverse of a modulo mod (coprime), by the extended Euclidean algorithm
static uint64_t h_invmod(uint64_t a, uint64_t mod)
{
    __int128 old_r = (__int128)(a % mod), r = (__int128)mod, old_c = 1, c = 0;
    while (r != 0) {
        const __int128 quo = old_r / r;
        const __int128 nr = old_r - quo * r;
        old_r = r;
        r = nr;
        const __int128 ncoef = old_c - quo * c;
        old_c = c;
        c = ncoef;
    }
    if (old_r != 1) return 0;                   // not coprime
    __int128 res = old_c % (__int128)mod;
    if (res < 0) res += mod;
    return (uint64_t)res;
}

static int log2_exact(int N)
{
    int b = 0;
    while ((1 << b) < N) ++b;
    return b;
}

static int bit_length64(uint64_t v)
{
    int b = 0;
    while (v) { ++b; v >>= 1; }
    return b;
}

// shape and modulus checks shared by every entry point; fills the reduction constants
// byte ranges [a, a + na) and [b, b + nb) share a byte
static bool ranges_overlap(const void *a, size_t na, const void *b, size_t nb)
{
    if (!a || !b || na == 0 || nb == 0) return false;
    const uintptr_t a0 = (uintptr_t)a, b0 = (uintptr_t)b;
    return a0 < b0 + nb && b0 < a0 + na;
}

static int rlwe_check(int N, int L, const uint64_t *moduli, RlweArgs *out)
{
    if (!moduli) return NIMBUS_COP_ERR_INVALID_ARG;
    if (N < 32 || N > 65536 || (N & (N - 1)) != 0) return NIMBUS_COP_ERR_INVALID_ARG;
    if (L < 1 || L > kMaxLimbs) return NIMBUS_COP_ERR_INVALID_ARG;
    RlweArgs a{};
    for (int l = 0; l < L; ++l) {
        const uint64_t q = moduli[l];
        if ((q & 1) == 0 || q >= (1ull << 62) || q < 3) return NIMBUS_COP_ERR_INVALID_ARG;
        if ((q - 1) % (2ull * (uint64_t)N) != 0) return NIMBUS_COP_ERR_INVALID_ARG;
        for (int j = 0; j < l; ++j)
            if (moduli[j] == q) return NIMBUS_COP_ERR_INVALID_ARG;
        const int b = bit_length64(q);
        Limb &P = a.limb[l].red;
        P.q = q;
        P.s1 = (uint32_t)(b - 1);
        P.mu = (uint64_t)((((u128)1) << (b + 63)) / q);
        P.pad = 0;
        if (b >= 35) {                  // fold(): only the kernels for moduli from 2^34 use it
            a.limb[l].fold_k = (uint32_t)(b - 33);
            a.limb[l].fold_m = (uint32_t)((((u128)1) << (64 + (b - 33))) / q);
        }
    }
    if (N > (1 << kRlweMaxLogN)) return NIMBUS_COP_ERR_UNSUPPORTED;
    *out = a;
    return NIMBUS_COP_OK;
}

// a primitive 2N-th root of unity: psi^N = -1.  Any of them gives the same products.
static bool find_psi(uint64_t q, int N, uint64_t *psi)
{
    const uint64_t e = (q - 1) / (2ull * (uint64_t)N);
    for (uint64_t g = 2; g < 2000 && g < q; ++g) {
        const uint64_t cand = h_powmod(g, e, q);
        if (h_powmod(cand, (uint64_t)N, q) == q - 1) {
            *psi = cand;
            return true;
        }
    }
    return false;
}

// Q and Delta = floor(Q / 2^t_bits) as four 64-bit words, least significant first
struct HostWide {
    uint64_t w[4] = {0, 0, 0, 0};
};

static HostWide hw_times(const HostWide &a, uint64_t m)
{
    HostWide r;
    u128 carry = 0;
    for (int i = 0; i < 4; ++i) {
        const u128 p = (u128)a.w[i] * m + carry;
        r.w[i] = (uint64_t)p;
        carry = p >> 64;
    }
    return r;
}

static HostWide hw_shift_right(const HostWide &a, int s)       // 0 < s < 64
{
    HostWide r;
    for (int i = 0; i < 4; ++i) {
        r.w[i] = a.w[i] >> s;
        if (i + 1 < 4) r.w[i] |= a.w[i + 1] << (64 - s);
    }
    return r;
}

static uint64_t hw_mod(const HostWide &a, uint64_t m)
{
    u128 rem = 0;
    for (int i = 3; i >= 0; --i) rem = ((rem << 64) | a.w[i]) % m;
    return (uint64_t)rem;
}

static double hw_to_double(const HostWide &a)
{
    double d = 0.0;
    for (int i = 3; i >= 0; --i) d = d * 18446744073709551616.0 + (double)a.w[i];
    return d;
}

struct Scaling {
    HostWide delta, half;
    double delta_inv;
};

// checks shared by decoding and encryption; max_limbs: what the caller can handle
static int scaling(int L, const uint64_t *moduli, int t_bits, Scaling *out)
{
    if (t_bits < 1 || t_bits > 32) return NIMBUS_COP_ERR_INVALID_ARG;
    for (int l = 0; l < L; ++l)
        if (moduli[l] <= (1ull << t_bits)) return NIMBUS_COP_ERR_INVALID_ARG;
    HostWide Q;
    Q.w[0] = 1;
    for (int l = 0; l < L; ++l) Q = hw_times(Q, moduli[l]);
    out->delta = hw_shift_right(Q, t_bits);
    out->half = hw_shift_right(out->delta, 1);
    out->delta_inv = 1.0 / hw_to_double(out->delta);
    return NIMBUS_COP_OK;
}

template <int SKIP>
static hipError_t launch_secret(const RlweArgs &a, int logN, int L, const int8_t *s,
                                Twiddle *tables, hipStream_t stream)
{
    if (logN == 15) {
        return launch(rlwe_secret_kernel<15, 1, 0>, dim3(2u * (unsigned)L), dim3(threads_for(14, 4)),
                      stream, a, s, tables);
    }
    NIMBUS_RLWE_DISPATCH(logN, (launch(rlwe_secret_kernel<LOGN, 0, LOGN >= kProductMinLogN && LOGN <= kProductMaxLogN ? SKIP : 0>,
                                       dim3((unsigned)L), dim3(threads_for(LOGN, 4)), stream, a, s, tables)));
}

}  // namespace nimbus

using namespace nimbus;

extern "C" {

size_t nimbus_rlwe_tables_bytes(int N, int L)
{
    if (N < (1 << kRlweMinLogN) || N > (1 << kRlweMaxLogN) || (N & (N - 1)) != 0) return 0;
    if (L < 1 || L > kMaxLimbs) return 0;
    return (size_t)L * limb_table_entries(N) * sizeof(Twiddle);
}

int nimbus_rlwe_setup(int N, int L, const uint64_t *moduli, const int8_t *s,
                      void *tables, size_t tables_bytes, void *stream)
{
    if (!s || !tables) return NIMBUS_COP_ERR_INVALID_ARG;
    RlweArgs a;
    const int rc = rlwe_check(N, L, moduli, &a);
    if (rc != NIMBUS_COP_OK) return rc;
    if (((uintptr_t)tables & 15u) != 0) return NIMBUS_COP_ERR_INVALID_ARG;
    if (tables_bytes < nimbus_rlwe_tables_bytes(N, L)) return NIMBUS_COP_ERR_BUFFER_SIZE;
    for (int l = 0; l < L; ++l) {
        const uint64_t q = moduli[l];
        uint64_t psi;
        if (!find_psi(q, N, &psi)) return NIMBUS_COP_ERR_INVALID_ARG;
        a.limb[l].psi = psi;
        a.limb[l].psi_inv = h_powmod(psi, 2ull * (uint64_t)N - 1, q);     // psi^(2N) = 1
        a.limb[l].n_inv = q - (q - 1) / (uint64_t)N;                      // N (q - (q-1)/N) = 1 mod q
    }
    const int logN = log2_exact(N);
    const unsigned total = (unsigned)N * (unsigned)L;
    if (launch(rlwe_powers_kernel, dim3((total + 255u) / 256u), dim3(256), (hipStream_t)stream,
               a, logN, L, (Twiddle *)tables) != hipSuccess)
        return NIMBUS_COP_ERR_LAUNCH;
    const dim3 grid((total + 255u) / 256u), block(256);
    if (product_kernel_applies(a, L, logN)) {
        if (launch_secret<2>(a, logN, L, s, (Twiddle *)tables, (hipStream_t)stream) != hipSuccess)
            return NIMBUS_COP_ERR_LAUNCH;
        const hipError_t e = launch(rlwe_product_set_kernel, dim3(grid.x, (unsigned)product_kinds(logN)), block,
                                    (hipStream_t)stream, a, (Twiddle *)tables, logN, L);
        return e == hipSuccess ? NIMBUS_COP_OK : NIMBUS_COP_ERR_LAUNCH;
    }
    if (launch_secret<0>(a, logN, L, s, (Twiddle *)tables, (hipStream_t)stream) != hipSuccess)
        return NIMBUS_COP_ERR_LAUNCH;
    // the same entries in the order of the product kernel: large batches, small batches
    const int pre = logN == 15 ? 1 : 0;
    const int maxs_of[kTableSets] = {0, logN == 15 ? 4 : stages_large_batch(logN),
                                     logN == 15 ? 4 : stages_small_batch(logN)};
    for (int set = 1; set < kTableSets; ++set) {
        if (launch(rlwe_table_set_kernel, grid, block, (hipStream_t)stream, (Twiddle *)tables, logN, L, pre,
                   maxs_of[set], set) != hipSuccess)
            return NIMBUS_COP_ERR_LAUNCH;
    }
    return NIMBUS_COP_OK;
}

int nimbus_rlwe_phase(const uint64_t *ct, int T, int N, int L, const uint64_t *moduli,
                      const void *tables, uint64_t *phi, void *stream)
{
    if (!ct || !tables || !phi || T < 0) return NIMBUS_COP_ERR_INVALID_ARG;
    PolyArgs a{};
    const int rc = rlwe_check(N, L, moduli, &a.limbs);
    if (rc != NIMBUS_COP_OK) return rc;
    if ((unsigned long long)T * (unsigned)L >= (1ull << 30)) return NIMBUS_COP_ERR_INVALID_ARG;
    if (T == 0) return NIMBUS_COP_OK;
    {
        const size_t poly_bytes = (size_t)L * (size_t)N * sizeof(uint64_t);
        if (ranges_overlap(phi, (size_t)T * poly_bytes, ct, 2u * (size_t)T * poly_bytes))
            return NIMBUS_COP_ERR_INVALID_ARG;
    }
    a.tables = (const Twiddle *)tables;
    a.L = L;
    a.src = ct;
    a.dst = phi;
    const hipError_t e = launch_product<false>(a, log2_exact(N), (size_t)T * L, (hipStream_t)stream);
    return e == hipSuccess ? NIMBUS_COP_OK : NIMBUS_COP_ERR_LAUNCH;
}

int nimbus_rlwe_decode(const uint64_t *phi, int T, int N, int L, const uint64_t *moduli,
                       int t_bits, uint64_t *m_hat, void *stream)
{
    if (!phi || !m_hat || T < 0) return NIMBUS_COP_ERR_INVALID_ARG;
    RlweArgs limbs;
    int rc = rlwe_check(N, L, moduli, &limbs);
    if (rc != NIMBUS_COP_OK) return rc;
    Scaling sc;
    rc = scaling(L, moduli, t_bits, &sc);
    if (rc != NIMBUS_COP_OK) return rc;
    const uint64_t total = (uint64_t)T * (uint64_t)N;
    if (total >= (1ull << 39)) return NIMBUS_COP_ERR_INVALID_ARG;
    // inverses of the Chinese remainder theorem; 0 = the moduli are not coprime
    uint64_t inv[kMaxLimbs][kMaxLimbs] = {};
    for (int j = 1; j < L; ++j)
        for (int i = 0; i < j; ++i) {
            inv[i][j] = h_invmod(moduli[i] % moduli[j], moduli[j]);
            if (inv[i][j] == 0) return NIMBUS_COP_ERR_INVALID_ARG;
        }
    if (T == 0) return NIMBUS_COP_OK;
    if (ranges_overlap(m_hat, (size_t)total * sizeof(uint64_t), phi, (size_t)total * (size_t)L * sizeof(uint64_t)))
        return NIMBUS_COP_ERR_INVALID_ARG;
    const dim3 grid((unsigned)((total + 255u) / 256u));
    DecodeArgs a{};
    a.phi = phi;
    a.m_hat = m_hat;
    a.logN = log2_exact(N);
    a.total = total;
    for (int j = 0; j < L; ++j) {
        const uint64_t q = moduli[j];
        a.q[j] = q;
        a.q_d[j] = (double)q;
        for (int i = 0; i < j; ++i) {
            a.inv[i][j] = Twiddle{inv[i][j], (uint64_t)(((u128)inv[i][j] << 64) / q)};
            a.above[i][j] = (moduli[i] / q + 1) * q;
        }
    }
    for (int i = 0; i < kMaxLimbs; ++i) {
        a.delta[i] = sc.delta.w[i];
        a.half[i] = sc.half.w[i];
    }
    a.half_d = hw_to_double(sc.half);
    a.delta_inv = sc.delta_inv;
    a.t_mask = (1ull << t_bits) - 1;
    hipError_t e;
    switch (L) {
    case 1: e = launch(rlwe_decode_kernel<1>, grid, dim3(256), (hipStream_t)stream, a); break;
    case 2: e = launch(rlwe_decode_kernel<2>, grid, dim3(256), (hipStream_t)stream, a); break;
    case 3: e = launch(rlwe_decode_kernel<3>, grid, dim3(256), (hipStream_t)stream, a); break;
    default: e = launch(rlwe_decode_kernel<4>, grid, dim3(256), (hipStream_t)stream, a); break;
    }
    return e == hipSuccess ? NIMBUS_COP_OK : NIMBUS_COP_ERR_LAUNCH;
}

int nimbus_rlwe_decrypt(const uint64_t *ct, int T, int N, int L, const uint64_t *moduli,
                        int t_bits, const void *tables, uint64_t *phi, uint64_t *m_hat,
                        void *stream)
{
    if (!ct || !tables || !phi || !m_hat || T < 0) return NIMBUS_COP_ERR_INVALID_ARG;
    // every check of the second step before the first one is enqueued
    RlweArgs limbs;
    int rc = rlwe_check(N, L, moduli, &limbs);
    if (rc != NIMBUS_COP_OK) return rc;
    Scaling sc;
    rc = scaling(L, moduli, t_bits, &sc);
    if (rc != NIMBUS_COP_OK) return rc;
    if ((uint64_t)T * (uint64_t)N >= (1ull << 39)) return NIMBUS_COP_ERR_INVALID_ARG;
    for (int j = 1; j < L; ++j)
        for (int i = 0; i < j; ++i)
            if (h_invmod(moduli[i] % moduli[j], moduli[j]) == 0) return NIMBUS_COP_ERR_INVALID_ARG;
    {
        const size_t words = (size_t)T * (size_t)N;
        if (ranges_overlap(m_hat, words * sizeof(uint64_t), ct, 2u * words * (size_t)L * sizeof(uint64_t)) ||
            ranges_overlap(m_hat, words * sizeof(uint64_t), phi, words * (size_t)L * sizeof(uint64_t)))
            return NIMBUS_COP_ERR_INVALID_ARG;
    }
    rc = nimbus_rlwe_phase(ct, T, N, L, moduli, tables, phi, stream);
    if (rc != NIMBUS_COP_OK) return rc;
    return nimbus_rlwe_decode(phi, T, N, L, moduli, t_bits, m_hat, stream);
}

int nimbus_rlwe_encrypt(const uint64_t *W, int k, int n, int t_bits, int N, int L,
                        const uint64_t *moduli, const void *tables, const uint64_t *a_poly,
                        const int8_t *e, uint64_t *ctW, void *stream)
{
    if (!W || !tables || !a_poly || !e || !ctW) return NIMBUS_COP_ERR_INVALID_ARG;
    if (k < 1 || n < 1) return NIMBUS_COP_ERR_INVALID_ARG;
    PolyArgs a{};
    int rc = rlwe_check(N, L, moduli, &a.limbs);
    if (rc != NIMBUS_COP_OK) return rc;
    Scaling sc;
    rc = scaling(L, moduli, t_bits, &sc);
    if (rc != NIMBUS_COP_OK) return rc;
    const unsigned long long Ch = ((unsigned long long)n + (unsigned)N - 1) / (unsigned)N;
    const unsigned long long polys = (unsigned long long)k * Ch * (unsigned)L;
    if (polys >= (1ull << 30) || Ch * (unsigned)N >= (1ull << 31)) return NIMBUS_COP_ERR_INVALID_ARG;
    {
        const size_t rows = (size_t)k * (size_t)Ch;
        const size_t ct_bytes = rows * 2u * (size_t)L * (size_t)N * sizeof(uint64_t);
        if (ranges_overlap(ctW, ct_bytes, W, (size_t)k * (size_t)n * sizeof(uint64_t)) ||
            ranges_overlap(ctW, ct_bytes, a_poly, ct_bytes / 2) ||
            ranges_overlap(ctW, ct_bytes, e, rows * (size_t)N))
            return NIMBUS_COP_ERR_INVALID_ARG;
    }
    for (int l = 0; l < L; ++l) {
        const uint64_t d = hw_mod(sc.delta, moduli[l]);
        a.limbs.limb[l].delta = Twiddle{d, (uint64_t)(((u128)d << 64) / moduli[l])};
    }
    a.tables = (const Twiddle *)tables;
    a.L = L;
    a.src = a_poly;
    a.dst = ctW;
    a.W = W;
    a.e = e;
    a.n = n;
    a.Ch = (int)Ch;
    const hipError_t err = launch_encrypt_rows(a, log2_exact(N), (size_t)polys, (hipStream_t)stream);
    return err == hipSuccess ? NIMBUS_COP_OK : NIMBUS_COP_ERR_LAUNCH;
}

}  // extern "C"
