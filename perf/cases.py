"""The work whose speed counts: the calls that the two parties of the protocol make.

Client, online (Algorithm 1 steps 2-4): one linear layer on prepared weights, share matrix in,
masked (and, where n <= N/2, packed) output ciphertexts out: kind "layer".  Several requests of
one shape at hand: kind "requests" (one staging and one matmul launch for all of them).  Weights
that are used once, without a setup pass: kind "canonical".
Client, setup: the re-layout of a layer's weight ciphertexts: kind "weights".
Server: encryption of the weight rows (setup, step 1), kind "encrypt", and decryption of the
returned ciphertexts (online, step 5), kind "decrypt".

Sizes: BERT-base linear layers (hidden 768, feed-forward 3072, fused QKV 2304) at 128 tokens and at
one token, the long-sequence layer (512 tokens, ring 8192, three limbs), the toy layer of the tests,
and the paper's own parameters (shares in Z_2^64, ring 8192, limbs of 59 and 55 bits).

Every result is an exact integer: the tolerance is equality.
"""
import math

import torch

import paper_2411_15707_amd as nc


# ---------------------------------------------------------------------------
# parameters
# ---------------------------------------------------------------------------
def _is_prime(n):
    """Miller-Rabin, deterministic below 3.3e24"""
    small = (2, 3, 5, 7, 11, 13, 17, 19, 23, 29, 31, 37, 41)
    if n < 2:
        return False
    for p in small:
        if n % p == 0:
            return n == p
    d, r = n - 1, 0
    while d % 2 == 0:
        d //= 2
        r += 1
    for a in small:
        x = pow(a, d, n)
        if x in (1, n - 1):
            continue
        for _ in range(r - 1):
            x = x * x % n
            if x == n - 1:
                break
        else:
            return False
    return True


def _q_bits(case):
    return [case["q0_bits"], case["q1_bits"], case["q2_bits"]][:case["L"]]


def _moduli(case):
    """per limb the largest prime of its width that is 1 modulo t and modulo 2N, all distinct"""
    step = 2 * case["N"]
    if case["x_bits"] <= 32:
        step = max(step, 1 << case["x_bits"])
    out = []
    for bits in _q_bits(case):
        q = (1 << bits) - step + 1
        while q in out or not _is_prime(q):
            q -= step
        out.append(q)
    return tuple(out)


def _chunks(case):
    return -(-case["n"] // case["N"])


def _columns(case):
    return _chunks(case) * 2 * case["L"] * case["N"]


def _packs(case):
    return 2 * case["n"] <= case["N"]


def _packed(case):
    return -(-case["m"] // (case["N"] // case["n"]))


def _case(kind, m, k, n, N, L, x_bits, q_bits, count=1):
    q = (list(q_bits) + [0, 0])[:3]
    return {"kind": kind, "m": m, "k": k, "n": n, "N": N, "L": L, "x_bits": x_bits,
            "q0_bits": q[0], "q1_bits": q[1], "q2_bits": q[2], "count": count}


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def listed():
    cases = []

    def add(name, *args, **kw):
        cases.append({"name": name, **_case(*args, **kw)})

    # the smallest layer anyone runs: eight tokens, packed into one ciphertext; latency only
    add("toy_layer", "layer", 8, 64, 64, 1024, 1, 16, [50])
    # generation: one token through the feed-forward up-projection
    add("one_token_ffn_up", "layer", 1, 768, 3072, 4096, 2, 20, [54, 54])
    # a BERT-base sequence of 128 tokens through both feed-forward projections; the second
    # packs five rows per ciphertext
    add("ffn_up", "layer", 128, 768, 3072, 4096, 2, 20, [54, 54])
    add("ffn_down", "layer", 128, 3072, 768, 4096, 2, 20, [54, 54])
    # the largest call: a long sequence, three limbs, two rows per packed ciphertext
    add("long_sequence", "layer", 512, 1024, 4096, 8192, 3, 24, [55, 55, 55])
    # the paper's own parameters: 64-bit shares, limbs of 59 and 55 bits, BERT-base up-projection
    add("wide_shares", "layer", 128, 768, 3072, 8192, 2, 64, [59, 55])
    # four requests of a ragged shape together: odd token count, odd inner size, output wider
    # than the ring (two chunks), the widest shares that one pass takes
    add("requests_ragged", "requests", 77, 1001, 5000, 4096, 1, 32, [54], count=4)
    # a QKV projection whose weights are used once: canonical layout, no setup pass
    add("qkv_unprepared", "canonical", 128, 768, 2304, 4096, 2, 20, [54, 54])
    # setup of the up-projection: the client's re-layout of the weights, the server's encryption
    add("weights_ffn_up", "weights", 1, 768, 3072, 4096, 2, 20, [54, 54])
    add("encrypt_ffn_up", "encrypt", 1, 768, 3072, 4096, 2, 20, [54, 54])
    # the server's online step: the 128 output rows of the up-projection, and the 256 packed
    # ciphertexts of the long-sequence layer
    add("decrypt_ffn_up", "decrypt", 128, 768, 3072, 4096, 2, 20, [54, 54])
    add("decrypt_long_sequence", "decrypt", 256, 1024, 4096, 8192, 3, 24, [55, 55, 55])
    return cases


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    # (half of the draws are layers: they are what runs for every query)
    kind = rng.choice(["layer", "layer", "layer", "layer", "layer", "requests", "canonical",
                       "weights", "encrypt", "decrypt"])
    while True:
        N = rng.choice([1024, 2048, 4096, 4096, 8192, 8192])
        L = rng.choice([1, 2, 2, 3])
        x_bits = rng.choice([16, 20, 24, 32])
        q_bits = [rng.randint(50, 55) for _ in range(L)]
        if kind == "layer" and rng.random() < 0.2:
            x_bits = rng.choice([48, 64])
            q_bits = [rng.randint(55, 59) for _ in range(L)]
        m = _log_int(rng, 1, 512)
        k = _log_int(rng, 48, 3072)
        n = _log_int(rng, 48, 2 * N)
        count = rng.randint(2, 8) if kind == "requests" else 1
        case = _case(kind, m, k, n, N, L, x_bits, q_bits, count)
        # no more byte products, and no more weights, than the largest listed layer has
        products = -(-x_bits // 8) * 8
        if m * k * _columns(case) * count * products > 512 * 1024 * 49152 * 24:
            continue
        if k * _columns(case) * count > 1024 * 49152:
            continue
        if kind == "canonical" and m * k * _columns(case) > 128 * 1024 * 49152:
            continue
        return case


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
class _Draws:
    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(seed)

    def below(self, shape, bound):
        return torch.randint(0, bound, shape, dtype=torch.int64, device="cuda", generator=self.gen)

    def shares(self, m, k, bits):
        """uniform shares of Z_2^bits as raw 64-bit words"""
        if bits < 63:
            return self.below((m, k), 1 << bits)
        return (self.below((m, k), 1 << 32) << 32) | self.below((m, k), 1 << 32)

    def residues(self, lead, moduli, N):
        """[*lead][L][N], limb l uniform below moduli[l] (ciphertexts and masks are uniform)"""
        out = torch.empty((*lead, len(moduli), N), dtype=torch.int64, device="cuda")
        for l, q in enumerate(moduli):
            out[..., l, :] = self.below((*lead, N), q)
        return out

    def error(self, shape, sigma=3.2):
        e = torch.empty(shape, dtype=torch.float32, device="cuda").normal_(0.0, sigma, generator=self.gen)
        bound = int(6 * sigma)
        return e.round_().clamp_(-bound, bound).to(torch.int8)

    def secret(self, N):
        return (self.below((N,), 3) - 1).to(torch.int8)


def _words(*shape):
    return torch.empty(shape, dtype=torch.int64, device="cuda")


def _bytes(count):
    return torch.empty(count, dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    draws = _Draws(seed)
    m, k, n, N, L = case["m"], case["k"], case["n"], case["N"], case["L"]
    x_bits, kind = case["x_bits"], case["kind"]
    moduli, Ch = _moduli(case), _chunks(case)
    st = {"kind": kind, "m": m, "k": k, "n": n, "N": N, "L": L, "x_bits": x_bits, "moduli": moduli}

    def weights():
        return draws.residues((k, Ch, 2), moduli, N)

    def prepared():
        ctW = weights()
        buf = _bytes(nc.nimbus_cop_prepared_bytes(k, n, N, L, moduli))
        nc.nimbus_cop_prepare(ctW, k, n, N, L, moduli, buf)
        return buf

    def mask(rows, chunks):
        return draws.residues((rows, chunks, 2), moduli, N)

    def workspace():
        return _bytes(nc.nimbus_cop_workspace_bytes(m, k, x_bits))

    def tables():
        buf = _bytes(nc.nimbus_rlwe_tables_bytes(N, L))
        nc.nimbus_rlwe_setup(N, L, moduli, draws.secret(N), buf)
        return buf

    if kind == "layer":
        st["X"] = draws.shares(m, k, x_bits)
        st["prepared"], st["workspace"] = prepared(), workspace()
        st["out"] = _words(m, Ch, 2, L, N)
        if _packs(case):
            T = nc.nimbus_cop_packed_count(m, n, N)
            st["packed_mask"], st["packed"] = mask(T, 1), _words(T, 1, 2, L, N)
        else:
            st["mask"] = mask(m, Ch)
    elif kind == "requests":
        count = range(case["count"])
        st["X"] = [draws.shares(m, k, x_bits) for _ in count]
        st["prepared"] = [prepared() for _ in count]
        st["workspace"] = [workspace() for _ in count]
        st["mask"] = [mask(m, Ch) for _ in count]
        st["out"] = [_words(m, Ch, 2, L, N) for _ in count]
    elif kind == "canonical":
        st["X"] = draws.shares(m, k, x_bits)
        st["ctW"], st["mask"], st["out"] = weights(), mask(m, Ch), _words(m, Ch, 2, L, N)
    elif kind == "weights":
        st["ctW"] = weights()
        st["prepared"] = _bytes(nc.nimbus_cop_prepared_bytes(k, n, N, L, moduli))
    elif kind == "encrypt":
        st["W"] = draws.below((k, n), 1 << x_bits)
        st["a"], st["e"] = draws.residues((k, Ch), moduli, N), draws.error((k, Ch, N))
        st["tables"], st["ctW"] = tables(), _words(k, Ch, 2, L, N)
    elif kind == "decrypt":
        st["ct"], st["tables"] = draws.residues((m, 2), moduli, N), tables()
        st["phi"], st["m_hat"] = _words(m, L, N), _words(m, N)
    else:
        raise ValueError(kind)
    return st


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def run(st):
    m, k, n, N, L = st["m"], st["k"], st["n"], st["N"], st["L"]
    x_bits, moduli, kind = st["x_bits"], st["moduli"], st["kind"]
    if kind == "layer":
        nc.nimbus_cop_matmul_prepared(st["X"], m, k, x_bits, st["prepared"], n, N, L, moduli,
                                      st.get("mask"), st["out"], st["workspace"])
        if "packed" not in st:
            return st["out"]
        nc.nimbus_cop_pack(st["out"], m, n, N, L, moduli, st["packed_mask"], st["packed"])
        return st["packed"]
    if kind == "requests":
        nc.nimbus_cop_stage_shares_batch(st["X"], m, k, x_bits, st["workspace"])
        nc.nimbus_cop_matmul_staged_batch(st["workspace"], m, k, x_bits, st["prepared"], n, N, L,
                                          moduli, st["mask"], st["out"])
        return st["out"]
    if kind == "canonical":
        nc.nimbus_cop_matmul(st["X"], m, k, x_bits, st["ctW"], n, N, L, moduli, st["mask"], st["out"])
        return st["out"]
    if kind == "weights":
        nc.nimbus_cop_prepare(st["ctW"], k, n, N, L, moduli, st["prepared"])
        return st["prepared"]
    if kind == "encrypt":
        nc.nimbus_rlwe_encrypt(st["W"], k, n, x_bits, N, L, moduli, st["tables"], st["a"], st["e"],
                               st["ctW"])
        return st["ctW"]
    nc.nimbus_rlwe_decrypt(st["ct"], m, N, L, moduli, x_bits, st["tables"], st["phi"], st["m_hat"])
    return st["phi"], st["m_hat"]


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def work(case):
    """bytes: every input once, every output once.  flops: for the matmuls two per 8-bit x 8-bit
    product of the operands' bytes; for the server side the 64-bit integer operations of the
    textbook transform (a modular product is three, a sum or difference one)."""
    m, k, n, N, L = case["m"], case["k"], case["n"], case["N"], case["L"]
    kind, count = case["kind"], case["count"]
    C, Ch = _columns(case), _chunks(case)
    residue_bytes = -(-max(_q_bits(case)) // 8)         # of a prepared weight
    limb_products = sum(-(-b // 8) for b in _q_bits(case)) * (C // L) * -(-case["x_bits"] // 8)
    if kind in ("layer", "requests", "canonical"):
        weight = 8 if kind == "canonical" else residue_bytes
        packed = kind == "layer" and _packs(case)
        outputs = (_packed(case) if packed else m) * C
        return {"bytes": count * (8 * m * k + weight * k * C + 16 * outputs),
                "flops": count * 2 * m * k * limb_products}
    if kind == "weights":
        return {"bytes": k * C * (8 + residue_bytes), "flops": 2 * k * C}
    log_n = N.bit_length() - 1
    product = L * (N * log_n * 5 + N * 3)               # two transforms and the pointwise product
    if kind == "encrypt":
        rows = k * Ch
        return {"bytes": 8 * k * n + rows * N * (1 + 8 * L + 16 * L), "flops": rows * product}
    return {"bytes": 8 * m * N * (2 * L + L + 1), "flops": m * product}


def tolerance(case):
    return "exact"
