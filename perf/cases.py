"""The calls a program makes of this library, as timed cases: exact integer products end to end
and on stored planes, residue products, and the residue route for wide integers, from the smallest
calls to the benchmark's largest.

``listed()`` names the cases, ``draw()`` gives further ones of the same ranges; a case is a dict of
plain values.  ``kind`` selects the call:

* ``exact``     C = A B through awe_gemm_exact: encode A, encode B, products, reconstruction
* ``stored_b``  B's planes are kept (a weight matrix encoded once), a pass encodes A and multiplies
* ``stored_a``  the same with A kept (the INT4 side of INT4 x INT8 is A)
* ``mod``       C = A B mod m through awe_gemm_mod
* ``crt``       the exact product of int64 matrices through residues, awe_gemm_crt

All results are integers (or correctly rounded doubles), so every output is compared exactly.
"""
import torch

from paper_2609_24519_amd import awe

# Products per scheme (the FP4 / FP6 products whose work a pass cannot do without).
PRODUCTS = {"awe6": 6, "awe4": 4, "b13": 9, "ternary": 3, "fp16_12": 12, "fp6p4": 4}
# Input ranges of the two sides.
RANGES = {"awe6": ((-128, 127), (-128, 127)), "awe4": ((-8, 7), (-128, 127)), "b13": ((-128, 127), (-128, 127)),
          "ternary": ((-1, 1), (-128, 127)), "fp16_12": ((-2048, 2047), (-2048, 2047)),
          "fp6p4": ((-128, 127), (-128, 127))}
BITS = 53  # magnitude of the int64 entries of the residue route (the FP64 significand)
# The FP64-significand residue set (pairwise coprime, its product above 2 K 2^106 up to K = 16384)
# and its products in all: 6 moduli of one product, 14 of three and 3 of four.
MODULI = [5, 7, 8, 9, 11, 13, 31, 37, 41, 43, 47, 53, 59, 61, 67, 71, 73, 79, 83, 89, 149, 151, 157]
MODULI_PRODUCTS = 60


def listed():
    return [
        # The smallest call in use: one 256^3 int8 product (the first benchmark workload); its time
        # is launches and the latency of one short reduction.
        {"name": "int8_256", "kind": "exact", "enc": "awe6", "M": 256, "N": 256, "K": 256, "out": "i32"},
        # An int8 product of odd sizes, rows unaligned in memory and ragged against every tile.
        {"name": "int8_ragged", "kind": "exact", "enc": "awe6", "M": 1001, "N": 1537, "K": 2049, "out": "i32"},
        # The ordinary square int8 product.
        {"name": "int8_2048", "kind": "exact", "enc": "awe6", "M": 2048, "N": 2048, "K": 2048, "out": "i32"},
        # The headline workload.
        {"name": "int8_8192", "kind": "exact", "enc": "awe6", "M": 8192, "N": 8192, "K": 8192, "out": "i32"},
        # A long reduction (a Gram-like product), whose sums need int64.
        {"name": "int8_longk", "kind": "exact", "enc": "awe6", "M": 2048, "N": 2048, "K": 65536, "out": "i64"},
        # Decoding a batch of 16 tokens against a stored int8 weight matrix.
        {"name": "int8_decode16", "kind": "stored_b", "enc": "awe6", "M": 16, "N": 8192, "K": 8192, "out": "i32"},
        # INT4 weights kept as planes, a prompt of 512 tokens of int8 activations.
        {"name": "int4_prefill512", "kind": "stored_a", "enc": "awe4", "M": 8192, "N": 512, "K": 8192,
         "out": "i32"},
        # The nine-product baseline encoding on a middling product.
        {"name": "base13_1024", "kind": "exact", "enc": "b13", "M": 1024, "N": 1024, "K": 1024, "out": "i32"},
        # The FP6 scheme with its limb weights in the block scales, the fastest for int8 operands.
        {"name": "fp6_4096", "kind": "exact", "enc": "fp6p4", "M": 4096, "N": 4096, "K": 4096, "out": "i32"},
        # 12-bit significands of FP16 values as integers.
        {"name": "fp16sig_2048", "kind": "exact", "enc": "fp16_12", "M": 2048, "N": 2048, "K": 2048, "out": "i64"},
        # One modulus of the residue set at the size of the residue workload.
        {"name": "mod89_4096", "kind": "mod", "m": 89, "M": 4096, "N": 4096, "K": 4096},
        # The integer layer of an emulated FP64 product: 53-bit entries, 23 moduli.
        {"name": "crt53_1024", "kind": "crt", "M": 1024, "N": 1024, "K": 4096},
    ]


_MOST = 6 * 8192 ** 3  # product MACs of the largest listed case


def _size(rng, lo, hi):
    """Log-uniform in [lo, hi]; half the draws are whole multiples of 64 where that fits."""
    v = int(round(lo * (hi / lo) ** rng.random()))
    if rng.random() < 0.5 and v >= 64:
        v = v // 64 * 64
    return max(lo, min(hi, v))


def draw(rng):
    kind = rng.choice(["exact", "exact", "exact", "stored_b", "stored_a", "mod", "crt"])
    while True:
        if kind == "exact":
            enc = rng.choice(["awe6", "awe6", "awe4", "b13", "ternary", "fp16_12", "fp6p4"])
            case = {"kind": kind, "enc": enc, "M": _size(rng, 32, 8192), "N": _size(rng, 32, 8192),
                    "K": _size(rng, 64, 65536)}
        elif kind in ("stored_b", "stored_a"):
            enc = rng.choice(["awe6", "awe4", "fp6p4"])
            few, many = _size(rng, 1, 1024), _size(rng, 512, 8192)
            case = {"kind": kind, "enc": enc, "M": few if kind == "stored_b" else many,
                    "N": many if kind == "stored_b" else few, "K": _size(rng, 512, 16384)}
        elif kind == "mod":
            case = {"kind": kind, "m": rng.choice(MODULI), "M": _size(rng, 32, 4096), "N": _size(rng, 32, 4096),
                    "K": _size(rng, 64, 16384)}
        else:
            case = {"kind": kind, "M": _size(rng, 32, 2048), "N": _size(rng, 32, 2048), "K": _size(rng, 64, 16384)}
        macs = case["M"] * case["N"] * case["K"]
        limit = _MOST // 8 if kind == "crt" else _MOST // 2  # the wide route's other passes cost more per MAC
        elements = case["K"] * (case["M"] + case["N"]) + case["M"] * case["N"]
        if macs * _products(case) > limit or elements > (1 << 26 if kind == "crt" else 1 << 28):
            continue
        if kind in ("exact", "stored_b", "stored_a"):
            (alo, _), (blo, _) = RANGES[case["enc"]]
            wide = alo * blo * case["K"] > 2 ** 31 - 1
            case["out"] = "i64" if wide or rng.random() < 0.25 else "i32"
        return case


def _products(case):
    if case["kind"] == "mod":
        return awe.get_encoding_info(awe.ENC_MOD, case["m"])["r"]
    return MODULI_PRODUCTS if case["kind"] == "crt" else PRODUCTS[case["enc"]]


def _inputs(case, seed):
    """Operands uniform over the encoding's range, A then B from one generator."""
    M, N, K = case["M"], case["N"], case["K"]
    if case["kind"] == "mod":
        (alo, ahi), (blo, bhi), dt = (0, case["m"] - 1), (0, case["m"] - 1), torch.uint8
    elif case["kind"] == "crt":
        b = 2 ** BITS - 1
        (alo, ahi), (blo, bhi), dt = (-b, b), (-b, b), torch.int64
    else:
        (alo, ahi), (blo, bhi) = RANGES[case["enc"]]
        dt = torch.int16 if case["enc"] == "fp16_12" else torch.int8
    g = torch.Generator(device="cuda").manual_seed(seed)
    A = torch.randint(alo, ahi + 1, (M, K), dtype=dt, device="cuda", generator=g)
    B = torch.randint(blo, bhi + 1, (K, N), dtype=dt, device="cuda", generator=g)
    return A, B


def prepare(case, seed):
    kind, M, N, K = case["kind"], case["M"], case["N"], case["K"]
    A, B = _inputs(case, seed)
    s = {"case": case, "A": A, "B": B, "flag": torch.zeros(1, dtype=torch.int32, device="cuda")}
    if kind == "crt":
        s["moduli"] = MODULI
        s["c128"] = torch.empty((M, N, 2), dtype=torch.int64, device="cuda")
        s["c64"] = torch.empty((M, N), dtype=torch.float64, device="cuda")
        s["ws_n"] = awe.crt_workspace_bytes(s["moduli"], M, N, K)
    elif kind == "mod":
        s["C"] = torch.empty((M, N), dtype=torch.int32, device="cuda")
        s["ws_n"] = awe.workspace_bytes(awe.ENC_MOD, case["m"], M, N, K)
    else:
        enc = awe.ENCODINGS[case["enc"]]
        s["C"] = torch.empty((M, N), dtype=torch.int64 if case["out"] == "i64" else torch.int32, device="cuda")
        if kind == "exact":
            s["ws_n"] = awe.workspace_bytes(enc, 0, M, N, K)
        else:
            s["pa"] = torch.empty(awe.plane_bytes(enc, 0, awe.SIDE_A, M, K), dtype=torch.uint8, device="cuda")
            s["pb"] = torch.empty(awe.plane_bytes(enc, 0, awe.SIDE_B, N, K), dtype=torch.uint8, device="cuda")
            if kind == "stored_b":
                awe.encode(enc, 0, awe.SIDE_B, B, N, K, N, s["pb"])
                del s["B"]
            else:
                awe.encode(enc, 0, awe.SIDE_A, A, M, K, K, s["pa"])
                del s["A"]
    if "ws_n" in s:
        s["ws"] = torch.empty(max(s["ws_n"], 1), dtype=torch.uint8, device="cuda")
    return s


def run(s):
    case = s["case"]
    kind, M, N, K = case["kind"], case["M"], case["N"], case["K"]
    if kind == "crt":
        b = 2 ** BITS - 1
        awe.gemm_crt(M, N, K, s["A"], K, s["B"], N, b, b, s["moduli"], s["c128"], s["c64"], N, s["ws"], s["ws_n"],
                     s["flag"])
        return {"c128": s["c128"], "c64": s["c64"], "flag": s["flag"]}
    if kind == "mod":
        awe.gemm_mod(case["m"], M, N, K, s["A"], K, s["B"], N, s["C"], N, s["ws"], s["ws_n"], s["flag"])
        return {"C": s["C"], "flag": s["flag"]}
    enc = awe.ENCODINGS[case["enc"]]
    c_type = awe.I64 if case["out"] == "i64" else awe.I32
    if kind == "exact":
        awe.gemm_exact(enc, M, N, K, s["A"], K, s["B"], N, s["C"], N, c_type, s["ws"], s["ws_n"], s["flag"])
        return {"C": s["C"], "flag": s["flag"]}
    if kind == "stored_b":
        awe.encode(enc, 0, awe.SIDE_A, s["A"], M, K, K, s["pa"], s["flag"])
    else:
        awe.encode(enc, 0, awe.SIDE_B, s["B"], N, K, N, s["pb"], s["flag"])
    awe.gemm_planes(enc, 0, M, N, K, s["pa"], s["pb"], s["C"], N, c_type)
    return {"C": s["C"], "flag": s["flag"]}


def work(case):
    kind, M, N, K = case["kind"], case["M"], case["N"], case["K"]
    flops = 2.0 * _products(case) * M * N * K
    if kind == "crt":
        return {"bytes": 8 * K * (M + N) + 24 * M * N, "flops": flops}
    if kind == "mod":
        return {"bytes": K * (M + N) + 4 * M * N, "flops": flops}
    esize = 2 if case["enc"] == "fp16_12" else 1
    c = M * N * (8 if case["out"] == "i64" else 4)
    enc = awe.ENCODINGS[case["enc"]]
    a, b = esize * M * K, esize * K * N
    if kind == "stored_b":
        b = awe.plane_bytes(enc, 0, awe.SIDE_B, N, K)
    elif kind == "stored_a":
        a = awe.plane_bytes(enc, 0, awe.SIDE_A, M, K)
    return {"bytes": a + b + c, "flops": flops}


def tolerance(case):
    return "exact"


def _wide_product(A, B):
    """(low, high) words of the exact product of int64 matrices with |entries| < 2^54, through
    18-bit limbs: a product of limbs summed over K <= 16384 stays below 2^50, exact in a double."""
    def limbs(X):
        out = []
        for _ in range(2):
            low = ((X + (1 << 17)) & ((1 << 18) - 1)) - (1 << 17)
            out.append(low)
            X = (X - low) >> 18
        return out + [X]

    la, lb = limbs(A), limbs(B)
    sums = [0] * 5
    for i in range(3):
        for j in range(3):
            p = torch.matmul(la[i].double(), lb[j].double()).to(torch.int64)
            sums[i + j] = sums[i + j] + p
    # X = sum_d sums[d] 2^(18 d): add into two's-complement words (lo, hi)
    lo = torch.zeros_like(sums[0])
    hi = torch.zeros_like(sums[0])
    flip = torch.tensor(-2 ** 63, dtype=torch.int64, device=lo.device)
    for d in range(5):
        sh = 18 * d
        if sh < 64:
            add_lo = sums[d] << sh
            add_hi = sums[d] >> (64 - sh) if sh else sums[d] >> 63
        else:
            add_lo = torch.zeros_like(lo)
            add_hi = sums[d] << (sh - 64)
        new = lo + add_lo
        hi = hi + add_hi + ((new ^ flip) < (lo ^ flip)).to(torch.int64)
        lo = new
    return lo, hi


def _nearest_double(lo, hi):
    """The nearest double (ties to even) of the integer hi 2^64 + lo, |X| < 2^127."""
    neg = hi < 0
    mlo = torch.where(neg, -lo, lo)
    mhi = torch.where(neg, ~hi + (lo == 0).to(torch.int64), hi)
    # 4 bits of 32-bit digits, from the top, gathered into the leading 60 bits and a sticky bit
    d = [(mhi >> 32) & 0xffffffff, mhi & 0xffffffff, (mlo >> 32) & 0xffffffff, mlo & 0xffffffff]
    out = torch.zeros(lo.shape, dtype=torch.float64, device=lo.device)
    done = torch.zeros(lo.shape, dtype=torch.bool, device=lo.device)
    for nbits in range(127, 0, -1):  # numbers with exactly nbits significant bits
        top = nbits - 1
        here = ~done & (((d[3 - top // 32] >> (top % 32)) & 1) == 1)
        if not bool(here.any()):
            continue
        done |= here
        h, l = mhi[here], mlo[here]
        s = max(0, nbits - 60)  # keep 60 bits
        if s == 0:
            v = l
        elif s < 64:
            v = ((l >> s) & ((1 << (64 - s)) - 1)) | (h << (64 - s))
            v = v | ((l & ((1 << s) - 1)) != 0).to(torch.int64)
        else:
            v = h >> (s - 64)
            rest = (l != 0) | ((h & ((1 << (s - 64)) - 1)) != 0)
            v = v | rest.to(torch.int64)
        out[here] = v.to(torch.float64) * (2.0 ** s)
    return torch.where(neg, -out, out)


def exact(case, seed):
    A, B = _inputs(case, seed)
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    if case["kind"] == "crt":
        lo, hi = _wide_product(A, B)
        return {"c128": torch.stack([lo, hi], dim=-1), "c64": _nearest_double(lo, hi), "flag": flag}
    C = torch.matmul(A.double(), B.double())  # every sum stays below 2^53: exact
    if case["kind"] == "mod":
        return {"C": torch.remainder(C, case["m"]).to(torch.int32), "flag": flag}
    return {"C": C.to(torch.int64 if case["out"] == "i64" else torch.int32), "flag": flag}
