"""What a program that uses this library has it do, for timing.

A message under a table of key pairs is encrypted or decrypted through the
public binding (Context, Plan, Server): the forms on device buffers, the
blinded form, the batched form over mixed key sizes, the form on host buffers
and the request server.  Sizes are those of the repository's workloads
(inputs.CONFIGS, inputs.TABLE_BITS): 16 KiB under 512-bit keys up to 100 MiB
under 2048-bit keys, 1024- to 4096-bit keys mixed, and the per-size table's
100 KB under 2048- to 8192-bit keys.
"""
import functools
import hashlib
import math

import numpy as np
import torch

from paper_2111_11924_amd import binding, inputs

MiB = 1 << 20

# Primes of the key pairs: prime i of a size is the i-th odd start value (a
# hash, top two bits set) plus 2 x its entry here, the distance to the first
# prime p with gcd(65537, p - 1) = 1.  A key pair is a pair of them, so one
# short list gives a whole key table without a search; what an operation costs
# depends on the size of the primes, not on how they were drawn.
_PRIMES = {
    256: (137, 123, 108, 168, 296, 171, 18, 22),
    512: (98, 21, 70, 41, 99, 17, 46, 13, 78, 69, 523, 47, 130, 126, 119, 161, 244, 398, 144, 95, 242, 10, 450, 42),
    768: (218, 124, 265, 338, 917, 72, 414, 273),
    1024: (250, 167, 114, 415, 74, 491, 694, 84, 71, 106, 72, 402, 114, 301, 21, 527, 42, 615, 392, 818, 776, 192, 0,
           240),
    1280: (509, 623, 1, 256, 415, 239, 1229, 39),
    1536: (421, 21, 119, 110, 1051, 689, 2467, 615, 55, 438, 848, 429, 280, 1281, 371, 29, 629, 238, 439, 261, 167,
           530, 151, 220),
    2048: (1664, 1295, 160, 718, 7, 594, 54, 552, 1667, 38, 201, 83, 505, 497, 50, 1582, 1269, 1460, 616, 180, 504,
           662, 593, 734),
    3072: (490, 607, 2832, 757, 4726, 2761, 217, 905),
    4096: (2722, 1661, 783, 6070, 6331, 1769, 344, 83),
}
MIXED = (1024, 2048, 3072, 4096)


@functools.lru_cache(maxsize=None)
def _prime(bits, i):
    x = int.from_bytes(hashlib.shake_256(f"prime/{bits}/{i}".encode()).digest(bits // 8), "big")
    return (x | (3 << (bits - 2)) | 1) + 2 * _PRIMES[bits][i]


@functools.lru_cache(maxsize=None)
def _key(bits, i, j):
    return inputs.key_from_primes(_prime(bits // 2, i), _prime(bits // 2, j), bits=bits)


def _pairs(bits):
    n = len(_PRIMES[bits // 2])
    return [(i, j) for i in range(n) for j in range(i + 1, n)]


def _keys(case, shape, rng):
    """The case's key table: `keys` different pairs of its size, or of sizes drawn from MIXED."""
    sizes = [case["bits"]] * case["keys"] if case["bits"] else [int(b) for b in shape.choice(MIXED, case["keys"])]
    pick = {b: rng.permutation(len(_pairs(b))) for b in sorted(set(sizes))}
    used = dict.fromkeys(pick, 0)
    out = []
    for b in sizes:
        out.append(_key(b, *_pairs(b)[pick[b][used[b]]]))
        used[b] += 1
    return out


def _key_map(case, keys, rng):
    """Chunk i under key i mod K, or under a random key; as many chunks as the message needs."""
    caps = np.array([k.bits // 8 - 4 for k in keys], dtype=np.int64)
    most = case["bytes"] // int(caps.min()) + 1
    km = rng.integers(0, len(keys), most) if case["map"] == "random" else np.arange(most) % len(keys)
    ends = np.cumsum(caps[km])
    return km[: int(np.searchsorted(ends, case["bytes"])) + 1].astype(np.uint32)


def _bytes(rng, n):
    return rng.integers(0, 256, n, dtype=np.uint8)


def _requests(case, keys, shape, rng):
    """(op, message, key map) of each request: log-uniform sizes, up to 64 keys each, half encrypt."""
    caps = np.array([k.bits // 8 - 4 for k in keys], dtype=np.int64)
    out = []
    for i in range(case["requests"]):
        size = int(round(math.exp(shape.uniform(math.log(1024), math.log(case["bytes"])))))
        subset = shape.choice(len(keys), size=int(shape.integers(1, min(64, len(keys)) + 1)), replace=False)
        km = subset[np.arange(size // int(caps.min()) + 1) % len(subset)]
        km = km[: int(np.searchsorted(np.cumsum(caps[km]), size)) + 1].astype(np.uint32)
        out.append((i % 2, _bytes(rng, size), km))
    return out


def _host_inputs(case, seed):
    # the case alone gives the sizes (key sizes, key map, requests), the seed the keys and bytes
    shape = np.random.Generator(np.random.PCG64([case["bits"], case["keys"], case["bytes"]]))
    rng = np.random.Generator(np.random.PCG64([seed, 7]))
    keys = _keys(case, shape, rng)
    if case["op"] == "serve":
        return keys, _requests(case, keys, shape, rng)
    km = _key_map(case, keys, shape)
    return keys, (km, _bytes(rng, case["bytes"]), rng)


def listed():
    return [
        # the smallest call: a 16 KiB message, a handful of tiles, all of it latency
        dict(name="dec-512b-16K", op="decrypt", bits=512, keys=8, bytes=16 * 1024, map="round_robin"),
        # a 1 MB file under 64 keys (the paper's smallest file), both directions; an odd length
        dict(name="enc-2048b-1M", op="encrypt", bits=2048, keys=64, bytes=1_000_003, map="round_robin"),
        dict(name="dec-2048b-1M", op="decrypt", bits=2048, keys=64, bytes=1 * MiB, map="round_robin"),
        # the paper's per-size experiment: 100 KB under 16 keys, large moduli
        dict(name="dec-4096b-100K", op="decrypt", bits=4096, keys=16, bytes=102_400, map="round_robin"),
        dict(name="dec-8192b-100K", op="decrypt", bits=8192, keys=16, bytes=102_400, map="round_robin"),
        # the paper's largest file: throughput, both directions
        dict(name="enc-2048b-100M", op="encrypt", bits=2048, keys=256, bytes=100 * MiB, map="round_robin"),
        dict(name="dec-2048b-100M", op="decrypt", bits=2048, keys=256, bytes=100 * MiB, map="round_robin"),
        # the scheme's blinded decryption of a 25 MB file
        dict(name="blind-dec-2048b-25M", op="blind_decrypt", bits=2048, keys=256, bytes=25 * MiB, map="round_robin"),
        # a table of mixed key sizes, chunks under random keys, through the batched form
        dict(name="batch-enc-mixed-25M", op="batch_encrypt", bits=0, keys=256, bytes=25 * MiB, map="random"),
        dict(name="batch-dec-mixed-25M", op="batch_decrypt", bits=0, keys=256, bytes=25 * MiB, map="random"),
        # a 10 MB file from and to host memory, encrypted and decrypted
        dict(name="host-2048b-10M", op="host", bits=2048, keys=64, bytes=10_000_000, map="round_robin"),
        # requests of 1 KiB to 10 MiB to the server, all in flight at once
        dict(name="serve-24", op="serve", bits=0, keys=128, bytes=10 * MiB, requests=24, map="random"),
    ]


# range of message sizes of each operation's drawn cases
_RANGE = {"encrypt": (1024, 100 * MiB), "decrypt": (1024, 100 * MiB), "blind_decrypt": (4096, 25 * MiB),
          "batch_encrypt": (64 * 1024, 25 * MiB), "batch_decrypt": (64 * 1024, 25 * MiB), "host": (64 * 1024, 25 * MiB),
          "serve": (64 * 1024, 10 * MiB)}


def draw(rng):
    op = rng.choice(["encrypt", "decrypt", "decrypt", "decrypt", "blind_decrypt", "batch_encrypt", "batch_decrypt", "host",
                     "serve"])
    lo, hi = _RANGE[op]
    case = dict(op=op, bits=0, keys=0, bytes=0, map=rng.choice(["round_robin", "random"]))
    if op in ("batch_encrypt", "batch_decrypt", "serve"):
        case["keys"] = rng.randint(8, 256)
    else:
        case["bits"] = rng.choice([512, 1024, 1536, 2048, 2048, 2560, 3072, 4096, 6144, 8192])
        case["keys"] = rng.randint(1, min(256, len(_pairs(case["bits"]))))
    case["bytes"] = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if op == "serve":
        case["requests"] = rng.randint(4, 24)
    # no dearer than the largest listed case (large moduli: fewer bytes)
    most = max(work(c)["flops"] for c in listed())
    while work(case)["flops"] > most / 2:
        case["bytes"] = case["bytes"] * 2 // 3
    return case


class _State:
    """A context with its key table, a plan or server, and the buffers of the call."""


def prepare(case, seed):
    keys, given = _host_inputs(case, seed)
    st = _State()
    st.op = case["op"]
    st.ctx = binding.Context(0)
    st.ctx.load_keys(keys)
    if st.op == "serve":
        st.requests = []
        for op, msg, km in given:
            data = msg
            if op == binding.PMK_OP_DECRYPT:
                plan = st.ctx.plan(km, len(msg))
                data = plan.encrypt(torch.from_numpy(msg).cuda())[: plan.ct_len].cpu().numpy()
                plan.close()
            st.requests.append((op, data, len(msg), km))
        st.server = st.ctx.server()
        return st
    km, msg, rng = given
    st.plan = st.ctx.plan(km, len(msg))
    if st.op == "host":
        st.msg = torch.from_numpy(msg).pin_memory()
        st.ct = torch.empty(st.plan.ct_len, dtype=torch.uint8, pin_memory=True)
        st.back = torch.empty(len(msg), dtype=torch.uint8, pin_memory=True)
        return st
    d_msg = torch.from_numpy(msg).cuda()
    if st.op in ("encrypt", "batch_encrypt"):
        st.given, st.out = d_msg, torch.empty(st.plan.ct_len, dtype=torch.uint8, device="cuda")
    elif st.op == "blind_decrypt":
        # a factor below N and, like any odd number that no prime of the key divides, invertible
        r = _bytes(rng, st.plan.ct_len)
        at = np.concatenate([[0], np.cumsum([keys[k].bits // 8 for k in km.tolist()])])
        r[at[:-1]] &= 0x7F
        r[at[1:] - 1] |= 1
        st.given = st.plan.encrypt_blinded(d_msg, torch.from_numpy(r).cuda())
        st.out = torch.empty(len(msg), dtype=torch.uint8, device="cuda")
    else:
        st.given, st.out = st.plan.encrypt(d_msg), torch.empty(len(msg), dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    return st


def run(state):
    op = state.op
    if op == "encrypt" or op == "batch_encrypt":
        return state.plan.encrypt(state.given, state.out, batch=op == "batch_encrypt")
    if op == "decrypt" or op == "batch_decrypt":
        return state.plan.decrypt(state.given, state.out, batch=op == "batch_decrypt")
    if op == "blind_decrypt":
        return state.plan.decrypt_blinded(*state.given, state.out)
    if op == "host":
        for rc in (state.plan.encrypt_host(state.msg, state.ct), state.plan.decrypt_host(state.ct, state.back)):
            if rc != binding.PMK_OK:
                raise binding.PmkError(rc)
        return state.ct, state.back
    sent = [state.server.submit(*r) for r in state.requests]
    for ticket, _ in sent:
        if state.server.wait(ticket)["status"] != binding.PMK_OK:
            raise RuntimeError("request failed")
    return [out for _, out in sent]


def _products(bits):
    """32-bit products of one encryption with e = 65537 and of one CRT decryption, counted as
    word-by-word Montgomery products (2 s^2 + s) with windows of five bits."""
    def mm(s):
        return 2 * s * s + s

    s, h = bits // 32, bits // 64
    half = (32 + 6 * (math.ceil(bits / 10) - 1)) * mm(h)
    return 19 * mm(s), 2 * half + 6 * mm(h) + h * h


def work(case):
    """Bytes in and out, and two operations per 32-bit product."""
    sizes = MIXED if not case["bits"] else (case["bits"],)
    # mixed sizes: every size gets the same number of chunks
    total = case["bytes"]
    if case["op"] == "serve":  # mean of a log-uniform size
        total = case["requests"] * (case["bytes"] - 1024) / math.log(case["bytes"] / 1024)
    chunks = total / sum(b // 8 - 4 for b in sizes)
    ct = sum(chunks * (b // 8) for b in sizes)
    enc = sum(chunks * _products(b)[0] for b in sizes)
    dec = sum(chunks * _products(b)[1] for b in sizes)
    parts = {"encrypt": (1, 0, 1), "batch_encrypt": (1, 0, 1), "decrypt": (0, 1, 1), "batch_decrypt": (0, 1, 1),
             "blind_decrypt": (0, 1.2, 2), "host": (1, 1, 2), "serve": (0.5, 0.5, 1)}[case["op"]]
    return {"bytes": float(total + parts[2] * ct), "flops": 2 * (parts[0] * enc + parts[1] * dec)}


def _cipher(keys, km, msg):
    """The ciphertext by Python's integers."""
    out, at = [], 0
    for k in km.tolist():
        key = keys[k]
        t = min(key.bits // 8 - 4, len(msg) - at)
        c = pow(int.from_bytes(msg[at : at + t].tobytes(), "big"), key.e, key.n)
        out.append(c.to_bytes(key.bits // 8, "big"))
        at += t
    return np.frombuffer(b"".join(out), dtype=np.uint8)


def exact(case, seed):
    keys, given = _host_inputs(case, seed)
    if case["op"] == "serve":
        return [msg if op == binding.PMK_OP_DECRYPT else None for op, msg, _ in given]
    km, msg, _ = given
    if case["op"] in ("encrypt", "batch_encrypt", "host"):
        ct = _cipher(keys, km, msg) if work(case)["flops"] / 2 < 6e10 * (0.03 if case["op"] == "host" else 0.1) else None
        return (ct, msg) if case["op"] == "host" else ct
    return msg
