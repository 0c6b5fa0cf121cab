"""GPU parity of the CRT halves whose reduction runs on the matrix cores (fold
forms): at the edges of their tiles and groups of tiles, for primes shorter
than their size class, at extreme operands, and at several units per wave.
Exact comparison: decryptions against the message (its ciphertext comes from
the encryption kernels, which reduce another way) and whole decrypted blocks
against the oracle."""
import json
import os
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

import oracle
from paper_2111_11924_amd import binding, inputs

pytestmark = pytest.mark.gpu

GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "large_keys.json")


@pytest.fixture(scope="module")
def torch():
    import torch as t

    assert t.cuda.is_available(), "GPU tests need a GPU"
    return t


@pytest.fixture(scope="module")
def ctx(torch):
    c = binding.Context(0)
    yield c
    c.close()


def keys_of(bits, count):
    """`count` keys of a size: generated up to 1536 bits, the stored key repeated above (the
    table keeps a record for each)."""
    if bits > 1536:
        with open(GOLDEN) as f:
            k = [k for k in json.load(f)["keys"] if k["bits"] == bits]
        return [inputs.RsaKey.from_json(k[0])] * count
    return inputs.make_keys([bits] * count, 700 + bits // 64)


def roundtrip(torch, ctx, km, msg):
    plan = ctx.plan(km, len(msg))
    ct = plan.encrypt(torch.from_numpy(msg).cuda())
    back = [plan.decrypt(ct), plan.decrypt(ct, batch=True)]
    assert plan.check() == binding.PMK_OK
    plan.close()
    return [b[: len(msg)].cpu().numpy() for b in back]


# A number in one lane (lanes 1): tiles of 64 chunks, in groups of up to two
# (1024 / 2048 bits) or four (3072 / 4096) under one key; over a block (lanes 4, 8):
# parts of 16 chunks.  Counts around those edges; grid caps: one wave, fewer
# waves than a block has, blocks that walk several units.
@pytest.mark.parametrize("cap", [0, 1, 3, 9])
@pytest.mark.parametrize("bits,lanes", [(1024, 1), (1088, 1), (1536, 1), (2048, 1), (3072, 1), (4096, 1), (1024, 4),
                                        (1536, 8), (2048, 8), (3072, 8), (4096, 8), (6144, 8), (8192, 8)])
def test_tile_and_group_edges(torch, ctx, bits, lanes, cap):
    if lanes > 1:
        counts = [1, 15, 16, 17, 65] if not cap else [33, 1]
    else:
        counts = [1, 63, 64, 65, 129, 257] if not cap else [129, 1]
    keys = keys_of(bits, len(counts))
    km = np.repeat(np.arange(len(counts), dtype=np.uint32), counts)
    msg = inputs.make_message(len(km) * (bits // 8 - 4) - 7, bits)
    ctx.load_keys(keys)
    old = ctx.lanes(bits)
    ctx.set_lanes(bits, lanes, old[1])
    ctx.set_grid_limit(cap)
    try:
        for got in roundtrip(torch, ctx, km, msg):
            np.testing.assert_array_equal(got, msg)
    finally:
        ctx.set_grid_limit(0)
        ctx.set_lanes(bits, *old)


def test_partial_round_by_blocks(torch, ctx):
    """4096-bit keys past a full round of one-lane blocks: the last groups run
    spread over blocks, in the same half buffer."""
    import torch as t

    rounds = 4 * 64 * (t.cuda.get_device_properties(0).multi_processor_count // 2)  # chunks of a round
    km = np.zeros(rounds + 64 * 5 + 3, dtype=np.uint32)
    msg = inputs.make_message(len(km) * 508 - 1, 77)
    ctx.load_keys(keys_of(4096, 1))
    for got in roundtrip(torch, ctx, km, msg)[:1]:
        np.testing.assert_array_equal(got, msg)


@pytest.mark.parametrize("bits,lanes,win", [(1024, 1, 4), (1024, 4, 4), (2048, 1, 2), (2048, 1, 6), (2048, 8, 5),
                                            (3072, 1, 5), (3072, 8, 5), (4096, 1, 5), (4096, 8, 5), (6144, 8, 5),
                                            (8192, 8, 5)])
def test_extreme_blocks(torch, ctx, bits, lanes, win):
    """Blocks whose residues and digits are extreme: 0, 1, N - 1, multiples of one
    prime, all-ones and alternating bytes, powers of two around limb edges; whole
    blocks equal the oracle's CRT decryption."""
    k = keys_of(bits, 1)[0]
    vals = [0, 1, k.n - 1, k.p, k.p * (k.q - 1), k.q * (k.p - 1), (1 << (bits - 1)) - 1]
    vals += [int(h * (bits // 8), 16) % k.n for h in ("7f", "80", "55", "ff")]
    if bits <= 4096:
        vals += [1 << e for e in (28, 29, bits // 2 - 1, bits // 2 + 20, bits - 2)] + [(1 << (bits // 2 + 20)) - 1]
    ctx.load_keys([k])
    old = ctx.lanes(bits), ctx.window(bits)
    ctx.set_lanes(bits, lanes, old[0][1])
    ctx.set_window(bits, win)
    try:
        kb = bits // 8
        plan = ctx.plan(np.zeros(len(vals), dtype=np.uint32), len(vals) * (kb - 4))
        plan.set_decrypt_output(binding.PMK_DEC_BLOCKS)
        ct = np.frombuffer(b"".join(v.to_bytes(kb, "big") for v in vals), dtype=np.uint8).copy()
        out = plan.decrypt(torch.from_numpy(ct).cuda())
        assert plan.check() == binding.PMK_OK
        got = out[: len(ct)].cpu().numpy().tobytes()
        plan.close()
    finally:
        ctx.set_lanes(bits, *old[0])
        ctx.set_window(bits, old[1])
    table = oracle.KeyTable([k])
    with ThreadPoolExecutor(8) as ex:
        want = list(ex.map(lambda v: oracle.rsa_int(table, 0, "crt", v), vals))
    assert [int.from_bytes(got[i * kb : (i + 1) * kb], "big") for i in range(len(vals))] == want


@pytest.mark.parametrize("cap", [0, 3])
@pytest.mark.parametrize("bits,win", [(1024, 2), (1536, 4), (2048, 5), (3072, 5), (4096, 5)])
def test_blinded_tile_and_group_edges(torch, ctx, bits, win, cap):
    """Both exponents in one chain per prime, at the edges of tiles and groups; a
    blinding factor that one of the primes divides is flagged and harms no other chunk."""
    counts = [1, 63, 64, 65, 129, 257] if not cap else [129, 1]
    keys = keys_of(bits, len(counts))
    kb = bits // 8
    km = np.repeat(np.arange(len(counts), dtype=np.uint32), counts)
    msg = inputs.make_message(len(km) * (kb - 4) - 7, bits + 1)
    ctx.load_keys(keys)
    old = ctx.lanes(bits), ctx.window(bits)
    ctx.set_lanes(bits, 1, old[0][1])
    ctx.set_window(bits, win)
    ctx.set_grid_limit(cap)
    try:
        plan = ctx.plan(km, len(msg))
        for bad in (None, keys[0].p, keys[0].q * 2):
            rblk = inputs.make_blinding(keys, km, bits)
            if bad:
                rblk[:kb] = np.frombuffer(bad.to_bytes(kb, "big"), np.uint8)
            cs, cr = plan.encrypt_blinded(torch.from_numpy(msg).cuda(), torch.from_numpy(rblk).cuda())
            assert plan.check() == binding.PMK_OK
            got = plan.decrypt_blinded(cs, cr)
            assert plan.check() == (binding.PMK_EBLIND if bad else binding.PMK_OK)
            skip = kb - 4 if bad else 0
            np.testing.assert_array_equal(got[skip : len(msg)].cpu().numpy(), msg[skip:])
        plan.close()
    finally:
        ctx.set_grid_limit(0)
        ctx.set_window(bits, old[1])
        ctx.set_lanes(bits, *old[0])


@pytest.mark.parametrize("bits,waves", [(1024, 3), (2048, 2)])
def test_partial_round_a_wave_per_simd(torch, ctx, bits, waves):
    """Past full rounds of one-lane blocks the last groups run a wave per SIMD, two units
    per block: an odd number of groups and a last group of one tile, plain and blinded."""
    import torch as t

    n = 128 * t.cuda.get_device_properties(0).multi_processor_count * waves + 64 * 4 + 3
    keys = keys_of(bits, 2)
    km = (np.arange(n) >= n - 64 * 7).astype(np.uint32)
    msg = inputs.make_message(n * (bits // 8 - 4) - 5, bits + 2)
    ctx.load_keys(keys)
    np.testing.assert_array_equal(roundtrip(torch, ctx, km, msg)[0], msg)
    plan = ctx.plan(km, len(msg))
    rblk = torch.from_numpy(inputs.make_blinding(keys, km, bits)).cuda()
    got = plan.decrypt_blinded(*plan.encrypt_blinded(torch.from_numpy(msg).cuda(), rblk))
    assert plan.check() == binding.PMK_OK
    np.testing.assert_array_equal(got[: len(msg)].cpu().numpy(), msg)
    plan.close()
