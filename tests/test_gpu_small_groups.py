"""Decryption under many keys with few tiles each: groups of one to three tiles, in
every form that such a launch takes, past one round of its blocks, each key
another.  Exact: the message comes back, plain, batched and blinded."""
import numpy as np
import pytest

from paper_2111_11924_amd import binding, inputs
from perf import cases

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    c = binding.Context(0)
    yield c
    c.close()


def keys_of(bits, count):
    """`count` keys: the pairs of a short list of primes, repeated where it has fewer,
    neighbours always different."""
    pairs = cases._pairs(bits)
    return [cases._key(bits, *pairs[i * 7 % len(pairs)]) for i in range(count)]


def check(ctx, bits, keys, chunks, blinded, mixed=0):
    import torch

    ks = keys_of(bits, keys)
    counts = np.full(keys, chunks)
    if mixed:  # groups of different sizes
        counts[::3] += mixed
    km = np.repeat(np.arange(keys, dtype=np.uint32), counts)
    msg = inputs.make_message(len(km) * (bits // 8 - 4) - 5, bits + keys)
    ctx.load_keys(ks)
    plan = ctx.plan(km, len(msg))
    d = torch.from_numpy(msg).cuda()
    if blinded:
        r = inputs.make_message(len(km) * (bits // 8), 9).reshape(len(km), bits // 8).copy()
        r[:, 0] = 0
        outs = [plan.decrypt_blinded(*plan.encrypt_blinded(d, torch.from_numpy(r.reshape(-1)).cuda()))]
    else:
        ct = plan.encrypt(d)
        outs = [plan.decrypt(ct), plan.decrypt(ct, batch=True)]
    assert plan.check() == binding.PMK_OK
    for o in outs:
        np.testing.assert_array_equal(o[: len(msg)].cpu().numpy(), msg)
    plan.close()


# one tile per key: past a wave per SIMD (1024, 2048), past three blocks (3072) and one
# block (4096) per compute unit; two and three tiles; groups of mixed sizes
@pytest.mark.parametrize("bits,keys,chunks,mixed", [
    (1024, 520, 33, 0), (1024, 522, 129, 0), (2048, 520, 20, 0), (2048, 140, 129, 70), (3072, 390, 20, 0),
    (3072, 260, 65, 0), (3072, 130, 129, 64), (4096, 130, 17, 0), (4096, 131, 65, 0), (4096, 90, 129, 64)])
def test_few_tiles_per_key(ctx, bits, keys, chunks, mixed):
    check(ctx, bits, keys, chunks, False, mixed)


@pytest.mark.parametrize("bits,keys,chunks,mixed", [
    (1024, 522, 129, 0), (2048, 520, 20, 0), (3072, 390, 20, 0), (3072, 130, 129, 64), (4096, 131, 65, 0)])
def test_few_tiles_per_key_blinded(ctx, bits, keys, chunks, mixed):
    check(ctx, bits, keys, chunks, True, mixed)


# numbers over blocks: tiles with one, two and all of their four parts, past one step of
# every block
@pytest.mark.parametrize("bits,keys,chunks,mixed", [(1024, 280, 7, 0), (2048, 140, 16, 0), (3072, 70, 20, 0),
                                                    (4096, 70, 16, 33), (6144, 40, 16, 17), (8192, 40, 17, 0)])
def test_few_parts_per_key(ctx, bits, keys, chunks, mixed):
    check(ctx, bits, keys, chunks, False, mixed)


# so many keys that Montgomery products are the faster form: one lane per number (1024 to
# 4096 bits), four lanes (6144, 8192); blinded also two lanes (4096)
@pytest.mark.parametrize("bits,keys,chunks", [(1024, 520, 65), (3072, 400, 33), (3072, 270, 65), (4096, 330, 49),
                                              (6144, 257, 49), (8192, 130, 49)])
def test_montgomery_form(ctx, bits, keys, chunks):
    check(ctx, bits, keys, chunks, False)


@pytest.mark.parametrize("bits,keys,chunks", [(3072, 400, 33), (4096, 140, 20), (4096, 257, 20)])
def test_montgomery_form_blinded(ctx, bits, keys, chunks):
    check(ctx, bits, keys, chunks, True)


@pytest.mark.parametrize("bits,keys", [(3072, 400), (4096, 330)])
def test_montgomery_form_edges(ctx, bits, keys):
    """Blocks 0, 1, N - 1, a multiple of one prime, and one of N itself, which is flagged and
    decrypts to zero bytes; the others equal c^d mod N."""
    import torch

    ks, kb, per = keys_of(bits, keys), bits // 8, 49
    ctx.load_keys(ks)
    km = np.repeat(np.arange(keys, dtype=np.uint32), per)
    plan = ctx.plan(km, len(km) * (kb - 4))
    plan.set_decrypt_output(binding.PMK_DEC_BLOCKS)
    ct = np.zeros((len(km), kb), np.uint8)
    at = [0, 1, 2, 3, per * keys - 1]
    k, last = ks[0], ks[-1]
    vals = [1, k.n - 1, k.p * 5, k.n, last.q * (last.p - 1)]
    for i, v in zip(at, vals):
        ct[i] = np.frombuffer(v.to_bytes(kb, "big"), np.uint8)
    out = plan.decrypt(torch.from_numpy(ct.reshape(-1)).cuda())
    assert plan.check() == binding.PMK_ERANGE
    got = out[: ct.size].cpu().numpy().reshape(ct.shape)
    want = np.zeros_like(ct)
    for i, v in zip(at, vals):
        key = ks[int(km[i])]
        want[i] = np.frombuffer((0 if v >= key.n else pow(v, key.d, key.n)).to_bytes(kb, "big"), np.uint8)
    np.testing.assert_array_equal(got, want)
    plan.close()


def test_blinded_tables_of_single_tiles(ctx):
    """124 keys with two chunks each: the window tables of blinded decryption hold two odd-power
    tables of 2^4 numbers of 40 limbs for each of the 248 waves, 81 MB, not twice that."""
    import torch

    keys, per = 124, 2
    ctx.load_keys(keys_of(2048, keys))
    win = ctx.window(2048)

    def run(n):
        km = np.repeat(np.arange(n, dtype=np.uint32), per)
        msg = inputs.make_message(len(km) * 252, n)
        r = inputs.make_message(len(km) * 256, 3).reshape(len(km), 256).copy()
        r[:, 0] = 0
        plan = ctx.plan(km, len(msg))
        args = plan.encrypt_blinded(torch.from_numpy(msg).cuda(), torch.from_numpy(r.reshape(-1)).cuda())
        before = torch.cuda.mem_get_info()[0]
        out = plan.decrypt_blinded(*args)
        assert plan.check() == binding.PMK_OK
        used = before - torch.cuda.mem_get_info()[0]
        np.testing.assert_array_equal(out[: len(msg)].cpu().numpy(), msg)
        plan.close()
        return used

    ctx.set_window(2048, 5)
    try:
        run(2)  # what the first launch of these kernels makes once
        assert run(keys) <= 124 * 2 * 2 * 16 * 40 * 64 * 4 + (8 << 20)
    finally:
        ctx.set_window(2048, win)


# past full rounds of the lane form, the last groups in each of the forms that take them,
# plain and batched
@pytest.mark.parametrize("bits,keys,chunks,mixed", [(1024, 40, 2560, 70), (2048, 36, 1920, 70), (3072, 70, 1024, 70),
                                                    (4096, 66, 512, 70)])
def test_partial_rounds(ctx, bits, keys, chunks, mixed):
    check(ctx, bits, keys, chunks, False, mixed)


@pytest.mark.parametrize("bits,keys,chunks,mixed", [(1024, 40, 2560, 70), (2048, 36, 1920, 70)])
def test_partial_rounds_blinded(ctx, bits, keys, chunks, mixed):
    check(ctx, bits, keys, chunks, True, mixed)


@pytest.mark.parametrize("bits,lanes", [(2048, 1), (2048, 8), (3072, 1), (3072, 8), (4096, 1), (4096, 8), (6144, 4),
                                        (6144, 8), (8192, 4), (8192, 8)])
def test_edges_under_different_keys(ctx, bits, lanes):
    """Tiles, groups and parts around their edges, each key another, so that a wrong key or
    fold table shows."""
    import torch

    counts = [1, 15, 17, 63, 64, 65, 129, 257] if bits <= 4096 else [1, 15, 17, 65]
    ctx.load_keys(keys_of(bits, len(counts)))
    km = np.repeat(np.arange(len(counts), dtype=np.uint32), counts)[::-1].copy()
    msg = inputs.make_message(len(km) * (bits // 8 - 4) - 7, bits + lanes)
    old = ctx.lanes(bits)
    ctx.set_lanes(bits, lanes, old[1])
    try:
        plan = ctx.plan(km, len(msg))
        ct = plan.encrypt(torch.from_numpy(msg).cuda())
        for out in (plan.decrypt(ct), plan.decrypt(ct, batch=True)):
            assert plan.check() == binding.PMK_OK
            np.testing.assert_array_equal(out[: len(msg)].cpu().numpy(), msg)
        plan.close()
    finally:
        ctx.set_lanes(bits, *old)


# the last step of the group form has fewer jobs: tiles with up to two parts, each in its
# quarter of the blocks, and tiles with most of their four
@pytest.mark.parametrize("bits,keys,chunks", [
    (1024, 270, 25), (2048, 228, 25), (2048, 131, 16), (2048, 90, 90), (3072, 100, 25), (3072, 66, 16), (3072, 18, 300),
    (4096, 100, 25), (4096, 65, 64), (6144, 50, 25), (8192, 33, 17)])
def test_last_step_of_group_blocks(ctx, bits, keys, chunks):
    check(ctx, bits, keys, chunks, False)
