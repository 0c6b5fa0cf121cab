"""GPU test of key tables whose fold tables do not fit the device's memory: they load,
and decryption (plain, batched, blinded, without allocation) runs on Montgomery products."""
import numpy as np
import pytest

from paper_2111_11924_amd import binding, inputs
from perf import cases

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits,count", [(2048, 16500), (4096, 4600)])
def test_tables_that_do_not_fit(bits, count):
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    pairs = cases._pairs(bits)
    keys = [cases._key(bits, *pairs[i % len(pairs)]) for i in range(count)]
    kb = bits // 8
    km = np.repeat(np.array([0, 5, 9, count - 1], np.uint32), [1, 65, 20, 130])
    msg = inputs.make_message(len(km) * (kb - 4) - 3, bits)
    r = inputs.make_message(len(km) * kb, 4).reshape(len(km), kb).copy()
    r[:, 0] = 0
    d, d_r = torch.from_numpy(msg).cuda(), torch.from_numpy(r.reshape(-1)).cuda()
    ctx = binding.Context(0)
    ctx.load_keys(keys[:1])
    torch.cuda.synchronize()
    hog = [torch.empty(torch.cuda.mem_get_info()[0] - (1280 << 20), dtype=torch.uint8, device="cuda")]
    try:
        with pytest.raises(torch.cuda.OutOfMemoryError):  # more than what is reported free can be had
            while len(hog) < 64:
                hog.append(torch.empty(256 << 20, dtype=torch.uint8, device="cuda"))
        del hog[-5:]
        torch.cuda.empty_cache()  # 1.3 to 1.5 GiB are free
        ctx.load_keys(keys)  # 105,984 and 384,512 bytes of fold tables per key: 1.6 GiB
        with pytest.raises(torch.cuda.OutOfMemoryError):  # as little as before: no fold tables
            hog.append(torch.empty(1536 << 20, dtype=torch.uint8, device="cuda"))
        hog.append(torch.empty(1024 << 20, dtype=torch.uint8, device="cuda"))
        del hog[-1]
        torch.cuda.empty_cache()
        plan = ctx.plan(km, len(msg))
        ct = plan.encrypt(d)
        outs = [plan.decrypt(ct), plan.decrypt(ct, batch=True),
                plan.decrypt_blinded(*plan.encrypt_blinded(d, d_r))]
        assert plan.check() == binding.PMK_OK
        outs.append(torch.empty_like(d))
        torch.cuda.synchronize()
        assert binding.pmk_decrypt_noalloc(ctx.handle, ct, plan.ct_len, km, outs[-1], len(msg)) == binding.PMK_OK
        for o in outs:
            np.testing.assert_array_equal(o[: len(msg)].cpu().numpy(), msg)
        plan.close()
    finally:
        del hog
        torch.cuda.empty_cache()
        ctx.close()


def test_reload_frees_the_previous_tables():
    """A table whose fold tables fit only once: loading it again keeps them."""
    import torch

    pairs = cases._pairs(2048)
    keys = [cases._key(2048, *pairs[i % len(pairs)]) for i in range(6600)]  # 0.65 GiB of fold tables
    ctx = binding.Context(0)
    ctx.load_keys(keys[:1])
    torch.cuda.synchronize()
    hog = [torch.empty(torch.cuda.mem_get_info()[0] - (1280 << 20), dtype=torch.uint8, device="cuda")]
    try:
        with pytest.raises(torch.cuda.OutOfMemoryError):
            while len(hog) < 64:
                hog.append(torch.empty(256 << 20, dtype=torch.uint8, device="cuda"))
        del hog[-5:]
        torch.cuda.empty_cache()
        for _ in range(2):
            ctx.load_keys(keys)
            with pytest.raises(torch.cuda.OutOfMemoryError):  # the tables are there
                hog.append(torch.empty(768 << 20, dtype=torch.uint8, device="cuda"))
        del hog[-2:]
        torch.cuda.empty_cache()
        km = np.repeat(np.array([0, 6599], np.uint32), [30, 40])
        msg = inputs.make_message(len(km) * 252, 6)
        plan = ctx.plan(km, len(msg))
        out = plan.decrypt(plan.encrypt(torch.from_numpy(msg).cuda()))
        assert plan.check() == binding.PMK_OK
        np.testing.assert_array_equal(out[: len(msg)].cpu().numpy(), msg)
        plan.close()
    finally:
        del hog
        torch.cuda.empty_cache()
        ctx.close()
