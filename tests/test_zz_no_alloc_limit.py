"""GPU test of the allocation-free decryption at the edge of its scratch: 2048-bit
chunks whose data (descriptors, packed words and canonical halves, 53,252 bytes
per tile) and one window table just fit 64 MiB, and a few tiles more."""
import numpy as np
import pytest

from paper_2111_11924_amd import binding, inputs
from perf import cases

pytestmark = pytest.mark.gpu


def test_as_many_tiles_as_fit_64_mib():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    most = 1257  # tiles, of one chunk each
    pairs = cases._pairs(2048)
    keys = [cases._key(2048, *pairs[i % len(pairs)]) for i in range(most + 6)]
    ctx = binding.Context(0)
    try:
        ctx.load_keys(keys)
        for n, rc in ((most, binding.PMK_OK), (most + 6, binding.PMK_ESIZE)):
            km = np.arange(n, dtype=np.uint32)
            msg = inputs.make_message(n * 252, n)
            plan = ctx.plan(km, len(msg))
            ct = plan.encrypt(torch.from_numpy(msg).cuda())
            torch.cuda.synchronize()
            out = torch.zeros(len(msg), dtype=torch.uint8, device="cuda")
            assert binding.pmk_decrypt_noalloc(ctx.handle, ct, n * 256, km, out, len(msg)) == rc
            if rc == binding.PMK_OK:
                np.testing.assert_array_equal(out.cpu().numpy(), msg)
            plan.close()
    finally:
        ctx.close()
