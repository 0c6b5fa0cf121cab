"""GPU test of the request server's rounds: the default bound on a round's chunks
holds two rounds of 2048-bit CRT halves with three waves per SIMD."""
import numpy as np
import pytest

from paper_2111_11924_amd import binding, inputs

pytestmark = pytest.mark.gpu


def test_default_round_holds_two_chip_filling_rounds():
    import torch

    n = 12 * 64 * torch.cuda.get_device_properties(0).multi_processor_count  # 196,608 on 256 compute units
    ctx = binding.Context(0)
    ctx.load_keys(inputs.make_keys([256], 871))
    srv = ctx.server(staging_bytes=64 << 20)
    try:
        rounds = []
        for chunks in (n, n + 1):
            msg = inputs.make_message(chunks * 28, chunks)
            before = srv.stats()["rounds"]
            ticket, out = srv.submit(binding.PMK_OP_ENCRYPT, msg, len(msg), np.zeros(chunks, np.uint32))
            assert srv.wait(ticket)["status"] == binding.PMK_OK
            rounds.append(srv.stats()["rounds"] - before)
        assert rounds == [1, 2]
    finally:
        srv.stop()
        ctx.close()
