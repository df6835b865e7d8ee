"""The consumer's LDS ring (one-wave workgroups, direct calls) on the GPU, at
the edges of its batches (1024 elements of a sum, 2048 of a copy) and of the 6
rounds in flight per wave, bit-exact against the oracle's sum."""
import numpy as np
import pytest

import oracle
import paper_2504_19519_amd as fo
import workloads
from gpu_util import empty16, from_dev, say, to_dev, torch_mod, zeros_u32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
@pytest.mark.parametrize("length,blocks", [(n, b) for b in (1, 3, 256) for n in (
    1, 8, 1023, 1024, 1025, 2047, 2049, 6 * 1024, 7 * 1024 + 9, 12 * 1024, 13 * 1024 + 511, 36 * 1024 + 5)] + [
        (256 * 13 * 1024 + 7, 256)])
def test_ring(length, blocks, dtype):
    torch = torch_mod()
    say(f"[consume ring] len={length} blocks={blocks} {dtype}")
    src, peer = workloads.uniform_bits(length, 41, dtype, -4, 4), workloads.uniform_bits(length, 42, dtype, -4, 4)
    dS, dP, ctr = to_dev(src), to_dev(peer), zeros_u32(1)
    ctr.fill_(2)
    total = oracle.encode(oracle.decode(src, dtype) + oracle.decode(peer, dtype), dtype)
    for q, want in ((dP, total), (None, src)):
        dst = empty16(length + 8, dtype)     # the elements past the segment stay as they are
        fo.consume_group(dS, q, dst, length, dtype, ctr, 2, opts={"consumer_blocks": blocks})
        torch.cuda.synchronize()
        got = from_dev(dst)
        np.testing.assert_array_equal(got[:length], want)
        assert np.all(got[length:length + 8] == {"fp16": 0x7E00, "bf16": 0x7FC0}[dtype])
