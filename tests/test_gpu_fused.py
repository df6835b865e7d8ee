"""The post-reorder's forms and its fusion with the consumer, on the GPU.

A run on one stream consumes and restores in one pass; rows are handled by one
wave or by a workgroup, held in registers or read twice. Each at the edges of
its range, against the oracle: what the consumer's buffer gets and every output
without RMSNorm are exact.
"""
import numpy as np
import pytest

import oracle
import paper_2504_19519_amd as fo
import workloads
from gpu_util import assert_close_bits, dev_plan, empty16, from_dev, say, to_dev, torch_mod, zeros_u32

pytestmark = pytest.mark.gpu

K = 64
# M, N: chunks per row (N / 8) at 256, 512 and 1024 and just past them, the widest row held in registers (2048)
# and the first that is not, few and many rows
SHAPES = [(64, 2048), (576, 2048), (512, 4096), (576, 4160), (64, 8192), (64, 8256), (64, 16384), (64, 16448),
          (192, 320)]


def setup(M, N, pattern, dtype, seed):
    rng = np.random.default_rng(seed)
    nd = {"tile": 0, "rowmajor": 0, "subtile": 4, "subtoken": 3}[pattern]
    sigma = rng.permutation(nd) if pattern == "subtile" else None
    bucket = rng.integers(0, nd, M) if pattern == "subtoken" else None
    T = -(-(M // 64) * (N // 64) // 100)
    kw = dict(pattern=pattern, num_dest=nd, num_cus=100, order="xcd", sizes=[1] * T, unit="waves")
    plan = fo.plan_groups(M, N, K, dtype=dtype, tile_m=64, tile_n=64, dest_perm=sigma, row_bucket=bucket, **kw)
    o = oracle.make_plan(M, N, 64, 64, group_m=4, num_xcds=8, sigma=sigma, bucket=bucket, **kw)
    A = to_dev(workloads.to_bits(rng.uniform(-1, 1, (M, K)), dtype))
    W = to_dev(workloads.to_bits(rng.uniform(-1, 1, (N, K)) / 8, dtype))
    peer = workloads.uniform_bits(M * N + 8, seed + 1, dtype) if pattern != "subtoken" else None
    return plan, o, dev_plan(plan), A, W, peer


def serial(plan, dp, A, W, C, peer, dst, out, bias=None, gamma=None, norm=False):
    torch = torch_mod()
    status = zeros_u32(1)
    fo.run_overlapped(plan, dp, A, W, C, peer, dst, out, bias, gamma, 1e-6, norm, None, status)   # null stream
    torch.cuda.synchronize()
    assert int(status.cpu()[0]) == 0


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("pattern,dtype", [("tile", "fp16"), ("subtile", "bf16"), ("subtoken", "fp16"),
                                           ("rowmajor", "bf16")])
def test_forms(shape, pattern, dtype):
    torch = torch_mod()
    M, N = shape
    n = M * N
    say(f"[post forms] {M}x{N} {pattern} {dtype}")
    plan, o, dp, A, W, peer = setup(M, N, pattern, dtype, M + N)
    bias, gamma = workloads.uniform_bits(N, 33, dtype, -0.1, 0.1), workloads.uniform_bits(N, 34, dtype, 0.5, 1.5)
    dB, dG, dP = to_dev(bias), to_dev(gamma), to_dev(peer) if peer is not None else None
    for b, g, norm in [(None, None, False), (dB, None, False), (None, None, True), (dB, dG, True), (None, dG, True)]:
        C, dst, out = empty16(n, dtype), empty16(n, dtype), empty16(n, dtype)
        serial(plan, dp, A, W, C, dP, dst, out, b, g, norm)
        want = oracle.apply_consumer(o, from_dev(C)[:n], None if peer is None else peer[:n], dtype)
        np.testing.assert_array_equal(from_dev(dst)[:n], want)
        x = want[oracle.post_index(o)].reshape(M, N)
        plain = empty16(n, dtype)
        fo.post_reorder(plan, dp, dst, plain, b, g, 1e-6, norm)
        torch.cuda.synchronize()
        for what, y in (("fused", out), ("alone", plain)):
            got = from_dev(y)[:n].reshape(M, N)
            if b is None and not norm:
                np.testing.assert_array_equal(got, x, err_msg=what)
                continue
            ref = oracle.rmsnorm(x, dtype, bias=bias if b is not None else None,
                                 gamma=gamma if g is not None else None, eps=1e-6, do_norm=norm)
            if norm:
                assert_close_bits(got, ref, dtype, what)
            else:
                np.testing.assert_array_equal(got, ref, err_msg=what)


def test_buffers_that_keep_the_passes_apart():
    # out on the GEMM's output or on the peer's partial (both free once the
    # consumer has read them), and a peer partial off the 16-byte grid: the run
    # takes its passes one after the other and gives the same bits
    M, N = 576, 2048
    n = M * N
    say("[fused: aliased and unaligned buffers]")
    plan, o, dp, A, W, peer = setup(M, N, "subtile", "fp16", 5)
    C, dst, out = empty16(n), empty16(n), empty16(n)
    dP = to_dev(peer)
    serial(plan, dp, A, W, C, dP, dst, out)
    Cr, want_dst, want = from_dev(C), from_dev(dst), from_dev(out)
    np.testing.assert_array_equal(want_dst[:n], oracle.apply_consumer(o, Cr[:n], peer[:n], "fp16"))
    for case in ("C", "peer", "unaligned"):
        C, dst, out, dP = empty16(n), empty16(n), empty16(n), to_dev(peer)
        if case == "unaligned":
            dP = to_dev(np.concatenate([peer[:1], peer]))
            arg = dP.data_ptr() + 2
        else:
            arg, out = dP, C if case == "C" else dP
        serial(plan, dp, A, W, C, arg, dst, out)
        np.testing.assert_array_equal(from_dev(dst)[:n], want_dst[:n], err_msg=case)
        np.testing.assert_array_equal(from_dev(out)[:n], want[:n], err_msg=case)
