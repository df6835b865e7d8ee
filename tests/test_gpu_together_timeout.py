"""A timed-out overlapped run whose groups are consumed together, on the GPU.

The consumer and post-reorder of such a run are one launch on the consumer
stream, so nothing but the run's gate word keeps it behind the GEMM stream. Once
a wait of the run has given up (host-shortened limit, one of the streams held
well past it) that launch must write neither dst nor out: later work of the GEMM
stream may be using both.
"""
import pytest

import paper_2504_19519_amd as fo
from gpu_util import dev_plan, empty16, say, streams_apart, torch_mod, zeros_u32

pytestmark = pytest.mark.gpu

HOLD = 500_000_000          # cycles: about 200 ms
LIMIT = {"poll_timeout_us": 20000}


@pytest.fixture(scope="module")
def pair():
    assert torch_mod().cuda.is_available(), "no GPU visible"
    return streams_apart()


# rows: the launch's workgroups counted one by one, and by a kernel behind it (more than 512)
@pytest.mark.parametrize("norm", [False, True])
@pytest.mark.parametrize("M", [512, 4096])
@pytest.mark.parametrize("held", ["gemm_stream", "comm_stream"])
def test_nothing_is_written_after_a_wait_gave_up(held, M, norm, pair):
    torch = torch_mod()
    N, K = 512, 128
    s1, s2 = pair
    say(f"[together, timed out] {M}x{N}x{K} held={held} norm={norm}")
    tiles = M // 64 * N // 64
    plan = fo.plan_groups(M, N, K, dtype="fp16", tile_m=64, tile_n=64, pattern="tile",
                          sizes=[tiles // 4, tiles // 4, tiles // 2], unit="tiles")
    dp = dev_plan(plan)
    A, W, peer = (torch.randn(n, device="cuda").half() for n in (M * K, N * K, M * N))
    C, dst, out = (empty16(M * N, "fp16") for _ in range(3))
    counters, status = zeros_u32(plan.num_counters), zeros_u32(1)

    def run(**kw):
        fo.run_overlapped(plan, dp, A, W, C, peer, dst, out, None, None, 1e-6, norm, counters, status, s1, s2, **kw)

    C2, dst2, out2 = (empty16(M * N, "fp16") for _ in range(3))
    fo.run_overlapped(plan, dp, A, W, C2, peer, dst2, out2, None, None, 1e-6, norm)
    torch.cuda.synchronize()
    for k in range(2):
        for t in (C, dst, out):
            t.fill_(0x7E00)
        status.zero_()
        torch.cuda.synchronize()
        with torch.cuda.stream(s1 if held == "gemm_stream" else s2):
            torch.cuda._sleep(HOLD)
        with torch.cuda.stream(s1):          # a reader of what an earlier run left there
            read = [t.clone() for t in (dst, out)]
        run(opts=LIMIT)
        with torch.cuda.stream(s1):          # the layer behind this one uses the buffers
            dst.fill_(17)
            out.fill_(18)
        torch.cuda.synchronize()
        assert int(status.cpu()[0]) & 1 == 1, f"round {k}"
        assert all(bool((t == 0x7E00).all()) for t in read), f"round {k}: written ahead of the GEMM stream's reader"
        assert bool((dst == 17).all()) and bool((out == 18).all()), f"round {k}: written after the wait gave up"
        # the caller clears the status; the next run on the same counters is whole
        status.zero_()
        torch.cuda.synchronize()
        run()
        torch.cuda.synchronize()
        assert int(status.cpu()[0]) == 0, f"round {k}"
        for what, x, y in (("C", C, C2), ("dst", dst, dst2), ("out", out, out2)):
            assert torch.equal(x, y), f"round {k}: {what}"
        assert counters[:plan.P].tolist() == list(plan.targets)
        assert int(counters[plan.P + fo.DISPENSER_WORDS]) == 0, "gate word"


def test_the_next_run_is_whole(pair):
    # the consumer stream is held; a run with a short limit and one with the normal
    # limit are queued back to back on the same buffers. The first gives up and its
    # late launch finds the second run's tag; the second waits for its own.
    torch = torch_mod()
    M, N, K = 512, 512, 128
    s1, s2 = pair
    say(f"[together, timed out back-to-back] {M}x{N}x{K}")
    plan = fo.plan_groups(M, N, K, dtype="fp16", tile_m=64, tile_n=64, pattern="tile", sizes=[16, 16, 32], unit="tiles")
    dp = dev_plan(plan)
    As = [torch.randn(M * K, device="cuda").half() for _ in range(2)]
    W, peer = (torch.randn(n, device="cuda").half() for n in (N * K, M * N))
    C, dst, first, out, C2, dst2, out2 = (empty16(M * N, "fp16") for _ in range(7))
    counters, status = zeros_u32(plan.num_counters), zeros_u32(1)
    fo.run_overlapped(plan, dp, As[1], W, C2, peer, dst2, out2)
    torch.cuda.synchronize()
    with torch.cuda.stream(s2):
        torch.cuda._sleep(HOLD)
    for A, o, opts in ((As[0], first, LIMIT), (As[1], out, None)):
        fo.run_overlapped(plan, dp, A, W, C, peer, dst, o, counters=counters, status_word=status, gemm_stream=s1,
                          comm_stream=s2, opts=opts)
    torch.cuda.synchronize()
    assert int(status.cpu()[0]) & 1 == 1
    assert bool((first == 0x7E00).all())
    for what, x, y in (("C", C, C2), ("dst", dst, dst2), ("out", out, out2)):
        assert torch.equal(x, y), what
