"""Runs captured into a graph and replayed, on the GPU: groups consumed
together, a launch per group, and on one stream. Every replay works on other
operands and is checked against an eager run on one stream with buffers of its
own, with the host waiting in between."""
import pytest

import paper_2504_19519_amd as fo
from gpu_util import dev_plan, empty16, say, torch_mod, zeros_u32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", ["together", "per group", "one stream"])
def test_replays(form):
    torch = torch_mod()
    M, N, K = 512, 512, 256
    say(f"[graph] {form}")
    plan = fo.plan_groups(M, N, K, dtype="fp16", tile_m=64, tile_n=64, pattern="tile", sizes=[16, 16, 32], unit="tiles")
    dp = dev_plan(plan)
    A, W, peer = (torch.randn(n, device="cuda").half() for n in (M * K, N * K, M * N))
    C, dst, out = (empty16(M * N, "fp16") for _ in range(3))
    counters, status = zeros_u32(plan.num_counters), zeros_u32(1)
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    comm = s1 if form == "one stream" else s2
    # (waits bounded well below the default: a replay that hangs on a handoff ends in the status bit)
    opts = {"poll_timeout_us": 200000, "consumer_blocks": 255 if form == "per group" else 256}

    def run():
        fo.run_overlapped(plan, dp, A, W, C, peer, dst, out, counters=counters, status_word=status, gemm_stream=s1,
                          comm_stream=comm, opts=opts)

    torch.cuda.synchronize()
    run()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s1):
        s2.wait_stream(s1)
        run()
        s1.wait_stream(s2)
    for k in range(5):
        A.copy_(torch.randn(M * K, device="cuda"))
        for t in (C, dst, out):
            t.fill_(0x7E00)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        C2, dst2, out2 = (empty16(M * N, "fp16") for _ in range(3))
        fo.run_overlapped(plan, dp, A, W, C2, peer, dst2, out2)
        torch.cuda.synchronize()
        assert int(status.cpu()[0]) == 0, f"replay {k}"
        for what, x, y in (("C", C, C2), ("dst", dst, dst2), ("out", out, out2)):
            assert torch.equal(x, y), f"replay {k}: {what}"
