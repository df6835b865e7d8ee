"""The stream handoffs of test_gpu_handoff, with a consumer launch per group.

Short runs consume all groups together when the options leave the consumer
launches alone, so these small runs would not reach the per-group launches and
their final launch's count. With another consumer grid as the process default
they do. All tests run on one pair of streams that are on different hardware
queues (kernels of streams that share a queue run one after another, and a held
stream then holds the other one too).
"""
import itertools

import pytest

import paper_2504_19519_amd as fo
from gpu_util import torch_mod
from test_gpu_handoff import (gpu, test_a_held_stream_is_waited_for,  # noqa: F401
                              test_a_timed_out_run_does_not_count_for_the_next, test_back_to_back_runs_share_buffers,
                              test_stale_counter_words_do_not_reach_a_run, test_timed_out_handoffs_raise_the_status_bit,
                              test_two_plans_alternate_on_the_same_streams)

pytestmark = pytest.mark.gpu


def _apart(torch, a, b):
    """Whether b runs while a is held, and a while b is."""
    for held, free in ((a, b), (b, a)):
        torch.cuda.synchronize()
        eh, ef = torch.cuda.Event(), torch.cuda.Event()
        with torch.cuda.stream(held):
            torch.cuda._sleep(20_000_000)
        eh.record(held)
        ef.record(free)
        ef.synchronize()
        if eh.query():
            return False
    torch.cuda.synchronize()
    return True


@pytest.fixture(scope="module", autouse=True)
def a_launch_per_group(gpu):  # noqa: F811
    torch = torch_mod()
    streams = [torch.cuda.Stream() for _ in range(6)]
    pair = next(p for p in itertools.combinations(streams, 2) if _apart(torch, *p))
    old, Stream = fo.get_consumer_grid(), torch.cuda.Stream
    fo.set_consumer_grid(255, 64)
    turn = itertools.cycle(pair)
    torch.cuda.Stream = lambda **kw: Stream(**kw) if kw else next(turn)
    yield
    torch.cuda.Stream = Stream
    fo.set_consumer_grid(*old)
