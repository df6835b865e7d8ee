"""The stream handoffs of test_gpu_handoff, with a consumer launch per group.

Short runs consume all groups together when the options leave the consumer
launches alone, so these small runs would not reach the per-group launches and
their final launch's count. With another consumer grid as the process default
they do. All tests run on one pair of streams that are on different hardware
queues.
"""
import itertools

import pytest

import paper_2504_19519_amd as fo
import test_gpu_handoff
from gpu_util import streams_apart, torch_mod
from test_gpu_handoff import (gpu, test_a_held_stream_is_waited_for,  # noqa: F401
                              test_a_timed_out_run_does_not_count_for_the_next, test_back_to_back_runs_share_buffers,
                              test_stale_counter_words_do_not_reach_a_run, test_timed_out_handoffs_raise_the_status_bit,
                              test_two_plans_alternate_on_the_same_streams)

pytestmark = pytest.mark.gpu


class _With:
    """An object with some of its attributes replaced."""

    def __init__(self, base, **attributes):
        self.__dict__.update(attributes, _base=base)

    def __getattr__(self, name):
        return getattr(self._base, name)


@pytest.fixture(scope="module")
def pair(gpu):  # noqa: F811
    return streams_apart()


@pytest.fixture(autouse=True)
def a_launch_per_group(pair, monkeypatch):
    # (the tests' own module sees a torch whose new streams are the pair's)
    torch, turn = torch_mod(), itertools.cycle(pair)
    view = _With(torch, cuda=_With(torch.cuda, Stream=lambda: next(turn)))
    monkeypatch.setattr(test_gpu_handoff, "torch_mod", lambda: view)
    old = fo.get_consumer_grid()
    fo.set_consumer_grid(255, 64)
    yield
    fo.set_consumer_grid(*old)
