"""The step's overlapped plan on small mini-batches, which take the serial order by
themselves: the chain and graph tests of the overlapped step run again with the size rule
lowered to zero edges."""
import pytest
import torch

from paper_2406_06022_amd import chain
from tests import test_gpu_chain, test_gpu_graph

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("index", [1, 2, 4])
def test_overlapped_plan_matches_serial_step(index, monkeypatch):
    monkeypatch.setattr(chain.MiniBatchStack, "overlap_min_edges", 0)
    calls = []
    stream = torch.cuda.Stream
    monkeypatch.setattr(torch.cuda, "Stream", lambda *a, **k: calls.append(1) or stream(*a, **k))
    test_gpu_chain.test_overlapped_plan_matches_serial_step(index)
    assert calls   # the second stream was made: the overlapped order ran


@pytest.mark.parametrize("index", [2, 4])
def test_graph_of_an_overlapped_step(index, monkeypatch):
    monkeypatch.setattr(chain.MiniBatchStack, "overlap_min_edges", 0)
    test_gpu_graph.test_graph_replays_match_eager_step(index)
