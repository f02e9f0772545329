"""The host side of SRLinear: which quantizers its calls get.  The entry points are replaced by ones that record them."""
import pytest
import torch

from paper_2511_00874_amd import lib as L
from paper_2511_00874_amd import train

M, N, K = 48, 32, 16


@pytest.fixture
def calls(monkeypatch):
    got = []

    def record(*args, **kw):
        got.extend(a for a in args if isinstance(a, (L.Quant, L.srq_quant)) and a is not train.NOQ)
        return None, None

    monkeypatch.setattr(L, "absmax_scales", lambda pairs: torch.ones(len(pairs)))
    for name in ("sr_linear_fwd", "sr_linear_fwd_stash", "sr_linear_bwd", "sr_linear_bwd_data", "sr_linear_bwd_stashed"):
        monkeypatch.setattr(L, name, record)
    return got


def _step(layer):
    x = torch.zeros((M, K), requires_grad=True)
    layer(x).backward(torch.zeros((M, N)))


@pytest.mark.parametrize("objective", train.OBJECTIVES)
def test_a_position_on_the_device_is_not_read_by_the_host(objective, calls):
    _step(train.SRLinear(K, N, 7, device="cpu", objective=objective))
    host = [(q.kind, q.round, q.seed, q.counter_offset) for q in calls]
    calls.clear()
    layer = train.SRLinear(K, N, 7, device="cpu", objective=objective)
    layer.position = torch.tensor([0], dtype=torch.int64)
    _step(layer)
    assert all(isinstance(q, L.Quant) and isinstance(q.counter_offset, torch.Tensor) for q in calls)  # (marshalled as device counters)
    assert [(q.kind, q.round_mode, q.seed, int(q.counter_offset)) for q in calls] == host
