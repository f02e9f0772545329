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


@pytest.mark.parametrize("objective", train.OBJECTIVES)
def test_a_subclass_sees_every_write_of_the_layers_state(objective, calls):
    seen = []

    class Property(train.SRLinear):
        position = property(lambda self: self._position, lambda self, v: object.__setattr__(self, "_position", v))
        have_grad = property(lambda self: self._have, lambda self, v: object.__setattr__(self, "_have", v))

    class Watched(train.SRLinear):
        def __setattr__(self, name, value):
            if name in ("position", "have_grad"):
                seen.append((name, value))
            super().__setattr__(name, value)

    plain = train.SRLinear(K, N, 7, device="cpu", objective=objective)
    _step(plain)
    for cls in (Property, Watched):
        layer = cls(K, N, 7, device="cpu", objective=objective)
        seen.clear()
        _step(layer)
        assert (layer.position, layer.have_grad) == (plain.position, True) and plain.have_grad
        assert not {"position", "have_grad"} & set(vars(layer)) or cls is Watched
    assert ("position", plain.position) in seen and ("have_grad", True) in seen
    plain.register_buffer("kept", torch.zeros(1))
    with pytest.raises(TypeError):
        plain.kept = 3  # as a module refuses it
    plain.position = torch.nn.Parameter(torch.zeros(1))
    assert "position" in dict(plain.named_parameters())
