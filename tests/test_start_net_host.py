"""Host side of the start network's parameter handling (no device needed)."""
import numpy as np
import torch

from paper_2508_05400_amd import learned_start as L


def _net(monkeypatch):
    """A network with its parameters in host memory, and the Adam calls it makes."""
    net, calls = L.StartNet.__new__(L.StartNet), []
    net.torch, net.t = torch, 0
    net.w, net.b = L.StartNet._parameters(torch.zeros(L.PARAMS))
    net.m, net.v = (sum(L.StartNet._views(torch.zeros(L.PARAMS)), []) for _ in range(2))
    monkeypatch.setattr(L.B, "rks_net_adam", lambda *a: calls.append(a))
    return net, calls


def test_adam_takes_device_addresses_and_short_lists(monkeypatch):
    """What the binding takes as a buffer is an address or anything with a
    data_ptr(); a list shorter than the parameters updates the leading ones."""
    net, calls = _net(monkeypatch)
    gw, gb = L.StartNet._views(torch.zeros(L.PARAMS))
    net.adam([g.data_ptr() for g in gw], [g.data_ptr() for g in gb], 1e-3)
    assert [c[1] for c in calls] == [g.data_ptr() for g in gw + gb] and net.t == 1
    calls.clear()
    net.adam(gw[:2], [], 1e-3)
    assert [c[4] for c in calls] == [net.w[0].numel(), net.w[1].numel()]
    calls.clear()
    net.adam([], [], 1e-3)
    assert not calls and net.t == 3
    net.adam(gw, gb, 1e-3)
    assert [c[4] for c in calls] == [L.PARAMS]


def test_parameters_are_tensors_of_their_own(monkeypatch):
    """Writing to one parameter does not invalidate what autograd saved of another."""
    net, _ = _net(monkeypatch)
    assert not any(t._is_view() for t in net.w + net.b)
    net.w[0].requires_grad_()
    loss = (net.w[0] * net.w[0]).sum()
    net.w[1].mul_(0.5)
    net.b[0].add_(1.0)
    loss.backward()
    assert net.b[1].abs().max() == 0 and net.b[0].min() == 1  # of one buffer, without overlap
