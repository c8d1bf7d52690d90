"""Host side of the start network's parameter handling (no device needed)."""
import numpy as np
import pytest
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


def test_load_takes_any_shape_of_the_right_size(monkeypatch, tmp_path):
    """Saved arrays replace the parameters entry by entry, in whatever shape they
    are; another number of entries is refused rather than broadcast."""
    net, _ = _net(monkeypatch)
    monkeypatch.setattr(L.StartNet, "__init__", lambda self, seed=0: self.__dict__.update(net.__dict__))
    rng = np.random.default_rng(1)
    arrs = {f"w{i}": rng.standard_normal((o, c * 9)).astype(np.float32) for i, (c, o, _) in enumerate(L.LAYERS)}
    arrs.update({f"b{i}": rng.standard_normal((o, 1)).astype(np.float32) for i, (_, o, _) in enumerate(L.LAYERS)})
    np.savez(tmp_path / "a.npz", **arrs)
    got = L.StartNet.load(str(tmp_path / "a.npz"))
    for i in range(len(L.LAYERS)):
        assert np.array_equal(got.w[i].numpy().ravel(), arrs[f"w{i}"].ravel())
        assert np.array_equal(got.b[i].numpy().ravel(), arrs[f"b{i}"].ravel())
    np.savez(tmp_path / "b.npz", **dict(arrs, b0=np.float32(1.0)))
    with pytest.raises(RuntimeError):
        L.StartNet.load(str(tmp_path / "b.npz"))
