"""The start network's parameters lie in one buffer: one Adam launch over them
equals one per tensor, with the network's own tensors and with replaced ones."""
import numpy as np
import pytest

import paper_2508_05400_amd as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("replace", [None, "w", "g", "m"])
def test_adam_over_all_parameters(lib, cuda, replace):
    from paper_2508_05400_amd.learned_start import StartNet
    torch = cuda
    net = StartNet(seed=5)
    x = torch.randn((2, 2, 64, 64), generator=torch.Generator().manual_seed(1)).cuda()
    V = torch.linalg.qr(torch.randn((2, 4096, 17), generator=torch.Generator().manual_seed(2)))[0].contiguous().cuda()
    ref = [[t.clone() for t in q] for q in (net.w + net.b, net.m, net.v)]
    for step in (1, 2):
        acts = net.forward(x)
        _, du = net.loss_and_grad(acts[-1], V)
        gw, gb = net.backward(acts, du)
        if replace == "w":
            net.w[2] = net.w[2].clone()
        elif replace == "g":
            gb = [g.clone() for g in gb]
        elif replace == "m":
            net.m[3] = net.m[3].clone()
        for p, g, m, v in zip(ref[0], list(gw) + list(gb), ref[1], ref[2]):
            P.rks_net_adam(p, g, m, v, p.numel(), 1e-2, step)
        net.adam(gw, gb, 1e-2)
        for got, want in zip((net.w + net.b, net.m, net.v), ref):
            for a, b in zip(got, want):
                assert np.array_equal(a.cpu().numpy(), b.cpu().numpy())
