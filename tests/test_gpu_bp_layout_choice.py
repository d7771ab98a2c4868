"""The BP layout chosen by batch size and weights, and the logarithm of the
exact rule: either side of each line gives the results of both layouts."""
import pytest
import torch

import oracle as O
from paper_1609_09358_amd import binding as PB

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,B", [(512, 5), (1024, 1), (1024, 768), (1024, 769), (2048, 256), (2048, 257), (4096, 3)])
@pytest.mark.parametrize("weights", ["none", "column", "node"])
@pytest.mark.parametrize("stop", [0, 1, 2])
def test_automatic_layout_equals_both(N, B, weights, stop):
    code = PB.PolarCode(N, N // 2, 16, 0, 2.0)
    g = torch.Generator(device="cuda").manual_seed(N + B)
    x = PB.polar_encode(code, torch.randint(0, 2, (B, code.K), generator=g, device="cuda", dtype=torch.uint8)).float()
    s2 = O.sigma2(2.0, 0.5)
    llr = (2.0 * (1.0 - 2.0 * x + s2 ** 0.5 * torch.randn(x.shape, generator=g, device="cuda")) / s2).contiguous()
    T = 8
    W = None
    if weights != "none":
        shape = (T, 2, code.n) + ((N,) if weights == "node" else ())
        W = torch.rand(shape, generator=g, device="cuda") * 0.4 + 0.7
    a = PB.bp_decode_batch(code, llr, max_iter=T, stop=stop, weights=W, soft=True)
    for v in (2, 3):
        b = PB.bp_decode_batch(code, llr, max_iter=T, stop=stop, weights=W, soft=True, variant=v)
        for k in ("u_hat", "iters", "ok", "llr_u"):
            assert torch.equal(a[k], b[k]), (k, v)
