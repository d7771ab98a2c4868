"""hybrid_decode_batch reads its buffers when its kernels run: contents changed
in place between calls, and one call recorded in a caller's own graph and
replayed, each against a fresh decoder on copies of the same contents."""
import pytest
import torch

import oracle as O
from paper_1609_09358_amd import binding as PB

pytestmark = pytest.mark.gpu

N, K, C, L, T = 256, 128, 16, 32, 12


def batch(code, B, ebn0, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = PB.polar_encode(code, torch.randint(0, 2, (B, K), generator=g, device="cuda", dtype=torch.uint8)).float()
    s2 = O.sigma2(ebn0, K / N)
    return (2.0 * (1.0 - 2.0 * x + s2 ** 0.5 * torch.randn(x.shape, generator=g, device="cuda")) / s2).contiguous()


@pytest.mark.parametrize("B", [1, 700, 3000])
@pytest.mark.parametrize("how", ["calls", "graph", "static graph"])
def test_contents_changed_in_place(B, how):
    code = PB.PolarCode(N, K, C, 0, 2.0, da_bits=60)
    W = torch.full((T, 2, code.n), 0.94, device="cuda")
    dec = PB.HybridDecoder(code, max_iter=T, L=L, stop=2, weights=W)
    llr = batch(code, B, 2.0, 1)
    out = dict(info=torch.empty((B, K), dtype=torch.uint8, device="cuda"),
               used_scl=torch.empty(B, dtype=torch.uint8, device="cuda"))
    stats = torch.zeros(8, dtype=torch.int64, device="cuda")

    def call():
        if how == "static graph":
            PB.hybrid_decode_batch_static(code, llr, dec.params, L, out=out, stats=stats)
        else:
            dec(llr, out=out, stats=stats)

    if how != "calls":
        call()  # the decoder's workspace and the library's kernels are there before the capture
        torch.cuda.synchronize()
        stats.zero_()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            call()
    total = torch.zeros_like(stats)
    for j, (e, w) in enumerate(((2.0, 0.94), (1.0, 0.94), (3.0, 0.8), (0.0, 0.9), (2.0, 0.94))):
        llr.copy_(batch(code, B, e, 10 + j))
        W.fill_(w)
        out["info"].fill_(7)
        out["used_scl"].fill_(7)
        call() if how == "calls" else g.replay()
        PB.bp_decode_batch(code, llr, max_iter=3)  # unrelated work after it
        st = torch.zeros_like(stats)
        ref = PB.HybridDecoder(code, max_iter=T, L=L, stop=2, weights=W.clone())(llr.clone(), stats=st)
        total += st
        assert torch.equal(out["info"], ref["info"]), j
        assert torch.equal(out["used_scl"], ref["used_scl"]), j
        assert torch.equal(stats, total), j
    assert B == 1 or 0 < int(total[2]) < 5 * B
