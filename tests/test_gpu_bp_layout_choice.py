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


@pytest.mark.parametrize("N,c", [(8, 0), (16, 0), (32, 8), (64, 8), (128, 8), (256, 8), (512, 16)])
@pytest.mark.parametrize("variant", [2, 3])
@pytest.mark.parametrize("stop", [1, 2])
def test_short_blocks_match_oracle(N, c, variant, stop):
    """Blocks of at most one wavefront a frame, several frames a wavefront with one left over: verdicts, iterations,
    decisions and the hybrid's information bits."""
    if stop == 2 and c == 0:
        pytest.skip("the CRC stop needs a CRC")
    K, B, T = max(1, N // 2 - (c if N <= 32 else 0)), 67, 12
    code = PB.PolarCode(N, K, c, 0, 2.0)
    poly = {0: 0, 8: 0x07, 16: 0x1021}[c]
    g = torch.Generator(device="cuda").manual_seed(N + stop)
    x = PB.polar_encode(code, torch.randint(0, 2, (B, K), generator=g, device="cuda", dtype=torch.uint8)).float()
    s2 = O.sigma2(2.0, 0.5)
    llr = (2.0 * (1.0 - 2.0 * x + s2 ** 0.5 * torch.randn(x.shape, generator=g, device="cuda")) / s2).contiguous()
    h = llr.cpu().numpy()
    for s in {0, stop}:
        ref = O.bp_batch(h, code.frozen, c, poly, max_iter=T, stop=s, prec="f32")
        out = PB.bp_decode_batch(code, llr, max_iter=T, stop=s, variant=variant)
        for k in ("u_hat", "iters", "ok"):
            assert (out[k].cpu().numpy() == ref[k]).all(), (k, s)
    ref = O.hybrid_batch(h, code.frozen, K, c, poly, T, 4, prec="f32", stop=stop)
    out = PB.HybridDecoder(code, max_iter=T, L=4, stop=stop, variant=variant)(llr)
    assert (out["info"].cpu().numpy() == ref["info"]).all()
    assert (out["used_scl"].cpu().numpy() == ref["used_scl"]).all()


@pytest.mark.parametrize("N,per_cu", [(1024, 8), (2048, 3), (4096, 1)])
@pytest.mark.parametrize("kind", ["plain", "exact", "column"])
@pytest.mark.parametrize("stop", [0, 1, 2])
def test_kernels_of_full_and_partial_chips_agree(N, per_cu, kind, stop):
    """The last batch of the kernels for a chip that is not full and the first one beyond give each frame the same
    results, soft outputs included."""
    if N == 1024 and (kind == "column" or stop == 0):
        per_cu = 6
    B = per_cu * torch.cuda.get_device_properties(0).multi_processor_count
    code = PB.PolarCode(N, N // 2, 16, 0, 2.0)
    g = torch.Generator(device="cuda").manual_seed(N + stop)
    x = PB.polar_encode(code, torch.randint(0, 2, (B + 1, code.K), generator=g, device="cuda", dtype=torch.uint8)).float()
    s2 = O.sigma2(2.0, 0.5)
    llr = (2.0 * (1.0 - 2.0 * x + s2 ** 0.5 * torch.randn(x.shape, generator=g, device="cuda")) / s2).contiguous()
    T = 6
    kw = dict(max_iter=T, stop=stop, soft=True, variant=3, rule=1 if kind == "exact" else 0)
    if kind == "column":
        kw["weights"] = torch.rand((T, 2, code.n), generator=g, device="cuda") * 0.4 + 0.7
    a = PB.bp_decode_batch(code, llr, **kw)
    b = PB.bp_decode_batch(code, llr[:B].contiguous(), **kw)
    for k in ("u_hat", "iters", "ok", "llr_u"):
        assert torch.equal(a[k][:B], b[k]), k
