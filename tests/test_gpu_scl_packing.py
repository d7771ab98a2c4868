"""Several frames per wavefront in the list decoder: batches large enough that
wavefronts take two or more frames, with a remainder in the last one, against
the same frames decoded in batches small enough to take one each, and against
the oracle at small block lengths."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_1609_09358_amd import binding as PB
from paper_1609_09358_amd import inputs

pytestmark = pytest.mark.gpu

POLY = {0: 0, 8: 0x07, 16: 0x1021, 24: 0x864CFB}
KEYS = ("u_hat", "crc_ok", "pm")


def cus():
    return torch.cuda.get_device_properties(0).multi_processor_count


def llrs(code, B, ebn0, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    bits = torch.randint(0, 2, (B, code.K), generator=g, device="cuda", dtype=torch.uint8)
    x = PB.polar_encode(code, bits).float()
    s2 = O.sigma2(ebn0, code.K / code.N)
    return (2.0 * (1.0 - 2.0 * x + s2 ** 0.5 * torch.randn(x.shape, generator=g, device="cuda")) / s2).contiguous()


# frames per wavefront: 2 with the first count, more (as many as lists fit) with the second
@pytest.mark.parametrize("N,c", [(8, 0), (16, 0), (32, 8), (64, 8), (128, 8), (256, 16), (512, 16), (1024, 24),
                                 (2048, 16), (4096, 16)])
@pytest.mark.parametrize("L", [1, 2, 4, 8, 16, 32])
@pytest.mark.parametrize("per_cu,extra", [(8, 3), (56, 5)])
def test_packed_equals_single(N, c, L, per_cu, extra):
    B = per_cu * cus() + extra
    if N * B * L > 1 << 30:
        B = 8 * cus() + extra  # two frames each
    code = PB.PolarCode(N, N // 2 - (c if N <= 32 else 0), c, 0, 2.0, da_bits=N // 8)
    llr = llrs(code, B, 1.5, N + L)
    # a few exact ties at every list boundary: LLRs on a coarse grid
    llr[: B // 4] = torch.round(llr[: B // 4] * 2) / 2
    all_ = PB.scl_decode_batch(code, llr, L)
    step = 4 * cus()
    for f in range(0, B, step):
        one = PB.scl_decode_batch(code, llr[f: f + step].contiguous(), L)
        for k in KEYS:
            assert torch.equal(all_[k][f: f + step], one[k]), (k, f)


@pytest.mark.parametrize("N,K,c,L", [(16, 8, 0, 8), (64, 32, 8, 32), (128, 64, 8, 8), (256, 100, 16, 16)])
def test_packed_matches_oracle(N, K, c, L):
    B = 24 * cus() + 1
    code = PB.PolarCode(N, K, c, 0, 2.0)
    llr = llrs(code, B, 1.5, 3)
    out = {k: v.cpu().numpy() for k, v in PB.scl_decode_batch(code, llr, L).items()}
    rows = np.r_[0:20, B // 2: B // 2 + 20, B - 20: B]
    ref = O.scl_batch(llr.cpu().numpy()[rows], code.frozen, L, c, POLY[c], prec="f32")
    assert np.array_equal(out["u_hat"][rows], ref["u_hat"])
    assert np.array_equal(out["crc_ok"][rows], ref["crc_ok"])
    assert np.array_equal(out["pm"][rows], ref["pm"].astype(np.float32))


def test_packed_frame_ids_and_ranking_modes():
    N, K, c, L, rows = 128, 64, 8, 8, 30 * 256
    code = PB.PolarCode(N, K, c, 0, 2.0)
    llr = llrs(code, rows, 1.5, 11)
    ids = torch.randperm(rows, device="cuda", generator=torch.Generator(device="cuda").manual_seed(1))[: rows - 77]
    ref = PB.scl_decode_batch(code, llr, L)
    try:
        for mode in (0, 1, 2, 3):
            PB.polar_set_scl_ranking(mode)
            out = PB.scl_decode_batch(code, llr, L, frame_ids=ids.to(torch.int32).contiguous())
            for k in KEYS:
                assert torch.equal(out[k][ids], ref[k][ids]), (mode, k)
            untouched = torch.ones(rows, dtype=torch.bool, device="cuda")
            untouched[ids] = False
            assert int(out["u_hat"][untouched].sum()) == 0
    finally:
        PB.polar_set_scl_ranking(0)


def test_infinite_and_huge_llrs_stay_in_bounds():
    """Infinite and very large LLRs: the decode ends, packed and single agree where the arithmetic has no NaN."""
    N, K, c, L = 64, 32, 8, 8
    B = 20 * cus()
    code = PB.PolarCode(N, K, c, 0, 2.0)
    llr = llrs(code, B, 1.5, 2)
    llr[::3] *= 1e30
    out = PB.scl_decode_batch(code, llr, L)
    one = PB.scl_decode_batch(code, llr[: 4 * cus()].contiguous(), L)
    for k in KEYS:
        assert torch.equal(out[k][: 4 * cus()], one[k])
    llr[::5, ::7] = float("inf")
    out = PB.scl_decode_batch(code, llr, L)
    torch.cuda.synchronize()
    assert int((out["u_hat"] > 1).sum()) == 0


def test_mixed_queue_of_several_codes_packs_per_code():
    """More failed frames than wavefronts in a plan whose codes share one block length."""
    codes = [PB.PolarCode(64, K, 8, 0, 2.0) for K in (16, 32, 44)]
    B = 30 * cus() + 7
    rng = np.random.default_rng(4)
    cf = rng.integers(0, 3, B).astype(np.int32)
    plan = PB.MixedPlan(codes, B, max_iter=2, L=8)
    llr_off, out_off, nl, nk = plan.layout(cf)
    llr = torch.empty(nl, device="cuda")
    rows = [llrs(code, B, 1.0, 20 + i) for i, code in enumerate(codes)]
    idx = torch.from_numpy(cf.astype(np.int64)).cuda()
    allr = torch.stack(rows)[idx, torch.arange(B, device="cuda")]
    llr.copy_(allr.reshape(-1))
    info = torch.zeros(nk, dtype=torch.uint8, device="cuda")
    used = torch.zeros(B, dtype=torch.uint8, device="cuda")
    stats = torch.zeros(8, dtype=torch.int64, device="cuda")
    plan(llr, torch.from_numpy(cf).cuda(), torch.from_numpy(llr_off).cuda(), torch.from_numpy(out_off).cuda(), info,
         used, stats, graph=True)
    info, used = info.cpu().numpy(), used.cpu().numpy()
    assert int(used.sum()) > 8 * cus()
    for c, code in enumerate(codes):
        sel = np.flatnonzero(cf == c)
        dec = PB.HybridDecoder(code, max_iter=2, L=8)
        st = dec(rows[c][torch.from_numpy(sel).cuda()].contiguous())
        gi, gu = st["info"].cpu().numpy(), st["used_scl"].cpu().numpy()
        assert np.array_equal(used[sel], gu)
        got = np.stack([info[out_off[f]: out_off[f] + code.K] for f in sel])
        assert np.array_equal(got, gi)


@pytest.mark.parametrize("N,c", [(32, 8), (256, 16)])
@pytest.mark.parametrize("L", [8, 32])
@pytest.mark.parametrize("per_cu,extra", [(1, 3), (8, 3), (16, 5), (20, 1), (56, 5)])
def test_ranking_modes_agree(N, c, L, per_cu, extra):
    """Counting and threshold selection against the network with one to four frames per wavefront, ties included."""
    B = per_cu * cus() + extra
    code = PB.PolarCode(N, N // 2 - (c if N <= 32 else 0), c, 0, 2.0, da_bits=N // 8)
    llr = llrs(code, B, 1.5, N + L)
    llr[: B // 2] = torch.round(llr[: B // 2])
    llr[: B // 8] = torch.sign(llr[: B // 8])
    ref = PB.scl_decode_batch(code, llr, L)
    try:
        for mode in (1, 3):
            PB.polar_set_scl_ranking(mode)
            out = PB.scl_decode_batch(code, llr, L)
            for k in KEYS:
                assert torch.equal(out[k], ref[k]), (mode, k)
    finally:
        PB.polar_set_scl_ranking(0)


@pytest.mark.parametrize("made,used", [(0, 3), (0, 1), (3, 0), (1, 3)])
def test_ranking_mode_changed_after_a_mixed_plan(made, used):
    """A mixed plan keeps the selection it was made with."""
    code = PB.PolarCode(64, 32, 8, 0, 2.0)
    B = 30 * cus() + 7
    llr = llrs(code, B, 1.0, 9)
    cf = np.zeros(B, np.int32)
    got = []
    try:
        for m in ((0, 0), (made, used)):
            PB.polar_set_scl_ranking(m[0])
            plan = PB.MixedPlan([code], B, max_iter=2, L=32)
            PB.polar_set_scl_ranking(m[1])
            llr_off, out_off, _, nk = plan.layout(cf)
            info = torch.zeros(nk, dtype=torch.uint8, device="cuda")
            plan(llr.reshape(-1), torch.from_numpy(cf).cuda(), torch.from_numpy(llr_off).cuda(),
                 torch.from_numpy(out_off).cuda(), info)
            got.append(info)
    finally:
        PB.polar_set_scl_ranking(0)
    assert torch.equal(got[0], got[1])


@pytest.mark.parametrize("N,aided,per_cu", [(256, True, 8), (512, False, 10), (512, True, 12), (1024, False, 10),
                                            (1024, True, 12), (2048, True, 8), (4096, False, 12)])
@pytest.mark.parametrize("extra", [0, 1])
def test_list_of_32_at_the_second_frame(N, aided, per_cu, extra):
    """The last batch of one frame per wavefront and the first of two at L = 32, by block length and decision aiding,
    against small batches."""
    B = per_cu * cus() + extra
    code = PB.PolarCode(N, N // 2, 16, 0, 2.0, da_bits=N // 4 if aided else 0)
    llr = llrs(code, B, 1.5, N)
    all_ = PB.scl_decode_batch(code, llr, 32)
    for f in range(0, B, 4 * cus()):
        one = PB.scl_decode_batch(code, llr[f: f + 4 * cus()].contiguous(), 32)
        for k in KEYS:
            assert torch.equal(all_[k][f: f + 4 * cus()], one[k]), (k, f)


@pytest.mark.parametrize("per_cu", [13, 63, 65, 257])
def test_pipelined_lists_of_32_by_batch_size(per_cu):
    """Pipelined batches on either side of the sizes at which the list decoder beside BP packs frames sooner."""
    B = per_cu * cus() + 1
    code = PB.PolarCode(128, 64, 16, 0, 2.0, da_bits=40)
    ll = [llrs(code, B, e, 30 + j) for j, e in enumerate((1.0, 3.0, 0.0))]
    stats = torch.zeros(8, dtype=torch.int64, device="cuda")
    outs = PB.HybridPipeline(code, max_iter=5, L=32, stop=2)(ll, stats=stats, want_used=True)
    st = torch.zeros(8, dtype=torch.int64, device="cuda")
    for o, x in zip(outs, ll):
        ref = PB.HybridDecoder(code, max_iter=5, L=32, stop=2)(x, stats=st)
        assert torch.equal(o["info"], ref["info"]) and torch.equal(o["used_scl"], ref["used_scl"])
    assert torch.equal(stats, st) and int(st[2]) > 8 * cus()


@pytest.mark.parametrize("N,K,c", [(8, 4, 0), (16, 9, 0), (32, 20, 8), (128, 64, 8), (256, 128, 16)])
@pytest.mark.parametrize("scale", [0.0, 1.0, 3e38])
def test_list_of_one_matches_oracle(N, K, c, scale):
    """A list of one, which decides without a ranking, with LLRs of three values: metrics that tie, LLRs of zero,
    metrics too large for a penalty to change."""
    B = 300
    code = PB.PolarCode(N, K, c, 0, 2.0, da_bits=K // 4)
    g = torch.Generator(device="cuda").manual_seed(N)
    llr = torch.randint(-1, 2, (B, N), generator=g, device="cuda").float()
    if scale > 1:
        llr[:, ::3] *= 1e9
    elif scale == 0:
        llr[: B // 2] = 0.0
    out = {k: v.cpu().numpy() for k, v in PB.scl_decode_batch(code, llr.contiguous(), 1).items()}
    ref = O.scl_batch(llr.cpu().numpy(), code.frozen, 1, c, POLY[c], prec="f32", da=code.decision_aided)
    for k in KEYS:
        assert np.array_equal(out[k], ref[k].astype(out[k].dtype)), k


# A hybrid plans for its batch, whose frames may share wavefronts, while a launch
# with few frames left gives each its own: the same words as a plan made for those alone
@pytest.mark.parametrize("N,c,L", [(64, 8, 8), (1024, 24, 8), (1024, 24, 32), (4096, 16, 32)])
@pytest.mark.parametrize("failing", [1, 3, 700])
def test_shared_plan_with_one_frame_each(N, c, L, failing):
    B = 24 * cus() + 1
    code = PB.PolarCode(N, N // 2, c, 0, 2.0, da_bits=N // 8)
    llr = llrs(code, B, 9.0, N + L)
    bad = torch.randperm(B, device="cuda", generator=torch.Generator(device="cuda").manual_seed(L))[:failing]
    llr[bad] = llrs(code, failing, -6.0, N - L)
    bp = PB.bp_decode_batch(code, llr, max_iter=20, stop=2)
    left = torch.nonzero(bp["ok"] == 0).flatten()
    assert 0 < left.numel() <= 4 * cus()
    out = PB.HybridDecoder(code, max_iter=20, L=L, stop=2)(llr)
    one = PB.HybridDecoder(code, max_iter=20, L=L, stop=2)(llr[left].contiguous())
    assert torch.equal(out["info"][left], one["info"])
    assert torch.equal(out["used_scl"], (bp["ok"] == 0).to(torch.uint8))
    assert bool(one["used_scl"].all())


# Threshold selection of one frame a wavefront ends its search early: metrics far apart, close together,
# equal (few distinct values, all zero) and beyond the largest float
@pytest.mark.parametrize("L", [8, 32])
@pytest.mark.parametrize("scale,step", [(1.0, 0), (1.0, 0.5), (1.0, 4.0), (0.0, 0), (1e-30, 0), (1e37, 0), (3e38, 0)])
def test_threshold_of_one_frame_equals_network(L, scale, step):
    code = PB.PolarCode(256, 128, 8, 0, 2.0)
    llr = llrs(code, 9, 0.0, L)
    if step:
        llr = torch.round(llr / step) * step
    llr = torch.clamp(llr * scale, -3.4e38, 3.4e38)
    try:
        PB.polar_set_scl_ranking(2)
        ref = PB.scl_decode_batch(code, llr, L)
        PB.polar_set_scl_ranking(3)
        out = PB.scl_decode_batch(code, llr, L)
    finally:
        PB.polar_set_scl_ranking(0)
    for k in KEYS:
        assert torch.equal(out[k], ref[k]), k
