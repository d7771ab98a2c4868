"""Encoder and channel kernels at the edges of their layouts: every block
length, batches that leave a wavefront's last frames empty or walk the grid more
than once, rates from one bit to all positions, rows and buffers off their
natural alignment."""
import ctypes as C

import numpy as np
import pytest
import torch

import oracle as O
from paper_1609_09358_amd import binding as PB
from paper_1609_09358_amd import inputs

pytestmark = pytest.mark.gpu

POLY = {0: 0, 8: 0x07, 16: 0x1021, 24: 0x864CFB}


def at(nbytes, shift, dtype=torch.uint8):
    """A device buffer whose first element lies `shift` elements past a 256-byte boundary, 64 spare elements after."""
    t = torch.full((nbytes + shift + 64,), 7, dtype=dtype, device="cuda")
    assert t.data_ptr() % 256 == 0
    return t, t[shift: shift + nbytes]


@pytest.mark.parametrize("N", [8, 16, 32, 64, 128, 256, 512, 1024, 2048, 4096])
@pytest.mark.parametrize("shift", [0, 3])
def test_encode_every_layout(N, shift):
    fpw = max(1, 1024 // N) if N >= 16 else 64
    for K, c, B in ((1, 0, 1), (N - 1, 0, 2 * fpw + 1), (N // 2 - 1 if N > 16 else 3, 0, 67),
                    (N - 24 if N >= 64 else N // 2, 24 if N >= 64 else 0, 130), (N // 4 + 1, 8 if N >= 32 else 0, 300)):
        code = PB.PolarCode(N, K, c, 0, 2.0)
        info = inputs.info_bits(B, K, seed=N + K)
        u_ref, x_ref = O.encode_batch(info, K, c, POLY[c], code.frozen)
        whole_i, di = at(B * K, shift)
        di.copy_(torch.from_numpy(info.reshape(-1)).cuda())
        whole_u, u = at(B * N, shift)
        whole_x, x = at(B * N, shift)
        s = C.c_void_p(torch.cuda.current_stream().cuda_stream)
        p = [C.c_void_p(t.data_ptr()) for t in (di, u, x)]
        PB._check(PB.lib().polar_encode(code.handle, p[0], B, p[1], p[2], s))
        torch.cuda.synchronize()
        assert np.array_equal(u.cpu().numpy().reshape(B, N), u_ref), (N, K, c, B)
        assert np.array_equal(x.cpu().numpy().reshape(B, N), x_ref), (N, K, c, B)
        for whole in (whole_u, whole_x):  # nothing outside the rows
            assert int((whole[:shift] != 7).sum()) == 0 and int((whole[shift + B * N:] != 7).sum()) == 0


def test_encode_walks_the_grid():
    N, K, c, B = 128, 61, 8, 256 * 8 * 4 * 8 + 13  # more frames than resident wavefronts hold
    code = PB.PolarCode(N, K, c, 0, 2.0)
    info = inputs.info_bits(B, K, seed=5)
    x = PB.polar_encode(code, torch.from_numpy(info).cuda()).cpu().numpy()
    assert np.array_equal(x, O.encode_batch(info, K, c, POLY[c], code.frozen)[1])


@pytest.mark.parametrize("N,B", [(1, 5), (2, 9), (4, 3), (8, 33), (12, 7), (1024, 3), (4096, 2)])
def test_channel_vector_form_equals_the_general_one(N, B):
    """The four-element form gives the bits of the one-element form (reached with buffers off its alignment)."""
    xb = torch.from_numpy(inputs.info_bits(B, N, seed=2)).cuda()
    z = torch.from_numpy(inputs.noise(B, N, seed=2, dtype=np.float32)).cuda()
    s2 = torch.linspace(0.05, 3.0, B, device="cuda")
    out = PB.polar_channel_awgn(xb, z, s2)
    _, zo = at(B * N, 1, torch.float32)
    zo.copy_(z.reshape(-1))
    _, lo = at(B * N, 1, torch.float32)
    s = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    PB._check(PB.lib().polar_channel_awgn(C.c_void_p(xb.data_ptr()), C.c_void_p(zo.data_ptr()),
                                          C.c_void_p(s2.data_ptr()), B, N, C.c_void_p(lo.data_ptr()), s))
    torch.cuda.synchronize()
    assert torch.equal(out.reshape(-1), lo)
