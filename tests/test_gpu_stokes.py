"""Unfused detection over whole periods of one channel (powers of two up to
64, where a wave holds whole periods) and just past it, Stokes I and IQUV, at
sizes that end inside a wave and inside a block, against 64-bit sums.

Bound: each parameter is a sum of 4 t_int products (8 with the factor two
taken as exact), each step off by at most 2^-24 of the sum of magnitudes:
(4 t_int + 4) 2^-24 sum(|X|^2 + |Y|^2).
"""
import pytest

torch = pytest.importorskip("torch")

from paper_1105_0661_amd import lbf  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("product", [lbf.STOKES_I, lbf.STOKES_IQUV], ids=["I", "IQUV"])
@pytest.mark.parametrize("t_int", [1, 2, 4, 8, 16, 32, 64, 128])
def test_periods(t_int, product):
    for C, B, P in ((1, 1, 1), (3, 5, 7), (2, 9, 131)):
        T = P * t_int
        g = torch.Generator().manual_seed(t_int * 1000 + P)
        y = torch.randn((C, B, T, 2, 2), generator=g) * 100.0
        # the output's neighbours stay as they were
        K = lbf.n_stokes(product)
        buf = torch.full((C * B * P * K + 64,), -7.0, device="cuda")
        out = buf[32:32 + C * B * P * K].view(C, B, P, K)
        lbf.stokes(y.cuda(), product, t_int, 1, out=out)
        d = y.double()
        x, z = torch.view_as_complex(d[..., 0, :].contiguous()), torch.view_as_complex(d[..., 1, :].contiguous())
        xx, zz, xz = x.abs() ** 2, z.abs() ** 2, x * z.conj()
        ref = torch.stack([xx + zz, xx - zz, 2 * xz.real, 2 * xz.imag], -1)[..., :K]
        ref = ref.reshape(C, B, P, t_int, K).sum(3)
        bound = (4 * t_int + 4) * 2.0 ** -24 * (xx + zz).reshape(C, B, P, t_int).sum(3)
        assert ((out.cpu().double() - ref).abs() <= bound[..., None]).all(), (C, B, P)
        assert (buf[:32] == -7.0).all() and (buf[32 + C * B * P * K:] == -7.0).all()
