"""Voltages of the FP16/BF16 worker, whose stores are turned through LDS so that
lanes write whole cache lines: sizes that end inside a turn of 8 samples, a
tile and a beam group, every item shape, against 64-bit sums.

int8 samples and the weights as given are exact operands and their products
exact in FP32, so a component is off by the roundings of its 2 S additions:
(2 S + 2) 2^-24 sum |w||x|.
"""
import pytest

torch = pytest.importorskip("torch")

from paper_1105_0661_amd import lbf  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture
def streams():
    yield lbf.set_tile_streams
    lbf.set_tile_streams(0)


@pytest.mark.parametrize("ns", [0, 1, 2, 4])
@pytest.mark.parametrize("S,T,B", [(1, 1, 1), (8, 7, 33), (40, 70, 8), (52, 70, 16), (64, 70, 9), (33, 100, 129), (64, 41, 300), (20, 800, 65)])
@pytest.mark.parametrize("xt", [torch.int8, torch.int16], ids=["ci8", "ci16"])
@pytest.mark.parametrize("wt", [torch.float16, torch.bfloat16], ids=["f16", "bf16"])
def test_stores(S, T, B, xt, wt, ns, streams):
    C = 3
    g = torch.Generator().manual_seed(S + B)
    x = torch.randint(-128, 128, (S, C, T, 2, 2), generator=g).to(xt)
    w = torch.randn((C, B, S, 2), generator=g).to(wt)
    buf = torch.full((C * B * T * 4 + 128,), -7.0, device="cuda")
    out = buf[64:64 + C * B * T * 4].view(C, B, T, 2, 2)
    streams(ns)
    lbf.beamform(x.cuda(), w.cuda(), lbf.VOLTAGES, out=out)
    xd, wd = torch.view_as_complex(x.double().contiguous()), torch.view_as_complex(w.double().contiguous())
    xs = xd.permute(1, 0, 2, 3).reshape(C, S, T * 2).contiguous()
    ref = torch.view_as_real(torch.bmm(wd, xs)).reshape(C, B, T, 2, 2)
    xa = x.double().abs().sum(-1).permute(1, 0, 2, 3).reshape(C, S, T * 2).contiguous()
    mag = torch.bmm(w.double().abs().sum(-1), xa).reshape(C, B, T, 2, 1)
    assert ((out.cpu().double() - ref).abs() <= (2 * S + 2) * 2.0 ** -24 * mag).all()
    assert (buf[:64] == -7.0).all() and (buf[-64:] == -7.0).all()
