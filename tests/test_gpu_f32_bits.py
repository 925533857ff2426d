"""FP32 blocks hold every bit of their weights and samples: what one live
station leaves of a product that FP32 holds exactly is that product."""
import math

import pytest

torch = pytest.importorskip("torch")

from paper_1105_0661_amd import lbf  # noqa: E402

pytestmark = pytest.mark.gpu

X = {"ci8": torch.int8, "ci16": torch.int16, "cf32": torch.float32}


def _phases(shape, seed, amplitude=1.0):
    g = torch.Generator().manual_seed(seed)
    a = torch.rand(shape, generator=g, dtype=torch.float64) * (2.0 * math.pi)
    return torch.stack([torch.cos(a), -torch.sin(a)], dim=-1).mul(amplitude).float()


def _voltages(x, w):
    return lbf.beamform(x.cuda(), w.cuda().contiguous(), lbf.VOLTAGES).cpu()          # [C][B][T][2][2]


@pytest.mark.parametrize("xt", ["ci8", "ci16", "cf32"])
@pytest.mark.parametrize("S", [1, 16, 17, 32, 40, 64])
def test_a_weight_keeps_its_24_bits(S, xt):
    # station s sends 2^k in one component of its own sample, all else is
    # silent: each voltage is one weight component times 2^k, exactly
    C, B = 2, 70
    x = torch.zeros((S, C, S, 2, 2), dtype=X[xt])
    k = torch.arange(S) % 7
    for s in range(S):
        x[s, :, s, 0, 0] = 2.0 ** k[s]
        x[s, :, s, 1, 1] = -(2.0 ** k[s])
    w = _phases((C, B, S), S, 0.7)
    got = _voltages(x, w)
    p = (2.0 ** k)[None, None, :, None]
    assert torch.equal(got[:, :, :, 0], w * p)
    assert torch.equal(got[:, :, :, 1], torch.stack([w[..., 1], -w[..., 0]], dim=-1) * p)


@pytest.mark.parametrize("S", [1, 16, 20, 40, 64])
def test_a_float_sample_keeps_its_24_bits(S):
    # one station's weight is 2^k, the others' are zero: each voltage is that
    # station's sample times 2^k, exactly
    C, T = 2, 70
    g = torch.Generator().manual_seed(S)
    x = torch.randn((S, C, T, 2, 2), generator=g) * 100.0
    w = torch.zeros((C, S, S, 2))
    k = torch.arange(S) % 5
    for s in range(S):
        w[:, s, s, 0] = 2.0 ** k[s]
    got = _voltages(x, w)                                                               # beam s: station s
    assert torch.equal(got, x.permute(1, 0, 2, 3, 4) * (2.0 ** k)[None, :, None, None, None])


def _levels(S, C, T, seed):
    """Float samples whose level jumps between 32-sample tiles by factors beyond any shared exponent."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.randn((S, C, T, 2, 2), generator=g, device="cuda")
    e = torch.tensor([0, 0, 0, 0, 9, 9, -14, 3, 3, 20, -3, -3], device="cuda").repeat_interleave(32)
    x.mul_(torch.exp2(e.float()).repeat((T + e.numel() - 1) // e.numel())[:T, None, None])
    x[S // 2].mul_(2.0 ** -13)
    return x


@pytest.mark.parametrize("S,product,t_int", [(20, lbf.STOKES_IQUV, 1), (64, lbf.STOKES_IQUV, 4)])
def test_float_results_do_not_depend_on_the_passes(S, product, t_int):
    # the whole block's staging is larger than the 64 MiB scratch: passes of
    # fewer channels, whose items are cut into other time segments
    C, T, B = 256, 768, 128
    fp = lbf.block_footprint(S, C, T, B, lbf.CF32, lbf.F32, product, t_int)
    assert fp.staging_bytes > (64 << 20)
    x = _levels(S, C, T, S)
    w = _phases((C, B, S), S).cuda()
    assert torch.equal(lbf.beamform(x, w, product, t_int), lbf.beamform_noalloc(x, w, product, t_int))


def test_a_channel_does_not_see_its_neighbour():
    # a ragged last tile reads on into the next channel: its level, or NaN there, changes no bit
    S, T, B = 32, 75, 40
    x = _levels(S, 2, T, 3).cpu()
    w = _phases((2, B, S), 3)
    want = _voltages(x, w)[0]
    for v in (2.0 ** 30, 2.0 ** -30, float("nan")):
        y = x.clone()
        y[:, 1] *= v
        assert torch.equal(_voltages(y, w)[0], want)


def _check_voltages64(x, w, got, chans):
    """Voltages of some channels against 64-bit sums: 2 S roundings of a chain of sums, and two more."""
    S = x.shape[0]
    xs = x[:, chans].double().permute(1, 0, 2, 3, 4)                                      # [c][s][t][p][ri]
    ws = w[chans].double()                                                                # [c][b][s][ri]
    y = torch.einsum("cbs,cstp->cbtp", torch.view_as_complex(ws), torch.view_as_complex(xs.contiguous()))
    mag = torch.einsum("cbs,cstp->cbtp", ws.abs().sum(-1), xs.abs().sum(-1))[..., None]
    assert ((got[chans].double() - torch.view_as_real(y)).abs() <= (2 * S + 2) * 2.0 ** -24 * mag).all()


@pytest.mark.parametrize("S,xt,B", [(5, "ci16", 70), (17, "ci8", 40), (40, "ci16", 10), (44, "ci8", 130), (64, "ci16", 70)])
def test_weights_far_apart_in_long_items(S, xt, B):
    # 25 tiles in items of 24 and 1: beams whose stations differ by 2^20 in
    # every beam of a channel, in one beam of it, in none
    C, T = 260, 779
    g = torch.Generator().manual_seed(S)
    x = (torch.randn((S, C, T, 2, 2), generator=g) * 30.0).round().clamp(-127, 127).to(X[xt])
    x[S - 1, :, ::3] = 0
    w = _phases((C, B, S), S)
    w[0::3, :, S // 2] *= 2.0 ** -20
    w[1::3, 3, 0] *= 2.0 ** 20
    _check_voltages64(x, w, _voltages(x, w), [0, 1, 2, C - 2, C - 1])


def _rms(S, xt, live, weights, seed):
    """Relative rms error of the voltages against 64 bits, and what a chain of FP32 products and sums leaves."""
    C, T, B = 4, 256, 48
    g = torch.Generator().manual_seed(seed)
    x = (torch.randn((S, C, T, 2, 2), generator=g) * 20.0).round().clamp(-127, 127).to(X[xt])
    w = _phases((C, B, S), seed)
    if weights == "equal":
        w = (torch.rand((C, B, 1, 1), generator=g) + 0.5) * torch.tensor([1.0, 0.0]).expand_as(w)
    mask = torch.zeros(S)
    mask[live] = 1.0
    w = w * mask[:, None]
    xs = x.float().permute(1, 0, 2, 3, 4)
    y = torch.view_as_real(torch.einsum("cbs,cstp->cbtp", torch.view_as_complex(w.double()),
                                        torch.view_as_complex(xs.double().contiguous())))
    re, im = torch.zeros(y.shape[:-1]), torch.zeros(y.shape[:-1])
    for s in live:                                                # products and sums each rounded once
        wr, wi = w[:, :, s, 0, None, None], w[:, :, s, 1, None, None]
        xr, xi = xs[:, None, s, ..., 0], xs[:, None, s, ..., 1]
        re = (re.double() + wr.double() * xr.double()).float()
        re = (re.double() - wi.double() * xi.double()).float()
        im = (im.double() + wi.double() * xr.double()).float()
        im = (im.double() + wr.double() * xi.double()).float()
    chain = torch.stack([re, im], dim=-1).double()
    return ((_voltages(x, w).double() - y).norm() / y.norm()).item(), ((chain - y).norm() / y.norm()).item()


@pytest.mark.parametrize("xt", ["ci8", "ci16"])
@pytest.mark.parametrize("weights", ["phases", "equal"])
@pytest.mark.parametrize("S,live", [(1, [0]), (3, [0, 1, 2]), (17, list(range(17))), (64, [9]), (64, [3, 59]),
                                    (64, [5, 21, 37]), (64, list(range(0, 64, 8))), (64, list(range(8))), (64, list(range(64)))],
                         ids=lambda v: str(v) if isinstance(v, int) else "%d live" % len(v))
def test_no_further_off_than_a_chain_of_fp32_sums(S, live, weights, xt):
    # over 98304 values; 2 % for the spread of an rms over them
    got, chain = _rms(S, xt, live, weights, 7 * S + len(live))
    assert got <= 1.02 * chain
