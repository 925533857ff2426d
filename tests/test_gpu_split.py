"""FP32 results from FP16 pieces (the split worker): station counts at the
edges of its K-steps and of its piece counts, samples over the whole int16
range (residuals beside the FP16 rounding), float samples whose level changes
by any factor, and weights and samples the pieces cannot hold (the exact
path), against 64-bit sums.

Bound: a chain of n FP32 operations on terms t_i is off by at most
n 2^-24 sum |t_i|.  A voltage component sums 2 S products; two roundings per
station for the FP32 chain, plus two units for the weight pieces, give
(4 S + 2) 2^-24 sum |w||x| as the bound that both worker paths keep.
"""
import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1105_0661_amd import lbf  # noqa: E402

pytestmark = pytest.mark.gpu

INT = {"ci8": (torch.int8, 127), "ci16": (torch.int16, 32767)}


def _case(S, C, T, B, xtype, sigma, seed, magnitude=None):
    """Samples [S][C][T][2][2] and FP32 weights [C][B][S][2] on the host."""
    g = torch.Generator().manual_seed(seed)
    dt, lim = INT[xtype]
    x = (torch.randn((S, C, T, 2, 2), generator=g) * sigma).round().clamp(-lim - 1, lim).to(dt)
    a = torch.rand((C, B, S), generator=g, dtype=torch.float64) * (2.0 * math.pi)
    m = torch.ones_like(a) if magnitude is None else magnitude
    return x, torch.stack([m * torch.cos(a), -m * torch.sin(a)], dim=-1).float()


def _voltages64(x, w):
    """[C][B][T][2][2] and the sums of magnitudes, in 64 bits: real products, so that infinities and NaN follow IEEE."""
    xd, wd = x.double().permute(1, 3, 0, 2, 4), w.double()              # [c][p][s][t][ri], [c][b][s][ri]

    def dot(a, b):                                                      # [c][b][s], [c][p][s][t] -> [c][b][t][p]
        return (a[:, :, None, :, None] * b[:, None]).sum(dim=3).permute(0, 1, 3, 2)
    re = dot(wd[..., 0], xd[..., 0]) + dot(-wd[..., 1], xd[..., 1])
    im = dot(wd[..., 0], xd[..., 1]) + dot(wd[..., 1], xd[..., 0])
    mag = dot(wd.abs().sum(-1), xd.abs().sum(-1))
    return torch.stack([re, im], dim=-1), mag[..., None]


def _voltages(x, w):
    return lbf.beamform(x.cuda(), w.cuda().contiguous(), lbf.VOLTAGES).cpu().double()


@pytest.mark.parametrize("xtype", ["ci8", "ci16"])
@pytest.mark.parametrize("S", [1, 8, 9, 16, 17, 32, 33, 40, 41, 56, 57, 64])
def test_stations_at_the_edges(S, xtype):
    B, T = (37, 100) if S % 2 else (70, 64)
    x, w = _case(S, 2, T, B, xtype, 30.0, 100 + S)
    ref, mag = _voltages64(x, w)
    got = _voltages(x, w)
    assert ((got - ref).abs() <= (4 * S + 2) * 2.0 ** -24 * mag).all()
    s = lbf.beamform(x.cuda(), w.cuda(), lbf.STOKES_IQUV, 4).cpu().double()            # [B][K][T'][C]
    p = (ref ** 2).sum(-1)                                                               # [c][b][t][p]
    i64 = p.sum(-1).reshape(2, B, T // 4, 4).sum(-1).permute(1, 2, 0)
    q64 = (p[..., 0] - p[..., 1]).reshape(2, B, T // 4, 4).sum(-1).permute(1, 2, 0)
    # each squared voltage is off by twice its own bound, the eight of a period and the sums by as many roundings
    bound = (2.0 * (4 * S + 2) + 16) * 2.0 ** -24 * (mag[..., 0] ** 2).sum(-1).reshape(2, B, T // 4, 4).sum(-1).permute(1, 2, 0)
    assert ((s[:, 0] - i64).abs() <= bound).all() and ((s[:, 1] - q64).abs() <= bound).all()


@pytest.mark.parametrize("S", [3, 24, 64])
def test_int16_over_its_whole_range(S):
    # residuals in every tile, in one sample of one tile only, and the extreme values themselves
    x, w = _case(S, 2, 200, 130, "ci16", 12000.0, S)
    x[0, 0, :4, 0, 0] = torch.tensor([-32768, 32767, 2049, -2049], dtype=torch.int16)
    quiet = _case(S, 2, 200, 130, "ci16", 40.0, S)[0]
    quiet[S // 2, 1, 70, 1, 1] = 30001
    for v in (x, quiet):
        ref, mag = _voltages64(v, w)
        assert ((_voltages(v, w) - ref).abs() <= (4 * S + 2) * 2.0 ** -24 * mag).all()


@pytest.mark.parametrize("xtype,S,B", [("ci8", 5, 40), ("ci16", 30, 140), ("ci16", 64, 40)])
def test_weights_outside_the_pieces(xtype, S, B):
    # magnitudes over 2^40 between stations, next to beams of ordinary weights and of tiny ones, a zero beam
    g = torch.Generator().manual_seed(S)
    m = torch.ones((2, B, S), dtype=torch.float64)
    m[:, 3] = torch.exp2(-40.0 * torch.rand((2, S), generator=g, dtype=torch.float64))
    m[:, 4] = 2.0 ** -100
    m[:, 5] = 0.0
    m[:, B - 1] = 2.0 ** 90
    x, w = _case(S, 2, 96, B, xtype, 50.0, 7, m)
    ref, mag = _voltages64(x, w)
    assert ((_voltages(x, w) - ref).abs() <= (4 * S + 2) * 2.0 ** -24 * mag).all()
    # infinities and NaN stay what the sums of products make of them, and in their beams
    w[0, 7, 0, 0] = float("inf")
    w[1, 8, S - 1, 1] = float("nan")
    x[0, 0, ::2] = 0
    ref, mag = _voltages64(x, w)
    got = _voltages(x, w)
    assert torch.equal(torch.isnan(got), torch.isnan(ref))
    assert torch.equal(torch.isposinf(got), torch.isposinf(ref)) and torch.equal(torch.isneginf(got), torch.isneginf(ref))
    fin = torch.isfinite(ref)
    err = torch.where(fin, got - ref, torch.zeros_like(ref)).abs()
    assert (err <= (4 * S + 2) * 2.0 ** -24 * torch.where(torch.isfinite(mag), mag, torch.zeros_like(mag))).all()


def _float_case(S, C, T, B, seed):
    g = torch.Generator().manual_seed(seed)
    x = torch.randn((S, C, T, 2, 2), generator=g) * 1000.0
    a = torch.rand((C, B, S), generator=g, dtype=torch.float64) * (2.0 * math.pi)
    return x, torch.stack([torch.cos(a), -torch.sin(a)], dim=-1).float()


@pytest.mark.parametrize("S", [19, 20, 32, 33, 40, 41, 48, 49, 57, 64])
def test_float_samples_at_the_edges(S):
    B, T = (37, 100) if S % 2 else (130, 72)
    x, w = _float_case(S, 2, T, B, S)
    ref, mag = _voltages64(x, w)
    assert ((_voltages(x, w) - ref).abs() <= (4 * S + 2) * 2.0 ** -24 * mag).all()
    s = lbf.beamform(x.cuda(), w.cuda(), lbf.STOKES_I, 4).cpu().double()[:, 0]
    i64 = (ref ** 2).sum((-1, -2)).reshape(2, B, T // 4, 4).sum(-1).permute(1, 2, 0)
    bound = (2.0 * (4 * S + 2) + 16) * 2.0 ** -24 * (mag[..., 0] ** 2).sum(-1).reshape(2, B, T // 4, 4).sum(-1).permute(1, 2, 0)
    assert ((s - i64).abs() <= bound).all()


@pytest.mark.parametrize("S,T", [(20, 1100), (64, 400)])
def test_float_samples_of_any_level(S, T):
    # levels from 2^-60 to 2^60 in turn, inside tiles and from tile to tile; a
    # burst in one sample, one weak station, a dead one, one dead polarisation,
    # silence over whole tiles, an item that begins with silence
    x, w = _float_case(S, 3, T, 70, S)
    level = torch.ones(T)
    for i, e in enumerate((0, 60, -60, 12, -9, 20)):
        level[i * 50:i * 50 + 50] = 2.0 ** e
    x[:, 0] *= level[None, :, None, None]
    x[:, 1, T // 2, 0, 1] *= 2.0 ** 30
    x[3] *= 2.0 ** -15
    x[4] = 0.0
    x[5, :, :, 1] = 0.0
    x[:, 2, :130] = 0.0
    x[:, 2, 200:210] *= 2.0 ** -110
    ref, mag = _voltages64(x, w)
    assert ((_voltages(x, w) - ref).abs() <= (4 * S + 2) * 2.0 ** -24 * mag + 2.0 ** -126).all()


@pytest.mark.parametrize("S", [24, 64])
def test_float_samples_not_finite(S):
    x, w = _float_case(S, 2, 160, 40, S)
    x[1, 0, 3, 0, 0] = float("inf")
    x[S - 1, 0, 70, 1, 1] = float("nan")
    x[2, 1, 159, 1, 0] = -float("inf")
    x[0, 1, 100] = 3.0e38
    ref, mag = _voltages64(x, w)
    got = _voltages(x, w)
    over = mag > 1.0e38                                     # where FP32 sums may overflow on the way
    fin = torch.isfinite(ref) & ~over.expand_as(ref)
    assert torch.equal(torch.isnan(got)[~over.expand_as(ref)], torch.isnan(ref)[~over.expand_as(ref)])
    assert not torch.isfinite(got)[~torch.isfinite(ref)].any()
    assert ((got - ref).abs() <= (4 * S + 2) * 2.0 ** -24 * mag)[fin].all()


def test_unit_weights_are_exact():
    x = torch.randint(-32768, 32768, (1, 3, 70, 2, 2), dtype=torch.int16)
    w = torch.zeros((3, 5, 1, 2))
    w[..., 0] = 1.0
    y = _voltages(x, w)
    assert torch.equal(y, x.double().permute(1, 0, 2, 3, 4).expand(3, 5, 70, 2, 2))
    assert np.isfinite(y.numpy()).all()
