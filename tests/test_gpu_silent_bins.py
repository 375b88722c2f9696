"""Groups of fold samples that cross one bin edge: each bin takes the sum of its
own samples.  Signals gated on for whole bins leave the others empty, whatever
the signal before the edge; a power beyond float16 counts in neither sum of its
group but its own."""
import numpy as np
import pytest

import oracle as O
import synth
from gpu_helpers import BW, EPS_HALF, F0, gpu_run, oracle_run
from test_real_path import gpu_real_run, oracle_real_run

pytestmark = pytest.mark.gpu

FS = BW * 1e6
UNIT = 2.0 ** -16  # of the fixed-point sums


def gated(seed, nsamp, nbins, per_bin):
    """Noise in two of every five bins, bins of per_bin samples: pairs of int8."""
    b = np.floor(np.arange(nsamp) / per_bin).astype(np.int64) % nbins
    on = b % 5 < 2
    return (synth.white_stream_int8(seed, nsamp).reshape(nsamp, 2) * on[:, None].astype(np.int8)).reshape(-1)


def check(prof, oprof, cnts, form):
    """Every bin: float32 sums, or float16 rounding (the silent samples then hold
    what the rounding of the others leaves: (EPS_HALF / 2)^2 of their power)."""
    assert prof.shape == oprof.shape
    mean = oprof.max()
    for p, w, m in zip(prof.astype(np.float64), oprof, cnts):
        if form == "fp32":
            tol = 1e-5 * w + UNIT
        else:
            tol = (1e-4 + 5 * EPS_HALF / np.sqrt(np.maximum(m, 1))) * w + 1e-4 * mean
        worst = int(np.argmax(np.abs(p - w) - tol))
        assert abs(p[worst] - w[worst]) <= tol[worst], (worst, p[worst], w[worst], m[worst])


# histograms in LDS and in global memory, sub-integrations that begin in silence,
# tiles of 16 and of 32 columns (2^20)
@pytest.mark.parametrize("form", ["fp32", "mixed_valu", "half", "mixed"])
@pytest.mark.parametrize("log2n,nbins,nsamp,subint", [(12, 64, 400_003, 0), (12, 64, 400_003, 65_539),
                                                      (12, 16_384, 1_300_003, 0), (20, 64, 4_000_003, 0)])
def test_empty_bins_stay_empty(log2n, nbins, nsamp, subint, form):
    per_bin = 25.6
    iq = gated(91, nsamp, nbins, per_bin)
    period = nbins * per_bin / FS
    oprof, _, r = oracle_run(iq, 0.0, 1 << log2n, nbins, period, subint=subint)
    assert (oprof < UNIT).sum() > 0.5 * oprof.size
    prof, _ = gpu_run(iq, 0.0, 1 << log2n, nbins, period, subint=subint, precision=form)
    check(prof, oprof, r["cnts"], form)


@pytest.mark.parametrize("form", ["fp32", "mixed_valu"])
@pytest.mark.parametrize("nbins,nsamp", [(64, 800_006), (16_384, 2_600_006)])
def test_empty_bins_stay_empty_real(nbins, nsamp, form):
    per_bin = 51.2
    raw = gated(92, nsamp, nbins, per_bin)
    period = nbins * per_bin / (2 * FS)
    oprof, _, r = oracle_real_run(raw, 0.0, 1 << 13, nbins, period, "lsb")
    assert (oprof < UNIT).sum() > 0.5 * oprof.size
    prof, _ = gpu_real_run(raw, 0.0, 1 << 13, nbins, period, "lsb", precision=form)
    check(prof, oprof, r["cnts"], form)


def matched(n, dm, at):
    """A strong int8 block of n samples whose dedispersed signal is one peak at sample
    `at` (whole or half) of the block, as a tensor of pairs: the conjugate filter's
    response (of modulus 1 / sqrt(0.9 n) where 0.9 n is smear), scaled until it clips."""
    import torch
    f = torch.fft.fftfreq(n, dtype=torch.float64, device="cuda") * BW
    turns = dm / (2.41e-10 * F0 * F0) * (f * f) / (F0 + f)
    turns -= (torch.arange(n, device="cuda") * round(2 * at)).remainder_(2 * n).double() / (2 * n)
    x = torch.fft.ifft(torch.polar(torch.ones_like(f), 2 * np.pi * turns.remainder_(1.0)))
    x = torch.view_as_real(x) * (400.0 * np.sqrt(0.9 * n))
    return x.round_().clamp_(-127, 127).to(torch.int8).reshape(-1)


# a peak of more than 65504 in the packed-float16 form (a block of 2^27 matched to
# the filter): infinite in the series, so in no bin's sum; the samples of its group
# on the other side of a bin edge are in theirs
@pytest.mark.parametrize("side", ["after", "before"])
def test_overflow_stays_on_its_side_of_the_edge(side):
    import torch
    import paper_1503_01405_amd as P
    n, nbins = 1 << 27, 1024
    dm = 0.9 * n / 61_100
    per_bin = 13_107.37
    period = nbins * per_bin / FS
    print("case: float16 overflow at a bin edge", side, flush=True)
    plan = P.Plan(F0, BW, dm, n, nbins, period, precision="half", max_batch=1, subint_nsamp=0, decim=1)
    try:
        info = plan.info()
        n_front, hop = info["n_front"], info["hop"]
        # an edge in the middle of a group, about half way: first sample `edge`
        q = int((n_front + hop / 2) / per_bin)
        while True:
            edge = int(np.ceil(q * per_bin)) - n_front
            if 5 <= edge % 16 <= 10:
                break
            q += 1
        at = edge + 2 if side == "after" else edge - 3
        x = matched(n, dm, at + n_front)
        _, ser = plan.process(x)
        ser = ser.cpu().numpy()
        status = plan.info()["status"]
        prof = plan.flush().cpu().numpy()[0].astype(np.float64)
    finally:
        plan.close()
    assert ser.size == hop and np.isinf(ser[at]) and np.isfinite(np.delete(ser, at)).all()
    assert status & P.POND_STATUS_NONFINITE
    # a group's samples of one bin are summed together
    bins = O.fold_bins(np.arange(hop), n_front, period, FS, nbins)
    cells = np.flatnonzero(np.diff(bins, prepend=-1) | (np.arange(hop) % 16 == 0))
    sums = np.add.reduceat(ser.astype(np.float64), cells)
    sums[~np.isfinite(sums)] = 0.0
    count = np.maximum(np.bincount(bins, minlength=nbins), 1)
    want = np.bincount(bins[cells], sums, nbins) / count
    groups = np.bincount(bins[cells], minlength=nbins) / count
    assert (np.abs(prof - want) <= 16 * 2.0 ** -24 * want + UNIT * groups).all()


# the range flag is of one contribution, the powers of a group that share a bin: a
# peak of 1.5e12 (2^40: 1.1e12) over two samples in different bins does not set it,
# on one sample it does
@pytest.mark.parametrize("where", ["two bins", "many bins", "one sample"])
def test_range_flag_of_contributions(where):
    import torch
    import paper_1503_01405_amd as P
    n = 1 << 26
    dm = 0.9 * n / 61_100
    nbins, per_bin = (64, 5.3) if where == "many bins" else (1024, 13_107.37)
    print("case: range flag,", where, flush=True)
    plan = P.Plan(F0, BW, dm, n, nbins, nbins * per_bin / FS, precision="fp32", max_batch=1, subint_nsamp=0, decim=16)
    try:
        info = plan.info()
        n_front, hop = info["n_front"], info["hop"]
        q = int((n_front + hop / 2) / per_bin)
        while True:
            at = int(np.ceil(q * per_bin)) - n_front  # an edge's first sample
            if at % 16 == 8:
                break
            q += 1
        peak = float(at) if where == "one sample" else at - 0.5
        _, ser = plan.process(matched(n, dm, peak + n_front))
        ser = ser.cpu().numpy()
        status = plan.info()["status"]
    finally:
        plan.close()
    assert ser.argmax() == at // 16 and ser.max() > 2.0 ** 40 and np.sort(ser)[-2] < 2.0 ** 39
    assert status == (P.POND_STATUS_RANGE if where == "one sample" else 0)
