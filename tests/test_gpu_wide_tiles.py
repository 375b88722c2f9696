"""Column passes on tiles of 32 columns against tiles of 16, and the fold of
groups at bin edges: launches of many blocks (wide) give the bits of launches
of one block (narrow at 2^20) and of samples that are not 4-byte aligned, and
the outputs match the oracle."""
import numpy as np
import pytest

import oracle as O
import synth

pytestmark = pytest.mark.gpu

F0, BW = 326.5, 16.0
N = 1 << 20


def gpu(x, dm, form, batch, nbins, period, subint=0, decim=16, nfft=N):
    import torch
    import paper_1503_01405_amd as P
    plan = P.Plan(F0, BW, dm, nfft, nbins, period, precision=form, max_batch=batch, subint_nsamp=subint, decim=decim)
    prof, ser = plan.process(x)
    last = plan.flush()
    nf = plan.info()["n_front"]
    torch.cuda.synchronize()
    plan.close()
    return np.concatenate([prof.cpu().numpy(), last.cpu().numpy()]), ser.cpu().numpy(), nf


# DMs whose n_front leaves remainders 0, even and odd modulo 16, with blocks
# that overlap by half (chained) and by a quarter or less
@pytest.mark.parametrize("form", ["half", "mixed"])
@pytest.mark.parametrize("dm", [0.0, 2.0, 3.1, 6.007, 8.2])
def test_wide_and_narrow_tiles_agree(dm, form):
    import torch
    nsamp = 12_000_003
    iq = synth.white_stream_int8(70, nsamp)
    x = torch.from_numpy(iq).cuda()
    pad = torch.empty(x.numel() + 2, dtype=torch.int8, device="cuda")
    pad[2:] = x                      # 2-byte aligned only
    want = gpu(x, dm, form, 1, 128, 0.0123)
    for y, batch in ((x, 16), (x, 11), (pad[2:], 16)):
        got = gpu(y, dm, form, batch, 128, 0.0123)
        assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1]), (dm, batch, want[2] % 16)


# bins of a whole number of samples (edges fall on samples), of 17.3 samples,
# and shorter than a group; sub-integrations that end inside groups
@pytest.mark.parametrize("form", ["fp32", "half", "mixed"])
@pytest.mark.parametrize("nbins,period,subint,decim", [(64, 0.0053, 0, 16), (64, 0.0053, 1_000_005, 8),
                                                       (1024, 1024 * 17.3 / 16e6, 777_777, 4),
                                                       (1024, 1024 * 9.5 / 16e6, 0, 1), (2000, 0.0021, 3_000_000, 2)])
def test_fold_edges(nbins, period, subint, decim, form):
    import torch
    nsamp = 7_000_001
    iq = synth.white_stream_int8(71, nsamp)
    r = O.run(iq, F0, BW, 6.007, N, nbins, period, subint_nsamp=subint, decim=decim)
    prof, ser, _ = gpu(torch.from_numpy(iq).cuda(), 6.007, form, 0, nbins, period, subint, decim)
    k = len(prof)
    assert prof.shape[0] == r["profiles"][:k].shape[0] and ser.shape == r["series"].shape
    eps = 0.0 if form == "fp32" else 5e-3  # per-sample rounding of a detected power
    n_out = r["n_out"]
    sizes = [subint] * (k - 1) + [n_out - (k - 1) * subint] if subint else [n_out]
    for p, w, m in zip(prof, r["profiles"], sizes):
        tol = 1e-6 if form == "fp32" else 1e-4 + 3 * eps / np.sqrt(m / nbins)
        assert np.linalg.norm(p - w) <= tol * np.linalg.norm(w)
    assert np.linalg.norm(ser - r["series"]) <= (1e-5 if form == "fp32" else 1e-2) * np.linalg.norm(r["series"])


# a call whose first sample is an odd one of the stream, on a buffer that keeps the
# stream's alignment: a pair of columns lies half in the carried tail, half in the
# call's input
@pytest.mark.parametrize("form", ["half", "mixed"])
@pytest.mark.parametrize("first", [3_000_001, 3_000_002, N + 1, 2 * N - 1])
def test_odd_carry(first, form):
    import torch
    import paper_1503_01405_amd as P
    nsamp = 12_000_003
    x = torch.from_numpy(synth.white_stream_int8(72, nsamp)).cuda()
    want = gpu(x, 6.007, form, 16, 128, 0.0123)
    plan = P.Plan(F0, BW, 6.007, N, 128, 0.0123, precision=form, max_batch=16, subint_nsamp=0, decim=16)
    # fill the other carry with samples of its own first
    plan.process(torch.full((2 * (first + 1),), 77, dtype=torch.int8, device="cuda"))
    plan.flush()
    ser = [plan.process(y)[1].cpu().numpy() for y in (x[:2 * first], x[2 * first:2 * first + 2 * 5_000_001],
                                                      x[2 * first + 2 * 5_000_001:])]
    prof = plan.flush().cpu().numpy()
    plan.close()
    assert np.array_equal(np.concatenate(ser), want[1]) and np.array_equal(prof, want[0])
