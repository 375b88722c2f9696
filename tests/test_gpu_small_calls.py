"""Launches of short calls: a segment whose blocks take one launch or several,
its histograms in LDS or not, and samples carried between calls from buffers
and in pieces of any even alignment, against one call on an aligned buffer."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

F0, BW = 326.5, 16.0


@pytest.mark.parametrize("form", ["fp32", "mixed_valu"])
@pytest.mark.parametrize("nsamp,nbins", [(4096, 1), (40_001, 63), (40_001, 64), (40_001, 65), (40_001, 8192),
                                         (300_007, 129), (100, 64)])
def test_segment_launches(nsamp, nbins, form):
    import torch
    import paper_1503_01405_amd as P
    dm, nfft, period = 0.03, 1 << 12, 0.0021
    x = torch.from_numpy(synth.white_stream_int8(82, nsamp)).cuda()
    plan = P.Plan(F0, BW, dm, nfft, nbins, period, precision=form, max_batch=16, subint_nsamp=0, decim=16)
    _, ser = plan.process(x)
    want = plan.flush().cpu().numpy()
    want_s = ser.cpu().numpy()
    plan.close()
    want = want[0] if len(want) else np.zeros(nbins, np.float32)
    for _ in range(2):
        prof = torch.full((nbins,), -1.0, device="cuda")
        got_s = torch.empty(max(want_s.size, 1), device="cuda")
        n = P.pond_dedisperse_segment_noalloc(F0, BW, dm, nfft, nbins, period, P.FORMS[form], x, nsamp, 16, prof,
                                              got_s, want_s.size)
        torch.cuda.synchronize()
        assert n == want_s.size
        # integer sums of the same powers: the same bits
        assert np.array_equal(prof.cpu().numpy(), want) and np.array_equal(got_s.cpu().numpy()[:n], want_s)


@pytest.mark.parametrize("pieces", [[1, 7, 8, 9], [4095, 4097, 3], [16_411], [2048 + 5, 13, 30_000]])
def test_carried_samples(pieces):
    import torch
    import paper_1503_01405_amd as P
    nsamp, nbins = 60_003, 50
    iq = synth.white_stream_int8(83, nsamp)
    x = torch.from_numpy(iq).cuda()

    def run(parts):
        plan = P.Plan(F0, BW, 0.03, 1 << 12, nbins, 0.0021, precision="fp32", max_batch=16, subint_nsamp=0, decim=16)
        sers = [plan.process(p)[1].cpu().numpy() for p in parts]
        prof = plan.flush().cpu().numpy()
        plan.close()
        return prof, np.concatenate(sers)

    parts, at, k = [], 0, 0
    while at < nsamp:
        c = min(pieces[k % len(pieces)] if k < 300 else nsamp, nsamp - at)
        buf = torch.empty(2 * c + 16, dtype=torch.int8, device="cuda")
        off = 2 * (k % 8)
        buf[off:off + 2 * c] = x[2 * at:2 * (at + c)]
        parts.append(buf[off:off + 2 * c])
        at += c
        k += 1
    got, want = run(parts), run([x])
    assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])
