"""Launches of short calls and short blocks: a segment whose blocks take one
launch or several, its histograms in LDS or not; samples carried between calls
from buffers and in pieces of any even alignment, against one call on an aligned
buffer; the library's own count of blocks per launch against a stated one."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

F0, BW = 326.5, 16.0


@pytest.mark.parametrize("form", ["fp32", "mixed_valu"])
@pytest.mark.parametrize("nsamp,nbins", [(4096, 1), (40_001, 63), (40_001, 64), (40_001, 65), (40_001, 8192),
                                         (300_007, 129), (100, 64),
                                         (8_000_011, 64)])
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


# the library's own count of short blocks per launch against 16: whole stream,
# sub-integrations that launches cut (few and many bins), histograms in global
# memory, a stream in pieces
@pytest.mark.parametrize("form", ["fp32", "half", "mixed", "mixed_valu", "bf16"])
@pytest.mark.parametrize("log2n,nbins,subint", [(10, 64, 0), (12, 64, 50_001), (14, 3000, 400_000), (16, 9000, 0),
                                                (16, 9000, 700_001), (17, 128, 0)])
def test_default_launches(log2n, nbins, subint, form):
    import torch
    import paper_1503_01405_amd as P
    nsamp = 4_000_003
    x = torch.from_numpy(synth.white_stream_int8(84, nsamp)).cuda()
    outs = []
    for batch, piece in ((16, nsamp), (0, nsamp), (0, 1_500_001)):
        try:
            plan = P.Plan(F0, BW, 0.005, 1 << log2n, nbins, 0.0123, precision=form, max_batch=batch,
                          subint_nsamp=subint, decim=16)
        except P.PondError:
            pytest.skip("the form has no columns this short")
        prof, ser = [], []
        for at in range(0, nsamp, piece):
            a, b = plan.process(x[2 * at:2 * min(at + piece, nsamp)])
            prof.append(a.cpu().numpy())
            ser.append(b.cpu().numpy())
        prof.append(plan.flush().cpu().numpy())
        plan.close()
        outs.append((np.concatenate(prof), np.concatenate(ser)))
    for got in outs[1:]:
        assert np.array_equal(got[0], outs[0][0]) and np.array_equal(got[1], outs[0][1])


@pytest.mark.parametrize("log2n", [11, 15, 18])
@pytest.mark.parametrize("form", ["fp32", "mixed_valu"])
def test_default_launches_of_real_input(log2n, form):
    import torch
    import paper_1503_01405_amd as P
    nsamp = 4_000_002
    x = torch.from_numpy(synth.white_stream_int8(85, nsamp)).cuda()
    outs = []
    for batch in (16, 0):
        plan = P.Plan(F0, BW, 0.005, 1 << log2n, 100, 0.0123, precision=form, max_batch=batch, subint_nsamp=1_000_002,
                      decim=32, sideband="lsb")
        prof, ser = plan.process(x)
        outs.append((np.concatenate([prof.cpu().numpy(), plan.flush().cpu().numpy()]), ser.cpu().numpy()))
        plan.close()
    assert np.array_equal(outs[1][0], outs[0][0]) and np.array_equal(outs[1][1], outs[0][1])


@pytest.mark.parametrize("form", ["fp32", "half"])
def test_default_launches_of_a_search(form):
    import torch
    import paper_1503_01405_amd as P
    nsamp = 2_000_003
    x = torch.from_numpy(synth.white_stream_int8(86, nsamp)).cuda()
    dms, outs = [0.0, 0.01, 0.05, 0.2, 0.6], []
    for batch in (16, None):
        h = P.pond_search_create(F0, BW, dms, 100, 0.0123, 1 << 12, 1 << 18, P.FORMS[form], max_batch=batch)
        prof = torch.empty(len(dms), 100, device="cuda")
        assert P.pond_search_run(h, x, nsamp, prof) == P.POND_OK
        torch.cuda.synchronize()
        P.pond_search_destroy(h)
        outs.append(prof.cpu().numpy())
    assert np.array_equal(outs[1], outs[0])


# the float16 forms' power scale, measured at creation: mean powers are those of
# the float32 form (float16 rounding of random sign; one part in a thousand)
@pytest.mark.parametrize("form", ["half", "mixed"])
@pytest.mark.parametrize("log2n", [12, 17, 22, 23])
def test_power_scale(log2n, form):
    import torch
    import paper_1503_01405_amd as P
    nsamp = 3 << log2n
    x = torch.from_numpy(synth.white_stream_int8(87, nsamp)).cuda()
    means = []
    for f in ("fp32", form):
        plan = P.Plan(F0, BW, 0.01, 1 << log2n, 64, 0.0123, precision=f, max_batch=0, decim=16)
        means.append(plan.process(x)[1].double().mean().item())
        plan.close()
    assert abs(means[1] / means[0] - 1) < 1e-3


# calls whose blocks are no multiple of a launch: one launch of up to twice the
# cached count, several of about the same size
@pytest.mark.parametrize("form,log2n", [("fp32", 22), ("half", 23)])
@pytest.mark.parametrize("nblocks", [1, 4, 5, 7, 9])
def test_uneven_launches(nblocks, form, log2n):
    import torch
    import paper_1503_01405_amd as P
    n = 1 << log2n
    nsamp = n + (nblocks - 1) * (n // 2)
    dm = 20.0 * n / (1 << 22)
    x = torch.from_numpy(synth.white_stream_int8(88, nsamp)).cuda()
    outs = []
    for batch in (1, 0):
        plan = P.Plan(F0, BW, dm, n, 100, 0.0123, precision=form, max_batch=batch, subint_nsamp=0, decim=16)
        ser = plan.process(x)[1].cpu().numpy()
        outs.append((plan.flush().cpu().numpy(), ser))
        plan.close()
    assert outs[0][1].size == nblocks * (n // 2) // 16
    assert np.array_equal(outs[1][0], outs[0][0]) and np.array_equal(outs[1][1], outs[0][1])
