"""The work area of short blocks: small in a plan or search that has only run short
calls, grown by the first longer one, with the same bits; a call captured before it
grew replays afterwards, and one captured first runs on what there is."""
import numpy as np
import pytest

import synth
from gpu_helpers import BW, F0

pytestmark = pytest.mark.gpu

NBINS, PERIOD = 64, 0.0053


def used():
    import torch
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    free, total = torch.cuda.mem_get_info()
    return total - free


@pytest.mark.parametrize("form", ["fp32", "half", "mixed_valu"])
def test_short_calls_hold_little(form):
    import torch
    import paper_1503_01405_amd as P
    x = torch.from_numpy(synth.white_stream_int8(96, 60_000)).cuda()  # under 32 blocks
    # 24 MB of fold partials, 16 of work area, the rest: tables, carried samples, rounding
    before, plans = used(), []
    for _ in range(8):
        plans.append(P.Plan(F0, BW, 0.03, 1 << 12, NBINS, PERIOD, precision=form, subint_nsamp=0, decim=16))
        plans[-1].process(x)
        plans[-1].flush()
    each = (used() - before) / 8
    for p in plans:
        p.close()
    assert each < 56e6, each
    before, searches = used(), []
    prof = torch.empty(2, NBINS, device="cuda")
    for _ in range(4):
        searches.append(P.pond_search_create(F0, BW, [0.01, 0.03], NBINS, PERIOD, 1 << 12, 1 << 12, P.FORMS[form]))
        assert P.pond_search_run(searches[-1], x, 60_000, prof) == P.POND_OK
    each = (used() - before) / 4
    for h in searches:
        P.pond_search_destroy(h)
    assert each < 56e6, each


@pytest.mark.parametrize("form,log2n", [("fp32", 12), ("half", 14), ("mixed_valu", 17), ("mixed", 12)])
def test_growth_gives_the_same_bits(form, log2n):
    import torch
    import paper_1503_01405_amd as P
    n = 1 << log2n
    dm = 0.8 * n / 2 / 61_100
    hop = P.pond_geometry(F0, BW, dm, n)[2]
    area = (1 << 24) // (n * (8 if form == "fp32" else 4))  # blocks there are at first
    x = torch.from_numpy(synth.white_stream_int8(97, 7 * area * hop)).cuda()
    outs = []
    for batch in (16, 0):
        plan = P.Plan(F0, BW, dm, n, NBINS, PERIOD, precision=form, max_batch=batch, subint_nsamp=0, decim=16)
        got, other = [], torch.cuda.Stream()
        for blocks, stream in ((3, None), (area, other), (area + 1, None), (6 * area, other), (7, None)):
            s = stream or torch.cuda.current_stream()
            with torch.cuda.stream(s):
                got.append(plan.process(x[:2 * (n + (blocks - 1) * hop)])[1].cpu().numpy())
                got.append(plan.flush().cpu().numpy())
        plan.close()
        outs.append(got)
    for a, b in zip(*outs):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("form", ["fp32", "half"])
def test_graphs_before_growth(form):
    import torch
    import paper_1503_01405_amd as P
    n, dm = 1 << 13, 0.05
    x = torch.from_numpy(synth.white_stream_int8(98, 1200 * n)).cuda()
    short, long = 30 * n, 1200 * n
    h = P.pond_plan_create(F0, BW, dm, n, NBINS, PERIOD, P.FORMS[form])
    s = torch.cuda.Stream()
    prof = torch.zeros((1, NBINS), device="cuda")
    out = {}
    for nsamp in (short, long):
        out[nsamp] = torch.zeros(P.pond_plan_expect(h, nsamp, 0)[1] // 16, device="cuda")

    def step(nsamp):
        ser = out[nsamp]
        stream = torch.cuda.current_stream()
        r, k = P.pond_dedisperse_series(h, x, nsamp, 0, prof, 0, 16, ser, ser.numel(), stream)
        assert r == 0 and k == ser.numel()
        assert P.pond_dedisperse_fold(h, None, 0, 0, prof, 1, stream) == 1

    try:
        graphs = {}
        for nsamp in (short, long):  # captured first: on the area there is at first
            graphs[nsamp] = torch.cuda.CUDAGraph()
            torch.cuda.synchronize()
            with torch.cuda.graph(graphs[nsamp], stream=s):
                step(nsamp)
        want = {}
        for nsamp in (long, short):  # eager: grows
            with torch.cuda.stream(s):
                step(nsamp)
            torch.cuda.synchronize()
            want[nsamp] = (prof.cpu().numpy(), out[nsamp].cpu().numpy())
        for _ in range(3):
            for nsamp in (short, long):
                prof.fill_(-1.0)
                out[nsamp].fill_(-1.0)
                torch.cuda.synchronize()
                graphs[nsamp].replay()
                torch.cuda.synchronize()
                assert np.array_equal(prof.cpu().numpy(), want[nsamp][0])
                assert np.array_equal(out[nsamp].cpu().numpy(), want[nsamp][1])
                with torch.cuda.stream(s):
                    step(long)
                torch.cuda.synchronize()
        graphs.clear()
    finally:
        P.pond_plan_destroy(h)


@pytest.mark.parametrize("form", ["fp32", "half"])
def test_search_growth(form):
    import torch
    import paper_1503_01405_amd as P
    x = torch.from_numpy(synth.white_stream_int8(99, 2_000_003)).cuda()
    dms, outs = [0.0, 0.01, 0.05, 0.2], []
    for batch in (16, None):
        h = P.pond_search_create(F0, BW, dms, NBINS, PERIOD, 1 << 12, 1 << 16, P.FORMS[form], max_batch=batch)
        got = []
        for nsamp in (100_000, 2_000_003, 300_001):
            prof = torch.empty(len(dms), NBINS, device="cuda")
            assert P.pond_search_run(h, x, nsamp, prof) == P.POND_OK
            got.append(prof.cpu().numpy())
        P.pond_search_destroy(h)
        outs.append(got)
    for a, b in zip(*outs):
        assert np.array_equal(a, b)
