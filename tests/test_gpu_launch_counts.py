"""Launches of a call whose sub-integrations bound its launch sizes: the library's
own sizes take no more launches than 16 blocks at a time, and give the same bits."""
import numpy as np
import pytest

import synth
from gpu_helpers import BW, F0

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form,log2n,nblocks,nbins,hops", [
    ("fp32", 12, 127, 1024, 20), ("half", 12, 127, 256, 4), ("mixed_valu", 14, 127, 256, 1.5),
    ("half", 18, 47, 1024, 20), ("half", 18, 47, 256, 4), ("mixed", 18, 47, 64, 0.5), ("fp32", 18, 33, 1000, 1.5),
    ("mixed_valu", 18, 47, 64, 1.5), ("half", 16, 100, 3000, 2.5)])
def test_no_more_launches_than_at_sixteen_blocks(form, log2n, nblocks, nbins, hops):
    import torch
    import paper_1503_01405_amd as P
    n = 1 << log2n
    dm = 0.9 * n / 2 / 61_100
    hop = P.pond_geometry(F0, BW, dm, n)[2]
    nsamp = n + (nblocks - 1) * hop + 5
    x = torch.from_numpy(synth.white_stream_int8(95, nsamp)).cuda()
    got = []
    for batch in (16, 0):
        plan = P.Plan(F0, BW, dm, n, nbins, 0.0123, precision=form, max_batch=batch, subint_nsamp=int(hops * hop) | 1,
                      decim=16)
        P.pond_plan_set_timing(plan.handle, True)
        prof, ser = plan.process(x)
        launches = P.pond_plan_kernel_times(plan.handle)["k1_unpack_colfft"][1]
        prof = torch.cat([prof, plan.flush()])
        got.append((launches, prof.cpu().numpy(), ser.cpu().numpy()))
        plan.close()
    assert got[1][0] <= got[0][0], (got[0][0], got[1][0])
    assert np.array_equal(got[1][1], got[0][1]) and np.array_equal(got[1][2], got[0][2])
