"""The search's inverse rows over several blocks per workgroup: every length
group and form gives the bits of one block per workgroup, whatever the
blocks per launch leave as the last, shorter chain, and matches the oracle."""
import numpy as np
import pytest

import oracle as O
import synth

pytestmark = pytest.mark.gpu

F0, BW, NBINS, PERIOD = 326.5, 16.0, 64, 4.1e-3


def search(x, nsamp, dms, log2n, form, batch):
    import torch
    import paper_1503_01405_amd as P
    h = P.pond_search_create(F0, BW, dms, NBINS, PERIOD, 1 << log2n, 1 << log2n, P.FORMS[form], max_batch=batch)
    prof = torch.empty((len(dms), NBINS), device="cuda")
    assert P.pond_search_run(h, x, nsamp, prof) == 0
    torch.cuda.synchronize()
    P.pond_search_destroy(h)
    return prof.cpu().numpy()


# rows of 2^5 .. 2^13 and 2^14: short rows (several per workgroup, the last
# group ragged), every last radix, the longest
@pytest.mark.parametrize("form", ["fp32", "mixed_valu", "half", "mixed"])
@pytest.mark.parametrize("log2n", [10, 13, 15, 17, 18, 19, 20, 21, 22, 23, 24])
def test_chained_inverse_rows(log2n, form):
    import torch
    n = 1 << log2n
    dms = [0.0, 0.4 * n / 2 / 61100, 0.9 * n / 2 / 61100]
    nblocks = 37 if log2n <= 18 else 7
    nsamp = n + (nblocks - 1) * (n // 2)
    iq = synth.white_stream_int8(50 + log2n, nsamp)
    x = torch.from_numpy(iq).cuda()
    one = search(x, nsamp, dms, log2n, form, 1)
    # the launch's blocks in chains of every shape the batch gives
    for batch in (nblocks, 5, 16):
        assert np.array_equal(search(x, nsamp, dms, log2n, form, batch), one), batch
    if log2n <= 19:
        want, _ = O.search(iq, F0, BW, dms, NBINS, PERIOD, n, n)
        m = (nblocks * n // 2) / NBINS  # samples per bin
        tol = 1e-6 if form == "fp32" else 1e-4 + 3 * 5e-3 / np.sqrt(m)
        for t in range(len(dms)):
            assert np.linalg.norm(one[t] - want[t]) <= tol * np.linalg.norm(want[t])
