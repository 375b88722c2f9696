"""Histogram sizes at which K3 changes its shape, each side of the line: 32-column
tiles to 16 (matrix-core form), two workgroups per CU to one (packed float16), LDS to
global memory.  Columns of 2^10 and 2^9, launches of many blocks and of two, against
the oracle and each other."""
import functools

import numpy as np
import pytest

import oracle as O
import synth
from gpu_helpers import BW, F0, gpu_run, profile_rel_l2, rel_l2
from test_gpu_parity import TOL, profile_tol

pytestmark = pytest.mark.gpu

PERIOD = 0.0891


@functools.lru_cache(maxsize=None)
def stream(log2n):
    """Twelve blocks and the oracle's powers of them."""
    n = 1 << log2n
    dm = 0.5 * n / 2 / 61_100
    g = O.plan_geometry(F0, BW, dm, n)
    iq = synth.white_stream_int8(102, n + 11 * g["hop"] + 3)
    r = O.run(iq, F0, BW, dm, n, 1, PERIOD, workers=8, keep_power=True)
    return dm, iq, g["n_front"], r["power"], r["series"]


# 160 KB of LDS; 67,632 B of tile and tables with columns of 2^10 (65,536 more with 32
# columns; 131,072 in float32), 34,208 with 2^9; 12 B an entry; at most 8,192 in LDS
@pytest.mark.parametrize("form,log2n,nbins", [
    ("half", 20, 1190), ("half", 20, 1191), ("half", 20, 8017), ("half", 20, 8018),
    ("mixed", 20, 2556), ("mixed", 20, 2557), ("mixed", 20, 8017), ("mixed", 20, 8018),
    ("half", 18, 3976), ("half", 18, 3977), ("half", 18, 8192), ("half", 18, 8193),
    ("fp32", 20, 2730), ("fp32", 20, 2731), ("fp32", 18, 8192), ("fp32", 18, 8193)])
def test_histogram_limits(form, log2n, nbins):
    dm, iq, n_front, power, series = stream(log2n)
    sums, cnts, _ = O.fold(power, 0, n_front, PERIOD, BW * 1e6, nbins, 0)
    want = O.profiles_from(sums, cnts)
    print(f"case: histogram limit {form} 2^{log2n} {nbins} bins", flush=True)
    got = [gpu_run(iq, dm, 1 << log2n, nbins, PERIOD, precision=form, max_batch=mb) for mb in (0, 2)]
    ep, es = profile_rel_l2(got[0][0], want), rel_l2(got[0][1], series)
    tp = profile_tol(form, power.size, 0, nbins)
    print(f"{form}: profile rel-L2 {ep:.3e} (tol {tp:.1e}) series rel-L2 {es:.3e}")
    assert ep <= tp and es <= TOL[form][1]
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])


def test_launches_beyond_the_cache():
    """Float32 launches of more than 256 MB of work area read the next column tile
    ahead: the same bits as launches of one block."""
    n, hop = 1 << 22, 1 << 21
    iq = synth.white_stream_int8(103, n + 8 * hop)  # 9 blocks of 32 MB
    got = [gpu_run(iq, 20.0, n, 100, PERIOD, max_batch=mb) for mb in (9, 1)]
    assert got[0][1].size == 9 * hop // 16
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])
