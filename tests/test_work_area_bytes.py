"""Bytes charged for a served stream: the work area is of the blocks that its calls
launch at once, not of more."""
import pytest

from gpu_helpers import BW, F0


# blocks of the area: one at a time for the split middle pass, else fewer than two
# launches of what stays cached
@pytest.mark.parametrize("form,log2n,blocks", [("half", 25, 1), ("fp32", 26, 1), ("fp32", 23, 5), ("half", 23, 7),
                                               ("fp32", 22, 7), ("half", 20, 16), ("fp32", 12, 16)])
def test_stream_bytes_hold_the_launches(form, log2n, blocks):
    import paper_1503_01405_amd as P
    n = 1 << log2n
    d = P.stream_desc(F0, BW, 0.5 * n / 2 / 61_100, n, 64, 0.1, 0, 1 << 20, P.FORMS[form])
    elem = 8 if form == "fp32" else 4
    got = P.pond_server_stream_bytes(d)
    # carried samples, at most 8 B of tables a point (and short ones), partials, slots
    rest = 4 * n + (2 * 2 + 16) * (1 << 20) + 12 * (1 << 21)
    assert blocks * n * elem < got < blocks * n * elem + rest + 8 * n + (8 << 20)
