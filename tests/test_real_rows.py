"""The real path's middle pass: the 2 x 2 step over a bin and its partner
against the real transform it stands for (CPU), and row lengths of every last
radix on the GPU against the oracle."""
import numpy as np
import pytest

import oracle as O
from test_real_path import check, real_stream


@pytest.mark.parametrize("sideband", ["lsb", "usb"])
def test_two_by_two_step_is_the_filtered_real_transform(sideband):
    """Z' = a Z + b G and G' = d G - b Z, G[k] = conj Z[N-k], with the rows'
    partner values from conjugated input under the same four-step twiddle."""
    n1, n2 = 32, 16
    N = n1 * n2
    rng = np.random.default_rng(3)
    x = rng.standard_normal(2 * N)
    M = O.real_chirp(2 * N, 326.5, 16.0, 0.01, sideband, 0.2)
    want = np.fft.irfft(np.fft.rfft(x) * M, n=2 * N)
    z = x[0::2] + 1j * x[1::2]
    cols = np.fft.fft(z.reshape(n2, n1), axis=0)          # [k2][n]: length n2, stride n1
    k1, n = np.arange(n1), np.arange(n1)
    out = np.zeros((n2, n1), dtype=complex)
    for k2 in range(n2 // 2 + 1):
        rb = 0 if k2 == 0 else n2 - k2
        tw = np.exp(-2j * np.pi * k2 * n / N)
        Z = np.fft.fft(cols[k2] * tw)
        G = np.fft.fft(np.conj(cols[rb]) * tw)
        k = k2 + n2 * k1
        P, Q = (M[k] + np.conj(M[N - k])) / 2, (M[k] - np.conj(M[N - k])) / 2
        t = np.pi * k / N
        a, d, b = P - np.sin(t) * Q, P + np.sin(t) * Q, 1j * np.cos(t) * Q
        out[k2] = np.fft.ifft(a * Z + b * G) * np.conj(tw)
        if rb != k2:
            out[rb] = np.conj(np.fft.ifft(d * G - b * Z) * np.conj(tw))
    got = np.fft.ifft(out, axis=0).reshape(-1)
    assert np.allclose(got.real, want[0::2], atol=1e-12) and np.allclose(got.imag, want[1::2], atol=1e-12)


@pytest.mark.gpu
@pytest.mark.parametrize("log2n", [12, 14, 15, 17, 18, 19, 21])
def test_gpu_rows_of_every_last_radix(log2n):
    n = 1 << log2n
    dm = 0.4 * n / 4 / 61100
    raw = real_stream(60 + log2n, 5 * n + 2 * 777, dm, 2.1e-3, "lsb", nfft_gen=max(1 << 16, n))
    check(raw, dm, n, 32, 2.1e-3, "lsb", ["fp32", "mixed_valu"], decim=4)
