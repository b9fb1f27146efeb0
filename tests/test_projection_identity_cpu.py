"""The identity behind the fused pipeline's projection, checked on the CPU.

k_pipe_b forms the amplitudes of a column from the closed form of the inverse
transform, P(y) = prod_b (1 + (-1)^(y_b) w_b conj(t_b(y mod 2^b))), rotates them
by s_y and takes the uncompute's projection on clock 0 as beta sum_y s_y |P|^2.
Pinned against the circuit's own steps: the inverse QFT of the phase state, the
rotation, the forward QFT, the conjugate phases and the sum over the clock.
Tolerance: 2^c terms of size at most 2^c, each within a few roundings.
"""
import numpy as np
import pytest


def inverse_cascade(v, c):
    a = np.array(v, dtype=complex)
    for b in range(c):
        h = 1 << b
        y = np.arange(1 << c)
        lo = y[(y & h) == 0]
        t = np.exp(2j * np.pi * (lo % h) / (2 * h))
        a0, a1 = a[lo].copy(), a[lo | h] * np.conj(t)
        a[lo], a[lo | h] = a0 + a1, a0 - a1
    return a


def forward_cascade(v, c):
    a = np.array(v, dtype=complex)
    for b in range(c - 1, -1, -1):
        h = 1 << b
        y = np.arange(1 << c)
        lo = y[(y & h) == 0]
        t = np.exp(2j * np.pi * (lo % h) / (2 * h))
        a0, a1 = a[lo].copy(), a[lo | h].copy()
        a[lo], a[lo | h] = a0 + a1, (a0 - a1) * t
    return a


@pytest.mark.parametrize("signed", [False, True])
@pytest.mark.parametrize("c", range(1, 10))
def test_projection_is_the_weighted_norm(c, signed):
    rng = np.random.default_rng(17 * c + signed)
    y = np.arange(1 << c)
    w = np.exp(2j * np.pi * rng.random(c))
    beta = complex(*rng.standard_normal(2))
    ph = np.ones(1 << c, dtype=complex)
    P = np.ones(1 << c, dtype=complex)
    for b in range(c):
        ph *= np.where((y >> b) & 1, w[b], 1.0)
        P *= 1.0 + np.where((y >> b) & 1, -1.0, 1.0) * w[b] * np.conj(np.exp(2j * np.pi * (y % (1 << b)) / (2 << b)))
    assert np.abs(inverse_cascade(ph, c) - P).max() <= 1e-13 * c * 2.0 ** c
    ys = np.where(signed & (y >> (c - 1) == 1), y - (1 << c), y).astype(float)
    s = np.zeros(1 << c)
    s[1:] = 1.0 / ys[1:]
    z_circuit = np.sum(np.conj(ph) * forward_cascade(s * beta * inverse_cascade(ph, c), c))
    z_norm = beta * np.sum(s * np.abs(P) ** 2)
    assert abs(z_circuit - z_norm) <= 1e-13 * c * 4.0 ** c * abs(beta)
