"""Shots from two-level prefix sums (segments within blocks) against the oracle:
states below, at and above one block, draws at both ends, and states whose
amplitudes vanish over segments, blocks and the end of the state."""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def Q():
    from paper_2310_17739_amd import qsim
    return qsim


@pytest.mark.parametrize("dtype", ["complex128", "complex64"])
@pytest.mark.parametrize("n", [1, 3, 4, 8, 11, 12, 13, 18])
@pytest.mark.parametrize("zeros", ["none", "tail", "head", "segments", "one"])
def test_shots(Q, dtype, n, zeros):
    psi = W.random_state(n, n).astype(dtype)
    N = 1 << n
    x = np.arange(N)
    if zeros == "tail":
        psi[max(1, N - N // 3):] = 0
    elif zeros == "head":
        psi[:N // 2] = 0
    elif zeros == "segments":
        psi[(x // 16) % 3 == 1] = 0
        psi[x // 4096 == 1] = 0
    elif zeros == "one":
        psi[x != (5 * N) // 7] = 0
    if not np.any(psi):
        psi[0] = 1
    u = np.concatenate([np.random.default_rng(n).random(3000), [0.0, np.nextafter(1.0, 0.0), 0.5, 2.0 ** -60]])
    print(f"sample dtype={dtype} n={n} zeros={zeros}", flush=True)
    sv = Q.StateVector(n, dtype)
    sv.qsim_set_state(psi)
    got = sv.qsim_sample(u).astype(np.int64)
    p = np.abs(psi.astype(np.complex128)) ** 2
    assert np.all(p[got] > 0)
    want = oracle.sample(n, psi.astype(np.complex128), u).astype(np.int64)
    # the oracle's sums are taken in another order: a draw within rounding of a
    # step may fall on the other side of it
    c = np.cumsum(p)
    edge = np.zeros(len(u), dtype=bool)
    for s in np.flatnonzero(got != want):
        a, b = sorted((got[s], min(want[s], N - 1)))
        edge[s] = c[b] - p[b] - c[a] <= 1e-12 * c[-1] and abs(u[s] * c[-1] - c[a]) <= 1e-12 * c[-1]
    assert np.all((got == want) | edge)
    assert len(sv.qsim_sample(np.zeros(0))) == 0
    sv.close()
