"""Pauli sums of thousands of terms (sorted by digits, planned in blocks, searches
that end early) against the oracle: masks of all kinds, many equal ones, all equal."""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def Q():
    from paper_2310_17739_amd import qsim
    return qsim


@pytest.mark.parametrize("n,count", [(10, 255), (10, 256), (10, 3000), (12, 2048), (12, 5000), (16, 3000)])
@pytest.mark.parametrize("masks", ["random", "few", "one", "diagonal", "ascending"])
def test_many_terms(Q, n, count, masks):
    rng = np.random.default_rng(n + count)
    t = np.zeros(count, dtype=W.PAULI_DTYPE)
    N = 1 << n
    t["zmask"] = rng.integers(0, N, count)
    t["xmask"] = {"random": rng.integers(0, N, count), "few": rng.integers(0, N, 7)[rng.integers(0, 7, count)],
                  "one": np.full(count, N - 2), "diagonal": np.zeros(count), "ascending": np.arange(count) % N}[masks]
    t["coeff"] = rng.normal(size=count)
    psi = W.random_state(n, 4)
    print(f"many terms n={n} count={count} {masks}", flush=True)
    sv = Q.StateVector(n, "complex128")
    sv.qsim_set_state(psi)
    # FP64 sums of at most a few hundred partial sums each: 2^-53 of each partial
    assert abs(sv.qsim_expval(t) - oracle.expval(n, psi, t)) < 1e-13 * np.abs(t["coeff"]).sum()
    sv.close()
