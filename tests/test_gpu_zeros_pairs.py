"""Qubits that several controlled rotations leave definite are so on the GPU: a reset,
and a forced outcome of probability 0."""
import numpy as np
import pytest

import oracle
import workloads as W
from test_gpu_span import tol
from test_host_span import norm_error
from test_host_zeros import A, surroundings
from test_host_zeros_pairs import GADGETS

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def Q():
    from paper_2310_17739_amd import qsim
    return qsim


@pytest.mark.parametrize("dtype,n,tile", [("complex128", 10, None), ("complex64", 14, None), ("complex128", 15, 11),
                                          ("complex64", 16, 12)])
@pytest.mark.parametrize("name", sorted(GADGETS))
def test_definite_qubits(Q, dtype, n, tile, name, monkeypatch):
    monkeypatch.setenv("QSIM_SPAN", "2")   # span passes whatever they cost
    recs, value = GADGETS[name]
    g = W.gates(surroundings(n, 1, 2) + list(recs))
    print(f"definite qubit dtype={dtype} n={n} {name}", flush=True)
    want, _, _ = oracle.run(n, g)
    sv = Q.StateVector(n, dtype)
    sv.qsim_apply(g, tile_qubits=tile)
    got = sv.qsim_get_state()
    assert norm_error(got, want) < tol(dtype, len(g))
    assert np.all(got.reshape(-1, 2)[:, 1 - value] == 0)
    with pytest.raises(Q.QsimError) as e:
        sv.qsim_measure_assert(A, 1 - value)
    assert e.value.code == Q.E_ZERO_PROB
    sv.qsim_reset(A)
    sv.close()
