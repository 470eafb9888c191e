"""Qubits that a circuit leaves definite are definite to the last bit on the GPU:
resets, assertions and forced outcomes, decided by the host and by the device."""
import numpy as np
import pytest

import oracle
import workloads as W
from test_gpu_span import tol
from test_host_span import norm_error
from test_host_zeros import A, GADGETS, surroundings

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
    head = surroundings(n, 1, 2) + list(recs)
    g = W.gates(head)
    print(f"definite qubit dtype={dtype} n={n} {name}", flush=True)
    sv = Q.StateVector(n, dtype)
    sv.qsim_apply(g, tile_qubits=tile)
    want, _, _ = oracle.run(n, g)
    got = sv.qsim_get_state()
    assert norm_error(got, want) < tol(dtype, len(g))
    assert np.all(got.reshape(-1, 2)[:, 1 - value] == 0)
    with pytest.raises(Q.QsimError) as e:
        sv.qsim_measure_assert(A, 1 - value)
    assert e.value.code == Q.E_ZERO_PROB
    assert sv.qsim_measure_assert(A, value) == 1.0
    sv.qsim_reset(A)
    want, _, _ = oracle.run(n, W.gates(head + [(W.KIND_X, (A,), ())] * value))
    assert norm_error(sv.qsim_get_state(), want) < 2 * tol(dtype, len(g))
    sv.close()
    progs = [head + [(W.KIND_RESET, (A,), ())], head + [(W.KIND_MEASURE, (A,), (), 0)], head + [(W.KIND_ASSERT0, (A,), (), 0)]]
    b = Q.Batch([{"n": n, "n_states": 2, "gates": W.gates(p), "uniforms": np.full((2, 1), 0.5),
                  "forced": np.array([[value], [1 - value]]), "n_slots": 1} for p in progs], dtype=dtype, tile_qubits=tile)
    b.qsim_batch_run()
    for i in range(3):
        r = b.qsim_batch_results(i)
        fails = [False, False] if i == 0 else [False, True] if i == 1 else [value == 1] * 2
        assert list(r["status"]) == [Q.E_ZERO_PROB if f else 0 for f in fails]
        for s in range(2):
            flipped = [(W.KIND_X, (A,), ())] * value if i == 0 else []
            want, _, _ = oracle.run(n, W.gates(head + flipped))
            assert norm_error(b.qsim_batch_get_state(i, s), want) < 2 * tol(dtype, len(g))
    b.close()
