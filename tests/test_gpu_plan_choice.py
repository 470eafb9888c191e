"""Programs and batches compare the plans of a circuit that lowers to rotations and
run the cheaper one; both give the oracle's state."""
import numpy as np
import pytest

import oracle
import workloads as W
from test_gpu_span import tol
from test_host_plan_choice import controlled_layers, exponentials, qft, rotation_layers
from test_host_span import norm_error, spanned

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def Q():
    from paper_2310_17739_amd import qsim
    return qsim


@pytest.mark.parametrize("dtype,n", [("complex128", 13), ("complex64", 16)])
@pytest.mark.parametrize("family,spans", [(rotation_layers, False), (qft, None), (controlled_layers, None), (exponentials, True)])
def test_programs_and_batches(Q, dtype, n, family, spans, monkeypatch):
    g = family(n)
    print(f"plan choice dtype={dtype} n={n} {family.__name__}", flush=True)
    for mode in ("1", "2", "0"):
        monkeypatch.setenv("QSIM_SPAN", mode)
        want, _, _ = oracle.run(n, g)
        sv = Q.StateVector(n, dtype)
        p = Q.Program(n, g, dtype)
        p.qsim_run(sv)
        st = p.qsim_program_stats()
        assert norm_error(sv.qsim_get_state(), want) < tol(dtype, len(g))
        b = Q.Batch([{"n": n, "n_states": 2, "gates": g}], dtype=dtype)
        b.qsim_batch_run()
        for s in range(2):
            assert norm_error(b.qsim_batch_get_state(0, s), want) < tol(dtype, len(g))
        if mode == "1" and spans is not None:
            assert spanned(st) == spans and spanned(b.qsim_batch_group_stats(0)) == spans
        if mode == "2":
            assert spanned(st)
        if mode == "0":
            assert not spanned(st)
        b.close()
        p.close()
        sv.close()
