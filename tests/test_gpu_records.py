"""Batch programs with measurement records and per-state angles on the GPU
against the oracle: whole states in one tile, states below and above."""
import numpy as np
import pytest

import oracle
import workloads as W
from test_gpu_batch import test_assertion_failure_marks_only_that_state as assertion_failure
from test_gpu_batch import test_joined_measure_reset_zero_probability as joined_measure_reset
from test_gpu_span import measured_program, tol
from test_host_records import as_template, failing_program
from test_host_span import norm_error

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def Q():
    from paper_2310_17739_amd import qsim
    return qsim


@pytest.mark.parametrize("dtype", ["complex128", "complex64"])
@pytest.mark.parametrize("n", [9, 10, 11, 12, 13, 14, 15])
def test_records_of_templates(Q, dtype, n):
    states = 4
    g, slots = measured_program(n, 2, seed=n)
    g, th = as_template(g)
    rng = np.random.default_rng(n + 2)
    th = th + rng.normal(0.0, 0.1, (states, len(th)))
    u = rng.random((states, slots))
    print(f"records of templates dtype={dtype} n={n}", flush=True)
    b = Q.Batch([{"n": n, "n_states": states, "gates": g, "params": th, "uniforms": u, "n_slots": slots}], dtype=dtype)
    for _ in range(2):
        b.qsim_batch_run()
        r = b.qsim_batch_results(0)
        assert np.all(r["status"] == 0)
        for s in range(states):
            want, _, p = oracle.run(n, g, params=th[s], forced=r["outcomes"][s], n_slots=slots)
            # a projection onto a branch of probability p magnifies an error by 1 / sqrt(p)
            err = tol(dtype, len(g)) / np.sqrt(np.prod(p))
            assert np.max(np.abs(r["probs"][s] - p)) < 2 * err
            assert norm_error(b.qsim_batch_get_state(0, s), want) < err
    b.close()


@pytest.mark.parametrize("dtype,n", [("complex128", 11), ("complex64", 11), ("complex128", 13), ("complex64", 14),
                                     ("complex128", 15)])
@pytest.mark.parametrize("bad", ["assert", "reset", "forced"])
def test_failing_records_of_templates(Q, dtype, n, bad):
    upto, prog, code = failing_program(n, bad)
    prog, th = as_template(prog)
    forced = np.array([[0, 0], [1, 1]], dtype=np.int32)
    print(f"failing record of a template dtype={dtype} n={n} {bad}", flush=True)
    b = Q.Batch([{"n": n, "n_states": 2, "gates": prog, "params": np.stack([th, th]), "uniforms": np.full((2, 2), 0.25),
                  "forced": forced, "n_slots": 2}], dtype=dtype)
    b.qsim_batch_run()
    r = b.qsim_batch_results(0)
    for s in range(2):
        fails = bad != "forced" or s == 0
        assert r["status"][s] == (code if fails else 0)
        want, _, _ = oracle.run(n, upto if fails else prog, params=None if fails else th, forced=forced[s], n_slots=2)
        assert norm_error(b.qsim_batch_get_state(0, s), want) < 4 * tol(dtype, len(prog))
    b.close()


@pytest.mark.parametrize("dtype", ["complex128", "complex64"])
@pytest.mark.parametrize("n", [11, 13])
def test_zero_probability_in_whole_states(Q, dtype, n):
    """A forced outcome and an assertion of probability 0 in one state of four, its
    angle bound per state."""
    joined_measure_reset(Q, dtype, n, None)
    if dtype == "complex128":
        assertion_failure(Q, n)
