"""Host-only checks of batch programs with measurement records (no GPU needed):
one state emulated from the device tables of its plan, as a batch compiles and
binds it, against the oracle."""
import numpy as np
import pytest

import oracle
import workloads as W
from paper_2310_17739_amd import qsim
from test_gpu_span import measured_program
from test_host_span import norm_error

LINEAR = [W.KIND_RX, W.KIND_RY, W.KIND_RZ, W.KIND_RXX, W.KIND_RZZ]


def as_template(g):
    """The same gates with every plain rotation's angle in a parameter vector."""
    g = g.copy()
    at = np.flatnonzero(np.isin(g["kind"], LINEAR))
    g["slot"][at] = np.arange(len(at))
    return g, g["theta"][at, 0].copy()


def failing_program(n, bad):
    """Rotations and a permuting frame, qubit 5 made |1> for certain and carried
    on to qubit 8, a record that fails, and gates after it.  Returns the records
    up to the failing one, the whole program and the code."""
    head, _ = measured_program(n, 1, seed=3)
    head = head[head["kind"] < W.KIND_BARRIER]
    tail, _ = measured_program(n, 1, seed=4)
    tail = tail[tail["kind"] < W.KIND_BARRIER]
    fixed = W.gates([(W.KIND_MEASURE, (5,), (), 0), (W.KIND_RESET, (5,), ()), (W.KIND_X, (5,), ()), (W.KIND_SWAP, (5, 8), ())])
    rec = {"assert": (W.KIND_ASSERT0, (8,), (), 1), "reset": (W.KIND_RESET, (3,), ()),
           "forced": (W.KIND_MEASURE, (8,), (), 1)}[bad]
    upto = np.concatenate([head, fixed])
    code = qsim.E_NOT_DEFINITE if bad == "reset" else qsim.E_ZERO_PROB
    return upto, np.concatenate([upto, W.gates([rec]), tail]), code


# 10..14: whole states in one tile; 9: below the rotations' tiles; 15: passes between records
@pytest.mark.parametrize("dtype,n", [("complex128", 9), ("complex128", 10), ("complex64", 11), ("complex128", 12),
                                     ("complex128", 13), ("complex64", 14), ("complex128", 15)])
@pytest.mark.parametrize("params", [False, True])
def test_records(dtype, n, params):
    g, slots = measured_program(n, 2, seed=n)
    g, th = as_template(g) if params else (g, None)
    u = np.random.default_rng(n).random(slots)
    r = qsim.qsim_debug_emulate_batch(n, g, dtype, params=th, uniforms=u, n_slots=slots)
    assert r["status"] == 0
    want, o, p = oracle.run(n, g, params=th, forced=r["outcomes"], n_slots=slots)
    # at most nine rotations per gate and two roundings of 2^-53 each, magnified by
    # 1 / sqrt(p) in a projection onto a branch of probability p
    tol = 2 * 9 * len(g) * 1.2e-16 / np.sqrt(np.prod(p))
    assert norm_error(r["state"], want) < tol
    assert np.max(np.abs(r["probs"] - p)) < 2 * tol
    is_measure = np.arange(slots) % 3 != 2
    assert np.all((r["outcomes"] == np.where(u < np.where(o == 0, p, 1 - p), 0, 1))[is_measure])


@pytest.mark.parametrize("dtype,n", [("complex128", 9), ("complex128", 10), ("complex64", 11), ("complex128", 13),
                                     ("complex64", 14), ("complex128", 15)])
@pytest.mark.parametrize("params", [False, True])
@pytest.mark.parametrize("bad", ["assert", "reset", "forced"])
def test_failing_records(dtype, n, params, bad):
    """The state stays as the failing record found it, its qubits in the order
    that the gates before left."""
    upto, prog, code = failing_program(n, bad)
    prog, th = as_template(prog) if params else (prog, None)
    forced = np.array([0, 0], dtype=np.int32)
    r = qsim.qsim_debug_emulate_batch(n, prog, dtype, params=th, uniforms=np.full(2, 0.25), forced=forced, n_slots=2)
    assert r["status"] == code
    want, _, _ = oracle.run(n, upto, forced=forced, n_slots=2)
    assert norm_error(r["state"], want) < 4 * 2 * 9 * len(prog) * 1.2e-16
