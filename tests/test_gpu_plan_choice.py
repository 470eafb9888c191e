"""Programs and batches compare the plans of a circuit that lowers to rotations and
run the cheaper one; both give the oracle's state."""
import numpy as np
import pytest

import oracle
import workloads as W
from test_gpu_span import tol
from test_host_plan_choice import controlled_layers, exchange_layers, exponentials, qft, rotation_layers
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


def attempts(Q, group, **kw):
    """Allocations and compiles that creating a batch asks for."""
    for after in range(200):
        Q.qsim_debug_fail_alloc(after)
        try:
            Q.Batch([group], **kw).close()
            return after
        except Q.QsimError as e:
            assert e.code == Q.E_NOMEM
        finally:
            Q.qsim_debug_fail_alloc(-1)
    raise AssertionError("no end")


def test_autotuning_times_the_form_that_runs(Q):
    """A program whose records keep its frame from cancelling runs as fused
    operators, though its gates alone lower to rotations: every fusion width of
    them is timed."""
    n = 12
    rng = np.random.default_rng(1)
    recs = []
    for k in range(3):
        recs += [(W.KIND_RY, (q,), (float(rng.normal()),)) for q in range(1, n)]
        recs += [(W.KIND_RXX, (q, q + 1), (float(rng.normal()),)) for q in range(1, n - 1)]
        recs += [(W.KIND_H, (0,), ()), (W.KIND_MEASURE, (0,), (), k), (W.KIND_H, (0,), ())]
    g = W.gates(recs)
    group = {"n": n, "n_states": 2, "gates": g, "uniforms": np.full((2, 3), 0.3), "n_slots": 3}
    print("autotune with records", flush=True)
    b = Q.Batch([group], dtype="complex64", autotune=True)
    assert not spanned(b.qsim_batch_group_stats(0))
    b.qsim_batch_run()
    r = b.qsim_batch_results(0)
    for s in range(2):
        want, _, _ = oracle.run(n, g, forced=r["outcomes"][s], n_slots=3)
        assert norm_error(b.qsim_batch_get_state(0, s), want) < 4 * tol("complex64", len(g))
    b.close()
    # widths 2 to 5, and the three tables of the timed plans
    assert attempts(Q, group, dtype="complex64", autotune=True) - attempts(Q, group, dtype="complex64") >= 4 + 3


def test_autotuning_times_every_width(Q):
    """At width 2 these layers run as rotations, at 3 to 5 as fused operators: all of
    them are timed, and the batch runs what the fastest width gave."""
    n, kw = 20, {"dtype": "complex64", "max_width": 2}
    g = exchange_layers(n)
    group = {"n": n, "n_states": 1, "gates": g}
    print("autotune over widths", flush=True)
    for w in (2, 3, 4, 5):
        b = Q.Batch([group], dtype="complex64", max_width=w, tile_qubits=12)
        assert spanned(b.qsim_batch_group_stats(0)) == (w == 2)
        b.close()
    b = Q.Batch([group], autotune=True, tile_qubits=12, **kw)
    st = b.qsim_batch_group_stats(0)
    assert spanned(st) == (st["tuned_width"] == 2)
    b.qsim_batch_run()
    want, _, _ = oracle.run(n, g)
    assert norm_error(b.qsim_batch_get_state(0, 0), want) < tol("complex64", len(g))
    b.close()
    # widths 2 to 5, the three tables of the timed plans, and the program a second time
    kw["tile_qubits"] = 12
    assert attempts(Q, group, autotune=True, **kw) - attempts(Q, group, **kw) >= 4 + 3 + 1
