"""Host-only: circuits that lower to rotations run as span passes or as tiled passes
of fused operators, whichever is modelled to be cheaper; a circuit that runs once
only compares where that can repay a second compile."""
import numpy as np
import pytest

import workloads as W
from paper_2310_17739_amd import qsim
from test_host_span import spanned


def rotation_layers(n, layers=12):
    rng = np.random.default_rng(5)
    return W.gates([((W.KIND_RX, W.KIND_RY, W.KIND_RZ)[rng.integers(3)], (q,), (float(rng.normal()),))
                    for _ in range(layers) for q in range(n)])


def controlled_layers(n, layers=6):
    rng = np.random.default_rng(3)
    recs = []
    for _ in range(layers):
        recs += [(k, (q,), (float(rng.normal()),)) for k in (W.KIND_RY, W.KIND_RZ) for q in range(n)]
        recs += [(W.KIND_CRY, (q, (q + 1) % n), (float(rng.normal()),)) for q in range(n)]
    return W.gates(recs)


def exchange_layers(n, layers=6):
    recs = []
    for _ in range(layers):
        for q in range(n - 1):
            recs += [(W.KIND_RXX, (q, q + 1), (0.1,)), (W.KIND_RZZ, (q, q + 1), (0.15,))]
        recs += [(W.KIND_RY, (q,), (0.2,)) for q in range(n)]
    return W.gates(recs)


def ising_layers(n, layers=10):
    recs = []
    for _ in range(layers):
        recs += [(W.KIND_RZZ, (q, q + 1), (0.1,)) for q in range(n - 1)] + [(W.KIND_RX, (q,), (0.2,)) for q in range(n)]
    return W.gates(recs)


def qft(n):
    recs = []
    for i in range(n - 1, -1, -1):
        recs.append((W.KIND_H, (i,), ()))
        recs += [(W.KIND_CU1, (j, i), (np.pi / 2 ** (i - j),)) for j in range(i - 1, -1, -1)]
    return W.gates(recs)


def exponentials(n):
    return W.pauli_exponential_circuit(n, 200, seed=3)[0]


# run times of span passes over tiled ones at 30 qubits complex64: 2.4, 1.45, 1.6; 0.65, 0.86, 0.54
@pytest.mark.parametrize("family,spans", [(rotation_layers, False), (controlled_layers, False), (exchange_layers, False),
                                          (ising_layers, True), (qft, True), (exponentials, True)])
def test_the_cheaper_plan(family, spans, monkeypatch):
    n, dtype = 30, "complex64"
    assert spanned(qsim.qsim_debug_plan(n, family(n), dtype)) == spans
    monkeypatch.setenv("QSIM_SPAN", "2")
    assert spanned(qsim.qsim_debug_plan(n, family(n), dtype))
    monkeypatch.setenv("QSIM_SPAN", "0")
    assert not spanned(qsim.qsim_debug_plan(n, family(n), dtype))


def test_one_run_of_a_small_state_compiles_once():
    """120 us of span passes cannot repay 500 us of fusion."""
    assert spanned(qsim.qsim_debug_plan(16, rotation_layers(16), "complex64"))
    assert spanned(qsim.qsim_debug_plan(16, controlled_layers(16), "complex64"))


def test_a_qft_takes_few_rotations():
    """The single-qubit phases of its controlled ones add up: one rotation per
    controlled phase and two per qubit at most."""
    for n in (13, 20, 26):
        st = qsim.qsim_debug_plan(n, qft(n), "complex128")
        assert spanned(st) and st["fused_ops"] <= n * (n - 1) // 2 + 3 * n
