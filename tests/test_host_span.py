"""Host-only checks of Pauli programs (no GPU needed): circuits lowered to
rotations through a Clifford frame, planned into passes on subspace tiles and
run by qsim_debug_emulate from the device records, against the oracle."""
import numpy as np
import pytest

import oracle
import workloads as W
from paper_2310_17739_amd import qsim

SINGLES = [W.KIND_ID, W.KIND_H, W.KIND_X, W.KIND_Y, W.KIND_Z, W.KIND_S, W.KIND_SDG, W.KIND_T, W.KIND_TDG, W.KIND_SX,
           W.KIND_RX, W.KIND_RY, W.KIND_RZ, W.KIND_U1, W.KIND_U2, W.KIND_U3]
PAIRS = [W.KIND_CX, W.KIND_CY, W.KIND_CZ, W.KIND_SWAP, W.KIND_CRX, W.KIND_CRY, W.KIND_CRZ, W.KIND_CU1, W.KIND_RXX,
         W.KIND_RZZ]
CLIFFORD = {W.KIND_H, W.KIND_X, W.KIND_Y, W.KIND_Z, W.KIND_S, W.KIND_SDG, W.KIND_SX, W.KIND_CX, W.KIND_CY, W.KIND_CZ,
            W.KIND_SWAP}


def spanned(st):
    """A Pauli program takes none of the paper's fusion steps."""
    return st["ops_after"][1] == -1


def mixed_circuit(n, count, seed, p_clifford=0.04):
    """Gates of every kind that rotations can express, few enough of them
    Clifford gates that do not cancel; angles include the exact quarter turns
    and the neighbourhood of pi."""
    rng = np.random.default_rng(seed)
    rot = [k for k in SINGLES + PAIRS if k not in CLIFFORD and k != W.KIND_ID]
    cl = sorted(CLIFFORD)
    recs = []
    for _ in range(count):
        k = int(rng.choice(cl if rng.random() < p_clifford else rot))
        qs = [int(q) for q in rng.choice(n, W.KIND_QUBITS[k], replace=False)]
        th = rng.uniform(-2 * np.pi, 2 * np.pi, 3)
        if rng.random() < 0.2:
            th[0] = rng.choice([np.pi, -np.pi, 2 * np.pi, np.pi - 1e-9, 0.0, 1e-300])
        recs.append((k, qs, tuple(th)))
    return W.gates(recs)


def norm_error(got, want):
    return np.linalg.norm(got - want) / np.linalg.norm(want)


@pytest.mark.parametrize("dtype,n,tile", [("complex128", 14, 10), ("complex64", 15, 10), ("complex128", 15, 11),
                                          ("complex64", 16, 12), ("complex128", 16, 13), ("complex64", 17, 14)])
def test_mixed_circuits_equal_oracle(dtype, n, tile, monkeypatch):
    g = mixed_circuit(n, 160, seed=n + tile)
    psi0 = W.random_state(n, 3)
    want, _, _ = oracle.run(n, g, psi=psi0)
    st = qsim.qsim_debug_plan(n, g, dtype, tile_qubits=tile)
    assert spanned(st)
    got = qsim.qsim_debug_emulate(n, g, dtype, tile_qubits=tile, psi=psi0)
    # at most nine rotations per gate and two roundings of 2^-53 each
    assert norm_error(got, want) < 2 * 9 * 160 * 1.2e-16
    monkeypatch.setenv("QSIM_SPAN", "0")
    assert not spanned(qsim.qsim_debug_plan(n, g, dtype, tile_qubits=tile))


def test_every_kind_alone():
    """Each kind between two layers of rotations: its images in the frame, its
    phase and its cancellation against a later inverse."""
    n, tile = 15, 10
    rng = np.random.default_rng(5)
    layer = [(W.KIND_RX if q % 2 else W.KIND_RY, (q,), (float(rng.normal()),)) for q in range(n)]
    layer += [(W.KIND_RZ, (q,), (float(rng.normal()),)) for q in range(n)]
    for k in SINGLES + PAIRS:
        qs = (4, 9)[:W.KIND_QUBITS[k]]
        one = [(k, qs, (0.7, -1.1, 2.3))]
        for recs in (layer + one + layer, layer + one + [(W.KIND_RZ, (9,), (0.3,))] + one + layer):
            g = W.gates(recs)
            assert spanned(qsim.qsim_debug_plan(n, g, "complex128", tile_qubits=tile)), k
            want, _, _ = oracle.run(n, g)
            got = qsim.qsim_debug_emulate(n, g, "complex128", tile_qubits=tile)
            assert norm_error(got, want) < 1e-13, k


def test_quarter_turn_rotations_cancel():
    """exp(-i theta P / 2) written with Rx(+-pi/2) leaves nothing in the frame:
    one rotation per exponential."""
    n = 21
    g, _, strings = W.pauli_exponential_circuit(n, 500, seed=3)
    st = qsim.qsim_debug_plan(n, g, "complex128")
    assert spanned(st) and st["fused_ops"] == len(strings)


def test_left_to_the_matrix_lowering():
    """Circuits that rotations do not pay for, and options that ask for another
    plan, keep the fused operators; bad records keep their errors."""
    n = 16
    for g in (W.random_circuit(n, 300, seed=1), W.gates([(W.KIND_CCX, (0, 1, 2))] * 3)):
        assert not spanned(qsim.qsim_debug_plan(n, g, "complex128"))
    p, _, _ = W.pauli_exponential_circuit(n, 50, seed=1)
    for kw in ({"level": 4}, {"flags": qsim.F_ONE_OP_PER_PASS}, {"flags": qsim.F_NO_SPARSE},
               {"flags": qsim.F_REG_ENGINE}, {"tile_qubits": 9}):
        assert not spanned(qsim.qsim_debug_plan(n, p, "complex128", **kw))
    assert spanned(qsim.qsim_debug_plan(n, p, "complex128", flags=qsim.F_FULL_SUPPORT))
    for bad, code in (((W.KIND_RZ, (n,), (0.1,)), qsim.E_QUBIT), ((W.KIND_RZ, (0,), (np.nan,)), qsim.E_ARG),
                      ((W.KIND_CX, (2, 2), ()), qsim.E_QUBIT), ((W.KIND_RZ, (0,), (0.1,), 0), qsim.E_ARG)):
        with pytest.raises(qsim.QsimError) as e:
            qsim.qsim_debug_plan(n, np.concatenate([p, W.gates([bad])]), "complex128")
        assert e.value.code == code


@pytest.mark.parametrize("dtype,n", [("complex64", 10), ("complex128", 11), ("complex128", 13), ("complex64", 14)])
def test_whole_states_keep_a_permuting_frame(dtype, n):
    """A state that is one tile is stored through what CX, SWAP and X leave in
    the frame, whatever their number; a circuit of nothing else is one pass."""
    rng = np.random.default_rng(n)
    recs, perm = [], []
    for i in range(120):
        a, b = (int(q) for q in rng.choice(n, 2, replace=False))
        kind = [W.KIND_CX, W.KIND_SWAP, W.KIND_X][rng.integers(3)]
        perm.append((kind, (a, b)[:W.KIND_QUBITS[kind]], ()))
        recs += [perm[-1], (W.KIND_RY, (a,), (float(rng.normal()),)), (W.KIND_CRZ, (a, b), (float(rng.normal()),))]
    psi0 = W.random_state(n, 3)
    for g in (W.gates(recs), W.gates(perm)):
        st = qsim.qsim_debug_plan(n, g, dtype)
        assert spanned(st)
        want, _, _ = oracle.run(n, g, psi=psi0)
        assert norm_error(qsim.qsim_debug_emulate(n, g, dtype, psi=psi0), want) < 1e-12
    assert st["passes"] == 1 and st["fused_ops"] == 0
