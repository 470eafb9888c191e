"""Host-only: amplitudes that a circuit leaves at exactly 0.  A reset, an assertion
and a forced outcome test for them, so a qubit that permutations, controlled gates
or cancelling rotations leave definite has to be definite to the last bit.  The
plans are emulated from their device tables, multiply-adds fused as in the kernels."""
import numpy as np
import pytest

import oracle
import workloads as W
from paper_2310_17739_amd import qsim
from test_host_span import norm_error, spanned

A, B, C = 0, 3, 7     # the ancilla that ends up definite, a qubit that is |0>, one in superposition


def surroundings(n, seed, rounds=1):
    """Rotations that leave every qubit but A and B in superposition."""
    rng = np.random.default_rng(seed)
    recs = []
    for _ in range(rounds):
        for q in range(n):
            if q not in (A, B):
                recs.append((W.KIND_RY, (q,), (float(rng.uniform(0.3, 1.2)),)))
                recs.append((W.KIND_RZ, (q,), (float(rng.normal()),)))
        for q in range(n - 1):
            if not {q, q + 1} & {A, B}:
                recs.append((W.KIND_RZZ, (q, q + 1), (float(rng.normal()),)))
                recs.append((W.KIND_RXX, (q, q + 1), (float(rng.normal()),)))
    return recs


# gates after which A is definite: (records, its value)
GADGETS = {
    # permutations that nothing cancels, between gates that keep the frame from permuting
    "x": ([(W.KIND_X, (A,), ())], 1),
    "x_beside_h": ([(W.KIND_X, (A,), ()), (W.KIND_H, (C,), ())], 1),
    "y": ([(W.KIND_Y, (A,), ())], 1),
    "rx_pi": ([(W.KIND_RX, (A,), (np.pi,))], 1),
    "ry_minus_pi": ([(W.KIND_RY, (A,), (-np.pi,))], 1),
    "cx": ([(W.KIND_X, (B,), ()), (W.KIND_CX, (B, A), ()), (W.KIND_S, (C,), ())], 1),
    "cx_from_zero": ([(W.KIND_CX, (B, A), ()), (W.KIND_H, (C,), ())], 0),
    "cy": ([(W.KIND_X, (B,), ()), (W.KIND_CY, (B, A), ())], 1),
    "cz_between": ([(W.KIND_X, (A,), ()), (W.KIND_CZ, (A, C), ()), (W.KIND_SWAP, (A, B), ())], 0),
    "swap": ([(W.KIND_X, (B,), ()), (W.KIND_SWAP, (A, B), ()), (W.KIND_SX, (C,), ())], 1),
    # controlled rotations whose control is |0>
    "crx": ([(W.KIND_CRX, (B, A), (0.7,))], 0),
    "cry": ([(W.KIND_CRY, (B, A), (-1.9,))], 0),
    "cry_after_x": ([(W.KIND_X, (A,), ()), (W.KIND_CRY, (B, A), (2.6,))], 1),
    "crx_many": ([(W.KIND_CRX, (B, A), (0.1 + 0.3 * i,)) for i in range(5)] + [(W.KIND_CRY, (B, A), (0.9,))], 0),
    "crz_between_h": ([(W.KIND_H, (A,), ()), (W.KIND_CRZ, (B, A), (1.3,)), (W.KIND_H, (A,), ())], 0),
    "cry_along_a_frame": ([(W.KIND_CX, (C, A), ()), (W.KIND_CRY, (B, A), (0.8,)), (W.KIND_CX, (C, A), ())], 0),
    "rxx_pi": ([(W.KIND_RXX, (A, B), (np.pi,)), (W.KIND_H, (C,), ())], 1),
    # whole and half turns
    "rx_two_pi": ([(W.KIND_RX, (A,), (2 * np.pi,))], 0),
    "ry_minus_four_pi": ([(W.KIND_RY, (A,), (-4 * np.pi,))], 0),
    "ry_three_pi": ([(W.KIND_RY, (A,), (3 * np.pi,))], 1),
    "rx_next_to_nothing": ([(W.KIND_RX, (A,), (1e-100,))], 0),
    "u3_pi": ([(W.KIND_U3, (A,), (np.pi, 0.0, np.pi))], 1),
    "crx_two_pi": ([(W.KIND_CRX, (C, A), (2 * np.pi,))], 0),
    # rotations that cancel
    "rx_back": ([(W.KIND_RX, (A,), (0.7,))] + surroundings(8, 5) + [(W.KIND_RX, (A,), (-0.7,))], 0),
    "u3_back": ([(W.KIND_U3, (A,), (0.7, 0.3, -1.1)), (W.KIND_U3, (A,), (-0.7, 1.1, -0.3))], 0),
    "ry_in_three": ([(W.KIND_RY, (A,), (0.3,)), (W.KIND_RY, (A,), (0.5,)), (W.KIND_RY, (A,), (-0.8,))], 0),
    "ry_to_pi": ([(W.KIND_RY, (A,), (1.0,)), (W.KIND_RY, (A,), (np.pi - 1.0,))], 1),
    "rxx_back": ([(W.KIND_RXX, (A, C), (0.4,)), (W.KIND_RZ, (C,), (0.0,)), (W.KIND_RXX, (C, A), (-0.4,))], 0),
    "cry_back": ([(W.KIND_CRY, (C, A), (0.9,)), (W.KIND_CRY, (C, A), (-0.9,))], 0),
    "cry_between_ry": ([(W.KIND_RY, (A,), (0.4,)), (W.KIND_CRY, (C, A), (0.9,)), (W.KIND_CRY, (C, A), (-0.9,)),
                        (W.KIND_RY, (A,), (-0.4,))], 0),
    # a controlled rotation and a hopping term, written with CX and basis changes
    "cry_by_cx": ([(W.KIND_RY, (A,), (0.45,)), (W.KIND_CX, (B, A), ()), (W.KIND_RY, (A,), (-0.45,)),
                   (W.KIND_CX, (B, A), ())], 0),
    "hop": ([(W.KIND_RXX, (A, B), (0.6,)), (W.KIND_RX, (A,), (np.pi / 2,)), (W.KIND_RX, (B,), (np.pi / 2,)),
             (W.KIND_RZZ, (A, B), (0.6,)), (W.KIND_RX, (A,), (-np.pi / 2,)), (W.KIND_RX, (B,), (-np.pi / 2,))], 0),
}


def check(n, dtype, recs, value, tile=None):
    g = W.gates(surroundings(n, 1, 2) + list(recs))
    psi = np.zeros(1 << n, dtype=np.complex128)
    psi[0] = 1
    got = qsim.qsim_debug_emulate(n, g, dtype, psi=psi, tile_qubits=tile)
    want, _, _ = oracle.run(n, g)
    assert norm_error(got, want) < 2 * 9 * len(g) * 1.2e-16
    other = got.reshape(-1, 2)[:, 1 - value]
    assert np.all(other == 0)
    # with records: a reset succeeds, the other outcome has probability 0
    after = W.gates(surroundings(n, 1, 2) + list(recs) + [(W.KIND_RESET, (A,), ())] + surroundings(n, 2))
    r = qsim.qsim_debug_emulate_batch(n, after, dtype, tile_qubits=tile)
    want, _, _ = oracle.run(n, W.gates(surroundings(n, 1, 2) + list(recs) + [(W.KIND_X, (A,), ())] * value + surroundings(n, 2)))
    assert r["status"] == 0 and norm_error(r["state"], want) < 2 * 9 * len(after) * 1.2e-16
    for forced in (value, 1 - value):
        m = W.gates(surroundings(n, 1, 2) + list(recs) + [(W.KIND_MEASURE, (A,), (), 0)])
        r = qsim.qsim_debug_emulate_batch(n, m, dtype, uniforms=[0.5], forced=[forced], n_slots=1, tile_qubits=tile)
        assert r["status"] == (0 if forced == value else qsim.E_ZERO_PROB)
        if forced == value:
            assert r["probs"][0] == 1.0
    m = W.gates(surroundings(n, 1, 2) + list(recs) + [(W.KIND_ASSERT0, (A,), (), 0)])
    r = qsim.qsim_debug_emulate_batch(n, m, dtype, n_slots=1, tile_qubits=tile)
    assert r["status"] == (0 if value == 0 else qsim.E_ZERO_PROB)
    return qsim.qsim_debug_plan(n, g, dtype, tile_qubits=tile)


@pytest.mark.parametrize("dtype,n,tile", [("complex128", 10, None), ("complex64", 14, None), ("complex128", 15, 11)])
@pytest.mark.parametrize("name", sorted(GADGETS))
def test_definite_qubits(dtype, n, tile, name, monkeypatch):
    monkeypatch.setenv("QSIM_SPAN", "2")   # span passes whatever they cost
    assert spanned(check(n, dtype, *GADGETS[name], tile=tile))



@pytest.mark.parametrize("n", [10, 16])
def test_a_circuit_and_its_inverse_leave_nothing(n):
    """Whatever the number of distinct strings."""
    g, _, _ = W.pauli_exponential_circuit(n, 3000, seed=2)
    both = np.concatenate([g, W.inverse_circuit(g)])
    st = qsim.qsim_debug_plan(n, both, "complex128")
    assert spanned(st) and st["fused_ops"] == 0 and st["passes"] == 0


@pytest.mark.parametrize("n", [10, 15])
def test_nothing_but_a_phase(n):
    psi0 = W.random_state(n, 3)
    for recs in ([(W.KIND_RX, (1,), (2 * np.pi,))], [(W.KIND_RZZ, (1, 4), (-2 * np.pi,)), (W.KIND_RY, (3,), (6 * np.pi,))],
                 [(W.KIND_RX, (2,), (2 * np.pi,)), (W.KIND_X, (2,), ()), (W.KIND_RX, (2,), (2 * np.pi,))],
                 [(W.KIND_RY, (2,), (2 * np.pi,)), (W.KIND_RZ, (1,), (0.0,))]):
        g = W.gates(recs)
        want, _, _ = oracle.run(n, g, psi=psi0)
        # a few roundings of 2^-53 each
        assert norm_error(qsim.qsim_debug_emulate(n, g, psi=psi0), want) < 1e-15


@pytest.mark.parametrize("dtype,n", [("complex128", 11), ("complex64", 15), ("complex128", 17)])
@pytest.mark.parametrize("seed", range(4))
def test_rotations_that_add_up(dtype, n, seed):
    """Few strings, repeated with angles that cancel, add up to half turns or do
    neither, controlled or not, between gates that commute with some of them."""
    rng = np.random.default_rng(seed)
    angles = [0.3, -0.3, 0.9, -0.9, np.pi, -np.pi, np.pi / 2, 2 * np.pi, np.pi - 0.3, 0.0]
    recs = []
    for _ in range(200):
        k = int(rng.choice([W.KIND_RX, W.KIND_RY, W.KIND_RZ, W.KIND_RXX, W.KIND_RZZ, W.KIND_CRX, W.KIND_CRY, W.KIND_CRZ, W.KIND_CU1,
                            W.KIND_U3, W.KIND_T, W.KIND_TDG, W.KIND_CX]))
        if k == W.KIND_CX and rng.random() < 0.7:
            continue
        qs = tuple(int(q) for q in rng.choice(4, W.KIND_QUBITS[k], replace=False) * 3)
        recs.append((k, qs, tuple(float(a) for a in rng.choice(angles, 3))))
    g = W.gates(recs)
    psi0 = W.random_state(n, seed)
    want, _, _ = oracle.run(n, g, psi=psi0)
    got = qsim.qsim_debug_emulate(n, g, dtype, psi=psi0, tile_qubits=None if n < 15 else 11)
    # at most nine rotations per gate and two roundings of 2^-53 each
    assert norm_error(got, want) < 2 * 9 * len(g) * 1.2e-16
