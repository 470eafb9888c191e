"""Host-only: qubits that several controlled rotations, or rotations that half turns
and others separate, leave definite to the last bit."""
import numpy as np
import pytest

import workloads as W
from test_host_span import spanned
from test_host_zeros import A, B, C, check

D = 2     # a qubit in superposition


def by_cx(control, target, theta):
    """A controlled RY as it is written with CX."""
    return [(W.KIND_RY, (target,), (theta / 2,)), (W.KIND_CX, (control, target), ()), (W.KIND_RY, (target,), (-theta / 2,)),
            (W.KIND_CX, (control, target), ())]


# gates after which A is definite (B is |0>): (records, its value)
GADGETS = {
    # several controls
    "two_controls": ([(W.KIND_CRY, (B, A), (0.9,)), (W.KIND_CRY, (C, A), (0.7,)), (W.KIND_CRY, (D, A), (0.3,)),
                      (W.KIND_CRY, (C, A), (-0.7,)), (W.KIND_CRY, (D, A), (-0.3,))], 0),
    "two_controls_by_cx": (by_cx(B, A, 0.9) + by_cx(C, A, 0.7) + by_cx(B, A, -0.4) + by_cx(C, A, -0.7), 0),
    "controlled_by_the_same": ([(W.KIND_CRX, (B, A), (1.6,)), (W.KIND_RX, (B,), (0.4,)), (W.KIND_RX, (B,), (-0.4,)),
                                (W.KIND_CRX, (B, A), (1.6,))], 0),
    "two_axes": ([(W.KIND_CRX, (B, A), (1.234,)), (W.KIND_SDG, (A,), ()), (W.KIND_CRY, (B, A), (-0.9,)), (W.KIND_S, (A,), ())], 0),
    # controlled ones among others about the same axis
    "by_cx_between_ry": ([(W.KIND_RY, (A,), (0.4,))] + by_cx(B, A, 0.9) + [(W.KIND_RY, (A,), (-0.4,))], 0),
    "cry_then_ry": ([(W.KIND_CRY, (B, A), (0.9,)), (W.KIND_RY, (A,), (0.4,)), (W.KIND_CRY, (B, A), (0.5,)),
                     (W.KIND_RY, (A,), (-0.4,))], 0),
    "by_cx_and_back": (by_cx(C, A, 0.9) + by_cx(C, A, -0.9)[::-1], 0),
    "by_cx_twice": (by_cx(B, A, 0.9) + by_cx(B, A, 0.35), 0),
    "ry_to_pi_and_cry": ([(W.KIND_RY, (A,), (1.0,)), (W.KIND_CRY, (B, A), (0.3,)), (W.KIND_RY, (A,), (np.pi - 1.0,))], 1),
    # half and whole turns in between
    "u2_twice": ([(W.KIND_U2, (A,), (0.0, np.pi)), (W.KIND_U2, (A,), (0.0, np.pi))], 0),
    "u2_that_add_up": ([(W.KIND_U2, (A,), (1.1, 0.2)), (W.KIND_U2, (A,), (0.4, np.pi - 1.1))], 0),
    "whole_u1_between": ([(W.KIND_RX, (A,), (1.34,)), (W.KIND_U1, (A,), (2 * np.pi,)), (W.KIND_RX, (A,), (-1.34,))], 0),
    "half_u1_between": ([(W.KIND_RX, (A,), (0.9,)), (W.KIND_U1, (A,), (np.pi,)), (W.KIND_RX, (A,), (0.9,))], 0),
    "u3_pi_between": ([(W.KIND_RZ, (A,), (0.3,)), (W.KIND_RX, (A,), (0.9,)), (W.KIND_U3, (A,), (np.pi, 0.2, -0.4)),
                       (W.KIND_RZ, (A,), (-0.6,)), (W.KIND_RX, (A,), (0.9,)), (W.KIND_RZ, (A,), (1.1,))], 1),
}


@pytest.mark.parametrize("dtype,n,tile", [("complex128", 10, None), ("complex64", 14, None), ("complex128", 15, 11)])
@pytest.mark.parametrize("name", sorted(GADGETS))
def test_definite_qubits(dtype, n, tile, name, monkeypatch):
    monkeypatch.setenv("QSIM_SPAN", "2")   # span passes whatever they cost
    assert spanned(check(n, dtype, *GADGETS[name], tile=tile))


@pytest.mark.parametrize("dtype,n,tile", [("complex128", 10, None), ("complex64", 14, None), ("complex128", 15, 11)])
@pytest.mark.parametrize("kinds", [(W.KIND_CRY, W.KIND_CRY, W.KIND_CRY), (W.KIND_CRX, W.KIND_CRX, W.KIND_CRX), (None, None, None),
                                   (W.KIND_CRY, None, W.KIND_CRY), (W.KIND_CRX, W.KIND_CRY, W.KIND_CRX)])
def test_controls_that_are_zero(dtype, n, tile, kinds, monkeypatch):
    """Controlled rotations of one target from several qubits that are |0>, written
    as gates or with CX (None), in between rotations of the target that cancel."""
    from paper_2310_17739_amd import qsim
    monkeypatch.setenv("QSIM_SPAN", "2")
    recs = [(W.KIND_RY, (q,), (0.3 + q,)) for q in range(4, n)] + [(W.KIND_RXX, (q, q + 1), (0.7,)) for q in range(4, n - 1)]
    recs.append((W.KIND_RY, (0,), (0.8,)))
    for k, kind in enumerate(kinds):
        recs += by_cx(k + 1, 0, 0.9 - 0.35 * k) if kind is None else [(kind, (k + 1, 0), (0.9 - 0.35 * k,))]
    # (those about another axis let no rotation of the target pass)
    if W.KIND_CRX not in kinds:
        recs.append((W.KIND_RY, (0,), (-0.8,)))
    else:
        recs = [r for r in recs if r[:2] != (W.KIND_RY, (0,))]
    psi = np.zeros(1 << n, dtype=np.complex128)
    psi[0] = 1
    got = qsim.qsim_debug_emulate(n, W.gates(recs), dtype, psi=psi, tile_qubits=tile).reshape(-1, 16)
    assert np.all(got[:, 1:] == 0)


@pytest.mark.parametrize("n,tile", [(10, None), (13, 11)])
def test_half_turns_among_bound_angles(n, tile, monkeypatch):
    """Half turns that pass rotations bound per state turn their signs round."""
    import oracle
    from paper_2310_17739_amd import qsim
    from test_host_span import norm_error
    monkeypatch.setenv("QSIM_SPAN", "2")
    rng = np.random.default_rng(4)
    recs, th = [], []
    for k in range(60):
        q, r = (int(v) for v in rng.choice(n, 2, replace=False))
        kind = int(rng.choice([W.KIND_RX, W.KIND_RY, W.KIND_RZ, W.KIND_RXX, W.KIND_RZZ]))
        th.append(float(rng.normal()))
        recs.append((kind, (q, r)[:W.KIND_QUBITS[kind]], (0.0,)))
        if k % 4 == 0:
            recs.append((W.KIND_U3, (r,), (np.pi, 0.3, float(rng.normal()))))
        if k % 7 == 0:
            recs.append((W.KIND_MEASURE, (q,), (), k // 7))
    g = W.gates(recs)
    g["slot"][np.isin(g["kind"], [W.KIND_RX, W.KIND_RY, W.KIND_RZ, W.KIND_RXX, W.KIND_RZZ])] = np.arange(len(th))
    r = qsim.qsim_debug_emulate_batch(n, g, params=th, uniforms=rng.random(9), n_slots=9, tile_qubits=tile)
    want, _, p = oracle.run(n, g, params=th, forced=r["outcomes"], n_slots=9)
    # nine rotations per gate at most, two roundings of 2^-53 each, magnified by the projections
    assert r["status"] == 0 and norm_error(r["state"], want) < 2 * 9 * len(g) * 1.2e-16 / np.sqrt(np.prod(p))
