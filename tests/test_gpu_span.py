"""Passes of Pauli rotations (k_span) against the oracle: every tile width,
one and several stages, angles whose cosine vanishes, initial |0...0>, per-state
angles, and measurements between passes."""
import numpy as np
import pytest

import oracle
import workloads as W
from test_host_span import mixed_circuit, norm_error, spanned

pytestmark = pytest.mark.gpu
# norm of the rounding errors: at most two roundings per rotation and at most
# nine rotations per gate, each 2^-53 or 2^-24 of an amplitude
EPS = {"complex128": 1.2e-16, "complex64": 6e-8}


def tol(dtype, gates):
    return 2 * 9 * gates * EPS[dtype]


@pytest.fixture(scope="module")
def Q():
    from paper_2310_17739_amd import qsim
    return qsim


@pytest.mark.parametrize("dtype,n,tile", [("complex128", 14, 10), ("complex128", 15, 11), ("complex128", 16, 12),
                                          ("complex128", 17, 13), ("complex64", 15, 10), ("complex64", 16, 11),
                                          ("complex64", 15, 12), ("complex64", 16, 13), ("complex64", 17, 14)])
@pytest.mark.parametrize("count", [1, 5, 150])
def test_tile_widths(Q, dtype, n, tile, count):
    g = mixed_circuit(n, count, seed=tile + count, p_clifford=0.0 if count < 10 else 0.04)
    psi0 = W.random_state(n, 7)
    print(f"span tile dtype={dtype} n={n} tile={tile} gates={count}", flush=True)
    sv = Q.StateVector(n, dtype)
    sv.qsim_set_state(psi0)
    sv.qsim_apply(g, tile_qubits=tile)
    assert spanned(sv.qsim_last_stats())
    want, _, _ = oracle.run(n, g, psi=psi0.astype(dtype).astype(np.complex128))
    assert norm_error(sv.qsim_get_state(), want) < tol(dtype, count)
    sv.close()


@pytest.mark.parametrize("dtype", ["complex128", "complex64"])
def test_templates_with_any_angles(Q, dtype):
    """Per-state angles, bound on the device, from 0 to beyond a whole turn."""
    n, nexp, states = 15, 60, 5
    rng = np.random.default_rng(2)
    recs = []
    for e, (qs, letters) in enumerate(W.pauli_strings(n, nexp, rng)):
        W.compile_pauli_exponential(qs, letters, 0.0, e, recs)
    g = W.gates(recs)
    th = rng.uniform(-7, 7, (states, nexp))
    th[0] = np.pi
    th[1, ::2] = 0.0
    th[2] = np.pi / 2
    print(f"span template dtype={dtype}", flush=True)
    b = Q.Batch([{"n": n, "n_states": states, "gates": g, "params": th}], dtype=dtype, tile_qubits=11)
    assert spanned(b.qsim_batch_group_stats(0))
    b.qsim_batch_run()
    assert np.all(b.qsim_batch_results(0)["status"] == 0)
    for s in range(states):
        want, _, _ = oracle.run(n, g, params=th[s])
        assert norm_error(b.qsim_batch_get_state(0, s), want) < tol(dtype, nexp)
    b.close()


@pytest.mark.parametrize("dtype", ["complex128", "complex64"])
def test_measurements_between_passes(Q, dtype):
    """The projection filter as a batch: assertions and resets between the
    passes of rotations."""
    g, info = W.projection_filter(14, 3, seed=5, delta=0.3)
    n = info["n"]
    print(f"span filter dtype={dtype}", flush=True)
    b = Q.Batch([{"n": n, "n_states": 2, "gates": g, "n_slots": 3}], dtype=dtype, tile_qubits=11)
    assert spanned(b.qsim_batch_group_stats(0))
    b.qsim_batch_run()
    r = b.qsim_batch_results(0)
    want, _, p = oracle.run(n, g)
    assert np.all(r["status"] == 0)
    for s in range(2):
        # a projection onto a branch of probability p magnifies an error by 1 / sqrt(p)
        grow = 1 / np.sqrt(np.prod(p))
        assert np.max(np.abs(r["probs"][s] - p)) < 2 * grow * tol(dtype, 3 * 16)
        assert norm_error(b.qsim_batch_get_state(0, s), want) < grow * tol(dtype, 3 * 16)
    b.close()


@pytest.mark.parametrize("dtype", ["complex128", "complex64"])
@pytest.mark.parametrize("n", [9, 10, 11, 12, 13, 18])
@pytest.mark.parametrize("count", [1, 70, 300])
def test_pauli_sums(Q, dtype, n, count):
    """Terms of any weight, several groups and stages, X masks that repeat, the
    identity and diagonals; one state and a batch of two."""
    rng = np.random.default_rng(n + count)
    t = np.zeros(count, dtype=W.PAULI_DTYPE)
    t["xmask"] = rng.integers(0, 1 << n, count)
    t["zmask"] = rng.integers(0, 1 << n, count)
    t["xmask"][::5] = 0
    t["xmask"][1::7] = t["xmask"][min(1, count - 1)]
    t["zmask"][::15] = 0
    t["coeff"] = rng.normal(size=count)
    psi = (1.5 * W.random_state(n, 4)).astype(dtype)
    print(f"span pauli sum dtype={dtype} n={n} terms={count}", flush=True)
    sv = Q.StateVector(n, dtype)
    sv.qsim_set_state(psi)
    want = oracle.expval(n, psi.astype(np.complex128), t)
    # FP64 sums of at most a few hundred partial sums each: 2^-53 of each partial
    assert abs(sv.qsim_expval(t) - want) < 1e-13 * np.abs(t["coeff"]).sum()
    for k in range(min(count, 4)):
        one = t[k:k + 1]
        assert abs(sv.qsim_expval(one) - oracle.expval(n, psi.astype(np.complex128), one)) < 1e-13 * abs(one["coeff"][0])
    sv.close()
    g = mixed_circuit(n, 30, seed=n, p_clifford=0.0)
    b = Q.Batch([{"n": n, "n_states": 2, "gates": g, "terms": t}], dtype=dtype)
    b.qsim_batch_run()
    r = b.qsim_batch_results(0)
    for s in range(2):
        psi = b.qsim_batch_get_state(0, s).astype(np.complex128)
        assert abs(r["expvals"][s] - oracle.expval(n, psi, t)) < 1e-13 * np.abs(t["coeff"]).sum()
        assert abs(r["norms"][s] - np.vdot(psi, psi).real) < 1e-13
    b.close()


@pytest.mark.parametrize("dtype", ["complex128", "complex64"])
def test_growth_before_scaling(Q, dtype):
    """One pass of the largest growth: rotations by 45 degrees bound per state,
    a fixed one just under the limit, and cosines that vanish."""
    n, count = 12, 94
    rng = np.random.default_rng(8)
    recs = [(W.KIND_RX, (0,), (np.pi - 2.0 ** -18,))]
    for e, (qs, letters) in enumerate(W.pauli_strings(n, count - 2, rng)):
        W.compile_pauli_exponential(qs, letters, 0.0, e, recs)
    recs.append((W.KIND_RX, (1,), (np.pi,)))
    g = W.gates(recs)
    th = np.full((2, count - 2), np.pi / 2)
    th[1, 1::2] = np.pi
    print(f"span growth dtype={dtype}", flush=True)
    b = Q.Batch([{"n": n, "n_states": 2, "gates": g, "params": th}], dtype=dtype)
    assert spanned(b.qsim_batch_group_stats(0))
    b.qsim_batch_run()
    for s in range(2):
        want, _, _ = oracle.run(n, g, params=th[s])
        assert norm_error(b.qsim_batch_get_state(0, s), want) < tol(dtype, count)
    b.close()


def measured_program(n, rounds, seed):
    """Rotations and a frame of CX, SWAP and X that no record undoes; per round a
    measurement, a measured and reset qubit, an assertion, and a reset after it."""
    rng = np.random.default_rng(seed)
    recs, slot = [], 0
    for _ in range(rounds):
        for q in range(n):
            recs.append((W.KIND_RY, (q,), (float(rng.uniform(0.4, 1.2)),)))
            if rng.random() < 0.5:
                recs.append((W.KIND_RZ, (q,), (float(rng.normal()),)))
        for _ in range(n):
            a, b = (int(q) for q in rng.choice(n, 2, replace=False))
            k = [W.KIND_CX, W.KIND_CX, W.KIND_SWAP, W.KIND_X, W.KIND_CRY][rng.integers(5)]
            recs.append((k, (a, b)[:W.KIND_QUBITS[k]], (float(rng.normal()),) if k == W.KIND_CRY else ()))
        a, b, c = (int(q) for q in rng.choice(n, 3, replace=False))
        recs += [(W.KIND_MEASURE, (a,), (), slot), (W.KIND_MEASURE, (b,), (), slot + 1), (W.KIND_RESET, (b,), ()),
                 (W.KIND_BARRIER, (), ()), (W.KIND_ASSERT0, (c,), (), slot + 2), (W.KIND_RESET, (c,), ())]
        slot += 3
    return W.gates(recs), slot


@pytest.mark.parametrize("dtype,n", [("complex128", 10), ("complex64", 10), ("complex128", 11), ("complex64", 12),
                                     ("complex128", 13), ("complex64", 13), ("complex64", 14)])
def test_records_inside_whole_states(Q, dtype, n):
    rounds, states = 3, 6
    g, slots = measured_program(n, rounds, seed=n)
    u = np.random.default_rng(n + 1).random((states, slots))
    print(f"span records dtype={dtype} n={n}", flush=True)
    b = Q.Batch([{"n": n, "n_states": states, "gates": g, "uniforms": u, "n_slots": slots}], dtype=dtype)
    assert spanned(b.qsim_batch_group_stats(0))
    for _ in range(2):
        b.qsim_batch_run()
        r = b.qsim_batch_results(0)
        for s in range(states):
            assert r["status"][s] == 0
            want, o, p = oracle.run(n, g, forced=r["outcomes"][s])
            grow = 1 / np.sqrt(np.prod(p))
            err = grow * tol(dtype, len(g))
            assert np.max(np.abs(r["probs"][s] - p)) < 2 * err
            drawn = np.array([u[s][k] for k in range(slots)])
            clear = np.abs(drawn - np.where(o == 0, p, 1 - p)) > 2 * err
            is_measure = np.arange(slots) % 3 != 2
            assert np.all((r["outcomes"][s] == np.where(drawn < np.where(o == 0, p, 1 - p), 0, 1))[clear & is_measure])
            assert norm_error(b.qsim_batch_get_state(0, s), want) < err
    b.close()


@pytest.mark.parametrize("dtype", ["complex128", "complex64"])
@pytest.mark.parametrize("bad", ["assert", "reset", "forced"])
def test_failing_records_keep_the_state(Q, dtype, bad):
    """A record that fails leaves its state as it was before, in the order of the
    qubits that the gates before it left, and touches no other state."""
    n = 11
    g, slots = measured_program(n, 1, seed=3)
    head = g[g["kind"] != W.KIND_BARRIER][:-5]
    tail, _ = measured_program(n, 1, seed=4)
    tail = tail[(tail["kind"] < W.KIND_BARRIER)]
    # qubit 5 is |1> for certain, then carried on by the frame
    fixed = W.gates([(W.KIND_MEASURE, (5,), (), 0), (W.KIND_RESET, (5,), ()), (W.KIND_X, (5,), ()), (W.KIND_SWAP, (5, 8), ())])
    rec = {"assert": (W.KIND_ASSERT0, (8,), (), 1), "reset": (W.KIND_RESET, (3,), ()), "forced": (W.KIND_MEASURE, (8,), (), 1)}[bad]
    head = head[head["kind"] < W.KIND_BARRIER]
    prog = np.concatenate([head, fixed, W.gates([rec]), tail])
    forced = np.array([[0, 0], [1, 1]], dtype=np.int32)
    print(f"span failing record dtype={dtype} {bad}", flush=True)
    b = Q.Batch([{"n": n, "n_states": 2, "gates": prog, "uniforms": np.full((2, 2), 0.25), "forced": forced, "n_slots": 2}], dtype=dtype)
    assert spanned(b.qsim_batch_group_stats(0))
    b.qsim_batch_run()
    r = b.qsim_batch_results(0)
    code = Q.E_NOT_DEFINITE if bad == "reset" else Q.E_ZERO_PROB
    for s in range(2):
        fails = bad != "forced" or s == 0
        assert r["status"][s] == (code if fails else 0)
        upto = np.concatenate([head, fixed]) if fails else prog
        want, _, _ = oracle.run(n, upto, forced=forced[s], n_slots=2)
        assert norm_error(b.qsim_batch_get_state(0, s), want) < 4 * tol(dtype, len(prog))
    b.close()
