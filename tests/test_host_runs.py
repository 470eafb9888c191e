"""Runs of dense 2-qubit operators (one trip through LDS for those on four
positions together): the packed plan emulated on the CPU against the oracle."""
import numpy as np
import pytest

import oracle
import workloads as W
from paper_2310_17739_amd import qsim


def dense_pairs(n, layout, seed):
    """Random 2-qubit unitaries: layers on neighbours ("brick"), any pairs in any
    qubit order with 1- and 3-qubit ones between them ("mixed"), or often the same
    pair or three qubits ("few")."""
    rng = np.random.default_rng(seed)
    if layout == "brick":
        sites = [(q, q + 1) for layer in range(6) for q in range(layer % 2, n - 1, 2)]
    elif layout == "mixed":
        sites = [tuple(int(q) for q in rng.choice(n, size=k, replace=False)) for k in rng.choice([1, 2, 2, 2, 3], size=60)]
    else:
        sites = [tuple(int(q) for q in rng.permutation(3)[:2] + n - 3) for _ in range(20)]
    recs, mats = [], []
    for i, qs in enumerate(sites):
        d = 1 << len(qs)
        u, _ = np.linalg.qr(rng.normal(size=(d, d)) + 1j * rng.normal(size=(d, d)))
        recs.append((W.KIND_MAT, qs, ()))
        mats.append(u)
    return recs, mats


def records(recs, mats):
    g = W.gates(recs)
    off = 0
    for i, m in enumerate(mats):
        g["mat_off"][i] = off
        off += m.size
    return g, np.concatenate([m.ravel() for m in mats])


CASES = [("complex64", 12, None), ("complex64", 14, 12), ("complex64", 15, 13), ("complex64", 14, None), ("complex64", 13, 11),
         ("complex128", 12, None), ("complex128", 14, 12), ("complex128", 13, None), ("complex128", 14, 13)]


@pytest.mark.parametrize("dtype,n,tile", CASES)
@pytest.mark.parametrize("layout", ["brick", "mixed", "few"])
@pytest.mark.parametrize("width", [2, 4])
def test_runs_equal_the_oracle(dtype, n, tile, layout, width):
    g, mats = records(*dense_pairs(n, layout, n))
    psi0 = W.random_state(n, 3)
    want, _, _ = oracle.run(n, g, mats=mats, psi=psi0)
    got = qsim.qsim_debug_emulate(n, g, dtype, mats=mats, psi=psi0, tile_qubits=tile, max_width=width)
    # FP64 throughout; coefficients are FP64 for both types here
    assert np.max(np.abs(got - want)) < 1e-12
