"""Runs of dense 2-qubit operators in k_tile against the oracle: every tile width
that takes them, initial |0...0>, and records between them."""
import numpy as np
import pytest

import oracle
import workloads as W
from test_host_runs import CASES, dense_pairs, records

pytestmark = pytest.mark.gpu
# per operator a sum of at most 2^3 products: at most 2 * 8 roundings, each 2^-53
# or 2^-24 of an amplitude
EPS = {"complex128": 1.2e-16, "complex64": 6e-8}


@pytest.fixture(scope="module")
def Q():
    from paper_2310_17739_amd import qsim
    return qsim


@pytest.mark.parametrize("dtype,n,tile", CASES)
@pytest.mark.parametrize("layout", ["brick", "mixed", "few"])
def test_runs(Q, dtype, n, tile, layout):
    recs, m = dense_pairs(n, layout, n + 1)
    g, mats = records(recs, m)
    psi0 = W.random_state(n, 5)
    print(f"runs dtype={dtype} n={n} tile={tile} {layout}", flush=True)
    sv = Q.StateVector(n, dtype)
    for psi in (None, psi0):
        if psi is None:
            sv.qsim_init_zero()
        else:
            sv.qsim_set_state(psi)
        sv.qsim_apply(g, mats=mats, tile_qubits=tile, max_width=2 if layout == "mixed" else 4)
        want, _, _ = oracle.run(n, g, mats=mats, psi=None if psi is None else psi.astype(dtype).astype(np.complex128))
        assert np.linalg.norm(sv.qsim_get_state() - want) < 16 * len(g) * EPS[dtype]
    sv.close()


@pytest.mark.parametrize("dtype,n", [("complex64", 12), ("complex64", 14), ("complex128", 12)])
def test_runs_between_records(Q, dtype, n):
    """A whole state in one tile, three states, measurements with forced outcomes
    between the layers."""
    recs, m = dense_pairs(n, "brick", n + 2)
    half = len(recs) // 2
    recs = recs[:half] + [(W.KIND_MEASURE, (1,), (), 0)] + recs[half:] + [(W.KIND_MEASURE, (n - 1,), (), 1)]
    g, mats = records(recs, m[:half] + [np.zeros(0)] + m[half:] + [np.zeros(0)])
    forced = np.array([[0, 1], [1, 0], [1, 1]], dtype=np.int32)
    print(f"runs and records dtype={dtype} n={n}", flush=True)
    b = Q.Batch([{"n": n, "n_states": 3, "gates": g, "mats": mats, "forced": forced, "uniforms": np.zeros((3, 2)), "n_slots": 2}], dtype=dtype)
    b.qsim_batch_run()
    r = b.qsim_batch_results(0)
    assert np.all(r["status"] == 0)
    for s in range(3):
        want, _, p = oracle.run(n, g, mats=mats, forced=forced[s])
        # a projection onto a branch of probability p magnifies an error by 1 / sqrt(p)
        grow = 1 / np.sqrt(np.prod(p))
        assert np.linalg.norm(b.qsim_batch_get_state(0, s) - want) < grow * 16 * len(g) * EPS[dtype]
    b.close()
