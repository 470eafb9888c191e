"""Groups of one batch beside each other: small groups, which run at the same
time on buffers of their own, and groups that share a state buffer, which run one
after another in order."""
import numpy as np
import pytest

import oracle
import workloads as W
from test_gpu_span import tol
from test_host_span import mixed_circuit, norm_error

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def Q():
    from paper_2310_17739_amd import qsim
    return qsim


@pytest.mark.parametrize("dtype", ["complex128", "complex64"])
@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("shared", ["none", "all", "part"])
def test_groups(Q, dtype, graph, shared):
    import torch
    widths = [11, 13, 13, 14, 9, 15]
    states = [3, 2, 4, 1, 5, 2]
    tdt = getattr(torch, dtype)
    scratch = torch.empty(1 << 17, dtype=tdt, device="cuda")
    groups, terms = [], []
    for i, (n, k) in enumerate(zip(widths, states)):
        terms.append(W.pauli_sum(n, 6, seed=i))
        g = {"n": n, "n_states": k, "gates": mixed_circuit(n, 120, seed=i, p_clifford=0.0), "terms": terms[i]}
        if shared == "all" or (shared == "part" and i in (1, 2, 4)):
            # "part": the ends of the buffers of groups 1, 2 and 4 overlap, the others have their own
            at = 0 if shared == "all" else {1: 0, 2: 1 << 13, 4: (5 << 13) - 100}[i]
            g["states"] = scratch[at:at + (k << n)]
        groups.append(g)
    print(f"groups dtype={dtype} graph={graph} shared={shared}", flush=True)
    b = Q.Batch(groups, dtype=dtype, use_graph=graph)
    for _ in range(3):
        b.qsim_batch_run()
        for i, g in enumerate(groups):
            r = b.qsim_batch_results(i)
            want, _, _ = oracle.run(g["n"], g["gates"])
            assert np.all(r["status"] == 0)
            # an error e of the state changes <H> by at most 2 |H| e
            e = tol(dtype, 120)
            assert np.max(np.abs(r["norms"] - 1)) < 2 * e
            assert np.max(np.abs(r["expvals"] - oracle.expval(g["n"], want, terms[i]))) < 4 * e * np.abs(terms[i]["coeff"]).sum()
            if shared == "none" or i == len(groups) - 1:
                for s in range(states[i]):
                    assert norm_error(b.qsim_batch_get_state(i, s), want) < e
    b.close()


@pytest.mark.parametrize("n", [9, 11])
@pytest.mark.parametrize("terms", [0, 1, 7])
def test_results_one_at_a_time(Q, n, terms):
    """Outputs that are not asked for (NULL) change nothing in the others."""
    import ctypes as C
    states = 5
    g = mixed_circuit(n, 40, seed=n, p_clifford=0.0)
    th = np.random.default_rng(1).normal(size=(states, 1))
    g = np.concatenate([W.gates([(W.KIND_RX, (0,), (0.0,), 0)]), g])
    group = {"n": n, "n_states": states, "gates": g, "params": th}
    if terms:
        group["terms"] = W.pauli_sum(n, terms, seed=3)
    print(f"results one at a time n={n} terms={terms}", flush=True)
    b = Q.Batch([group], dtype="complex128")
    b.qsim_batch_run()
    r = b.qsim_batch_results(0)
    for s in range(states):
        want, _, _ = oracle.run(n, g, params=th[s])
        assert abs(r["norms"][s] - 1) < 2 * tol("complex128", 41)
        e = oracle.expval(n, want, group["terms"]) if terms else 0.0
        assert abs(r["expvals"][s] - e) < 4 * tol("complex128", 41) * max(terms, 1)
    for name, at, dt in (("expvals", 4, np.float64), ("norms", 5, np.float64), ("status", 6, np.int32)):
        out = np.full(states, -7, dtype=dt)
        args = [b.h, 0, None, None, None, None, None]
        args[at] = C.c_void_p(out.ctypes.data)
        Q.check(Q.lib().qsim_batch_results(*args))
        assert np.array_equal(out, r[name])
    b.close()
