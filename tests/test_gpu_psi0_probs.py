"""GPU parity of vqc_forward_ex: the optional initial state Psi_0 (Algorithm 1)
and the basis-state probabilities of the final state (Sec. 3), against the
double-precision oracle.

Bars: E as in the other parity tests (max abs 1e-5).  Probabilities: max abs
1e-5 per entry; since E_j is a signed sum of the probabilities, an error bar on
E of 1e-5 leaves each probability within the same bar whatever the state's
spread, and fp32 arithmetic on a unit-norm state stays far inside it at these
depths.  Gradients after a Psi_0 forward: the row max-norm bar of the other
parity tests.  Psi_0 is drawn in complex64 and reaches both sides as the same
values.
"""
import sys

import numpy as np
import pytest

import oracle
from paper_2607_11985_amd import workloads as W

pytestmark = pytest.mark.gpu

E_TOL = 1e-5
P_TOL = 1e-5
G_REL = 1e-4
G_FLOOR = 1e-6


@pytest.fixture(scope="module")
def torch_mod():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2607_11985_amd import _lib
    _lib.load()
    return torch


def note(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def run_ex(torch, ops, n, P, F, p, x, psi0, path="auto", engine="jit", training=False,
           want_E=True, want_probs=True):
    from paper_2607_11985_amd.api import Circuit
    circ = Circuit(ops, n, P, F, path=path, engine=engine)
    tp = torch.from_numpy(np.ascontiguousarray(p)).cuda()
    tx = torch.from_numpy(np.ascontiguousarray(x)).cuda()
    ts = torch.from_numpy(np.ascontiguousarray(psi0)).cuda() if psi0 is not None else None
    out = circ.forward_ex(tp, tx, ts, expvals=want_E, probs=want_probs, training=training)
    torch.cuda.synchronize()
    res = {"circ": circ, "p": tp, "x": tx}
    res["E"] = out[0].cpu().numpy() if out[0] is not None else None
    res["probs"] = out[1].cpu().numpy() if out[1] is not None else None
    if training:
        res["ws"] = out[2]
    return res


def check(a, ref, tol, what):
    err = float(np.max(np.abs(a.astype(np.float64) - ref))) if a.size else 0.0
    assert err <= tol, f"{what} max abs err {err:.3e}"
    return err


@pytest.mark.parametrize("n,B,kind", [(1, 5, "haar"), (2, 33, "haar"), (3, 37, "basis"),
                                      (4, 37, "haar"), (6, 9, "sparse"), (8, 7, "haar"),
                                      (9, 5, "haar"), (10, 4, "basis"), (12, 3, "haar"),
                                      (13, 2, "sparse")])
def test_resident_psi0_probs(torch_mod, n, B, kind):
    """Several samples per workgroup and a ragged last workgroup (small n), padding
    qubits (n < 4), and the tangent-form kernels (n >= 9)."""
    ops, P, F = W.random_circuit(n, 14 * n + 6, seed=300 + n)
    p, x = W.random_inputs(B, P, F, seed=310 + n)
    s0 = W.random_states(B, n, seed=320 + n, kind=kind)
    note(f"resident psi0 n={n} B={B} kind={kind}")
    r = run_ex(torch_mod, ops, n, P, F, p, x, s0)
    Er, st = oracle.forward(ops, n, p, x, want_state=True, psi0=s0)
    check(r["E"], Er, E_TOL, "E")
    check(r["probs"], np.abs(st) ** 2, P_TOL, "probs")


@pytest.mark.parametrize("n,B", [(5, 11), (11, 3), (14, 2)])
def test_probs_from_zero_state(torch_mod, n, B):
    """Probabilities without Psi_0 (the state starts from |0...0>); expvals not asked."""
    ops, P, F = W.random_circuit(n, 12 * n, seed=330 + n)
    p, x = W.random_inputs(B, P, F, seed=340 + n)
    note(f"probs from |0> n={n} B={B}")
    r = run_ex(torch_mod, ops, n, P, F, p, x, None, want_E=False)
    assert r["E"] is None
    check(r["probs"], oracle.probabilities(ops, n, p, x), P_TOL, "probs")


@pytest.mark.parametrize("n,B,path", [(14, 3, "stream"), (15, 2, "auto"), (16, 2, "auto")])
def test_streaming_psi0_probs(torch_mod, n, B, path):
    ops, P, F = W.random_circuit(n, 8 * n, seed=350 + n)
    p, x = W.random_inputs(B, P, F, seed=360 + n)
    s0 = W.random_states(B, n, seed=370 + n)
    note(f"streaming psi0 n={n} B={B} path={path}")
    r = run_ex(torch_mod, ops, n, P, F, p, x, s0, path=path)
    assert r["circ"].info()["path"] == 2
    Er, st = oracle.forward(ops, n, p, x, want_state=True, psi0=s0)
    check(r["E"], Er, E_TOL, "E")
    check(r["probs"], np.abs(st) ** 2, P_TOL, "probs")


@pytest.mark.parametrize("n,layers,B", [(14, 4, 517), (16, 4, 17), (17, 3, 9), (20, 2, 2)])
def test_streaming_probs_out_of_order(torch_mod, n, layers, B):
    """Entangled circuits whose last pass covers few entries of a line of the
    probabilities: from 2^20 (2^23 at 14 qubits) amplitudes on order_kernel puts them in
    order, below the pass stores them itself.  From an inference and a training call,
    whose backward then runs, with and without Psi_0; the first, a middle and the last
    row against the oracle, and the first rows equal bit for bit from a batch below
    the line."""
    torch = torch_mod
    from paper_2607_11985_amd.api import Circuit
    ops, P, F = W.strongly_entangling_circuit(n, layers)
    rows = sorted({0, B // 2, B - 1})
    p, x = W.random_inputs(B, P, F, seed=390 + n)
    cot = W.random_cotangent(B, n, seed=391 + n)
    states = W.random_states(len(rows), n, seed=392 + n)
    circ = Circuit(ops, n, P, F, path="stream")
    tp, tx, tg = (torch.from_numpy(np.ascontiguousarray(v)).cuda() for v in (p, x, cot))
    for s0 in (None, states):
        note(f"ordered probs n={n} layers={layers} B={B} psi0={s0 is not None}")
        ts = None
        if s0 is not None:
            ts = torch.from_numpy(s0).cuda()[torch.arange(B) % len(rows)]
            ts[rows] = torch.from_numpy(s0).cuda()
        dpr, _, Er = oracle.vjp(ops, n, p[rows], x[rows], cot[rows], psi0=s0)
        _, st = oracle.forward(ops, n, p[rows], x[rows], want_state=True, psi0=s0)
        E, pr = circ.forward_ex(tp, tx, ts, probs=True)
        E2, pr2, ws = circ.forward_ex(tp, tx, ts, probs=True, training=True)
        dp, _ = circ.backward(tp, tx, tg, ws)
        E1, pr1 = circ.forward_ex(tp[:1], tx[:1], None if ts is None else ts[:1], probs=True)
        torch.cuda.synchronize()
        assert torch.equal(E, E2) and torch.equal(pr, pr2)
        if n < 20:
            assert torch.equal(E1, E[:1]) and torch.equal(pr1, pr[:1])
        check(E[rows].cpu().numpy(), Er, E_TOL, "E")
        check(pr[rows].cpu().numpy(), np.abs(st) ** 2, P_TOL, "probs")
        err = np.max(np.abs(dp[rows].cpu().numpy() - dpr), axis=1)
        assert np.all(err <= G_REL * np.max(np.abs(dpr), axis=1)
                      + G_FLOOR * np.sum(np.abs(cot[rows]), axis=1)), err


@pytest.mark.parametrize("n,path", [(5, "auto"), (10, "auto"), (14, "stream")])
def test_interpreter_psi0_probs(torch_mod, n, path):
    ops, P, F = W.random_circuit(n, 10 * n, seed=380 + n)
    B = 4
    p, x = W.random_inputs(B, P, F, seed=390 + n)
    s0 = W.random_states(B, n, seed=400 + n)
    note(f"interpreter psi0 n={n} path={path}")
    r = run_ex(torch_mod, ops, n, P, F, p, x, s0, path=path, engine="interp")
    Er, st = oracle.forward(ops, n, p, x, want_state=True, psi0=s0)
    check(r["E"], Er, E_TOL, "E")
    check(r["probs"], np.abs(st) ** 2, P_TOL, "probs")


@pytest.mark.parametrize("n,path,engine", [(4, "auto", "jit"), (9, "auto", "jit"),
                                           (12, "auto", "interp"), (14, "stream", "jit")])
def test_gradients_after_psi0_forward(torch_mod, n, path, engine):
    """A training forward from Psi_0 saves the final state; the adjoint then gives
    the gradients of that forward (Psi_0 fixed)."""
    ops, P, F = W.random_circuit(n, 10 * n, seed=410 + n)
    B = 3
    p, x = W.random_inputs(B, P, F, seed=420 + n)
    s0 = W.random_states(B, n, seed=430 + n)
    cot = W.random_cotangent(B, n, seed=440 + n)
    note(f"gradients after psi0 forward n={n} path={path} engine={engine}")
    r = run_ex(torch_mod, ops, n, P, F, p, x, s0, path=path, engine=engine, training=True,
               want_probs=False)
    g = torch_mod.from_numpy(cot).cuda()
    dp, dx = r["circ"].backward(r["p"], r["x"], g, r["ws"])
    torch_mod.cuda.synchronize()
    dpr, dxr, Er = oracle.vjp(ops, n, p, x, cot, psi0=s0)
    check(r["E"], Er, E_TOL, "E")
    gg = np.concatenate([dp.cpu().numpy(), dx.cpu().numpy()], axis=1).astype(np.float64)
    gr = np.concatenate([dpr, dxr], axis=1)
    err = np.max(np.abs(gg - gr), axis=1)
    bar = G_REL * np.max(np.abs(gr), axis=1) + G_FLOOR * np.sum(np.abs(cot), axis=1)
    assert np.all(err <= bar), (err, bar)


def test_full_batch_config_sampled_rows(torch_mod):
    """The 8-qubit data re-uploading workload at its full batch, from Haar-random
    Psi_0, checked on sampled rows."""
    w = W.make_config(2)
    rows = [0, 1, w.batch // 2, w.batch - 1]
    s0 = W.random_states(w.batch, w.n_qubits, seed=450)
    note(f"config {w.name} full batch {w.batch} with psi0, rows {rows}")
    r = run_ex(torch_mod, w.ops, w.n_qubits, w.n_params, w.n_inputs, w.params, w.inputs, s0)
    Er, st = oracle.forward(w.ops, w.n_qubits, w.params[rows], w.inputs[rows], want_state=True,
                            psi0=s0[rows])
    check(r["E"][rows], Er, E_TOL, "E")
    check(r["probs"][rows], np.abs(st) ** 2, P_TOL, "probs")
    # properties at every row: probabilities sum to one, E is their signed marginal
    pr = r["probs"].astype(np.float64)
    assert np.max(np.abs(pr.sum(axis=1) - 1.0)) < 1e-4
    n = w.n_qubits
    sgn = np.array([[1 - 2 * ((k >> j) & 1) for j in range(n)] for k in range(1 << n)])
    assert np.max(np.abs(pr @ sgn - r["E"])) < 1e-4


def test_zero_state_psi0_and_errors(torch_mod):
    from paper_2607_11985_amd import _lib
    from paper_2607_11985_amd.api import Circuit
    torch = torch_mod
    n, B = 5, 6
    ops, P, F = W.random_circuit(n, 40, seed=460)
    p, x = W.random_inputs(B, P, F, seed=461)
    # Psi_0 = 0: the evolution is linear, everything stays zero
    z = np.zeros((B, 1 << n), dtype=np.complex64)
    r = run_ex(torch, ops, n, P, F, p, x, z)
    assert np.all(r["E"] == 0.0) and np.all(r["probs"] == 0.0)
    # |0...0> given explicitly equals the default start
    e0 = np.zeros((B, 1 << n), dtype=np.complex64)
    e0[:, 0] = 1.0
    r1 = run_ex(torch, ops, n, P, F, p, x, e0)
    r2 = run_ex(torch, ops, n, P, F, p, x, None)
    assert np.array_equal(r1["E"], r2["E"]) and np.array_equal(r1["probs"], r2["probs"])
    circ = Circuit(ops, n, P, F)
    tp = torch.from_numpy(p).cuda()
    tx = torch.from_numpy(x).cuda()
    E = torch.empty((B, n), device="cuda")
    s = torch.zeros((B, (1 << n) + 1), dtype=torch.complex64, device="cuda")
    with pytest.raises(_lib.VQCError):  # neither output asked for
        _lib.vqc_forward_ex(circ.handle, B, tp.data_ptr(), tx.data_ptr(), None, None, None,
                            None, 0, None)
    with pytest.raises(_lib.VQCError):  # misaligned Psi_0
        _lib.vqc_forward_ex(circ.handle, B, tp.data_ptr(), tx.data_ptr(), s.data_ptr() + 4,
                            E.data_ptr(), None, None, 0, None)
    # batch 0 is a no-op
    _lib.vqc_forward_ex(circ.handle, 0, None, None, None, None, None, None, 0, None)
    torch.cuda.synchronize()
