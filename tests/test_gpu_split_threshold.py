"""Streaming calls run two batch halves on two streams from 2048 tiles on and
stay on one stream below.  The same samples in a batch on either side of the
line, and in a batch of a few, give the same rows bit for bit: the training
step, the separate forward and backward, and the probabilities."""
import numpy as np
import pytest

from paper_2607_11985_amd import workloads as W
from tests.parity_util import note
from tests.test_gpu_parity import torch_mod  # noqa: F401

pytestmark = pytest.mark.gpu


def test_rows_do_not_depend_on_the_split(torch_mod):
    torch = torch_mod
    from paper_2607_11985_amd.api import Circuit
    n = 14
    ops, P, F = W.strongly_entangling_circuit(n, 2)
    c = Circuit(ops, n, P, F, path="stream", tile_qubits=12)
    at = 2048 >> (n - 12)  # the first batch that splits
    params, inputs = W.random_inputs(at + 1, P, F, seed=4242)
    cot = W.random_cotangent(at + 1, n, seed=4243)
    tp, tx, tg = (torch.from_numpy(v).cuda() for v in (params, inputs, cot))
    want = None
    for B in (3, at - 1, at, at + 1):
        note(f"split line n={n} B={B}")
        p, x, g = tp[:B].contiguous(), tx[:B].contiguous(), tg[:B].contiguous()
        E, dp, dx = c.train_step(p, x, "sum")
        E2, pr, ws = c.forward_ex(p, x, probs=True, training=True)
        dp2, dx2 = c.backward(p, x, g, ws)
        torch.cuda.synchronize()
        rows = [v[:3].cpu().numpy() for v in (E, dp, dx, E2, pr, dp2, dx2)]
        if want is None:
            want = rows
        for w, r in zip(want, rows):
            assert np.array_equal(w, r)
        if B >= at - 1:  # every row, against the batch one below the line
            full = [v[:at - 1].cpu().numpy() for v in (E, dp, dx, E2, dp2, dx2)]
            if B == at - 1:
                below = full
            for w, r in zip(below, full):
                assert np.array_equal(w, r)
