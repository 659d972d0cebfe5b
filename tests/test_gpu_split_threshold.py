"""Streaming calls run two batch halves on two streams from 2^25 amplitudes times
passes on and stay on one stream below (the step counts the passes of its
forward and its adjoint, the separate calls their own).  The same samples in
batches on either side of each line, and in a batch of a few, give the same
rows bit for bit: the training step, the separate forward and backward, and
the probabilities."""
import numpy as np
import pytest

from paper_2607_11985_amd import workloads as W
from tests.parity_util import note, split_line
from tests.test_gpu_parity import torch_mod  # noqa: F401

pytestmark = pytest.mark.gpu


def test_rows_do_not_depend_on_the_split(torch_mod):
    torch = torch_mod
    from paper_2607_11985_amd.api import Circuit
    n = 14
    ops, P, F = W.strongly_entangling_circuit(n, 2)
    c = Circuit(ops, n, P, F, path="stream", tile_qubits=12)
    lines = [split_line(c.info(), "step"), split_line(c.info(), "forward")]
    assert lines[0] < lines[1]
    top = lines[1] + 1
    params, inputs = W.random_inputs(top, P, F, seed=4242)
    cot = W.random_cotangent(top, n, seed=4243)
    tp, tx, tg = (torch.from_numpy(v).cuda() for v in (params, inputs, cot))
    below = None
    for B in (top, lines[1], lines[1] - 1, lines[0], lines[0] - 1, 3):
        note(f"split lines {lines} n={n} B={B}")
        p, x, g = tp[:B].contiguous(), tx[:B].contiguous(), tg[:B].contiguous()
        E, dp, dx = c.train_step(p, x, "sum")
        E2, pr, ws = c.forward_ex(p, x, probs=True, training=True)
        dp2, dx2 = c.backward(p, x, g, ws)
        torch.cuda.synchronize()
        rows = [v.cpu().numpy() for v in (E, dp, dx, E2, pr, dp2, dx2)]
        if below is not None:
            for w, r in zip(below, rows):
                assert np.array_equal(w[:B], r)
        below = rows
