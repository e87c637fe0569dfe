"""Operands of one training step that the split products hold only in part, where the loader
transforms them (SiLU' of the readout): against the float64 oracle, within the tolerances of the step."""
import copy

import numpy as np
import pytest

from helpers import TOL_W, banner, rel_l2

pytestmark = pytest.mark.gpu


def _step(b):
    import torch
    from paper_2604_15821_amd import janus
    d = janus.upload(b)
    ctx = janus.Context(b.model)
    nl = ctx.build_edges(d["pos"], d["cell"], d["offsets"])
    loss, E, F, dW = ctx.step(d["pos"], d["cell"], d["species"], d["offsets"], nl, d["W"], d["E_ref"], d["F_ref"])
    torch.cuda.synchronize()
    out = float(loss.cpu()[0]), E.cpu().numpy(), F.cpu().numpy(), janus.unpack(dW.cpu().numpy(), b.model)
    ctx.close()
    return out


def _batch(n):
    from paper_2604_15821_amd.synth import make_batch, subset
    b = copy.copy(subset(make_batch("tiny"), range(n)))
    b.weights = {k: v.copy() for k, v in b.weights.items()}
    return b


def _forward(b):
    from oracle.model import Params, build_graph_for, forward_energy, route_all
    P = Params.from_weights(b.weights, b.model)
    g = build_graph_for(b)
    return forward_energy(b.species, g, P, route_all(b.species, g, P))[1]


def test_readout_column_far_below_the_padding_of_its_chunk():
    """dW_o1 of one 32-atom cell cut to 20 atoms: a chunk shorter than one stage, whose padded rows must not
    set the scale of a column with SiLU'(z) = -3e-12 in every atom."""
    from oracle.model import training_step
    b = _batch(1)
    n = 20
    b.pos, b.species, b.F_ref = b.pos[:n], b.species[:n], b.F_ref[:n]
    b.offsets = np.array([0, n], np.int32)
    banner("split step, readout column", n)
    h = _forward(b)["h"][-1]
    b.weights["W_o1"][:, 7] = np.linalg.lstsq(h, np.full(n, -30.0), rcond=None)[0]
    ref = training_step(b)[3]["W_o1"][:, 7]
    got = _step(b)[3]["W_o1"][:, 7]
    assert 0 < np.abs(ref).max() < 1e-6
    # SiLU'(z) ~ z e^z: an error of z (z's fp32 rounding, 64 terms of |h w|) is the result's relative error
    dz = 64 * 2.0 ** -24 * (np.abs(h) @ np.abs(b.weights["W_o1"][:, 7])).max()
    assert dz < 1e-3
    assert rel_l2(got, ref) <= TOL_W + dz
