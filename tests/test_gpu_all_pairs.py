"""All-pairs neighbour search where its lanes and images can go wrong: 1 to 129 atoms (one
lane, the last lane of a wave, a second pass), cells with 27, 45 and 125 images (up to and beyond
the 32 that one mask holds), atoms outside their cell; bit for bit against the oracle."""
import numpy as np
import pytest

from helpers import banner
from oracle.neighbors import neighbor_list, reverse_map

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 129])
@pytest.mark.parametrize("sides", [(7.0, 8.0, 9.0), (3.0, 7.0, 8.0), (2.6, 2.5, 2.4), (40.0, 5.0, 41.0)])
@pytest.mark.parametrize("spread", [0.0, 1.5])
def test_matches_oracle(n, sides, spread):
    import dataclasses

    import torch

    from paper_2604_15821_amd import janus
    from paper_2604_15821_amd.synth import WORKLOADS
    banner("all pairs", n, sides, spread)
    rng = np.random.default_rng(n)
    sizes = [n, 3]
    pos = (rng.random((n + 3, 3)) * sides + spread * rng.integers(-1, 2, (n + 3, 3))).astype(np.float32)
    cell = np.stack([np.diag(sides), np.diag(sides[::-1])]).astype(np.float32)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    ei, ej, sh, rowptr = neighbor_list(pos, cell, off, 5.0)
    ctx = janus.Context(dataclasses.replace(WORKLOADS["tiny"].model, r_cut=5.0))
    ctx.set_edge_builder(2)
    nl = ctx.build_edges(torch.from_numpy(pos).cuda(), torch.from_numpy(cell).cuda(), torch.from_numpy(off).cuda())
    got = {k: getattr(nl, k).cpu().numpy() for k in ("ei", "ej", "shift", "rowptr", "rev")}
    ctx.close()
    for k, ref in (("ei", ei), ("ej", ej), ("shift", sh), ("rowptr", rowptr)):
        assert got[k].shape == ref.shape and (got[k] == ref).all(), k
    if ei.size:
        assert (got["rev"] == reverse_map(ei, ej, sh, n + 3)).all()
