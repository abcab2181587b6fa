"""The GAT layer's passes over the entries at every width class, with a row
of more entries than one wave takes, repeated entries, rows without halo
columns, and every workspace byte set before the first write."""
import numpy as np
import pytest

import oracle
from paper_2206_00057_amd import synth
from test_gpu_gat import Case, _need_gpu  # noqa: F401  (fixture)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# every lane-group layout with a partial last vector and with a full one
WIDTHS = [(4, 3, 16), (9, 29, 32), (5, 61, 64), (6, 66, 128), (7, 130, 256), (3, 257, 512)]


@pytest.mark.parametrize("widths", WIDTHS, ids=lambda w: "x".join(map(str, w)))
@pytest.mark.parametrize("longest", [0, 2500])
def test_gat_entries(widths, longest):
    cfg = synth.scaled(synth.CONFIGS["tiny"], 1200, widths=widths, classes=widths[-1])
    g = synth.make_graph(cfg, seed=2)
    part = synth.scramble_rows(synth.make_partition(cfg, g, 1), seed=5, long_row=longest)
    c = Case(g.n, part, widths, seed=2)
    c.ws.fill_(255)
    c.D.digest_partition_bind_workspace(c.h, c.ws)
    c.gws.fill_(255)
    c.D.digest_gat_bind_workspace(c.h, c.gws)
    for level in (0, 1):
        c.pull(level, synth.relu_normal((g.n, widths[level]), seed=20 + level))
    first = c.layer(1, oracle.RELU, "layer 1")
    second = c.layer(2, oracle.IDENTITY, "layer 2")
    # the layers keep their forward state apart, and repeat bit for bit
    for a, b in zip(first + second, c.layer(1, oracle.RELU, "again") +
                    c.layer(2, oracle.IDENTITY, "again")):
        np.testing.assert_array_equal(a.cpu().numpy().view(np.uint32),
                                      b.cpu().numpy().view(np.uint32))
