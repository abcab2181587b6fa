"""Aggregations out of the XCDs' L2s (column-sliced sources) against the CPU
oracle, at the edges of their rule and of their kernel: partial last slices,
widths that are no multiple of 4, rows of more entries than one wave takes,
blocks of 64 entries cut by the rows' ends, repeated entries, both product
orders with and without the ReLU mask."""
import dataclasses

import pytest

from paper_2206_00057_amd import synth
from test_gpu_parity import Case, _need_gpu, check_layer  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

# owned rows, mean endpoints drawn per row, widths, entries of the longest row
CASES = [
    (2504, 9, (600, 602, 48), 0),       # 6.03 MB of 602 floats, about 15 entries a row
    (4001, 30, (603, 256, 16), 5003),   # odd width, one row over a whole workgroup
    (8000, 24, (256, 192, 41), 2049),   # last slice of 9 columns, rows of 41 floats
    (12003, 40, (602, 128, 16), 0),     # a ReLU layer transformed first: D masked as it is laid out
    (15001, 12, (101, 101, 64), 0),     # scalar loads, one odd row past the strips
    (16500, 14, (96, 256, 256, 40), 2048),   # above the fused passes' row count
    # widths below the rule's narrowest that pad to it, no other width sliced
    (10003, 45, (100, 37), 0),
    (9001, 45, (100, 128, 39), 0),
]


@pytest.mark.parametrize("n,mean,widths,longest", CASES,
                         ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_sliced_layers(n, mean, widths, longest):
    cfg = dataclasses.replace(synth.CONFIGS["dense"], name="sliced", n=2 * n, blocks=2,
                              c=mean / 490.0, cap=n // 2, p_intra=0.85, widths=widths,
                              classes=widths[-1])
    g = synth.make_graph(cfg)
    part = synth.scramble_rows(synth.make_partition(cfg, g, 1), seed=7, repeat_frac=0.1,
                               long_row=longest)
    c = Case(cfg, g, part, ws_fill=0xFF)   # every workspace float NaN
    for layer in range(1, c.L + 1):
        check_layer(c, layer)
