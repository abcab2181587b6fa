"""Aggregations out of the XCDs' L2s (column-sliced sources) against the CPU
oracle, at the edges of their rule and of their kernel: partial last slices,
widths that are no multiple of 4, rows of more entries than one wave takes,
blocks of 64 entries cut by the rows' ends, repeated entries, both product
orders with and without the ReLU mask."""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2206_00057_amd import synth
from test_gpu_parity import Case, _need_gpu, check_layer, dev, host  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

# owned rows, mean endpoints drawn per row, widths, entries of the longest row
CASES = [
    (2504, 45, (600, 602, 48), 0),      # 6.03 MB of 602 floats
    (4001, 30, (603, 256, 16), 5003),   # odd width, one row over a whole workgroup
    (8000, 36, (256, 192, 41), 2049),   # last slice of 9 columns, rows of 41 floats
    (12003, 46, (602, 128, 16), 0),     # a ReLU layer transformed first: D masked as it is laid out
    (15001, 45, (101, 101, 64), 0),     # scalar loads, one odd row past the strips
    (16500, 18, (96, 256, 256, 40), 2048),   # above the fused passes' row count
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


@pytest.mark.parametrize("widths", [(96, 256, 41), (96, 256, 256)],
                         ids=lambda w: "x".join(map(str, w)))
def test_infinite_rows_stay_infinite(widths):
    """Sums that hold an infinite term as the row's last entry, over rows of
    every length: infinite like the oracle's, not NaN (nor, past a ReLU, zero)."""
    from paper_2206_00057_amd import digest as D
    import torch
    n, rng = 8100, np.random.default_rng(3)
    rows = [np.sort(rng.choice(n - 1, 31 + i % 67, replace=False)) for i in range(n)]
    rows = [np.concatenate([r, [n - 1] * (i % 3 == 0), [n] * (i % 2)]).astype(np.int64)
            for i, r in enumerate(rows)]
    indptr = np.concatenate([[0], np.cumsum([r.size for r in rows])])
    part = synth.Partition(owned=np.arange(n), halo=np.array([n]), indptr=indptr,
                           indices=np.concatenate(rows),
                           values=np.full(indptr[-1], 0.02, np.float32))
    cfg = dataclasses.replace(synth.CONFIGS["tiny"], n=n + 1, widths=widths, classes=widths[-1])
    c = Case(cfg, synth.Graph(n + 1, *[None] * 4), part, ws_fill=0xFF)
    store = synth.relu_normal((n + 1, 256), seed=1)
    D.digest_pull(c.h, 1, dev(store))
    c.op.pull(1, store)
    x, w = store[:n].copy(), np.abs(synth.normal((256, widths[2]), seed=2)) + 0.1
    dh = np.abs(synth.normal((n, widths[2]), seed=3))
    x[n - 1, 7] = dh[n - 1, 3] = np.inf
    for act in (oracle.RELU, oracle.IDENTITY):
        out, dx = torch.empty(n, widths[2], device="cuda"), torch.empty(n, 256, device="cuda")
        D.digest_layer_forward(c.h, 2, dev(x), dev(w), out, act)
        ref = c.op.forward(2, x, w, act)
        D.digest_layer_backward(c.h, 2, dev(x), dev(np.ones_like(ref)), dev(dh), dev(w),
                                torch.empty(w.shape, device="cuda"), dx)
        ref_dx = c.op.backward(2, x, w, np.ones_like(ref), dh, act, want_dh_in=True)[1]
        for got, r, name in ((host(out), ref, "forward"), (host(dx), ref_dx, "dH_in")):
            assert np.isinf(r).any() and np.isfinite(r).any(), name
            np.testing.assert_array_equal(got[~np.isfinite(r)], r[~np.isfinite(r)], err_msg=name)
            np.testing.assert_allclose(got[np.isfinite(r)], r[np.isfinite(r)], rtol=1e-4,
                                       err_msg=name)
