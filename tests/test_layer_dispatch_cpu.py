"""Which aggregation a layer call runs, and what it hands to it, on the CPU:
the library's host code linked with plain loops in place of its kernels
(``host_kernels.cpp``) against the oracle, over a workspace of NaN.  The
widths lie on both sides of the lines of the rule for aggregations out of
column slices: widths whose padding to whole vectors crosses a line, with no
other width of the network on the sliced side, and their neighbours."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import oracle
from conftest import ROOT
from paper_2206_00057_amd import build as B
from paper_2206_00057_amd import digest as D
from paper_2206_00057_amd import synth


@pytest.fixture(scope="module")
def library(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("host") / "libdigest_host.so")
    subprocess.run(["g++", *B.CXX_FLAGS, "-fopenmp", "-shared", "-Wl,-Bsymbolic",
                    os.path.join(B.CSRC, "digest_host.cpp"),
                    os.path.join(ROOT, "tests", "host_kernels.cpp"), "-o", lib], check=True)
    return lib


@pytest.fixture
def on_cpu(library, monkeypatch):
    """digest's functions over numpy arrays, in the host library."""
    def pointer(a, dtype, numel, name):
        assert a.dtype == np.float32 and a.flags.c_contiguous and a.size == numel, name
        return a.ctypes.data_as(ctypes.c_void_p)
    monkeypatch.setattr(D, "LIB_PATH", library)
    monkeypatch.setattr(D, "_lib", None)
    monkeypatch.setattr(D, "_dev", pointer)
    monkeypatch.setattr(D, "_stream", lambda s: ctypes.c_void_p(0))
    return D.lib()


def partition(n, mean, seed=0):
    """n owned rows, about mean distinct in-partition entries and two halo
    entries each (one row without entries)."""
    rng = np.random.default_rng(seed)
    n_halo = n // 4
    inside = np.sort(rng.integers(0, n, (n, mean)), 1)
    outside = n + rng.integers(0, n_halo, (n, 2))
    deg = np.full(n, mean + 2)
    deg[n // 2] = 0
    cols = np.concatenate([inside, outside], 1)[np.arange(n) != n // 2].reshape(-1)
    indptr = np.concatenate([[0], np.cumsum(deg)])
    values = rng.uniform(0.5, 1.5, cols.size).astype(np.float32) / mean
    return (n + n_halo, indptr, cols, values, np.arange(n), np.arange(n, n + n_halo))


# rows, entries a row, widths, layer, and whether its backward is sliced
CASES = [
    (8100, 34, (100, 39), 1, False),          # 39 -> 40, below the narrowest
    (8100, 34, (100, 37), 1, False),
    (8100, 34, (40, 128, 38), 2, False),      # lists exist, for another width
    (8100, 34, (100, 100, 39), 2, False),
    (8100, 34, (100, 40), 1, False),          # whole vectors need more entries a row
    (8100, 50, (100, 40), 1, True),
    (8100, 34, (100, 100, 41), 2, True),
    (7000, 80, (600, 214), 1, False),         # 214 -> 216 crosses 6 MB of rows
    (7000, 80, (600, 215), 1, True),
    (7000, 79, (600, 215), 1, False),         # just below 480 MB of gathered rows
    (8100, 34, (100, 39, 96), 2, False),      # aggregated first, 39 wide
    (8100, 34, (100, 41, 96), 2, True),
]


def close(got, ref, name):
    assert np.isfinite(got).all(), name
    # fp32 results of sums in 64 bits, against the oracle's
    assert np.abs(got - ref).max() <= 1e-5 * np.abs(ref).max(), name


@pytest.mark.parametrize("act", [oracle.RELU, oracle.IDENTITY], ids=["relu", "identity"])
@pytest.mark.parametrize("n,mean,widths,layer,sliced", CASES, ids=lambda v: str(v))
def test_layer_runs_what_its_plan_holds(on_cpu, n, mean, widths, layer, sliced, act):
    args = partition(n, mean)
    h = D.digest_partition_create(*args, widths)
    tf = D.digest_partition_plan(h, layer)["transform_first"]
    assert tf == (widths[layer - 1] > widths[layer])
    ws = np.full(h.workspace_bytes // 4 + 64, np.nan, np.float32)
    base = ws.ctypes.data + (-ws.ctypes.data) % 256
    D._check(on_cpu.digest_partition_bind_workspace(h.handle, base, h.workspace_bytes, None))
    op = oracle.OraclePartition(*args, list(widths))
    d_in, d_out = widths[layer - 1], widths[layer]
    store = synth.normal((args[0], d_in), seed=1)
    x, w = np.ascontiguousarray(store[:n]), synth.normal((d_in, d_out), seed=2)
    dh = synth.normal((n, d_out), seed=3)
    D.digest_pull(h, layer - 1, store)
    op.pull(layer - 1, store)
    out = np.full((n, d_out), np.nan, np.float32)
    D.digest_layer_forward(h, layer, x, w, out, act)
    ref = op.forward(layer, x, w, act)
    close(out, ref, "forward")
    counts = (ctypes.c_int * 2)()
    for want in ("dw", "dh_in", "dh_halo"):
        dw = np.full((d_in, d_out), np.nan, np.float32)
        dx = np.full((n, d_in), np.nan, np.float32) if want != "dw" else None
        if want == "dh_halo" and layer == 1:
            continue
        on_cpu.host_kernels_counts(ctypes.byref(counts, 0), ctypes.byref(counts, 4))
        if want == "dh_halo":
            dhalo = np.full((h.n_halo, d_in), np.nan, np.float32)
            D.digest_layer_backward_halo(h, layer, x, ref, dh, w, dw, dx, dhalo)
            close(dhalo, op.halo_gradient(layer, w, ref, dh, act), want)
        else:
            D.digest_layer_backward(h, layer, x, ref, dh, w, dw, dx)
        on_cpu.host_kernels_counts(ctypes.byref(counts, 0), ctypes.byref(counts, 4))
        ref_dw, ref_dx = op.backward(layer, x, w, ref, dh, act, want_dh_in=dx is not None)
        close(dw, ref_dw, want)
        if dx is not None:
            close(dx, ref_dx, want)
        # transformed first: one aggregation over P_in^T, with dh_halo one more
        # over P_out^T; aggregated first: none for dw, one over P_m^T for both
        assert tuple(counts) == ((sliced, (not sliced) + (want == "dh_halo")) if tf
                                 else (0, 0) if want == "dw"
                                 else (sliced, not sliced) if want == "dh_in" else (0, 1)), want
    D.digest_partition_destroy(h)


def test_gat_layout_is_planned_by_the_first_call_of_any_thread(on_cpu):
    """The lists of a dense partition's attention layer are built with the
    first query, not with the partition, and once."""
    from concurrent.futures import ThreadPoolExecutor
    sizes = []
    for mean in (70, 60):   # strips of rows from 64 entries a row on, and none
        h = D.digest_partition_create(*partition(2100, mean), (8, 16))
        with ThreadPoolExecutor(8) as pool:
            sizes.append(set(pool.map(lambda _: D.digest_gat_query(h), range(32))))
        nnz = h.nnz
        sizes[-1] = {s - 4 * nnz for s in sizes[-1]}   # less the weights
        D.digest_partition_destroy(h)
    dense, sparse = sizes
    assert len(dense) == len(sparse) == 1
    # a 16-byte block per strip (a row or more) and nothing else
    assert 16 * 2100 / 8 < min(dense) - min(sparse) <= 16 * 2100 + 512


@pytest.mark.parametrize("mean", [70, 60])   # with strips of rows to upload, and without
def test_gat_bind_waits_for_its_upload(on_cpu, mean):
    """The layers may be called on another stream than the bind."""
    h = D.digest_partition_create(*partition(2100, mean), (8, 16))
    ws = np.zeros((h.workspace_bytes + D.digest_gat_query(h)) // 4 + 128, np.float32)
    base = ws.ctypes.data + (-ws.ctypes.data) % 256
    D._check(on_cpu.digest_partition_bind_workspace(h.handle, base, h.workspace_bytes, None))
    before = on_cpu.host_kernels_pending()
    gat = base + -(-h.workspace_bytes // 256) * 256
    D._check(on_cpu.digest_gat_bind_workspace(h.handle, gat, D.digest_gat_query(h), None))
    assert on_cpu.host_kernels_pending() == (0 if mean == 70 else before)
    D.digest_partition_destroy(h)
