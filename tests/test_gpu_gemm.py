"""The dense products (three bf16 parts per operand) at the edges of their
tiles and K steps, against float64, and with operands no split can hold:
infinities, NaN and values that round past bf16's largest.  The partition's
matrix is the identity, so that a layer is its products alone."""
import numpy as np
import pytest

from paper_2206_00057_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def products(n, d_in, d_out, h, w, dh, h_out):
    """act(h W), h^T D and D W^T of layer 2 (ReLU), with D = dh [h_out > 0]."""
    from paper_2206_00057_amd import digest as D
    p = D.digest_partition_create(n, np.arange(n + 1), np.arange(n), np.ones(n, np.float32),
                                  np.arange(n), np.zeros(0, np.int64), [d_in, d_in, d_out, 3])
    ws = torch.full((p.workspace_bytes,), 255, dtype=torch.uint8, device="cuda")
    D.digest_partition_bind_workspace(p, ws)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    out = torch.empty(n, d_out, device="cuda")
    dw, dx = torch.empty(d_in, d_out, device="cuda"), torch.empty(n, d_in, device="cuda")
    x, wd = dev(h), dev(w)
    D.digest_layer_forward(p, 2, x, wd, out, D.ACT_RELU)
    D.digest_layer_backward(p, 2, x, dev(h_out), dev(dh), wd, dw, dx)
    return [t.cpu().numpy() for t in (out, dw, dx)]


def inputs(n, d_in, d_out):
    w = synth.normal((d_in, d_out), seed=3)
    return (synth.normal((n, d_in), seed=1), w, synth.normal((n, d_out), seed=2),
            synth.normal((n, d_out), seed=4))


def refs(h, w, dh, h_out):
    h, w = h.astype(np.float64), w.astype(np.float64)
    d = np.where(h_out > 0, dh, 0).astype(np.float64)
    return np.maximum(h @ w, 0), h.T @ d, d @ w.T


# rows, input and output widths: one K step and less, partial last steps,
# tiles cut in both directions, unaligned rows, the 128x128 tile's rows
SHAPES = [(1, 17, 65), (64, 32, 66), (65, 33, 129), (130, 95, 70), (500, 64, 256),
          (333, 602, 257), (20001, 101, 130)]


@pytest.mark.parametrize("n,d_in,d_out", SHAPES)
def test_products_match_float64(n, d_in, d_out):
    a = inputs(n, d_in, d_out)
    for name, got, ref in zip(("forward", "dW", "dH"), products(n, d_in, d_out, *a), refs(*a)):
        # each of K terms and one rounding per 16 of them: well below
        # sqrt(K) 2^-24 of the result's size, taken four times for the maximum
        K = {"forward": d_in, "dW": n, "dH": d_out}[name]
        scale = max(np.sqrt(np.mean(ref ** 2)), 1e-30)
        bound = 4 * (4 + np.sqrt(K)) * 2.0 ** -24 * max(scale, np.sqrt(K))
        assert np.abs(got - ref).max() <= bound, (name, np.abs(got - ref).max(), bound)


# binary exponents of h, w and D: each operand in turn as small as a normal
# float and as a subnormal one (whose parts are below every normal bf16)
SMALL = [(-118, 40, 40), (40, -118, 40), (40, 40, -118), (-139, 40, 40), (40, -139, 40),
         (40, 40, -139)]


@pytest.mark.parametrize("n,d_in,d_out", [(130, 95, 70), (333, 602, 257), (20001, 101, 130)])
@pytest.mark.parametrize("exps", SMALL, ids=lambda e: "_".join(map(str, e)))
def test_small_operands_keep_their_bits(n, d_in, d_out, exps):
    eh, ew, ed = exps
    h, w, dh, h_out = inputs(n, d_in, d_out)
    h, w, dh = np.ldexp(h, eh), np.ldexp(w, ew), np.ldexp(dh, ed)   # (subnormals are rounded)
    for name, got, ref, e in zip(("forward", "dW", "dH"), products(n, d_in, d_out, h, w, dh, h_out),
                                 refs(h, w, dh, h_out), (eh + ew, eh + ed, ed + ew)):
        K = {"forward": d_in, "dW": n, "dH": d_out}[name]
        # the bound of test_products_match_float64, for products of size 2^e
        bound = 4 * (4 + np.sqrt(K)) * 2.0 ** -24 * np.sqrt(K) * 2.0 ** e
        assert np.abs(got - ref).max() <= bound, (name, np.abs(got - ref).max(), bound)


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan, 3.4e38])
@pytest.mark.parametrize("n,d_in,d_out", [(130, 95, 70), (20001, 101, 130)])
def test_non_finite_operands_stay_where_they_belong(n, d_in, d_out, bad):
    h, w, dh, h_out = inputs(n, d_in, d_out)
    w[np.abs(w) < 1e-3] = 0.5
    h_out[7] = dh[7] = 1.0
    h[5, d_in - 1] = dh[7, 3] = bad
    with np.errstate(all="ignore"):
        ref = [r.astype(np.float32) for r in refs(h, w, dh, h_out)]
    for name, got, r in zip(("forward", "dW", "dH"), products(n, d_in, d_out, h, w, dh, h_out),
                            ref):
        if name == "forward":   # the ReLU is max(x, 0), which drops a NaN
            r = np.where(np.isnan(r), 0.0, r)
        np.testing.assert_array_equal(np.isnan(got), np.isnan(r), err_msg=name)
        np.testing.assert_array_equal(np.isinf(got), np.isinf(r), err_msg=name)
        fin = np.isfinite(r)
        assert (np.sign(got[~fin & ~np.isnan(r)]) == np.sign(r[~fin & ~np.isnan(r)])).all()
        rest = fin & (np.abs(r) < 1e30)
        np.testing.assert_allclose(got[rest], r[rest], rtol=1e-4, atol=1e-4 * np.sqrt(n),
                                   err_msg=name)


def test_a_diverged_layer_stays_a_fast_one():
    """Operands that are NaN throughout: each product again on the fp32
    instructions, not element by element (which took 100 times as long)."""
    n, d_in, d_out = 11250, 500, 256
    from paper_2206_00057_amd import digest as D
    p = D.digest_partition_create(n, np.arange(n + 1), np.arange(n), np.ones(n, np.float32),
                                  np.arange(n), np.zeros(0, np.int64), [d_in, d_out])
    ws = torch.empty(p.workspace_bytes, dtype=torch.uint8, device="cuda")
    D.digest_partition_bind_workspace(p, ws)
    x, dh = torch.randn(n, d_in, device="cuda"), torch.randn(n, d_out, device="cuda")
    w, out = torch.randn(d_in, d_out, device="cuda"), torch.empty(n, d_out, device="cuda")
    dw = torch.empty(d_in, d_out, device="cuda")

    def run():
        D.digest_layer_forward(p, 1, x, w, out, D.ACT_IDENTITY)
        D.digest_layer_backward(p, 1, x, out, dh, w, dw, None)

    def time():
        run()
        t = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        t[0].record()
        for _ in range(5):
            run()
        t[1].record()
        t[1].synchronize()
        return t[0].elapsed_time(t[1])

    finite = time()
    x.fill_(float("nan"))
    assert time() < 10 * finite
    assert torch.isnan(out).all() and torch.isnan(dw).all()
