"""GPU parity of the transformer layer (dcp_layer_fwd / dcp_layer_bwd: the HIP
attention, norm, projection and weight-gradient kernels, the other products in
rocBLAS) against the float64 layer oracle, and the recomputation contract: a backward that re-runs the forward
returns bitwise what a backward with the stashed activations returns.

Tolerance: every output, input gradient and weight gradient within 2e-2 of
the largest reference magnitude of its tensor.  The forward stores seven
intermediates in bf16 (y1; q, k, v; o; h; y2; u; a), each rounded to within
2^-8 relative, and the GEMMs take bf16 operands; the gradients are bounded
the same way as the attention gradients."""

import math

import numpy as np
import pytest

from oracle import layer as LY
from paper_2608_07524_amd import inputs as I

from gpu_util import GRAD_TOL, to_bits

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    t = pytest.importorskip("torch")
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2608_07524_amd as P
    P.load()
    return t


def _dev(torch, a):
    return torch.from_numpy(I.bf16_bits(np.asarray(a, dtype=np.float32)).view(np.int16)).view(torch.bfloat16).cuda()


def _setup(torch, lengths, H, D, causal, seed):
    import paper_2608_07524_amd as P
    rng = np.random.default_rng(seed)
    h = H * D
    cu = I.cu_from_lengths(lengths)
    T = int(cu[-1])
    W = {}
    for n, shape in P.layer_param_shapes(h).items():
        if n.startswith("norm"):
            W[n] = 1.0 + 0.2 * rng.standard_normal(shape)
        else:
            W[n] = rng.standard_normal(shape) / math.sqrt(shape[0])
    x = rng.standard_normal((T, h))
    dout = rng.standard_normal((T, h))
    # the bf16 values the GPU sees, widened for the oracle
    Wb = {n: I.bf16_to_f64(I.bf16_bits(v.astype(np.float32))) for n, v in W.items()}
    xb, db = (I.bf16_to_f64(I.bf16_bits(v.astype(np.float32))) for v in (x, dout))
    wd = {n: _dev(torch, v) for n, v in Wb.items()}
    gd = {n: torch.zeros(v.shape, dtype=torch.float32, device="cuda") for n, v in Wb.items()}
    layer = P.Layer(wd, gd, cu, H, D, causal, 1.0 / math.sqrt(D), 1e-6)
    return layer, cu, Wb, xb, db, _dev(torch, xb), _dev(torch, db)


def _run(torch, layer, x, dout, keep):
    for g in layer.grads.values():
        g.zero_()
    out = layer.fwd(x, keep=keep)
    dx = layer.bwd(x, dout)
    torch.cuda.synchronize()
    return to_bits(out), to_bits(dx), {n: g.cpu().numpy().copy() for n, g in layer.grads.items()}


@pytest.mark.parametrize("causal", [False, True])
def test_layer_matches_oracle(torch, causal):
    lengths = [300, 45, 17, 700, 1, 130]
    H, D = 2, 64
    layer, cu, Wb, xb, db, x, dout = _setup(torch, lengths, H, D, causal, 21 + causal)
    out, dx, grads = _run(torch, layer, x, dout, keep=True)
    ref_out, cache = LY.layer_forward(xb, Wb, cu, H, D, 1.0 / math.sqrt(D), causal, 1e-6)
    ref_dx, ref_g = LY.layer_backward(db, Wb, cache, cu, H, D, 1.0 / math.sqrt(D), causal)

    def rel(got, ref):
        return float(np.max(np.abs(got - ref)) / np.max(np.abs(ref)))

    errs = {"out": rel(I.bf16_to_f64(out), ref_out), "dx": rel(I.bf16_to_f64(dx), ref_dx)}
    errs.update({n: rel(grads[n].astype(np.float64), ref_g[n]) for n in LY.PARAMS})
    print(f"layer causal={causal}: " + " ".join(f"{k} {v:.1e}" for k, v in errs.items()), flush=True)
    assert max(errs.values()) <= GRAD_TOL, errs


# The weight gradients' output tiles are 192 x 192 and their token slices 32
# rows; with fewer than 256 tiles the tokens are split as well, in at least
# eight slices each.  Widths below, at and across the tile; one token, a slice
# and its neighbours, an uneven split; and a width with tiles enough for no
# split.  Gradients add to what is there.
@pytest.mark.parametrize("H,D,lengths", [(1, 64, [1]), (3, 64, [31, 2]), (3, 72, [32]), (5, 64, [900, 133]),
                                         (2, 128, [1025]), (16, 72, [33, 32])])
def test_weight_gradients(torch, H, D, lengths):
    layer, cu, Wb, xb, db, x, dout = _setup(torch, lengths, H, D, True, 31 + H)
    for g in layer.grads.values():
        g.fill_(3.0)
    layer.fwd(x)
    layer.bwd(x, dout)
    torch.cuda.synchronize()
    _, cache = LY.layer_forward(xb, Wb, cu, H, D, 1.0 / math.sqrt(D), True, 1e-6)
    _, ref = LY.layer_backward(db, Wb, cache, cu, H, D, 1.0 / math.sqrt(D), True)
    errs = {n: float(np.max(np.abs(layer.grads[n].cpu().numpy().astype(np.float64) - 3.0 - ref[n]))
                     / np.max(np.abs(ref[n]))) for n in LY.PARAMS if np.any(ref[n])}
    print(f"weight gradients H={H} D={D} {lengths}: " + " ".join(f"{k} {v:.1e}" for k, v in errs.items()), flush=True)
    # (3 + g is rounded to fp32: at most 2^-23 of 3, against gradients of order 0.1 and more)
    assert max(errs.values()) <= GRAD_TOL, errs


# At hidden 4,096 the weight gradients are six library products from 12,288 tokens
# on: the sum of the gradients of the batch's halves, which are not.
def test_weight_gradients_of_many_wide_tokens(torch):
    import paper_2608_07524_amd as P
    H, D, T = 32, 128, 12288
    gen = torch.Generator(device="cuda").manual_seed(3)
    rand = lambda *s: torch.randn(*s, generator=gen, device="cuda")
    W = {n: (rand(*s) / (math.sqrt(s[0]) if len(s) > 1 else 1.0)).to(torch.bfloat16)
         for n, s in P.layer_param_shapes(H * D).items()}
    x, dout = (rand(T, H * D).to(torch.bfloat16) for _ in range(2))

    def grads(rows):
        g = {n: torch.full(w.shape, 3.0, dtype=torch.float32, device="cuda") for n, w in W.items()}
        for lo in range(0, T, rows):
            layer = P.Layer(W, g, np.arange(0, rows + 1, 512), H, D, True, None, 1e-6)
            layer.fwd(x[lo:lo + rows])
            layer.bwd(x[lo:lo + rows], dout[lo:lo + rows])
            torch.cuda.synchronize()
        return g

    whole, halves = grads(T), grads(T // 2)
    errs = {n: float((whole[n] - halves[n]).abs().max() / (halves[n] - 3.0).abs().max()) for n in W}
    assert max(errs.values()) <= GRAD_TOL, errs


# Matrices that share one gradient buffer: it receives the sum, whether the
# tokens are split over workgroups (few tiles) or not.
@pytest.mark.parametrize("H,D,lengths", [(3, 64, [600, 141]), (16, 72, [33, 32])])
def test_shared_gradient_buffer(torch, H, D, lengths):
    from paper_2608_07524_amd import _native as N
    layer, cu, Wb, xb, db, x, dout = _setup(torch, lengths, H, D, True, 41 + H)
    shared = layer.grads["wq"]
    layer.grads["wk"] = layer.grads["wv"] = shared
    layer.grads["w_down"] = layer.grads["w_up"]  # (one buffer, two shapes)
    layer.g = N.LayerWeightsC(*[layer.grads[n].data_ptr() for n in N.LAYER_PARAMS])
    layer.fwd(x)
    layer.bwd(x, dout)
    torch.cuda.synchronize()
    _, cache = LY.layer_forward(xb, Wb, cu, H, D, 1.0 / math.sqrt(D), True, 1e-6)
    _, ref = LY.layer_backward(db, Wb, cache, cu, H, D, 1.0 / math.sqrt(D), True)
    want = {"wq": ref["wq"] + ref["wk"] + ref["wv"], "w_up": ref["w_up"] + ref["w_down"].reshape(ref["w_up"].shape),
            "wo": ref["wo"]}
    errs = {n: float(np.max(np.abs(layer.grads[n].cpu().numpy() - w)) / np.max(np.abs(w))) for n, w in want.items()}
    assert max(errs.values()) <= GRAD_TOL, errs


# The projections' tiles are 192 features x 64 or (more than 256 tiles) 128
# tokens, their slices 64 of the contraction.  Widths of one slice, of a slice
# and a remainder, across a feature tile; tokens at and around the counts from
# which GELU (512), dY1 (2,048) and, for short rows or full rounds of tiles, the
# others (6,144; 45,990 x 72 is 360 tiles) are taken, and at tile edges; both tile
# heights of every product.  (The wide ones: every count of 512-column chunks the
# RMSNorm backward is built for.)
@pytest.mark.parametrize("H,D,lengths", [(1, 64, [512]), (1, 72, [511, 1]), (3, 72, [513]), (4, 72, [2047, 66]),
                                         (2, 128, [1025, 1023]), (1, 72, [70] * 476), (1, 72, [70] * 657),
                                         (1, 72, [70] * 88), (16, 72, [300, 277]),
                                         (16, 128, [33]), (20, 128, [17]), (28, 128, [17])])
def test_projections(torch, H, D, lengths):
    layer, cu, Wb, xb, db, x, dout = _setup(torch, lengths, H, D, True, 51 + H)
    out, dx, grads = _run(torch, layer, x, dout, keep=True)
    ref_out, cache = LY.layer_forward(xb, Wb, cu, H, D, 1.0 / math.sqrt(D), True, 1e-6)
    ref_dx, ref = LY.layer_backward(db, Wb, cache, cu, H, D, 1.0 / math.sqrt(D), True)
    pairs = {"out": (I.bf16_to_f64(out), ref_out), "dx": (I.bf16_to_f64(dx), ref_dx)}
    pairs.update({n: (grads[n].astype(np.float64), ref[n]) for n in LY.PARAMS})
    errs = {n: float(np.max(np.abs(a - b)) / np.max(np.abs(b))) for n, (a, b) in pairs.items()}
    print(f"projections H={H} D={D} T={len(x)}: " + " ".join(f"{k} {v:.1e}" for k, v in errs.items()), flush=True)
    assert max(errs.values()) <= GRAD_TOL, errs


def test_recompute_is_bitwise_the_stashed_backward(torch):
    layer, cu, Wb, xb, db, x, dout = _setup(torch, [200, 37, 513, 9], 4, 72, False, 5)
    kept = _run(torch, layer, x, dout, keep=True)
    again = _run(torch, layer, x, dout, keep=True)
    recomputed = _run(torch, layer, x, dout, keep=False)
    for a, b, c in zip(kept[:2], again[:2], recomputed[:2]):
        assert np.array_equal(a, b) and np.array_equal(a, c)
    for n in LY.PARAMS:
        assert np.array_equal(kept[2][n], again[2][n]) and np.array_equal(kept[2][n], recomputed[2][n]), n


def test_stack_executor_recompute_patterns(torch):
    """Three layers: every recompute pattern (the planner's flags) gives the
    same input gradient and weight gradients, bit for bit."""
    from paper_2608_07524_amd import model as M
    st = M.Stack(3, [0, 150, 170, 400], 2, 64, causal=True, seed=4)
    results = []
    for flags in ([0, 0, 0], [1, 0, 0], [1, 1, 0], [1, 1, 1]):
        for layer in st.layers:
            for g in layer.grads.values():
                g.zero_()
        st.step(flags)
        torch.cuda.synchronize()
        dx = to_bits(st.dys[0])  # the first layer's input gradient
        grads = [layer.grads[n].cpu().numpy().copy() for layer in st.layers for n in LY.PARAMS]
        results.append((dx, grads, to_bits(st.xs[-1])))
    for dx, grads, out in results[1:]:
        assert np.array_equal(dx, results[0][0]) and np.array_equal(out, results[0][2])
        assert all(np.array_equal(a, b) for a, b in zip(grads, results[0][1]))
