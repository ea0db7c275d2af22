"""Matrix products on split operands (three bfloat16 parts, six products, two accumulators) at the edges of their tiles and
slabs, element by element against 64 bits; infinities and NaN; and forward propagation of any width and row stride."""
import numpy as np
import pytest
import torch

import workloads
from gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu
F = np.float32

# Short sums: what split_pick and split_dw_pays leave to the fp32 instruction is held to the same bound.
# (d_in, d_out, P, b): the 128x128, 64x128, 64x64, 32x128 and 32x32 tiles of 256 compute units, rows, columns and sums one
# below, at and one above a tile, a step (16) or a slab (32, 64); one row, one column of a tile, a sum of one
SHAPES = [
    (63, 2048, 16, 70), (64, 2047, 17, 128), (2048, 65, 16, 129),         # 128x128 forward; input gradient for the last
    (31, 2048, 16, 64), (2049, 33, 16, 33),                               # 64x128
    (32, 1024, 16, 40), (1023, 47, 16, 63),                               # 64x64
    (16, 2048, 16, 32), (2048, 100, 17, 1),                               # 32x128
    (1, 33, 2, 1), (15, 40, 3, 31), (65, 34, 2, 17), (300, 97, 5, 65),    # 32x32
    (127, 128, 40, 31), (128, 255, 33, 96), (515, 100, 32, 100),          # weight gradients with 64x128 tiles, sums ragged
]


def _operands(d_in, d_out, P, b, seed=7):
    rng = np.random.default_rng(seed)
    block = (d_in + 1) * d_out
    ld = block + (3 if d_in % 2 else 0)                                   # rows that start at any element
    # a wide range of magnitudes, so that in a short sum a part that is dropped or put to the wrong place shows in some
    # element (in a long one it does not: see test_long_sums_keep_every_part_of_either_operand)
    A = (rng.standard_normal((P, b, d_in)) * np.exp2(rng.integers(-6, 7, (P, b, d_in)))).astype(F)
    W = (rng.standard_normal((P, ld)) * np.exp2(rng.integers(-6, 7, (P, ld)))).astype(F)
    Z = (rng.standard_normal((P, b, d_out)) * 1e-3).astype(F)
    return A, W, Z, ld


def _products(kind, A, W, Z, d_in, d_out):
    """The product and the sum of absolute products per element, in 64 bits."""
    P, b = A.shape[:2]
    a, z = A.astype(np.float64), Z.astype(np.float64)
    w = W[:, :(d_in + 1) * d_out].reshape(P, d_in + 1, d_out).astype(np.float64)
    one = np.concatenate([a, np.ones((P, b, 1))], axis=2)
    if kind == 0:
        return one @ w, np.abs(one) @ np.abs(w), d_in + 1
    if kind == 1:
        t = one.transpose(0, 2, 1)
        return t @ z, np.abs(t) @ np.abs(z), b
    t = w[:, :d_in].transpose(0, 2, 1)
    gate = a > 0
    return (z @ t) * gate, (np.abs(z) @ np.abs(t)) * gate, d_out


def _run(hip, kind, A, W, Z, d_in, d_out, ld, width):
    P = A.shape[0]
    out = torch.full((P, width + 5), float("nan"), device="cuda")
    hip.easgd_layer_product(kind, d_in, d_out, to_dev(A), out, Wl=to_dev(W), dZ=to_dev(Z), ld=ld, out_ws=width + 5)
    got = to_host(out)
    assert np.isnan(got[:, width:]).all()
    return got[:, :width]


@pytest.mark.parametrize("d_in,d_out,P,b", SHAPES, ids=lambda v: str(v))
def test_every_element_against_64_bits(d_in, d_out, P, b):
    import paper_1708_02983_amd as hip
    A, W, Z, ld = _operands(d_in, d_out, P, b)
    for kind in (0, 1, 2):
        ref, mag, K = _products(kind, A, W, Z, d_in, d_out)
        got = _run(hip, kind, A, W, Z, d_in, d_out, ld, ref[0].size).reshape(ref.shape)
        # fp32 sums: at most K additions (the fp32 instruction, where a rule keeps it; one per sixteen and product in the
        # split form), each off by half an ulp of a partial sum; dropped products below 2^-24 of each term
        bound = (K + 8) * 2.0 ** -24 * mag
        worst = np.abs(got - ref) - bound
        assert (worst <= 0).all(), (kind, float((np.abs(got - ref) / np.maximum(mag, 1e-30)).max()))


@pytest.mark.parametrize("d_in,d_out,P,b", [(70, 2048, 16, 70), (65, 34, 2, 17)], ids=lambda v: str(v))
def test_infinities_and_nan_give_what_fp32_products_give(d_in, d_out, P, b):
    import paper_1708_02983_amd as hip
    A, W, Z, ld = _operands(d_in, d_out, P, b)
    A[0, 3, 5], A[0, 4, 64], A[1, 2, 0] = np.inf, -np.inf, np.nan
    W[0, 7 * d_out + 9] = np.inf
    W[1, (d_in - 1) * d_out + 33] = np.nan
    A[0, 5, 7] = 0.0                                                      # 0 * inf
    with np.errstate(invalid="ignore"):
        ref, _, _ = _products(0, A, W, Z, d_in, d_out)
    got = _run(hip, 0, A, W, Z, d_in, d_out, ld, ref[0].size).reshape(ref.shape)
    np.testing.assert_array_equal(np.isnan(got), np.isnan(ref))
    inf = np.isinf(ref)
    np.testing.assert_array_equal(got[inf], ref[inf].astype(F))
    assert np.isfinite(got[np.isfinite(ref)]).all()


# Sums of many slabs, so that the loop over whole slabs runs with the products whose loads were issued two slabs before: even
# and odd numbers of slabs, last slabs of every kind, all tiles (of 256 compute units) in forward and input-gradient form.
LONG_SHAPES = [
    (300, 2048, 16, 100), (351, 2048, 16, 128), (2048, 299, 16, 100), (2048, 416, 16, 90),   # 128x128: 10, 11; 10, 13 slabs
    (500, 2048, 16, 64), (1024, 300, 16, 128), (1024, 415, 16, 100),                         # 64x128
    (415, 768, 12, 192), (768, 333, 12, 150),                                                # 64x64
    (2100, 500, 17, 70), (500, 2101, 17, 70), (500, 641, 16, 128),                           # 64x64, both operands requested early
    (640, 2048, 16, 20),                                                                     # 32x128, the same
    (415, 2048, 17, 32), (2048, 300, 16, 20),                                                # 32x128
    (700, 97, 5, 65), (97, 700, 5, 65),                                                      # 32x32
]


def _three_parts(rng, shape):
    """24-bit numbers of either sign, all three bfloat16 parts of which are needed."""
    bits = rng.integers(1 << 23, 1 << 24, shape) | 1
    return (bits * rng.choice((-1.0, 1.0), shape) * 2.0 ** -23).astype(F)


@pytest.mark.parametrize("d_in,d_out,P,b", LONG_SHAPES, ids=lambda v: str(v))
def test_long_sums_keep_every_part_of_either_operand(d_in, d_out, P, b):
    """One nonzero 24-bit number per row of one operand, powers of two in the other: every result is one product and exact, so
    a part that is dropped, put to another place or multiplied by another slab's shows whatever the length of the sum.  Then
    ordinary operands against 64 bits."""
    import paper_1708_02983_amd as hip
    rng = np.random.default_rng(d_in + d_out)
    block = (d_in + 1) * d_out
    ld = block + (3 if d_in % 2 else 0)
    for kind in (0, 1, 2):
        for sparse_first in (True, False):
            # x (P, M, K) and y (P, K, N) of the product; the bias row of the weights stays zero
            M, K, n = {0: (b, d_in, d_out), 1: (d_in, b, d_out), 2: (b, d_out, d_in)}[kind]
            x, y = np.exp2(rng.integers(-3, 4, (P, M, K))).astype(F), np.exp2(rng.integers(-3, 4, (P, K, n))).astype(F)
            thin = np.zeros((P, M if sparse_first else n, K), dtype=F)
            at = (np.arange(thin.shape[1])[None, :] * 7 + np.arange(P)[:, None] * 5) % K
            np.put_along_axis(thin, at[:, :, None], _three_parts(rng, at.shape)[:, :, None], axis=2)
            if sparse_first: x = thin
            else: y = thin.transpose(0, 2, 1).copy()
            W = np.zeros((P, ld), dtype=F)
            A, Z = np.ones((P, b, d_in), dtype=F), np.zeros((P, b, d_out), dtype=F)
            if kind == 0: A, w = x, y
            elif kind == 1: A, Z, w = x.transpose(0, 2, 1).copy(), y, None
            else: Z, w = x, y.transpose(0, 2, 1)
            if w is not None: W[:, :d_in * d_out] = w.reshape(P, -1)
            ref, _, _ = _products(kind, A, W, Z, d_in, d_out)
            got = _run(hip, kind, A, W, Z, d_in, d_out, ld, ref[0].size).reshape(ref.shape)
            if kind == 1: got, ref = got[:, :d_in], ref[:, :d_in]         # (the bias row is a sum of many)
            np.testing.assert_array_equal(got, ref.astype(F), err_msg="kind %d sparse %s" % (kind, sparse_first))
        A, W, Z, _ = _operands(d_in, d_out, P, b)
        ref, mag, K = _products(kind, A, W, Z, d_in, d_out)
        got = _run(hip, kind, A, W, Z, d_in, d_out, W.shape[1], ref[0].size).reshape(ref.shape)
        assert (np.abs(got - ref) <= (K + 8) * 2.0 ** -24 * mag).all(), kind


def test_64x64_tiles_keep_their_bits_in_either_order_of_the_loads():
    """Sixteen workers have one block per compute unit and request both operands early, seventeen do not."""
    import paper_1708_02983_amd as hip
    d_in, d_out, P, b = 500, 641, 17, 128
    A, W, Z, ld = _operands(d_in, d_out, P, b)
    few = _run(hip, 2, A[:16], W[:16], Z[:16], d_in, d_out, ld, b * d_in)
    np.testing.assert_array_equal(_run(hip, 2, A, W, Z, d_in, d_out, ld, b * d_in)[:16], few)


RANGE_SHAPES = [(300, 2048, 16, 70), (2048, 100, 17, 40), (65, 34, 2, 17), (127, 128, 40, 31)]


def _scaled_operands(d_in, d_out, P, b, kind, sx, sy):
    """Operands of ordinary values times sx (the operand that is summed along its rows first) and sy; no bias."""
    A, W, Z, ld = _operands(d_in, d_out, P, b)
    W[:, d_in * d_out:(d_in + 1) * d_out] = 0.0
    Z *= F(1e3)
    with np.errstate(over="ignore"):
        if kind == 0:
            A, W = A * F(sx), W * F(sy)
        elif kind == 1:
            A, Z = A * F(sx), Z * F(sy)
        else:
            Z, W = Z * F(sx), W * F(sy)
    return A, W, Z, ld


@pytest.mark.parametrize("sx,sy", [(2.0 ** -120, 2.0 ** 60), (2.0 ** 60, 2.0 ** -120), (2.0 ** -138, 2.0 ** 100),
                                   (2.0 ** 100, 2.0 ** -40), (2.0 ** 30, 2.0 ** 70)], ids=lambda v: "2^%d" % np.log2(v))
@pytest.mark.parametrize("d_in,d_out,P,b", RANGE_SHAPES, ids=lambda v: str(v))
def test_small_and_large_operands_lose_nothing(d_in, d_out, P, b, sx, sy):
    """Down to denormal operands (whose products are not) and up to sums that only just are finite."""
    import paper_1708_02983_amd as hip
    for kind in (0, 1, 2):
        A, W, Z, ld = _scaled_operands(d_in, d_out, P, b, kind, sx, sy)
        ref, mag, K = _products(kind, A, W, Z, d_in, d_out)
        got = _run(hip, kind, A, W, Z, d_in, d_out, ld, ref[0].size).reshape(ref.shape)
        worst = np.abs(got - ref) - ((K + 8) * 2.0 ** -24 * mag + K * 2.0 ** -149)
        assert (worst <= 0).all(), (kind, float(np.nanmax(np.abs(got - ref) / np.maximum(mag, 1e-300))))


@pytest.mark.parametrize("d_in,d_out,P,b", RANGE_SHAPES, ids=lambda v: str(v))
def test_values_at_the_ends_of_the_range(d_in, d_out, P, b):
    """Finite values beyond the largest bfloat16 in either operand, times zeros and small values; infinities times denormal
    ones; NaN: all three products give what sums of fp32 products give."""
    import paper_1708_02983_amd as hip
    top, tiny = F(3.4e38), F(2.0 ** -140)
    for kind in (0, 1, 2):
        A, W, Z, ld = _scaled_operands(d_in, d_out, P, b, kind, 1.0, 1.0)
        w = W[:, :(d_in + 1) * d_out].reshape(P, d_in + 1, d_out)          # a view when the rows are packed, else a copy
        x, y = {0: (A, w), 1: (A.transpose(0, 2, 1), Z), 2: (Z, w.transpose(0, 2, 1))}[kind]    # x (P, M, K), y (P, K, N)
        y[0, 1, :] *= F(2.0 ** -40)
        x[0, 1, 1] = top                                                   # times small values: finite
        y[0, 2, 3] = top
        x[0, :, 2] = 0.0                                                   # times zero: nothing
        y[0, 4, 5] = tiny
        y[0, 4, 6] = -tiny
        x[0, 0, 4] = np.inf
        x[1, 3, 5] = np.nan
        x[1, 2, 0] = -np.inf
        W[:, :(d_in + 1) * d_out] = w.reshape(P, -1)
        with np.errstate(invalid="ignore"):
            ref, mag, K = _products(kind, A, W, Z, d_in, d_out)
            if kind == 2:                                                  # the gate replaces, it does not multiply
                z, t = Z.astype(np.float64), w[:, :d_in].transpose(0, 2, 1).astype(np.float64)
                ref, mag = np.where(A > 0, z @ t, 0.0), np.where(A > 0, np.abs(z) @ np.abs(t), 0.0)
        got = _run(hip, kind, A, W, Z, d_in, d_out, ld, ref[0].size).reshape(ref.shape)
        np.testing.assert_array_equal(np.isnan(got), np.isnan(ref), err_msg=str(kind))
        inf, fin = np.isinf(ref), np.isfinite(ref)
        np.testing.assert_array_equal(got[inf], ref[inf].astype(F), err_msg=str(kind))
        with np.errstate(invalid="ignore"):
            bound = (K + 8) * 2.0 ** -24 * mag
        assert (np.abs(got[fin] - ref[fin]) <= bound[fin]).all(), kind


@pytest.mark.parametrize("kind,d_in,d_out,P,b", [
    (0, 64, 512, 8, 50), (0, 127, 1024, 8, 256), (0, 640, 500, 15, 100),         # short; a grid that the fp32 tiles fill
    (2, 512, 64, 8, 50), (2, 1024, 100, 8, 256), (2, 500, 640, 15, 100),
    (1, 1024, 48, 32, 100), (1, 1024, 1024, 16, 16), (1, 255, 500, 3, 40),       # half empty tiles; a short slab; few blocks
], ids=lambda v: str(v))
def test_products_that_the_split_form_would_slow_down_keep_the_fp32_instruction(kind, d_in, d_out, P, b):
    """There the default gives the bits of the forced 64x64 tile."""
    import paper_1708_02983_amd as hip
    A, W, Z, ld = _operands(d_in, d_out, P, b)
    width = (b * d_out, (d_in + 1) * d_out, b * d_in)[kind]
    old = hip.get_option(hip.OPT_GEMM_TILE)
    try:
        got = []
        for tile in (0, 2):
            hip.set_option(hip.OPT_GEMM_TILE, tile)
            got.append(_run(hip, kind, A, W, Z, d_in, d_out, ld, width))
    finally:
        hip.set_option(hip.OPT_GEMM_TILE, old)
    np.testing.assert_array_equal(got[0], got[1])


@pytest.mark.parametrize("dims,P,b", [((63, 37, 41, 10), 3, 20), ((64, 65, 130, 20), 2, 33), ((33, 2048, 10), 16, 33)],
                         ids=lambda v: str(v).replace(" ", ""))
def test_row_stride_does_not_change_a_bit(dims, P, b):
    """Replicas packed back to back, so that rows and layers start at any element, against padded ones."""
    import paper_1708_02983_amd as hip
    N = workloads.mlp_num_params(dims)
    rng = np.random.default_rng(3)
    rows = (rng.standard_normal((P, N)) * 0.1).astype(F)
    X = to_dev(rng.standard_normal((P, b, dims[0])).astype(F))
    y = to_dev(rng.integers(0, dims[-1], (P, b)).astype(np.int32))
    got = []
    for ld in (N, N + 1, (N + 255) // 256 * 256):
        W = np.full((P, ld), np.nan, dtype=F)
        W[:, :N] = rows
        G = torch.full((P, ld), float("nan"), device="cuda")
        loss = torch.empty(P, device="cuda")
        hip.easgd_grad(dims, to_dev(W), X, y, G, loss)
        g = to_host(G)
        assert np.isnan(g[:, N:]).all()
        got.append((g[:, :N], to_host(loss)))
    for g, l in got[1:]:
        np.testing.assert_array_equal(g, got[0][0])
        np.testing.assert_array_equal(l, got[0][1])


def test_logits_of_replicas_beyond_the_last_level_cache_keep_the_fp32_instruction():
    """From 2^26 parameters in all replicas on every product does, the last layer's forward product included: the gradients
    have the bits of the forced fp32 64x64 tile (whose sums run in the same order)."""
    import paper_1708_02983_amd as hip
    dims, P, b = (2048, 1000), 33, 64
    N = workloads.mlp_num_params(dims)
    assert P * N >= 2 ** 26 > (P - 1) * N
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    W = torch.empty((P, N), device="cuda").normal_(0.0, 0.03, generator=gen)
    X = torch.rand((P, b, dims[0]), device="cuda", generator=gen)
    y = torch.randint(0, dims[1], (P, b), dtype=torch.int32, device="cuda", generator=gen)
    old = hip.get_option(hip.OPT_GEMM_TILE)
    got = []
    try:
        for tile in (0, 2):
            hip.set_option(hip.OPT_GEMM_TILE, tile)
            G, loss = torch.full_like(W, float("nan")), torch.empty(P, device="cuda")
            hip.easgd_grad(dims, W, X, y, G, loss)
            got.append((G, loss))
    finally:
        hip.set_option(hip.OPT_GEMM_TILE, old)
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
