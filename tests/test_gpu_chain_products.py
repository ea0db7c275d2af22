"""Products of small grids in 16x16 tiles of the fp32 matrix instruction: an element is a chain of fused multiply-adds in
ascending k whatever tile it is computed in, so every tile gives the bits of the 64x64 one (EASGD_OPT_GEMM_TILE 2).  Sizes one
below, at and above a tile, a slab (64 values of k) and the pipeline's first slabs; rows that start at any element."""
import numpy as np
import pytest
import torch

import workloads
from gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu
F = np.float32


def _with_tile(hip, tile, f):
    old = hip.get_option(hip.OPT_GEMM_TILE)
    hip.set_option(hip.OPT_GEMM_TILE, tile)
    try:
        return f()
    finally:
        hip.set_option(hip.OPT_GEMM_TILE, old)


# (dims, P, b): the tiles that 256 compute units take for the hidden layers
NETWORKS = [
    ((63, 33, 10), 2, 1), ((64, 48, 10), 3, 15), ((65, 65, 10), 2, 16),           # 32x32; sums of 64, 65, 66
    ((784, 500, 300, 10), 8, 50), ((255, 34, 257, 12), 5, 33), ((511, 130, 3), 4, 65),
    ((1023, 777, 333, 7), 6, 37), ((300, 1009, 10), 5, 48),                             # 16x64 (and 32x32 for 777->333)
    ((129, 1000, 16), 5, 17),                                                           # 32x32
    ((156, 1041, 10), 13, 17), ((129, 1520, 10), 4, 63), ((256, 513, 10), 7, 65),       # 32x64
    ((784, 640, 10), 12, 100),                                                          # the 64x64 tile itself
]


@pytest.mark.parametrize("dims,P,b", NETWORKS, ids=lambda v: str(v))
def test_hidden_layers_keep_the_bits_of_the_64x64_tile(dims, P, b):
    """The last layer's weight gradient [H 1]^T dZ takes the same kernel for either option and depends on every hidden unit."""
    import paper_1708_02983_amd as hip
    rng = np.random.default_rng(sum(dims) + b)
    N = workloads.mlp_num_params(dims)
    W = (rng.standard_normal((P, N)) * np.sqrt(2.0 / dims[0])).astype(F)
    X = rng.random((P, b, dims[0]), dtype=F)
    y = to_dev(rng.integers(0, dims[-1], (P, b)).astype(np.int32))
    last = (dims[-2] + 1) * dims[-1]
    dW, dX = to_dev(W), to_dev(X)

    def grad():
        G, loss = torch.full((P, N), float("nan"), device="cuda"), torch.empty(P, device="cuda")
        hip.easgd_grad(dims, dW, dX, y, G, loss)
        return to_host(G)[:, N - last:], to_host(loss)

    g, loss = _with_tile(hip, 0, grad)
    g2, loss2 = _with_tile(hip, 2, grad)
    np.testing.assert_array_equal(loss, loss2)
    np.testing.assert_array_equal(g, g2)
    assert np.isfinite(g).all() and (g != 0).any()


# (d_in, d_out, P, b): sums too short for the split form
INPUT_GRADIENTS = [(47, 2, 3, 1), (64, 31, 2, 16), (97, 36, 4, 33), (300, 64, 3, 37), (641, 68, 6, 37),   # 32x32
                   (321, 64, 24, 17), (353, 100, 23, 17),                                        # 32x64
                   (1024, 48, 16, 128),                                                          # the 64x64 tile itself
                   (321, 63, 24, 1),                                                             # 32x32 of the split form
                   # one to six slabs of 64, with 128-bit loads on the 64x64 path and without (sums below 40)
                   (828, 100, 3, 63), (403, 204, 19, 87), (1302, 33, 3, 43),                                # 32x32
                   (1766, 80, 20, 9), (995, 108, 15, 13), (767, 324, 11, 46), (1517, 312, 6, 45), (1062, 39, 13, 14),   # 16x64
                   (940, 172, 12, 31), (1752, 244, 5, 94), (901, 224, 9, 78), (1074, 248, 16, 70), (1768, 39, 18, 32)]  # 32x64


@pytest.mark.parametrize("d_in,d_out,P,b", INPUT_GRADIENTS, ids=lambda v: str(v))
def test_short_sums_of_input_gradients_keep_the_bits_of_the_64x64_tile(d_in, d_out, P, b):
    import paper_1708_02983_amd as hip
    rng = np.random.default_rng(d_in + d_out + b)
    ld = (d_in + 1) * d_out + 3
    A, W, Z = (to_dev(rng.standard_normal(s).astype(F)) for s in ((P, b, d_in), (P, ld), (P, b, d_out)))

    def product():
        out = torch.full((P, b * d_in + 5), float("nan"), device="cuda")
        hip.easgd_layer_product(2, d_in, d_out, A, out, Wl=W, dZ=Z, ld=ld, out_ws=b * d_in + 5)
        return to_host(out)

    got, ref = _with_tile(hip, 0, product), _with_tile(hip, 2, product)
    assert np.isnan(got[:, b * d_in:]).all()
    gate = to_host(A).reshape(P, -1) > 0
    exact = (to_host(Z).astype(np.float64) @ to_host(W)[:, :d_in * d_out].reshape(P, d_in, d_out).astype(np.float64).transpose(0, 2, 1)).reshape(P, -1)
    mag = (np.abs(to_host(Z)).astype(np.float64) @ np.abs(to_host(W))[:, :d_in * d_out].reshape(P, d_in, d_out).astype(np.float64).transpose(0, 2, 1)).reshape(P, -1)
    # at most d_out additions, each off by half an ulp of a partial sum
    assert (np.abs(got[:, :b * d_in] - np.where(gate, exact, 0.0)) <= (d_out + 8) * 2.0 ** -24 * mag).all()
    if d_out % 4 == 0 or d_out < 40:            # the split form starts at sums of 40 where a width rules out 128-bit loads
        np.testing.assert_array_equal(got[:, :b * d_in], ref[:, :b * d_in])


# 32x32 forward and, at a sum of 50, the split form's input gradient; 32x32, 16x64 and 32x64 input gradients
@pytest.mark.parametrize("d_in,d_out,P,b", [(65, 50, 3, 17), (65, 34, 3, 17), (1062, 39, 13, 14), (1768, 39, 18, 32)], ids=lambda v: str(v))
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_what_lies_behind_a_row_does_not_reach_a_sum(bad, d_in, d_out, P, b):
    """A 128-bit load at the end of a row brings the values behind it, and the last slab of a sum those of the next layer: none of
    them may meet a zero in a product (0 * inf is NaN)."""
    import paper_1708_02983_amd as hip
    rng = np.random.default_rng(3)
    A, Z = rng.standard_normal((P, b, d_in)).astype(F), rng.standard_normal((P, b, d_out)).astype(F)
    block = (d_in + 1) * d_out
    W = np.full((P, block + 70 * d_out), bad, dtype=F)
    W[:, :block] = rng.standard_normal((P, block))
    dA, dW, dZ = to_dev(A), to_dev(W), to_dev(Z)
    for kind, width in ((0, d_out), (2, d_in)):
        out = torch.empty((P, b * width), device="cuda")
        hip.easgd_layer_product(kind, d_in, d_out, dA, out, Wl=dW, dZ=dZ, ld=W.shape[1], out_ws=b * width)
        assert np.isfinite(to_host(out)).all(), kind


# (d_in, d_out, P, b): one, two tiles of sixteen columns; rows one below, at and above a wavefront's and a block's; sums one below,
# at and above a matrix instruction (4), a trip to memory (64) and two of them
NARROW = [(1, 1, 2, 1), (15, 3, 3, 3), (16, 10, 2, 4), (17, 16, 4, 5), (63, 10, 9, 63), (64, 12, 8, 64), (65, 2, 16, 65),
          (127, 17, 3, 30), (130, 31, 8, 129), (785, 10, 5, 130), (96, 32, 4, 40)]


@pytest.mark.parametrize("d_in,d_out,P,b", NARROW, ids=lambda v: str(v))
def test_narrow_weight_gradients_element_by_element(d_in, d_out, P, b):
    import paper_1708_02983_amd as hip
    rng = np.random.default_rng(d_in + d_out + b)
    A, Z = rng.standard_normal((P, b, d_in)).astype(F), rng.standard_normal((P, b, d_out)).astype(F)
    width = (d_in + 1) * d_out
    one = np.concatenate([A, np.ones((P, b, 1), F)], axis=2).astype(np.float64).transpose(0, 2, 1)
    ref, mag = (one @ Z.astype(np.float64)).reshape(P, -1), (np.abs(one) @ np.abs(Z).astype(np.float64)).reshape(P, -1)

    def product(A):
        out = torch.full((P, width + 5), float("nan"), device="cuda")
        hip.easgd_layer_product(1, d_in, d_out, to_dev(A), out, dZ=to_dev(Z), out_ws=width + 5)
        got = to_host(out)
        assert np.isnan(got[:, width:]).all()
        return got[:, :width]

    # b additions, each off by half an ulp of a partial sum
    assert (np.abs(product(A) - ref) <= (b + 8) * 2.0 ** -24 * mag).all()
    # an infinity in the last row of A reaches the first row of the result and no other
    A[:, b - 1, 0] = np.inf
    got = product(A).reshape(P, d_in + 1, d_out)
    assert not np.isfinite(got[:, 0]).any() and np.isfinite(got[:, 1:]).all()


# (kind, d_in, d_out, P, b): several blocks of a small tile per compute unit, at short sums, where the 64x64 tile is faster
SEVERAL_BLOCKS = [(0, 65, 1326, 27, 34), (0, 80, 1168, 8, 193), (2, 560, 64, 29, 115), (2, 896, 96, 10, 229)]


@pytest.mark.parametrize("kind,d_in,d_out,P,b", SEVERAL_BLOCKS, ids=lambda v: str(v))
def test_the_tile_that_is_picked_is_not_slower_than_the_64x64_tile(kind, d_in, d_out, P, b):
    """Small tiles took 1.5 to 1.8 times as long here.  Launches in a graph, both sides in turn, the best of nine; two runs of one side
    differ by a few percent."""
    import paper_1708_02983_amd as hip
    ld = (d_in + 1) * d_out
    A, W, Z = (torch.randn(s, device="cuda") for s in ((P, b, d_in), (P, ld), (P, b, d_out)))
    width = b * (d_out if kind == 0 else d_in)
    out = torch.empty((P, width), device="cuda")

    def product():
        hip.easgd_layer_product(kind, d_in, d_out, A, out, Wl=W, dZ=Z, ld=ld, out_ws=width, relu=kind == 0)

    def graph():
        product()
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            for _ in range(40): product()
        return g

    sides = [graph(), _with_tile(hip, 2, graph)]
    best = [float("inf"), float("inf")]
    for _ in range(9):
        for i, g in enumerate(sides):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            g.replay()
            e0.record()
            g.replay()
            e1.record()
            torch.cuda.synchronize()
            best[i] = min(best[i], e0.elapsed_time(e1))
    assert best[0] < 1.2 * best[1], best


# (d_in, d_out, P, b): more blocks of 64 rows than one (three) per compute unit, which take the 128x32 tile; four workers of them
# take the narrow kernel
MANY_NARROW = [(640, 12, 24, 132), (640, 16, 24, 192), (1023, 17, 50, 37), (1022, 32, 50, 65)]


@pytest.mark.parametrize("d_in,d_out,P,b", MANY_NARROW, ids=lambda v: str(v))
def test_narrow_weight_gradients_keep_the_bits_of_the_128x32_tile(d_in, d_out, P, b):
    import paper_1708_02983_amd as hip
    A, Z = torch.randn((P, b, d_in), device="cuda"), torch.randn((P, b, d_out), device="cuda")
    width = (d_in + 1) * d_out

    def product(P):
        out = torch.full((P, width), float("nan"), device="cuda")
        hip.easgd_layer_product(1, d_in, d_out, A[:P], out, dZ=Z[:P], out_ws=width)
        return to_host(out)

    np.testing.assert_array_equal(product(P)[:4], product(4))


def test_shared_launches_keep_the_bits_of_either_narrow_form():
    """The last layer's weight gradient in the launch of the hidden layer's input gradient: the 128x32 tile for all workers, the
    narrow kernel for four of them."""
    import paper_1708_02983_amd as hip
    dims, P, b = (20, 48, 640, 12), 24, 132
    N, last = workloads.mlp_num_params(dims), 641 * 12
    ld = (N + 3) // 4 * 4
    W, X = torch.randn((P, ld), device="cuda") * 0.1, torch.rand((P, b, 20), device="cuda")
    y = torch.randint(0, 12, (P, b), dtype=torch.int32, device="cuda")

    def grad(P):
        G = torch.full((P, ld), float("nan"), device="cuda")
        hip.easgd_grad(dims, W[:P], X[:P], y[:P], G)
        return to_host(G)[:, N - last:N]

    got = grad(P)
    assert np.isfinite(got).all()
    np.testing.assert_array_equal(got[:4], grad(4))
