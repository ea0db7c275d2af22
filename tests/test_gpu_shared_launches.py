"""An input-gradient product and the weight gradient of a narrow layer share a launch in every form that either of them
takes: fewer launches, the same bits."""
import numpy as np
import pytest
import torch

import workloads
from gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu
F = np.float32

# dims, P, b, EASGD_OPT_GEMM_TILE: the input gradient of the layer above the first as ...
CASES = [
    ((40, 2048, 300, 12), 16, 20, 0),         # split 32x128 tiles (a minibatch of at most 32 rows)
    ((71, 261, 303, 20), 3, 37, 0),           # split 32x32, a last layer without 128-bit loads
    ((72, 260, 304, 16), 3, 37, 0),           # split 32x32, a last layer with them
    ((72, 260, 200, 16), 3, 37, 2),           # fp32 64x64 tiles, forced
    ((72, 260, 48, 18), 3, 37, 2),            # the same, a last layer without 128-bit loads
    ((72, 1000, 48, 16), 9, 100, 0),          # a short sum
]


@pytest.mark.parametrize("dims,P,b,tile", CASES, ids=lambda v: str(v).replace(" ", ""))
def test_narrow_weight_gradients_share_a_launch(dims, P, b, tile):
    import paper_1708_02983_amd as hip
    N = workloads.mlp_num_params(dims)
    rng = np.random.default_rng(11)
    W = to_dev((rng.standard_normal((P, N)) * 0.1).astype(F))
    Wc, V = to_dev(to_host(W)[0].copy()), to_dev((rng.standard_normal((P, N)) * 1e-3).astype(F))
    X = to_dev(rng.standard_normal((P, b, dims[0])).astype(F))
    y = to_dev(rng.integers(0, dims[-1], (P, b)).astype(np.int32))
    old = hip.get_option(hip.OPT_GEMM_TILE), hip.get_option(hip.OPT_GEMM_PAIR)
    launches, outs = [], []
    try:
        hip.set_option(hip.OPT_GEMM_TILE, tile)
        for pair in (0, 1):
            hip.set_option(hip.OPT_GEMM_PAIR, pair)
            G, loss = torch.full_like(W, float("nan")), torch.full((P,), float("nan"), device="cuda")
            before = hip.launch_count()
            hip.easgd_grad(dims, W, X, y, G, loss)
            launches.append(hip.launch_count() - before)
            res = [to_host(G), to_host(loss)]
            for rule in ("easgd", "measgd"):
                rW, rV, rWc, rl = W.clone(), V.clone(), Wc.clone(), torch.full_like(loss, float("nan"))
                hip.easgd_mlp_round(dims, rW, rWc, X, y, 0.05, 0.05, V=rV if rule == "measgd" else None, delta=0.9, loss=rl)
                res += [to_host(rW), to_host(rV), to_host(rWc), to_host(rl)]
            outs.append(res)
    finally:
        hip.set_option(hip.OPT_GEMM_TILE, old[0])
        hip.set_option(hip.OPT_GEMM_PAIR, old[1])
    # the last layer's weight gradient with the input gradient of the layer below, and the weight gradients of the
    # layers below that where both take the same form
    assert launches[1] <= launches[0] - 1 - (tile == 2), launches
    for a, c in zip(*outs):
        assert np.isfinite(a).all()
        np.testing.assert_array_equal(a, c)


@pytest.mark.parametrize("dims,P,b,rides", [((3072, 593), 3, 124, True), ((2048, 1000), 16, 128, False)],
                         ids=lambda v: str(v).replace(" ", ""))
def test_center_rule_rides_on_wide_logits_where_their_tile_leaves_room(dims, P, b, rides):
    """One layer and more than 32 classes: the first forward product is the logits, as split tiles.  420 blocks of 64x128 fill
    three quarters of the chip's places for them, so the center rule is on extra blocks and not a launch of its own; 128x128
    tiles fill all of theirs.  The same bits either way."""
    import paper_1708_02983_amd as hip
    N = workloads.mlp_num_params(dims)
    rng = np.random.default_rng(12)
    W = to_dev((rng.standard_normal((P, N)) * 0.03).astype(F))
    Wc = to_dev(to_host(W)[0].copy())
    X = to_dev(rng.random((P, b, dims[0])).astype(F))
    y = to_dev(rng.integers(0, dims[-1], (P, b)).astype(np.int32))
    old = hip.get_option(hip.OPT_ROUND_OVERLAP)
    launches, outs = {}, []
    try:
        for overlap in (0, 1, 3):                   # a launch of its own; chosen; extra blocks
            hip.set_option(hip.OPT_ROUND_OVERLAP, overlap)
            rW, rWc, loss = W.clone(), Wc.clone(), torch.empty(P, device="cuda")
            before = hip.launch_count()
            hip.easgd_mlp_round(dims, rW, rWc, X, y, 0.05, 0.05, loss=loss)
            launches[overlap] = hip.launch_count() - before
            outs.append([to_host(rW), to_host(rWc), to_host(loss)])
    finally:
        hip.set_option(hip.OPT_ROUND_OVERLAP, old)
    assert launches[3] == launches[0] - 1 and (launches[1] == launches[3]) == rides, launches
    for res in outs[1:]:
        for a, c in zip(outs[0], res):
            np.testing.assert_array_equal(a, c)
