"""The calls of this library that are timed, and the ranges that they stand for.

A training program calls one of
  * ``easgd_mlp_round``: a whole Sync EASGD round of a dense ReLU network, forward and backward (kind "round");
  * ``easgd_grad``: the gradients of all workers, for a program that does something of its own with them before the
    exchange (kind "gradient");
  * ``easgd_sync_round`` / ``measgd_round`` / ``measgd_round_bf16``: the elastic exchange-and-update of replicas whose
    gradients come from elsewhere, for instance from convolutions (kind "update");
  * ``easgd_layer_product``: one product of a dense layer for all workers, forward or either direction of backward
    propagation (kind "layer").

``rows`` says how the program lays its replica matrices out: "padded" rows start at multiples of 256 elements, "packed"
rows follow one another as ``torch.empty(P, N)`` gives them, whatever N is.
"""
import math

import numpy as np
import torch

import paper_1708_02983_amd as hip

ETA, RHO, DELTA = 0.05, 0.05, 0.9
RULES = ("easgd", "measgd", "measgd_bf16")


def listed():
    return [
        # the smallest round there is in use: softmax regression on digits, a handful of workers; launches and latency
        {"name": "softmax_round", "kind": "round", "dims": "784-10", "P": 4, "b": 64, "rule": "easgd", "rows": "padded"},
        # the default benchmark workload: digit-sized inputs, two hidden layers
        {"name": "digits_round", "kind": "round", "dims": "784-1024-1024-10", "P": 16, "b": 128, "rule": "easgd", "rows": "padded"},
        # the largest training workload: image-sized inputs, momentum, a batch that fills no whole matrix tile
        {"name": "images_round_momentum", "kind": "round", "dims": "3072-2048-2048-10", "P": 32, "b": 100, "rule": "measgd", "rows": "padded"},
        # an ordinary small network whose parameter count is no multiple of four, replicas allocated without padding
        {"name": "packed_round_momentum", "kind": "round", "dims": "784-500-300-10", "P": 8, "b": 50, "rule": "measgd", "rows": "packed"},
        # widths that are multiples of nothing, more classes than the fused last layer takes, replicas without padding
        {"name": "odd_gradient", "kind": "gradient", "dims": "1023-777-333-100", "P": 6, "b": 37, "rows": "packed"},
        # single layers: a long sum with a large batch; a short sum with a large result; a ragged batch
        {"name": "layer_forward", "kind": "layer", "product": "forward", "d_in": 3072, "d_out": 2048, "P": 8, "b": 256, "rows": "padded"},
        {"name": "layer_weight_gradient", "kind": "layer", "product": "weight_gradient", "d_in": 1024, "d_out": 1024, "P": 16, "b": 128, "rows": "padded"},
        {"name": "layer_input_gradient", "kind": "layer", "product": "input_gradient", "d_in": 2048, "d_out": 2048, "P": 32, "b": 100, "rows": "padded"},
        # the exchange alone at the size the method was made for, plain and with momentum (the largest call)
        {"name": "alexnet_update", "kind": "update", "P": 8, "N": 61_000_000, "rule": "easgd", "rows": "padded"},
        {"name": "alexnet_update_momentum", "kind": "update", "P": 16, "N": 61_000_000, "rule": "measgd", "rows": "padded"},
        # the exchange of the default network's replicas as a program allocates them without thinking about padding
        {"name": "digits_update_packed", "kind": "update", "P": 16, "N": 1_863_690, "rule": "easgd", "rows": "packed"},
        # gradients and momentum buffers stored in 16 bits, at the larger network's size
        {"name": "images_update_bf16", "kind": "update", "P": 8, "N": 10_510_346, "rule": "measgd_bf16", "rows": "padded"},
    ]


def _dims(case):
    return tuple(int(d) for d in case["dims"].split("-"))


def _num_params(dims):
    return sum((dims[l] + 1) * dims[l + 1] for l in range(len(dims) - 1))


def _ld(case, n):
    return (n + 255) // 256 * 256 if case["rows"] == "padded" else n


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_once(rng):
    kind = rng.choice(("round", "round", "gradient", "layer", "update"))
    rows = rng.choice(("padded", "packed"))
    if kind == "update":
        return {"kind": kind, "P": _log_int(rng, 2, 32), "N": _log_int(rng, 5_000, 61_000_000), "rule": rng.choice(RULES), "rows": rows}
    P, b = _log_int(rng, 2, 32), _log_int(rng, 16, 256)
    if kind == "layer":
        return {"kind": kind, "product": rng.choice(("forward", "weight_gradient", "input_gradient")),
                "d_in": _log_int(rng, 64, 3072), "d_out": _log_int(rng, 48, 2048), "P": P, "b": b, "rows": rows}
    hidden = [_log_int(rng, 48, 2048) for _ in range(rng.randint(0, 3))]
    # most programs choose round widths, some do not
    if rng.random() < 0.5:
        hidden = [(h + 15) // 16 * 16 for h in hidden]
    d_in = rng.choice((784, 3072, _log_int(rng, 64, 3072)))
    classes = rng.choice((10, 10, _log_int(rng, 2, 1000)))
    case = {"kind": kind, "dims": "-".join(str(d) for d in (d_in, *hidden, classes)), "P": P, "b": b, "rows": rows}
    if kind == "round":
        case["rule"] = rng.choice(RULES[:2])
    return case


def draw(rng):
    largest_bytes = max(work(c)["bytes"] for c in listed())
    largest_flops = max(work(c)["flops"] for c in listed())
    while True:
        case = _draw_once(rng)
        w = work(case)
        if w["bytes"] <= largest_bytes and w["flops"] <= largest_flops:
            return case


# ---- inputs -------------------------------------------------------------------------------------------------------

class _Draws:
    """Seeded draws made on the GPU, and zero-filled matrices whose valid columns hold them."""

    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(seed)

    def normal(self, shape, std):
        return torch.empty(shape, dtype=torch.float32, device="cuda").normal_(0.0, std, generator=self.gen)

    def rows(self, P, n, ld, std):
        if ld == n:
            return self.normal((P, n), std)
        out = torch.zeros((P, ld), dtype=torch.float32, device="cuda")
        for i in range(P):
            out[i, :n].normal_(0.0, std, generator=self.gen)
        return out

    def labels(self, shape, classes):
        return torch.randint(0, classes, shape, dtype=torch.int32, device="cuda", generator=self.gen)


def _layer_std(d_in):
    return math.sqrt(2.0 / d_in)                                 # He-normal


def _network(case, seed):
    """Replicas that have drifted apart around the center, a minibatch per worker, momentum of earlier rounds."""
    dims, P, b = _dims(case), case["P"], case["b"]
    n = _num_params(dims)
    ld = _ld(case, n)
    d = _Draws(seed)
    Wc = torch.empty(n, dtype=torch.float32, device="cuda")
    W = torch.zeros((P, ld), dtype=torch.float32, device="cuda")
    off = 0
    for l in range(len(dims) - 1):
        size, bias = dims[l] * dims[l + 1], dims[l + 1]
        Wc[off:off + size] = d.normal((size,), _layer_std(dims[l]))
        Wc[off + size:off + size + bias] = d.normal((bias,), 0.05)
        off += size + bias
    for i in range(P):
        W[i, :n] = Wc * (1.0 + d.normal((n,), 0.05))
    X = torch.rand((P, b, dims[0]), dtype=torch.float32, device="cuda", generator=d.gen)   # pixels
    y = d.labels((P, b), dims[-1])
    V = d.rows(P, n, ld, 1e-4) if case.get("rule") == "measgd" else None
    return W, Wc, V, X, y


def _replicas(case, seed):
    P, n = case["P"], case["N"]
    ld = _ld(case, n)
    d = _Draws(seed)
    W, Wc = d.rows(P, n, ld, 0.01), d.normal((n,), 0.01)
    G = d.rows(P, n, ld, 1e-3)
    V = None if case["rule"] == "easgd" else d.rows(P, n, ld, 1e-4)
    if case["rule"] == "measgd_bf16":
        G, V = G.to(torch.bfloat16), V.to(torch.bfloat16)
    return W, V, G, Wc


def _layer(case, seed):
    P, b, d_in, d_out = case["P"], case["b"], case["d_in"], case["d_out"]
    block = (d_in + 1) * d_out
    d = _Draws(seed)
    A = d.normal((P, b, d_in), 1.0).clamp_(min=0.0)              # what a ReLU layer hands on
    Wl = d.rows(P, block, _ld(case, block), _layer_std(d_in))
    dZ = d.normal((P, b, d_out), 1e-3)
    return A, Wl, dZ


_PRODUCTS = {"forward": 0, "weight_gradient": 1, "input_gradient": 2}


def prepare(case, seed):
    state = {"case": case}
    if case["kind"] in ("round", "gradient"):
        dims = _dims(case)
        W, Wc, V, X, y = _network(case, seed)
        whole = case["kind"] == "round"
        size = (hip.easgd_mlp_round_workspace_bytes if whole else hip.easgd_grad_workspace_bytes)(dims, case["P"], case["b"])
        state.update(dims=dims, W=W, Wc=Wc, V=V, X=X, y=y,
                     G=None if whole else torch.zeros_like(W),
                     loss=torch.empty(case["P"], dtype=torch.float32, device="cuda"),
                     workspace=torch.empty(size, dtype=torch.uint8, device="cuda"))
    elif case["kind"] == "update":
        W, V, G, Wc = _replicas(case, seed)
        state.update(W=W, V=V, G=G, Wc=Wc)
    else:
        A, Wl, dZ = _layer(case, seed)
        width = {"forward": case["b"] * case["d_out"], "weight_gradient": (case["d_in"] + 1) * case["d_out"],
                 "input_gradient": case["b"] * case["d_in"]}[case["product"]]
        state.update(A=A, Wl=Wl, dZ=dZ, out=torch.empty((case["P"], width), dtype=torch.float32, device="cuda"))
    return state


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "round":
        hip.easgd_mlp_round(state["dims"], state["W"], state["Wc"], state["X"], state["y"], ETA, RHO, V=state["V"], delta=DELTA,
                            loss=state["loss"], workspace=state["workspace"])
        out = {"W": state["W"], "Wc": state["Wc"], "loss": state["loss"]}
        if state["V"] is not None:
            out["V"] = state["V"]
        return out
    if kind == "gradient":
        hip.easgd_grad(state["dims"], state["W"], state["X"], state["y"], state["G"], state["loss"], workspace=state["workspace"])
        return {"G": state["G"], "loss": state["loss"]}
    if kind == "update":
        W, V, G, Wc, n = state["W"], state["V"], state["G"], state["Wc"], case["N"]
        if case["rule"] == "easgd":
            hip.easgd_sync_round(W, G, Wc, ETA, RHO, N=n)
            return {"W": W, "Wc": Wc}
        if case["rule"] == "measgd":
            hip.measgd_round(W, V, G, Wc, ETA, RHO, DELTA, N=n)
        else:
            hip.measgd_round_bf16(W, V, G, Wc, ETA, RHO, DELTA, N=n)
        return {"W": W, "V": V, "Wc": Wc}
    hip.easgd_layer_product(_PRODUCTS[case["product"]], case["d_in"], case["d_out"], state["A"], state["out"], Wl=state["Wl"],
                            dZ=state["dZ"], ld=state["Wl"].shape[1], out_ws=state["out"].shape[1], relu=case["product"] == "forward")
    return {"out": state["out"]}


# ---- what a pass cannot do without --------------------------------------------------------------------------------

def work(case):
    P = case["P"]
    if case["kind"] == "update":
        per_worker = {"easgd": 12, "measgd": 20, "measgd_bf16": 14}[case["rule"]]
        flops = {"easgd": 6, "measgd": 8, "measgd_bf16": 8}[case["rule"]]
        return {"bytes": case["N"] * (per_worker * P + 8), "flops": case["N"] * P * flops}
    b = case["b"]
    if case["kind"] == "layer":
        d_in, d_out = case["d_in"], case["d_out"]
        a, w, z = b * d_in, (d_in + 1) * d_out, b * d_out
        moved = {"forward": a + w + z, "weight_gradient": a + z + w, "input_gradient": z + w + a + a}[case["product"]]
        return {"bytes": 4 * P * moved, "flops": 2 * P * b * d_in * d_out}
    dims = _dims(case)
    n = _num_params(dims)
    products = sum((2 if l == 0 else 3) * 2 * b * dims[l] * dims[l + 1] for l in range(len(dims) - 1))
    data = P * b * (dims[0] + 1) * 4 + P * 4
    if case["kind"] == "gradient":
        return {"bytes": P * n * 8 + data, "flops": P * products}
    state_bytes = P * n * (8 if case["rule"] == "easgd" else 16) + n * 8
    return {"bytes": state_bytes + data, "flops": P * (products + 8 * n)}


# ---- tolerances and the 64-bit results ----------------------------------------------------------------------------

def tolerance(case):
    """About four times what the fp32 kernels differ from the 64-bit results by, measured over listed and drawn cases."""
    if case["kind"] == "update":
        # element-wise: W and Wc 2.5e-8 (one rounding), with momentum 3.6e-8; in 16 bits the momentum codes that sit on
        # a rounding boundary differ: V 3.4e-4, and W by what that moves it
        return {"rel": 1.5e-3 if case["rule"] == "measgd_bf16" else 1.5e-7}
    if case["kind"] == "layer":
        return {"rel": 4e-6}                                     # 1.5e-7 (sum of 128) to 8.1e-7 (sum of 2048)
    units = case["P"] * case["b"] * sum(_dims(case)[1:-1])
    if case["kind"] == "round" and case["rule"] == "easgd":
        return {"rel": 1e-5}                                     # W moves little in a round: 3e-8 to 1.4e-6
    if units < 20_000:
        return {"rel": 4e-6}                                     # 3e-7 to 5.6e-7
    # A hidden unit whose input is within rounding of zero (about one in a million) is gated differently by different
    # correct sums, and each such sample and unit changes the gradient by about 1/sqrt(units) of its norm: with 1.3e7
    # units the momentum buffers differ from the 64-bit ones by 3.1e-4.
    return {"rel": 4.0 / math.sqrt(units)}


def _f(x):
    return float(np.float32(x))


def _elastic(W, V, G, Wc, n):
    """Both rules of the exchange in 64 bits, worker by worker; V16: momentum kept in bfloat16."""
    eta, rho, delta = _f(ETA), _f(RHO), _f(DELTA)
    c = Wc.double()
    total = torch.zeros_like(c)
    outW = torch.zeros(W.shape, dtype=torch.float64, device=W.device)
    outV = None if V is None else torch.zeros_like(outW)
    for i in range(W.shape[0]):
        w = W[i, :n].double()
        diff = w - c
        total += diff
        if V is None:
            outW[i, :n] = w - eta * (G[i, :n].double() + rho * diff)
            continue
        v = delta * V[i, :n].double() - eta * G[i, :n].double()
        if V.dtype == torch.bfloat16:
            v = v.to(torch.bfloat16).double()
        outV[i, :n] = v
        outW[i, :n] = w + v - eta * rho * diff
    out = {"W": outW, "Wc": c + eta * rho * total}
    if V is not None:
        out["V"] = outV
    return out


def _gradients(dims, W, X, y):
    """Softmax cross-entropy gradients of a ReLU network in 64 bits, packed like the replicas, and the mean losses."""
    P, b = X.shape[0], X.shape[1]
    G = torch.zeros(W.shape, dtype=torch.float64, device=W.device)
    loss = torch.empty(P, dtype=torch.float64, device=W.device)
    layers = len(dims) - 1
    for i in range(P):
        offs, blocks, off = [], [], 0
        for l in range(layers):
            size = (dims[l] + 1) * dims[l + 1]
            offs.append(off)
            blocks.append(W[i, off:off + size].double().view(dims[l] + 1, dims[l + 1]))
            off += size
        acts = [X[i].double()]
        for l in range(layers):
            z = acts[l] @ blocks[l][:-1] + blocks[l][-1]
            acts.append(z.clamp(min=0.0) if l < layers - 1 else z)
        logp = torch.log_softmax(acts[-1], dim=1)
        hot = torch.zeros_like(logp)
        hot.scatter_(1, y[i].long().view(-1, 1), 1.0)
        loss[i] = -(logp * hot).sum() / b
        dz = (logp.exp() - hot) / b
        for l in range(layers - 1, -1, -1):
            size = dims[l] * dims[l + 1]
            G[i, offs[l]:offs[l] + size] = (acts[l].t() @ dz).reshape(-1)
            G[i, offs[l] + size:offs[l] + size + dims[l + 1]] = dz.sum(dim=0)
            if l:
                dz = (dz @ blocks[l][:-1].t()) * (acts[l] > 0)
    return G, loss


def exact(case, seed):
    if case["kind"] == "update":
        if case["P"] * case["N"] > 600_000_000:
            return None                                          # tens of gigabytes in 64 bits
        W, V, G, Wc = _replicas(case, seed)
        return _elastic(W, V, G, Wc, case["N"])
    if case["kind"] == "layer":
        A, Wl, dZ = _layer(case, seed)
        d_in, d_out = case["d_in"], case["d_out"]
        outs = []
        for i in range(case["P"]):
            block = Wl[i, :(d_in + 1) * d_out].double().view(d_in + 1, d_out)
            a, z = A[i].double(), dZ[i].double()
            if case["product"] == "forward":
                o = (a @ block[:-1] + block[-1]).clamp(min=0.0)
            elif case["product"] == "weight_gradient":
                o = torch.cat((a.t() @ z, z.sum(dim=0, keepdim=True)))
            else:
                o = (z @ block[:-1].t()) * (a > 0)
            outs.append(o.reshape(-1))
        return {"out": torch.stack(outs)}
    dims = _dims(case)
    W, Wc, V, X, y = _network(case, seed)
    G, loss = _gradients(dims, W, X, y)
    if case["kind"] == "gradient":
        return {"G": G, "loss": loss}
    out = _elastic(W, V, G, Wc, _num_params(dims))
    out["loss"] = loss
    return out
