"""Performance cases of the N-D Winograd layers.

Each case is one piece of work a program gives this library, through the
public binding (paper_1611_06565_amd.wino): a layer's forward pass with its
transformed kernels kept, a layer's data or weight gradient, a whole training
step of a layer, the eight-layer C3D-style stack with its pools, and the 2-D
benchmark's chain of three layers.  The sizes are the layers of
``workloads``, the ones the benchmark runs, and generic ragged ones.

``listed`` gives the fixed cases, ``draw`` another one of the same ranges,
``prepare`` what a program holds before the call, ``run`` one pass, ``work``
the bytes and operations a pass cannot do without, ``tolerance`` what another
correct fp32 implementation may differ by, ``exact`` the outputs in float64.
"""
from __future__ import annotations

import math

import torch

from paper_1611_06565_amd.wino import Plan

# ---------------------------------------------------------------------------
# cases


def _layer(name, kind, N, m, r, batch, C, K, X, pad, tile=(0, 0, 0), act="none", bias=False,
           x_dist="relu_normal"):
    case = {"kind": kind, "N": N, "m": m, "r": r, "batch": batch, "C": C, "K": K, "pad": pad,
            "act": act, "bias": bias, "x_dist": x_dist}
    if name is not None:
        case["name"] = name
    for i in range(3):
        case[f"X{i}"] = X[i] if i < N else 1
        case[f"t{i}"] = tile[i]
    return case


def _stack(name, batch, depth, side):
    case = {"kind": "stack", "batch": batch, "depth": depth, "side": side}
    if name is not None:
        case["name"] = name
    return case


def _chain(name, batch, side):
    case = {"kind": "chain", "batch": batch, "side": side}
    if name is not None:
        case["name"] = name
    return case


def listed():
    return [
        # the smallest layer of the workloads: one call is launches and latency
        _layer("small_f2_3d", "forward", 3, 2, 3, 1, 16, 16, (16, 16, 16), 0, x_dist="normal"),
        # a C3D-style video layer, the benchmark's default: F(2^3, 3^3) forward
        _layer("video_f2_3d", "forward", 3, 2, 3, 8, 64, 128, (16, 56, 56), 1),
        # a 2-D layer of an image network, F(4^2, 3^2) forward
        _layer("image_f4_2d", "forward", 2, 4, 3, 64, 256, 256, (56, 56), 1),
        # a volumetric layer on one large sample, F(4^3, 3^3) forward
        _layer("volume_f4_3d", "forward", 3, 4, 3, 1, 32, 32, (128, 128, 128), 1, x_dist="uniform"),
        # odd extents and channel counts, a bias and a leaky ReLU, F(4^3, 3^3)
        # with more than 64 kernels
        _layer("ragged_f4_3d", "forward", 3, 4, 3, 3, 50, 100, (13, 45, 51), 1, act="leaky", bias=True),
        # the whole eight-layer stack on a batch of clips (inference)
        _stack("stack_b4", 4, 16, 112),
        # the paper's 2-D benchmark: three unpadded 4 x 4 layers, F(5^2, 4^2)
        _chain("chain_f5_2d_b20", 20, 224),
        # backward pass of the video layer, data side: new kernels each step
        _layer("video_dgrad_f2_3d", "dgrad", 3, 2, 3, 8, 64, 128, (16, 56, 56), 1, x_dist="normal"),
        # backward pass of the video layer, kernel side
        _layer("video_wgrad_f2_3d", "wgrad", 3, 2, 3, 8, 64, 128, (16, 56, 56), 1),
        # one training step of a small ragged 2-D layer: forward with bias and
        # both gradients, the kernels transformed anew as after an update
        _layer("train_f4_2d", "train", 2, 4, 3, 16, 96, 160, (27, 33), 1, bias=True),
        # per-axis tiles, short first axis: (2, 4, 4) on the video layer
        _layer("video_tile244", "forward", 3, 2, 3, 8, 64, 128, (16, 56, 56), 1, tile=(2, 4, 4), act="relu"),
        # a 4 x 4 x 4 kernel on a volume, F(5^3, 4^3)
        _layer("volume_f5x4_3d", "forward", 3, 5, 4, 1, 32, 32, (96, 96, 96), 1, x_dist="uniform"),
    ]


# the largest drawn case: direct FLOPs, floats of one transformed operand and
# of x or y within the listed cases' largest
_MAX_FLOPS = 2.0e11
_MAX_V = 2.4e8
_MAX_XY = 5.2e7


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        kind = rng.choice(["forward"] * 6 + ["dgrad", "wgrad", "train", "train", "stack", "chain"])
        if kind == "stack":
            return _stack(None, rng.randint(1, 4), rng.choice([8, 12, 16]), rng.choice([80, 88, 96, 104, 112]))
        if kind == "chain":
            return _chain(None, rng.randint(1, 20), rng.randint(96, 224))
        sizes = [(2, 4, 3), (3, 2, 3), (3, 2, 3), (3, 4, 3), (3, 4, 3), (2, 2, 3)]
        if kind == "forward":
            sizes += [(3, 5, 4), (2, 5, 4), (3, 0, 3)]
        N, m, r = rng.choice(sizes)
        tile = (0, 0, 0)
        if m == 0:
            m, tile = 2, rng.choice([(2, 4, 4), (4, 2, 2)])
        C, K = _logint(rng, 3, 512), _logint(rng, 8, 512)
        if r == 4:
            C, K = _logint(rng, 8, 64), _logint(rng, 8, 64)
        if N == 2:
            batch = _logint(rng, 1, 64)
            X = (_logint(rng, 7, 224), _logint(rng, 7, 224))
        else:
            batch = _logint(rng, 1, 8)
            X = (_logint(rng, 4, 96), _logint(rng, 7, 128), _logint(rng, 7, 128))
        case = _layer(None, kind, N, m, r, batch, C, K, X, rng.choice([0, 1, 1]), tile=tile,
                      act=rng.choice(["none", "relu", "leaky"]) if kind == "forward" else "none",
                      bias=rng.random() < 0.5 if kind in ("forward", "train") else False,
                      x_dist=rng.choice(["relu_normal", "normal", "uniform"]))
        sx, sy = _numel(case, "x"), _numel(case, "y")
        # gradients run up to three products: a third of the work each
        share = {"forward": 1.0, "dgrad": 1.0, "wgrad": 0.6, "train": 0.3}[kind]
        if (_direct_flops(case) <= share * _MAX_FLOPS and max(sx, sy) <= share * _MAX_XY
                and _transformed(case)[0] * max(C, K) <= share * _MAX_V
                and 1e6 <= work(case)["flops"] <= 5.2e10):
            return case


# ---------------------------------------------------------------------------
# geometry


def _extents(case):
    N = case["N"]
    X = [case[f"X{i}"] for i in range(N)]
    Y = [x + 2 * case["pad"] - case["r"] + 1 for x in X]
    tile = [case[f"t{i}"] or case["m"] for i in range(N)]
    return X, Y, tile


def _numel(case, what):
    X, Y, _ = _extents(case)
    if what == "x":
        return case["batch"] * case["C"] * math.prod(X)
    if what == "y":
        return case["batch"] * case["K"] * math.prod(Y)
    return case["K"] * case["C"] * case["r"] ** case["N"]


def _transformed(case):
    """(tiles x elements, elements) of the layer's transform."""
    _, Y, tile = _extents(case)
    T = case["batch"] * math.prod(-(-y // t) for y, t in zip(Y, tile))
    nxi = math.prod(t + case["r"] - 1 for t in tile)
    return T * nxi, nxi


def _direct_flops(case):
    return 2.0 * _numel(case, "y") * case["C"] * case["r"] ** case["N"]


def _stack_layers(case):
    """(C, K, X, pool window or None, m) of the eight 3x3x3 pad-1 layers."""
    X, C = [case["depth"], case["side"], case["side"]], 3
    widths = (64, 128, 256, 256, 512, 512, 512, 512)
    pools = {0: (1, 2, 2), 1: (2, 2, 2), 3: (2, 2, 2), 5: (2, 2, 2), 7: (2, 2, 2)}
    out = []
    for i, K in enumerate(widths):
        pool = pools.get(i)
        if pool is not None and min(x // p for x, p in zip(X, pool)) < 1:
            pool = (1, 2, 2)           # a clip too short to halve its first axis again
        # F(4^3) while the rows are long, F(2^3) on the small late layers
        out.append((C, K, tuple(X), pool, 4 if X[2] >= 28 and X[1] >= 28 else 2))
        if pool is not None:
            X = [x // p for x, p in zip(X, pool)]
        C = K
    return out


def _chain_layers(case):
    X, out = case["side"], []
    for _ in range(3):
        out.append(_layer(None, "forward", 2, 5, 4, case["batch"], 32, 32, (X, X), 0))
        X -= 3
    return out


# ---------------------------------------------------------------------------
# inputs


def _draw(gen, shape, dist, fan_in=1):
    t = torch.empty(shape, dtype=torch.float32, device="cuda")
    if dist == "uniform":
        return t.uniform_(generator=gen)
    t.normal_(generator=gen)
    if dist == "relu_normal":
        t.clamp_(min=0.0)
    elif dist == "he":
        t.mul_(math.sqrt(2.0 / fan_in))
    return t


def _inputs(case, seed):
    """Every random tensor of a case, from the seed alone."""
    gen = torch.Generator("cuda").manual_seed(int(seed))
    if case["kind"] == "stack":
        layers = _stack_layers(case)
        x = _draw(gen, (case["batch"], 3) + layers[0][2], "uniform")
        return {"x": x, "w": [_draw(gen, (K, C, 3, 3, 3), "he", 27 * C) for C, K, _, _, _ in layers]}
    if case["kind"] == "chain":
        layers = _chain_layers(case)
        x = _draw(gen, (case["batch"], 32, case["side"], case["side"]), "uniform")
        return {"x": x, "w": [_draw(gen, (32, 32, 4, 4), "he", 512) for _ in layers]}
    X, Y, _ = _extents(case)
    N, C, K, r = case["N"], case["C"], case["K"], case["r"]
    out = {"x": _draw(gen, (case["batch"], C, *X), case["x_dist"]),
           "w": _draw(gen, (K, C) + (r,) * N, "he", C * r ** N)}
    if case["bias"]:
        out["bias"] = _draw(gen, (K,), "normal").mul_(0.1)
    if case["kind"] in ("dgrad", "wgrad", "train"):
        out["dy"] = _draw(gen, (case["batch"], K, *Y), "normal")
    return out


_SLOPE = 0.1


def _plan(case):
    X, _, _ = _extents(case)
    N = case["N"]
    tile = tuple(case[f"t{i}"] for i in range(N))
    return Plan(N, case["m"], case["r"], case["C"], case["K"], [case["batch"], *X], pad=case["pad"],
                relu=case["act"] == "relu", leaky=_SLOPE if case["act"] == "leaky" else None,
                tile=tile if any(tile) else None)


def _buffer(nbytes):
    return torch.empty(max(nbytes, 4) // 4, dtype=torch.float32, device="cuda")


def _workspace(plan):
    need = plan.forward_workspace_bytes
    return _buffer(need) if need else None


def prepare(case, seed):
    st = _inputs(case, seed)
    st["case"] = case
    kind = case["kind"]
    if kind == "stack":
        # as a serving program keeps them: plans, transformed kernels,
        # workspaces and the layers' output buffers
        st["layers"] = []
        for (C, K, X, pool, m), w in zip(_stack_layers(case), st.pop("w")):
            plan = Plan(3, m, 3, C, K, [case["batch"], *X], pad=1, relu=True)
            shape = plan.pooled_shape(pool) if pool is not None else plan.output_shape
            y = torch.empty(shape, dtype=torch.float32, device="cuda")
            # the pool rides on the product where the library offers it
            fused = pool is not None and (m == 4 or pool == (2, 2, 2))
            pre = torch.empty(plan.output_shape, dtype=torch.float32, device="cuda") \
                if pool is not None and not fused else None
            st["layers"].append((plan, plan.transform_filter(w), pool, fused, _workspace(plan), pre, y))
        return st
    if kind == "chain":
        st["layers"] = []
        for layer, w in zip(_chain_layers(case), st.pop("w")):
            plan = _plan(layer)
            st["layers"].append((plan, plan.transform_filter(w), _workspace(plan)))
        return st
    plan = st["plan"] = _plan(case)
    if kind == "forward":
        st["U"] = plan.transform_filter(st.pop("w"))
        st["ws"] = _workspace(plan)
    if kind == "train":
        st["ws"] = _workspace(plan)
        st["U"] = plan.new_filter()
    if kind in ("dgrad", "train"):
        st["adj"] = plan.adjoint()
        st["adj_ws"] = _workspace(st["adj"])
        st["adj_U"] = st["adj"].new_filter()
    if kind in ("wgrad", "train"):
        st["wg_ws"] = _buffer(plan.weight_gradient_workspace_bytes)
    return st


def run(st):
    kind = st["case"]["kind"]
    if kind == "stack":
        from paper_1611_06565_amd.wino import maxpool3d
        x = st["x"]
        for plan, U, pool, fused, ws, pre, y in st["layers"]:
            if fused:
                plan.forward_pool(x, U, pool, y=y, workspace=ws)
            elif pool is not None:
                maxpool3d(plan.forward(x, U, y=pre, workspace=ws), pool, y)
            else:
                plan.forward(x, U, y=y, workspace=ws)
            x = y
        return x
    if kind == "chain":
        x = st["x"]
        for plan, U, ws in st["layers"]:
            x = plan.forward(x, U, workspace=ws)
        return x
    if kind == "forward":
        return st["plan"].forward(st["x"], st["U"], workspace=st["ws"], bias=st.get("bias"))
    out = {}
    if kind == "train":
        U = st["plan"].transform_filter(st["w"], U=st["U"])
        out["y"] = st["plan"].forward(st["x"], U, workspace=st["ws"], bias=st.get("bias"))
    if kind in ("dgrad", "train"):
        U = st["adj"].transform_filter_adjoint(st["w"], U=st["adj_U"])
        out["dx"] = st["adj"].forward(st["dy"], U, workspace=st["adj_ws"])
    if kind in ("wgrad", "train"):
        out["dw"] = st["plan"].weight_gradient(st["x"], st["dy"], workspace=st["wg_ws"])
    return out


# ---------------------------------------------------------------------------
# what a pass cannot do without


def work(case):
    """Bytes: inputs and outputs once, the transformed kernels where a program
    keeps them.  FLOPs: the products of the minimal algorithm at the case's
    tile (the transforms' additions left out)."""
    kind = case["kind"]
    if kind in ("stack", "chain"):
        bytes_ = flops = 0.0
        if kind == "chain":
            sub = _chain_layers(case)
            last = _numel(sub[-1], "y")
        else:
            sub = []
            for C, K, X, pool, m in _stack_layers(case):
                sub.append(_layer(None, "forward", 3, m, 3, case["batch"], C, K, X, 1))
            last = case["batch"] * 512 * math.prod(x // p for x, p in zip(X, pool))
        bytes_ += 4.0 * (_numel(sub[0], "x") + last)
        for s in sub:
            V, nxi = _transformed(s)
            flops += 2.0 * V * s["C"] * s["K"]
            bytes_ += 4.0 * nxi * s["C"] * s["K"]
        return {"bytes": bytes_, "flops": flops}
    V, nxi = _transformed(case)
    product = 2.0 * V * case["C"] * case["K"]
    x, y, w, U = (_numel(case, "x"), _numel(case, "y"), _numel(case, "w"), nxi * case["C"] * case["K"])
    if kind == "forward":
        return {"bytes": 4.0 * (x + y + U), "flops": product}
    if kind == "dgrad":
        return {"bytes": 4.0 * (x + y + w), "flops": product}
    if kind == "wgrad":
        return {"bytes": 4.0 * (x + y + w), "flops": product}
    return {"bytes": 4.0 * (2 * x + 2 * y + 2 * w), "flops": 3.0 * product}


# Errors against float64 grow with the tile and, at m = 4, with the layer's
# shape.  The bounds are about four times what the library shows against
# ``exact`` over the listed cases and drawn ones (largest relative error and
# largest difference over the result's size): m = 2 4.7e-7 and 3.2e-6, m = 4
# 4.2e-6 and 1.8e-4, m = 5 4.9e-6 and 9.6e-5; the weight gradient sums over
# every output position: 1.9e-6 and 1.1e-5 (m = 2), 5.6e-6 and 5.2e-5 (m = 4);
# stack 1.8e-6 and 7.5e-6, chain 2.3e-6 and 2.4e-5.
_TOL = {2: (2e-6, 1.4e-5), 4: (1.7e-5, 7e-4), 5: (2e-5, 4e-4)}
_TOL_DW = {2: (8e-6, 4.5e-5), 4: (2.2e-5, 2.2e-4), 5: (2.2e-5, 4e-4)}


def tolerance(case):
    kind = case["kind"]
    if kind == "stack":
        return {"rel": 7e-6, "max": 3e-5}
    if kind == "chain":
        return {"rel": 9e-6, "max": 1e-4}
    m = max([case["m"]] + [case[f"t{i}"] for i in range(3)])
    rel, largest = _TOL[m]
    if kind in ("wgrad", "train"):
        rel, largest = max(rel, _TOL_DW[m][0]), max(largest, _TOL_DW[m][1])
    return {"rel": rel, "max": largest}


# ---------------------------------------------------------------------------
# float64 reference: the correlation and its gradients, one kernel offset at a
# time as plain matrix products


def _offsets(r, N):
    return [tuple((i // r ** a) % r for a in reversed(range(N))) for i in range(r ** N)]


def _padded(x, pad, N):
    return torch.nn.functional.pad(x, (pad, pad) * N) if pad else x


def _window(xp, p, Y):
    sl = (slice(None), slice(None)) + tuple(slice(o, o + y) for o, y in zip(p, Y))
    return xp[sl].reshape(xp.shape[0], xp.shape[1], -1)


def _corr64(x, w, pad):
    N, r = x.dim() - 2, w.shape[-1]
    xp = _padded(x, pad, N)
    Y = [s - r + 1 for s in xp.shape[2:]]
    out = torch.zeros((x.shape[0], w.shape[0], math.prod(Y)), dtype=torch.float64, device=x.device)
    for p in _offsets(r, N):
        wp = w[(slice(None), slice(None)) + p].contiguous()
        for n in range(x.shape[0]):
            out[n].addmm_(wp, _window(xp[n:n + 1], p, Y)[0])
    return out.reshape(x.shape[0], w.shape[0], *Y)


def _dgrad64(dy, w, pad, X):
    N, r = dy.dim() - 2, w.shape[-1]
    Y = list(dy.shape[2:])
    out = torch.zeros((dy.shape[0], w.shape[1], *[x + 2 * pad for x in X]), dtype=torch.float64, device=dy.device)
    flat = dy.reshape(dy.shape[0], dy.shape[1], -1)
    for p in _offsets(r, N):
        wp = w[(slice(None), slice(None)) + p].t().contiguous()
        for n in range(dy.shape[0]):
            sl = (n, slice(None)) + tuple(slice(o, o + y) for o, y in zip(p, Y))
            out[sl] += (wp @ flat[n]).reshape(w.shape[1], *Y)
    return out[(slice(None), slice(None)) + tuple(slice(pad, pad + x) for x in X)].contiguous()


def _wgrad64(x, dy, pad, r):
    N = x.dim() - 2
    xp = _padded(x, pad, N)
    Y = list(dy.shape[2:])
    flat = dy.reshape(dy.shape[0], dy.shape[1], -1)
    out = torch.zeros((dy.shape[1], x.shape[1]) + (r,) * N, dtype=torch.float64, device=x.device)
    for p in _offsets(r, N):
        acc = torch.zeros((dy.shape[1], x.shape[1]), dtype=torch.float64, device=x.device)
        for n in range(x.shape[0]):
            acc.addmm_(flat[n], _window(xp[n:n + 1], p, Y)[0].t().contiguous())
        out[(slice(None), slice(None)) + p] = acc
    return out


def _pool64(x, window):
    return torch.nn.functional.max_pool3d(x, window, window)


def exact(case, seed):
    inp = _inputs(case, seed)
    kind = case["kind"]
    if kind == "stack":
        x = inp["x"].double()
        for (C, K, X, pool, m), w in zip(_stack_layers(case), inp["w"]):
            x = _corr64(x, w.double(), 1).clamp_(min=0.0)
            if pool is not None:
                x = _pool64(x, pool)
        return x
    if kind == "chain":
        x = inp["x"].double()
        for w in inp["w"]:
            x = _corr64(x, w.double(), 0)
        return x
    x, w = inp["x"].double(), inp["w"].double()
    X, _, _ = _extents(case)
    out = {}
    if kind in ("forward", "train"):
        y = _corr64(x, w, case["pad"])
        if case["bias"]:
            y += inp["bias"].double().view(1, -1, *[1] * case["N"])
        if case["act"] == "relu":
            y.clamp_(min=0.0)
        elif case["act"] == "leaky":
            slope = float(torch.tensor(_SLOPE, dtype=torch.float32))
            y = torch.where(y > 0, y, y * slope)
        if kind == "forward":
            return y
        out["y"] = y
    if kind in ("dgrad", "train"):
        out["dx"] = _dgrad64(inp["dy"].double(), w, case["pad"], X)
    if kind in ("wgrad", "train"):
        out["dw"] = _wgrad64(x, inp["dy"].double(), case["pad"], case["r"])
    return out
