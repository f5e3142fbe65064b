"""Performance cases of the WBMM library.

``listed()`` names the work a user of this package has it do, over the range
it is used in: single-image and tiny calls, training steps of the stage
shapes of a windowed-convolution backbone, dense-prediction maps, maps that
the windows do not tile, the float32 operator benchmark, the hierarchical
form, cached matrices and rectangular windows.  ``draw(rng)`` gives further
cases of the same ranges.  Every case runs through the package's public entry
points, as a program that uses them does: outputs are allocated by the call
and nothing is synchronised.

A case is a dict of plain values:
  kind   "infer"   y = wbmm_forward
         "train"   wbmm_forward, then wbmm_backward (both gradients)
         "autograd" the differentiable wbmm and its gradients
         "hier"    wbmm_hier_forward, then wbmm_hier_backward (window 2 wl)
         "cached"  wbmm_dense_forward with a matrix built once beforehand
         "rect"    wbmm_rect_forward / _backward_input / _backward_table
  dtype  "f32", "bf16" or "f16"
  B, C, H, W   the activation's shape
  wh, ww       the window (equal except for "cached" and "rect"; for "hier"
               the global window, twice the local one)
"""
import math

import torch

import paper_2607_02097_amd as wbmm_pkg

_DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}


def _case(name, kind, dtype, B, C, H, W, wh, ww=None):
    c = {"kind": kind, "dtype": dtype, "B": B, "C": C, "H": H, "W": W, "wh": wh, "ww": wh if ww is None else ww}
    return dict(name=name, **c) if name else c


def listed():
    return [
        # one training step of a toy layer: what a call costs when the GPU
        # work is next to nothing
        _case("tiny_train_f32_w7", "train", "f32", 1, 8, 28, 28, 7),
        # one image through a first-stage layer at inference
        _case("single_infer_f16_w7", "infer", "f16", 1, 96, 56, 56, 7),
        # first stage of the small backbone in training
        _case("stage1_train_bf16_w7", "train", "bf16", 64, 96, 56, 56, 7),
        # second stage (the benchmark's headline shape)
        _case("stage2_train_bf16_w14", "train", "bf16", 64, 192, 28, 28, 14),
        # third stage: one window per image, more channels than compute units
        _case("stage3_train_bf16_w14", "train", "bf16", 128, 384, 14, 14, 14),
        # a dense-prediction map in training
        _case("dense_pred_train_bf16_w14", "train", "bf16", 16, 64, 112, 112, 14),
        # a detection feature map (800 x 1333 input at stride 8) that the
        # windows do not tile, with an odd width
        _case("ragged_train_bf16_w14", "train", "bf16", 8, 96, 100, 167, 14),
        # the operator benchmark: float32, 256 channels, batch 128
        _case("operator_infer_f32_w14", "infer", "f32", 128, 256, 56, 56, 14),
        # float32 training at the batch of the operator benchmark, through
        # autograd
        _case("stage2_autograd_f32_w14", "autograd", "f32", 128, 192, 28, 28, 14),
        # training of the hierarchical (global + local window) form
        _case("hier_train_bf16_w14", "hier", "bf16", 64, 192, 28, 28, 14),
        # inference with cached matrices, at the operator benchmark's batch
        _case("cached_infer_bf16_w14", "cached", "bf16", 128, 256, 28, 28, 14),
        # training with rectangular windows
        _case("rect_train_f16_w7x14", "rect", "f16", 32, 96, 56, 56, 7, 14),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["infer", "train", "train", "autograd", "hier", "cached", "rect"])
    dtype = rng.choice(["bf16", "bf16", "f16", "f32"])
    # windows of 7 and 14 are what the networks use; the library takes 1..16
    if kind == "hier":
        wh = ww = 2 * rng.choice([7, 7, 4, 5, 6, 8])
    elif kind == "rect":
        wh, ww = rng.choice([(7, 14), (14, 7), (4, 16), (5, 9), (8, 12), (16, 3)])
    else:
        wh = ww = rng.choice([7, 7, 14, 14, rng.randint(4, 16)])
    # elements of one activation: the matrix-product passes cost more per
    # element in float32 and with materialised matrices
    cap = {"cached": 20e6, "rect": 5e6}.get(kind, 25e6)
    if dtype == "f32":
        cap *= 0.5
    C = _log_int(rng, 8, 512)
    if rng.random() < 0.5:
        # a map that the windows tile
        H = wh * max(1, _log_int(rng, 14, 168) // wh)
        W = ww * max(1, _log_int(rng, 14, 168) // ww)
        if rng.random() < 0.5 and wh == ww:
            W = H
    else:
        H, W = _log_int(rng, 10, 170), _log_int(rng, 10, 170)
    while C * H * W > cap and H > 2 * wh and W > 2 * ww:
        H, W = max(H // 2, wh), max(W // 2, ww)
    B = _log_int(rng, 1, max(1, min(256, int(cap // (C * H * W)))))
    return _case(None, kind, dtype, B, C, H, W, wh, ww)


def _table_sizes(case):
    C, wh, ww = case["C"], case["wh"], case["ww"]
    sizes = [(C, (2 * wh - 1) * (2 * ww - 1))]
    if case["kind"] == "hier":
        sizes.append((C, (wh - 1) ** 2))  # local window wl = wh / 2
    return sizes


def _inputs(case, seed):
    """Unit-normal activations and upstream gradients, tables of standard
    deviation 0.02 (their initialisation)."""
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    dt = _DTYPES[case["dtype"]]
    shape = (case["B"], case["C"], case["H"], case["W"])

    def normal(size, std=1.0):
        return (torch.randn(size, generator=gen, device="cuda", dtype=torch.float32) * std).to(dt)

    inp = {"x": normal(shape), "tables": [normal(s, 0.02) for s in _table_sizes(case)]}
    if case["kind"] in ("train", "autograd", "hier", "rect"):
        inp["dy"] = normal(shape)
    return inp


def prepare(case, seed):
    s = _inputs(case, seed)
    s.update(kind=case["kind"], wh=case["wh"], ww=case["ww"])
    if case["kind"] == "cached":
        s["m"] = wbmm_pkg.wbmm_build_matrix(s["tables"][0], s["wh"], s["ww"])
    if case["kind"] == "autograd":
        s["x"].requires_grad_(True)
        s["tables"][0].requires_grad_(True)
    return s


def run(s):
    kind, x, t, w = s["kind"], s["x"], s["tables"][0], s["wh"]
    if kind == "infer":
        return {"y": wbmm_pkg.wbmm_forward(x, t, w)}
    if kind == "train":
        y = wbmm_pkg.wbmm_forward(x, t, w)
        dx, dt = wbmm_pkg.wbmm_backward(x, s["dy"], t, w)
        return {"y": y, "dx": dx, "dt": dt}
    if kind == "autograd":
        y = wbmm_pkg.wbmm(x, t, w)
        dx, dt = torch.autograd.grad(y, (x, t), s["dy"])
        return {"y": y.detach(), "dx": dx, "dt": dt}
    if kind == "hier":
        tl, wl = s["tables"][1], w // 2
        y = wbmm_pkg.wbmm_hier_forward(x, t, tl, wl)
        dx, dt, dtl = wbmm_pkg.wbmm_hier_backward(x, s["dy"], t, tl, wl)
        return {"y": y, "dx": dx, "dt": dt, "dtl": dtl}
    if kind == "cached":
        return {"y": wbmm_pkg.wbmm_dense_forward(x, s["m"], s["wh"], s["ww"])}
    y = wbmm_pkg.wbmm_rect_forward(x, t, s["wh"], s["ww"])
    dx = wbmm_pkg.wbmm_rect_backward_input(s["dy"], t, s["wh"], s["ww"])
    dt = wbmm_pkg.wbmm_rect_backward_table(x, s["dy"], s["wh"], s["ww"])
    return {"y": y, "dx": dx, "dt": dt}


def work(case):
    """One pass: every input read once and every output written once; two
    operations per product of a position with the d = wh ww positions of its
    window, for each of the forward and the two gradients."""
    es = 4 if case["dtype"] == "f32" else 2
    n = case["B"] * case["C"] * case["H"] * case["W"]
    d = case["wh"] * case["ww"]
    tab = sum(a * b for a, b in _table_sizes(case))
    kind = case["kind"]
    if kind == "infer":
        return {"bytes": (2 * n + tab) * es, "flops": 2 * n * d}
    if kind == "cached":
        return {"bytes": (2 * n + case["C"] * d * d) * es, "flops": 2 * n * d}
    dt_es = es if kind == "autograd" else 4
    # x, dy, the tables; y, dx, the tables' gradients
    return {"bytes": (4 * n + tab) * es + tab * dt_es, "flops": 6 * n * d}


def tolerance(case):
    # 16-bit: one rounding of a float32 sum; float32: the order of the sums
    # (measured against the 64-bit results below)
    if case["dtype"] == "bf16":
        return {"rel": 7e-3, "max": 3e-2}
    if case["dtype"] == "f16":
        return {"rel": 9e-4, "max": 4e-3}
    return {"rel": 3e-6, "max": 2e-5}


def _windows(v, wh, ww):
    """[B, C, H, W] -> [C, windows, wh ww] of the zero-padded map."""
    B, C, H, W = v.shape
    v = torch.nn.functional.pad(v, (0, -W % ww, 0, -H % wh))
    nh, nw = v.shape[2] // wh, v.shape[3] // ww
    v = v.reshape(B, C, nh, wh, nw, ww).permute(1, 0, 2, 4, 3, 5)
    return v.reshape(C, B * nh * nw, wh * ww).contiguous()


def _unwindows(v, shape, wh, ww):
    B, C, H, W = shape
    nh, nw = -(-H // wh), -(-W // ww)
    v = v.reshape(C, B, nh, nw, wh, ww).permute(1, 0, 2, 4, 3, 5)
    return v.reshape(B, C, nh * wh, nw * ww)[:, :, :H, :W].contiguous()


def _index(wh, ww, dev):
    """Table entry of (input position i, output position j)."""
    p = torch.arange(wh * ww, device=dev)
    h, x = p // ww, p % ww
    return (h[:, None] - h[None] + wh - 1) * (2 * ww - 1) + x[:, None] - x[None] + ww - 1


def exact(case, seed):
    inp = _inputs(case, seed)
    kind, wh, ww = case["kind"], case["wh"], case["ww"]
    d = wh * ww
    dev = inp["x"].device
    idx = _index(wh, ww, dev)
    same = None
    if kind == "hier":
        wl = wh // 2
        p = torch.arange(d, device=dev)
        part = (p // ww // wl) * 2 + (p % ww) // wl  # local sub-window of a position
        same = part[:, None] == part[None]
        h, x = p // ww % wl, p % ww % wl
        idxl = (h[:, None] - h[None] + wl - 1) * (2 * wl - 1) + x[:, None] - x[None] + wl - 1
        idxl = torch.where(same, idxl, torch.zeros_like(idxl))
    out = {}
    C = case["C"]
    step = max(1, int(4e7 // (case["B"] * case["H"] * case["W"])))  # channels at a time
    for c0 in range(0, C, step):
        sl = slice(c0, min(C, c0 + step))
        t = [v[sl].double() for v in inp["tables"]]
        m = t[0][:, idx]
        if same is not None:
            m = m + t[1][:, idxl] * same + 2.0 * torch.eye(d, device=dev, dtype=torch.float64)
        x = inp["x"][:, sl].double()
        xw = _windows(x, wh, ww)
        part_out = {"y": _unwindows(torch.bmm(xw, m.contiguous()), x.shape, wh, ww)}
        if "dy" in inp:
            gw = _windows(inp["dy"][:, sl].double(), wh, ww)
            part_out["dx"] = _unwindows(torch.bmm(gw, m.transpose(1, 2).contiguous()), x.shape, wh, ww)
            g = torch.bmm(xw.transpose(1, 2).contiguous(), gw)
            n = g.shape[0]
            z = torch.zeros((n, t[0].shape[1]), device=dev, dtype=torch.float64)
            part_out["dt"] = z.index_add_(1, idx.flatten(), g.reshape(n, d * d))
            if same is not None:
                z = torch.zeros((n, t[1].shape[1]), device=dev, dtype=torch.float64)
                part_out["dtl"] = z.index_add_(1, idxl.flatten(), (g * same).reshape(n, d * d))
        for k, v in part_out.items():
            out.setdefault(k, []).append(v)
    return {k: torch.cat(v, 1 if k in ("y", "dx") else 0) for k, v in out.items()}
