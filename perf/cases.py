"""Performance cases of the dynamic-volume-lines library: what a program that
uses it has it do, through the Python binding of the C ABI.

A case is one of seven pieces of work (``work`` key):

``tf``       a transfer-function edit on a resident volume: every field's alpha
             table is set and the volume line recomputed (the interactive loop;
             windows fixed, so from the second frame on the library may use
             what it keeps per window set).  ``window = drag`` moves the
             windows from frame to frame instead (a window slider), ``n_tf``
             above 256 uses fine tables.
``batch``    several resident volumes (an ensemble), each with a new TF, in one
             executor batch (``how = batch``) or one captured graph (``graph``).
``serve``    a burst of client requests on few volumes: several TF sets and
             plot widths per volume in one batch, bins copied to the host.
``order``    a new mesh: Hilbert ordering of the cells, keys and permutation
             exported for the 3D side, volume dropped again.
``load``     a new mesh up to its first plot: ordering, TFs, first update.
``step``     the next time step on the same mesh: every field's values
             replaced, then the update with the windows of the new data.
``explore``  brushing: bins selected, their cells masked in the 3D order, the
             region zoomed into a volume of its own and plotted, per-bin
             histograms and the raster of the plot.

Volumes are seeded AMR leaf sets (coarse grid, the top fraction of the cells of
each level by a smooth random function refined into 8), cells listed level by
level, with log-normal density, anti-correlated temperature, pressure, velocity
magnitude and further smooth fields, each with a little noise from cell to
cell.  Sizes and settings are those of the repository's workloads: 64^3 to
about 500 M cells, 1 to 8 fields, plots 1024 to 3840 wide, tables of 256
entries, P = 1 with minimum importance 0.025, and the options around them.
"""
import math

import numpy as np
import torch

from paper_2306_11612_amd import dvl

_DT = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
_DEF = dict(cells=0.0, refine="", fields=4, dtype="f32", n_bins=1920, n_tf=256, exponent=1.0, fmin=0.025,
            vmax="range", scale=1, scan="fp64", clamp=0, window="data", volumes=1, per=1, how="batch", alloc="hip")


def _full(case):
    c = dict(_DEF)
    c.update(case)
    return c


def listed():
    return [
        # the smallest interactive call: the single-level 64^3 grid, 1024 wide
        {"name": "tf_grid_64", "work": "tf", "cells": 262144.0, "n_bins": 1024},
        # the paper's setting: a three-level data set of some 12 M cells on a full-HD plot
        {"name": "tf_amr_12m", "work": "tf", "cells": 11.8e6, "refine": "0.3,0.15"},
        # the headline volume: five levels, some 500 M cells
        {"name": "tf_amr_500m", "work": "tf", "cells": 501e6, "refine": "0.4,0.3,0.2,0.1"},
        # a window slider dragged on a 50 M-cell volume: the values are read on every frame
        {"name": "tf_window_drag_50m", "work": "tf", "cells": 50e6, "refine": "0.3,0.3,0.3", "window": "drag"},
        # half-size storage with fine (1024-entry) tables, the largest of the serving volumes but one
        {"name": "tf_bf16_fine_150m", "work": "tf", "cells": 150e6, "refine": "0.3,0.3,0.3", "dtype": "bf16", "n_tf": 1024},
        # a small volume on a 4K-wide plot with an exponent, the exact maximum: more bins than tiles
        {"name": "tf_wide_exact_5m", "work": "tf", "cells": 5.1e6, "refine": "0.3,0.3", "n_bins": 3840, "exponent": 2.0,
         "vmax": "exact"},
        # an ensemble of eight small volumes of eight fields, one batch per frame
        {"name": "batch_8x2m", "work": "batch", "cells": 2.3e6, "refine": "0.3,0.3", "fields": 8, "n_bins": 2048, "volumes": 8},
        # a serving burst: two resident volumes, four clients each, bins to the host
        {"name": "serve_2x4_20m", "work": "serve", "cells": 20e6, "refine": "0.3,0.3,0.3", "volumes": 2, "per": 4},
        # a new mesh ordered, its keys and permutation handed to the 3D side
        {"name": "order_amr_50m", "work": "order", "cells": 50e6, "refine": "0.3,0.3,0.3", "alloc": "torch"},
        # a small new mesh up to its first plot
        {"name": "load_amr_1m", "work": "load", "cells": 1.1e6, "refine": "0.3", "dtype": "f16"},
        # the next time step of a simulation on the same mesh
        {"name": "step_amr_12m", "work": "step", "cells": 11.8e6, "refine": "0.3,0.15"},
        # brushing and zooming into a part of the plot
        {"name": "explore_amr_12m", "work": "explore", "cells": 11.8e6, "refine": "0.3,0.15"},
    ]


def _log_uniform(rng, lo, hi):
    return float(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    work = rng.choice(["tf", "tf", "tf", "batch", "serve", "order", "load", "step", "explore"])
    levels = rng.randint(1, 5)
    c = {"work": work,
         "refine": ",".join("%.2f" % rng.uniform(0.1, 0.4) for _ in range(levels - 1)),
         "dtype": rng.choice(["f32", "f32", "f16", "bf16"]),
         "fields": rng.choice([1, 2, 3, 4, 4, 4, 6, 8]),
         "n_bins": rng.choice([1024, 1920, 1920, 2048, 3840, rng.randint(200, 4000)])}
    if work == "tf":
        c["cells"] = _log_uniform(rng, 2e4, 2e8)
        c["window"] = rng.choice(["data", "data", "fixed", "drag"])
        c["n_tf"] = rng.choice([256, 256, 256, 64, 1000])
        c["exponent"] = rng.choice([1.0, 1.0, 1.0, 0.5, 2.0])
        c["vmax"] = rng.choice(["range", "range", "bound", "exact"])
        c["scan"] = rng.choice(["fp64", "fp64", "kahan"])
        c["clamp"] = rng.choice([0, 0, 1])
        c["fmin"] = rng.choice([0.025, 0.025, 0.1])
        c["scale"] = 3 if c["exponent"] == 1.0 and rng.random() < 0.2 else 1
    elif work == "batch":
        c["volumes"] = rng.randint(2, 8)
        c["cells"] = _log_uniform(rng, 1e5, 4e6)
        c["how"] = rng.choice(["batch", "graph"])
    elif work == "serve":
        c["volumes"] = rng.randint(1, 4)
        c["per"] = rng.randint(1, 8)
        c["cells"] = _log_uniform(rng, 2e5, 4e7)
    elif work == "order":
        c["cells"] = _log_uniform(rng, 2e5, 1e8)
        c["alloc"] = "torch"
    elif work == "load":
        c["cells"] = _log_uniform(rng, 2e4, 2e7)
        c["alloc"] = rng.choice(["hip", "torch"])
    elif work == "step":
        c["cells"] = _log_uniform(rng, 2e5, 6e7)
    else:
        c["cells"] = _log_uniform(rng, 2e5, 3e7)
    return c


# ------------------------------------------------------------------ inputs

def _fracs(case):
    return [float(f) for f in case["refine"].split(",") if f]


def _leaves_per_base_cell(fracs):
    g, mult = 0.0, 1.0
    for r in fracs:
        g += mult * (1.0 - r)
        mult *= 8.0 * r
    return g + mult


def _base_side(case):
    return max(4, int(round((case["cells"] / _leaves_per_base_cell(_fracs(case))) ** (1.0 / 3.0))))


def _n_cells(case):
    """Cells of one volume of the case (up to the rounding of the refined numbers)."""
    return _base_side(case) ** 3 * _leaves_per_base_cell(_fracs(case))


def _smooth(x, y, z, half, extent, rs, terms, kmax):
    """A smooth random function of the cell centres: cosines of random wave
    vectors, amplitudes falling with the wave number; about unit variance."""
    out = torch.zeros(x.shape, dtype=torch.float32, device=x.device)
    k = rs.uniform(-kmax, kmax, (terms, 3))
    amp = 1.0 / (1.0 + np.linalg.norm(k, axis=1))
    amp *= math.sqrt(2.0) / np.linalg.norm(amp)
    ph = rs.uniform(0.0, 2.0 * math.pi, terms)
    fx, fy, fz = ((a + half).float().mul_(2.0 * math.pi / extent) for a in (x, y, z))
    for i in range(terms):
        t = torch.mul(fx, float(k[i, 0]))
        t.add_(fy, alpha=float(k[i, 1])).add_(fz, alpha=float(k[i, 2])).add_(float(ph[i])).cos_()
        out.add_(t, alpha=float(amp[i]))
    return out


def _leaves(base, fracs, rs, dev):
    """Leaf cells (x, y, z int32 lower corners, level uint8), coarsest level first."""
    L = len(fracs)
    extent = base << L
    r = torch.arange(base, dtype=torch.int32, device=dev) << L
    cz, cy, cx = (g.reshape(-1) for g in torch.meshgrid(r, r, r, indexing="ij"))
    xs, ys, zs, ls = [], [], [], []
    seed = rs.randint(0, 1 << 30)
    for k, frac in enumerate(fracs):
        lev = L - k
        v = _smooth(cx, cy, cz, 1 << (lev - 1), extent, np.random.RandomState(seed), 20, 12.0)
        n_fine = int(round(frac * v.numel()))
        fine = torch.zeros(v.numel(), dtype=torch.bool, device=dev)
        fine[torch.sort(v).indices[v.numel() - n_fine:]] = True
        del v
        keep = ~fine
        for out, c in ((xs, cx), (ys, cy), (zs, cz)):
            out.append(c[keep])
        ls.append(torch.full((xs[-1].numel(),), lev, dtype=torch.uint8, device=dev))
        h = 1 << (lev - 1)
        off = torch.tensor([0, h], dtype=torch.int32, device=dev)
        o = torch.meshgrid(off, off, off, indexing="ij")
        cx, cy, cz = ((c[fine][:, None] + d.reshape(-1)[None]).reshape(-1) for c, d in ((cx, o[2]), (cy, o[1]), (cz, o[0])))
        del fine, keep
    xs.append(cx); ys.append(cy); zs.append(cz)
    ls.append(torch.zeros(cx.numel(), dtype=torch.uint8, device=dev))
    return torch.cat(xs), torch.cat(ys), torch.cat(zs), torch.cat(ls), extent


def _one_field(m, cache, x, y, z, half, extent, rs, gen):
    def g(terms):
        v = _smooth(x, y, z, half, extent, rs, terms, 6.0)
        return v.add_(torch.randn(v.shape, generator=gen, device=v.device, dtype=torch.float32), alpha=0.03)
    if m == 0:
        cache["rho"] = g(14).mul_(1.2).exp_()
        return cache["rho"]
    if m == 1:
        cache["temp"] = cache["rho"].rsqrt().mul_(g(8).mul_(0.2).exp_())
        return cache["temp"]
    if m == 2:
        return cache["rho"] * cache.pop("temp")
    if m == 3:
        return torch.hypot(g(8), g(8))
    return g(8)


def _fields(case, x, y, z, level, extent, rs, gen):
    half = torch.bitwise_right_shift(torch.bitwise_left_shift(torch.ones_like(x), level.int()), 1)
    cache, out = {}, []
    for m in range(case["fields"]):
        out.append(_one_field(m, cache, x, y, z, half, extent, rs, gen).to(_DT[case["dtype"]]))
    return out


def _table(rs, n_tf):
    """A piecewise-linear alpha table through 4 to 8 random control points."""
    k = rs.randint(4, 9)
    pos = np.sort(rs.uniform(0.0, 1.0, k))
    return np.interp((np.arange(n_tf) + 0.5) / n_tf, pos, rs.uniform(0.0, 1.0, k)).astype(np.float32)


def _tables(rs, M, n_tf):
    return np.stack([_table(rs, n_tf) for _ in range(M)])


def _inputs(case, seed):
    """The case's raw inputs: meshes, fields, tables, windows (from the seed alone)."""
    c = _full(case)
    dev = torch.device("cuda", torch.cuda.current_device())
    rs = np.random.RandomState(seed % (1 << 32))
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    fr = _fracs(c)
    vols = []
    for k in range(c["volumes"]):
        scaled = dict(c)
        if c["volumes"] > 1:   # volumes of unequal sizes
            scaled["cells"] = c["cells"] * (0.5 + k / (c["volumes"] - 1.0))
        x, y, z, level, extent = _leaves(_base_side(scaled), fr, rs, dev)
        F = _fields(c, x, y, z, level, extent, rs, gen)
        vols.append({"x": x, "y": y, "z": z, "level": level, "fields": F, "extent": extent,
                     "alpha": [_tables(rs, c["fields"], c["n_tf"]) for _ in range(c["per"])]})
    return c, vols, rs, gen


def _alpha_windows(c, v, rs):
    """Windows per frame: the data ranges (None), or for ``fixed`` and ``drag``
    an inner part of them, moved by a twentieth from one frame to the other."""
    if c["window"] == "data":
        return [None]
    out = []
    a, b = rs.uniform(0.0, 0.1), rs.uniform(0.8, 1.0)
    for shift in ((0.0, 0.05) if c["window"] == "drag" else (0.0,)):
        lo, hi = [], []
        for f in v["fields"]:
            l, h = float(f.min()), float(f.max())
            lo.append(np.float32(l + (h - l) * (a + shift)))
            hi.append(np.float32(l + (h - l) * (b + shift)))
        out.append((np.array(lo, np.float32), np.array(hi, np.float32)))
    return out


def _kw(c):
    return dict(exponent=c["exponent"], min_importance=c["fmin"], clamp_mode=c["clamp"], level_scale=c["scale"],
                vmax_mode={"range": dvl.VMAX_TF_RANGE, "bound": dvl.VMAX_TF_BOUND, "exact": dvl.VMAX_EXACT}[c["vmax"]],
                scan_mode={"fp64": dvl.SCAN_FP64, "kahan": dvl.SCAN_KAHAN_FP32}[c["scan"]])


def _widths(c):
    return [max(16, c["n_bins"] * w // 2) for w in (2, 1, 4, 2)]


def prepare(case, seed):
    c, vols, rs, gen = _inputs(case, seed)
    s = {"case": c, "kw": _kw(c), "frame": 0}
    work, M, W = c["work"], c["fields"], c["n_bins"]
    if work in ("order", "load"):
        s["in"] = vols[0]
        s["allocator"] = dvl.torch_allocator() if c["alloc"] == "torch" else None
        s["bins"] = dvl.Bins(W, M)
        return s
    s["alpha"] = [v["alpha"] for v in vols]
    s["windows"] = _alpha_windows(c, vols[0], rs)
    s["vol"] = [dvl.build_order(v["x"], v["y"], v["z"], v["level"], v["fields"]) for v in vols]
    if work == "step":
        v = vols[0]
        s["next"] = _fields(c, v["x"], v["y"], v["z"], v["level"], v["extent"], rs, gen)
    if work in ("tf", "step"):
        s["bins"] = dvl.Bins(W, M)
    elif work == "batch":
        s["bins"] = [dvl.Bins(W, M) for _ in vols]
        if c["how"] == "graph":
            s["graph"] = dvl.Graph([_request(s, i, 0, b) for i, b in enumerate(s["bins"])])
        else:
            s["executor"] = dvl.Executor()
    elif work == "serve":
        ws = _widths(c)
        s["bins"] = [[dvl.Bins(ws[k % len(ws)], M) for k in range(c["per"])] for _ in vols]
        s["executor"] = dvl.Executor()
    else:
        s["bins"] = dvl.Bins(W, M)
        s["zoom_bins"] = dvl.Bins(W, M)
        b0 = int(rs.randint(0, W // 2))
        s["brush"] = (b0, min(W - 1, b0 + W // 5))
        s["allocator"] = dvl.torch_allocator()
    return s


# ------------------------------------------------------------------ one pass

def _request(s, i, k, bins):
    return dvl.Request(s["vol"][i], s["alpha"][i][k], bins, **s["kw"])


def _set_tfs(V, alpha, window=None):
    for m in range(alpha.shape[0]):
        if window is None:
            V.set_tf(m, alpha[m])
        else:
            V.set_tf(m, alpha[m], float(window[0][m]), float(window[1][m]))


def _out(b):
    return {"first_cell": b.first_cell, "last_cell": b.last_cell, "mean": b.mean, "vmin": b.vmin, "vmax": b.vmax,
            "y": b.y, "f_total": b.f_total, "vmax_used": b.vmax_used}


def run(state):
    c = state["case"]
    return {"tf": _run_tf, "batch": _run_batch, "serve": _run_serve, "order": _run_order, "load": _run_load,
            "step": _run_step, "explore": _run_explore}[c["work"]](state, c)


def _run_tf(s, c):
    V = s["vol"][0]
    w = s["windows"][s["frame"] % len(s["windows"])]
    s["frame"] += 1
    _set_tfs(V, s["alpha"][0][0], w)
    V.update(s["bins"], **s["kw"])
    return _out(s["bins"])


def _run_batch(s, c):
    if c["how"] == "graph":
        s["graph"].set_tf_all([a[0] for a in s["alpha"]])
        s["graph"].launch()
    else:
        s["executor"].update_batch([_request(s, i, 0, b) for i, b in enumerate(s["bins"])])
    return [_out(b) for b in s["bins"]]


def _run_serve(s, c):
    reqs = [_request(s, i, k, b) for i, bs in enumerate(s["bins"]) for k, b in enumerate(bs)]
    s["executor"].update_batch(reqs)
    got = [r.vol.read_bins(r.bins) for r in reqs]
    keep = ("first", "last", "mean", "vmin", "vmax", "y")
    return {k: np.concatenate([g[k].reshape(-1) for g in got]) for k in keep}


def _run_order(s, c):
    v = s["in"]
    V = dvl.build_order(v["x"], v["y"], v["z"], v["level"], v["fields"], allocator=s["allocator"])
    keys, perm = V.export_order()
    ranges = [V.field_range(m) for m in range(c["fields"])]
    V.close()
    return {"keys": keys, "perm": perm, "ranges": np.array(ranges, np.float64)}


def _run_load(s, c):
    v = s["in"]
    V = dvl.build_order(v["x"], v["y"], v["z"], v["level"], v["fields"], allocator=s["allocator"])
    _set_tfs(V, v["alpha"][0])
    V.update(s["bins"], **s["kw"])
    V.close()
    return _out(s["bins"])


def _run_step(s, c):
    V = s["vol"][0]
    for m in range(c["fields"]):
        V.set_field(m, s["next"][m])
    _set_tfs(V, s["alpha"][0][0])
    V.update(s["bins"], **s["kw"])
    return _out(s["bins"])


def _run_explore(s, c):
    V, b = s["vol"][0], s["bins"]
    _set_tfs(V, s["alpha"][0][0])
    V.update(b, **s["kw"])
    first, last, klo, khi = V.select_bins(b, *s["brush"])
    mask = V.select_mask([(klo, khi)])
    Z = V.zoom(first, last, allocator=s["allocator"])
    _set_tfs(Z, s["alpha"][0][0])
    zb = s["zoom_bins"]
    Z.update(zb, **s["kw"])
    lo, hi = V.field_range(0)
    hist = V.bin_histograms(b, 0, 64, lo, hi if hi > lo else float(np.nextafter(np.float32(lo), np.float32(np.inf))))
    image = dvl.rasterize(zb.y, 256)
    Z.close()
    return {"bins": _out(b), "mask": mask, "zoom": _out(zb), "hist": hist, "image": image}


# ------------------------------------------------------------------ what a pass cannot do without

def work(case):
    """Bytes and operations of one pass, each input read once and each output
    written once.  A TF edit cannot do without one table index per cell and
    field (a byte for tables of 256 entries, the value where the windows move
    or the tables are finer); an operation is an add, multiply, compare or
    lookup of the per-cell arithmetic (quantiser 3, lookup 1, max and min 2 per
    field; scale, clamp and sum 4 per cell; 12 per bit of a Hilbert key)."""
    c = _full(case)
    n, M, eb, W = _n_cells(c), c["fields"], 4 if c["dtype"] == "f32" else 2, c["n_bins"]
    vals, out = n * M * eb, W * (8 + 16 * M) + 12
    index = n * M * (1 if c["n_tf"] <= 256 and c["window"] != "drag" else eb)
    upd = n * (6 * M + 4)
    bits = max(1.0, math.ceil(math.log2(_base_side(c) << len(_fracs(c)))))
    build = dict(bytes=n * 13 + vals + n * 13 + vals, flops=n * 3 * bits * 4)
    w = c["work"]
    if w == "tf":
        return {"bytes": index + out, "flops": upd}
    if w == "batch":
        return {"bytes": c["volumes"] * (n * M + out), "flops": c["volumes"] * upd}
    if w == "serve":
        ws = _widths(c)
        o = sum(ws[k % len(ws)] for k in range(c["per"])) * (8 + 16 * M)
        return {"bytes": c["volumes"] * (n * M + o), "flops": c["volumes"] * c["per"] * upd}
    if w == "order":
        return {"bytes": build["bytes"] + 12 * n, "flops": build["flops"]}
    if w == "load":
        return {"bytes": build["bytes"] + out, "flops": build["flops"] + upd}
    if w == "step":
        return {"bytes": vals + 4 * n + vals + out, "flops": upd}
    part = 0.2 * n   # cells of the brushed fifth of the plot, as a share of the plot
    return {"bytes": n * M + out + 12 * n + n + part * (13 + M * eb) * 2 + n * eb + W * 256 + 256 * M * W + out,
            "flops": 1.2 * upd + 4 * n}


# ------------------------------------------------------------------ the same in 64 bits

def _hilbert(x, y, z, level, bits):
    """Hilbert index of the cells' centroids (Skilling's transposed form)."""
    half = torch.bitwise_right_shift(torch.bitwise_left_shift(torch.ones_like(x), level.int()), 1)
    X = [x + half, y + half, z + half]
    for j in range(bits - 1, 0, -1):
        q, p = 1 << j, (1 << j) - 1
        for i in range(3):
            on = torch.bitwise_and(X[i], q) != 0
            t = torch.bitwise_and(torch.bitwise_xor(X[0], X[i]), p)
            t.masked_fill_(on, 0)
            if i:
                X[i] = torch.bitwise_xor(X[i], t)
            X[0] = torch.where(on, torch.bitwise_xor(X[0], p), torch.bitwise_xor(X[0], t))
            del on, t
    X[1] = torch.bitwise_xor(X[1], X[0])
    X[2] = torch.bitwise_xor(X[2], X[1])
    t = torch.zeros_like(X[0])
    for j in range(bits - 1, 0, -1):
        t = torch.where(torch.bitwise_and(X[2], 1 << j) != 0, torch.bitwise_xor(t, (1 << j) - 1), t)
    key = torch.zeros(x.shape, dtype=torch.int64, device=x.device)
    for j in range(bits):
        for i in range(3):
            b = torch.bitwise_and(torch.bitwise_right_shift(torch.bitwise_xor(X[i], t), j), 1).to(torch.int64)
            key = torch.bitwise_or(key, b << (3 * j + 2 - i))
    return key


def _order(v):
    bits = 1
    while (1 << bits) < v["extent"]:
        bits += 1
    key = _hilbert(v["x"], v["y"], v["z"], v["level"], bits)
    return torch.sort(key).indices


def _entry(x, lo, hi, n_tf):
    """The table entry of a value, by the library's stated rule: the fp32
    quantiser of the window, one rounding of x * s + b to fp32."""
    s = np.float32(n_tf / (float(hi) - float(lo)))
    b = np.float32(-float(lo) * float(s))
    t = (x.double() * float(s) + float(b)).float()
    return t.clamp_(0.0, float(n_tf - 1)).floor_().long()


def _windows_of(F):
    lo = np.array([float(f.min()) for f in F], np.float32)
    hi = np.array([float(f.max()) for f in F], np.float32)
    return lo, np.where(hi > lo, hi, np.nextafter(lo, np.float32(np.inf))).astype(np.float32)


def _exact_update(c, level, F, alpha, W, window=None, ranges=None, max_level=None):
    """One update in 64 bits on cells in Hilbert order (F: stored values)."""
    M, dev = len(F), F[0].device
    n_tf = alpha.shape[1]
    lo, hi = window if window is not None else _windows_of(F)
    vmax = torch.full((F[0].numel(),), -math.inf, dtype=torch.float64, device=dev)
    vmin = -vmax
    im, jm = [], []
    for m in range(M):
        e = _entry(F[m], lo[m], hi[m], n_tf)
        im.append(int(e.min())); jm.append(int(e.max()))
        a = torch.from_numpy(alpha[m].astype(np.float64)).to(dev)[e]
        vmax, vmin = torch.maximum(vmax, a), torch.minimum(vmin, a)
        del a, e
    V = vmax.sub_(vmin)
    del vmin
    A = alpha.astype(np.float64)
    bound = max(A[m, im[m]:jm[m] + 1].max() for m in range(M)) - min(A[m, im[m]:jm[m] + 1].min() for m in range(M))
    if c["vmax"] == "exact":
        vm = float(V.max())
    elif c["vmax"] == "bound":
        vm = bound
    else:
        part = A[:, min(im):max(jm) + 1]
        vm = float((part.max(0) - part.min(0)).max())
        vm = vm if vm > 0 else bound
    width = torch.pow(torch.tensor(2.0, dtype=torch.float64, device=dev), level.double() * c["scale"])
    r = V / vm if vm > 0 else torch.zeros_like(V)
    if c["clamp"]:
        f = (r.clamp_(min=c["fmin"]) * width) ** c["exponent"]
    else:
        f = ((r * width) ** c["exponent"]).clamp_(min=c["fmin"])
    del width, r, V
    end = torch.cumsum(f, 0)
    total = float(end[-1])
    start = (end - f).mul_(W / total)
    end.mul_(W / total)
    del f
    b = torch.arange(W, dtype=torch.float64, device=dev)
    first = torch.searchsorted(end, b, right=True).clamp_(max=F[0].numel() - 1)
    last = (torch.searchsorted(start, b + 1.0, right=False) - 1).clamp_(min=0)
    first = torch.minimum(first, last)
    del start, end
    cnt = last - first + 1
    pos = torch.repeat_interleave(first - (torch.cumsum(cnt, 0) - cnt), cnt)
    pos += torch.arange(pos.numel(), device=dev)
    mean = torch.empty(M, W, dtype=torch.float64, device=dev)
    mn, mx = torch.empty_like(mean), torch.empty_like(mean)
    for m in range(M):
        v = F[m].double()[pos]
        for o, how in ((mean, "mean"), (mn, "min"), (mx, "max")):
            o[m] = torch.segment_reduce(v, how, lengths=cnt)
        del v
    return {"first_cell": None, "last_cell": None, "mean": mean, "vmin": mn, "vmax": mx, "y": None,
            "f_total": torch.tensor([total], dtype=torch.float64),
            "vmax_used": torch.tensor([vm], dtype=torch.float64)}


def exact(case, seed):
    """What ``run`` returns, in 64 bits: integers and the heights (a table step
    at the mean) have no such value."""
    c, vols, rs, gen = _inputs(case, seed)
    work, W = c["work"], c["n_bins"]
    if work == "explore" or _n_cells(c) > 220e6:
        return None
    if work == "order":
        lo = [float(f.min()) for f in vols[0]["fields"]]
        hi = [float(f.max()) for f in vols[0]["fields"]]
        return {"keys": None, "perm": None, "ranges": np.array(list(zip(lo, hi)), np.float64)}
    windows = _alpha_windows(c, vols[0], rs) if work != "load" else [None]
    outs = []
    for i, v in enumerate(vols):
        o = _order(v)
        F = v["fields"]
        if work == "step":
            F = _fields(c, v["x"], v["y"], v["z"], v["level"], v["extent"], rs, gen)
        level = v["level"][o]
        F = [f[o] for f in F]
        del o
        ws = _widths(c)
        for k in range(c["per"]):
            outs.append(_exact_update(c, level, F, v["alpha"][k], ws[k % len(ws)] if work == "serve" else W, windows[0]))
        v.clear()
    if work == "serve":
        cat = lambda key: np.concatenate([o[key].cpu().numpy().reshape(-1) for o in outs])  # noqa: E731
        return {"first": None, "last": None, "mean": cat("mean"), "vmin": cat("vmin"), "vmax": cat("vmax"), "y": None}
    return outs if work == "batch" else outs[0]
