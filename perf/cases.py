"""The work that programs hand to this library, as a list of timed cases.

A case is one pass through the public entry points (binding, tp_binding, el_binding) with the
plan, the workspace and the tensors already on the GPU, as a training loop or a server holds them.
Seven kinds:

  serve     sc_forward_noalloc: the contraction alone, without a workspace (a serving loop)
  sc_step   sc_forward, then sc_backward with the grouping and the folded weights reused: the
            product basis of one training step
  sc_force  the same two calls, then sc_double_backward: a step whose loss contains forces
  tp_step   tp_forward and tp_backward: the message construction of one training step
  tp_force  the same, then tp_double_backward
  linear    el_forward and el_backward: the channel mixing between the two
  fused     el_sc_forward and el_sc_backward: channel mixing and product basis behind one call

Value distributions and element mix are those of paper_2504_10700_amd/workloads.py, drawn on the
device.  The ranges: 1 to 200 000 atoms, 64 to 256 channels (multiples of 64 and others), l up to
3, correlation order 2 and 3, outputs 0e to 0e+1o+2e+3o, fp32, fp64 and bfloat16 rows, batches in
the order of the data set or grouped by element, both layouts of the rows.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2504_10700_amd import binding as sc
from paper_2504_10700_amd import el_binding as el
from paper_2504_10700_amd import tp_binding as tp
from paper_2504_10700_amd import workloads

# output irreps (L, parity) by name
OUTPUTS = {
    "0e": ((0, 1),),
    "0e1o": ((0, 1), (1, -1)),
    "0e1o2e": ((0, 1), (1, -1), (2, 1)),
    "0e1o2e3o": ((0, 1), (1, -1), (2, 1), (3, -1)),
}
ROW_TYPE = {"f32": torch.float32, "f64": torch.float64, "bf16": torch.bfloat16}
WEIGHT_TYPE = {"f32": torch.float32, "f64": torch.float64, "bf16": torch.float32}
PLAN_TYPE = {"f32": sc.SC_F32, "f64": sc.SC_F64, "bf16": sc.SC_BF16}
ELEMENT_BYTES = {"f32": 4, "f64": 8, "bf16": 2}
ELEMENTS = 89
MEAN_DEGREE = 20


def _sc(name, kind, nodes, channels=128, l_max=3, nu=3, outputs="0e1o", dtype="f32", grouped=False,
        component_major=False):
    return {"name": name, "kind": kind, "nodes": nodes, "channels": channels, "l_max": l_max, "nu": nu,
            "outputs": outputs, "dtype": dtype, "grouped": grouped, "component_major": component_major}


def _tp(name, kind, nodes, channels=128, l_Y=3, l_h=1, L_max=3, dtype="f32"):
    return {"name": name, "kind": kind, "nodes": nodes, "channels": channels, "l_Y": l_Y, "l_h": l_h,
            "L_max": L_max, "dtype": dtype}


def _linear(name, nodes, k_in=128, k_out=128, l_max=3, dtype="f32"):
    return {"name": name, "kind": "linear", "nodes": nodes, "k_in": k_in, "k_out": k_out, "l_max": l_max,
            "dtype": dtype}


def _fused(name, nodes, k_in=128, channels=128, outputs="0e1o", dtype="f32"):
    return {"name": name, "kind": "fused", "nodes": nodes, "k_in": k_in, "channels": channels, "l_max": 3, "nu": 3,
            "outputs": outputs, "dtype": dtype}


def listed():
    return [
        # one small structure per call, the inner loop of molecular dynamics: latency and launches
        _sc("serve_61_atoms", "serve", 61),
        # the paper's batch: bins of 3072 atoms
        _sc("step_3072_atoms", "sc_step", 3072),
        # the training step that the benchmark quotes
        _sc("step_10k_atoms", "sc_step", 10_000),
        # ... and the large batch, bound by memory alone
        _sc("step_200k_atoms", "sc_step", 200_000),
        # a wide model with second-order features
        _sc("step_wide_2e", "sc_step", 50_000, channels=256, outputs="0e1o2e"),
        # rows stored as bfloat16
        _sc("step_bf16_rows", "sc_step", 10_000, dtype="bf16"),
        # training on forces: forward, backward and second-order pass
        _sc("force_10k_atoms", "sc_force", 10_000),
        # a smaller model (l <= 2) in double precision, as relaxations are run; a ragged batch
        _sc("step_l2_f64", "sc_step", 2_731, l_max=2, dtype="f64"),
        # messages of a middle layer (features 0e+1o), forward and backward
        _tp("messages_10k_atoms", "tp_step", 10_000),
        # messages of the layer after one with 0e+1o+2e outputs
        _tp("messages_2e_features", "tp_step", 3_001, l_h=2),
        # messages in training on forces
        _tp("force_messages", "tp_force", 10_000),
        # channel mixing, forward and backward
        _linear("linear_10k_atoms", 10_000),
    ]


def _log_size(rng, lo, hi):
    """A size spread evenly over its logarithm."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _drawn(case):
    del case["name"]
    return case


def draw(rng):
    kind = rng.choices(["serve", "sc_step", "sc_force", "tp_step", "tp_force", "linear", "fused"],
                       [2, 5, 2, 3, 2, 2, 1])[0]
    if kind in ("serve", "sc_step", "sc_force"):
        dtype = rng.choices(["f32", "f64", "bf16"], [6, 2, 2])[0]
        l_max, nu = rng.choices([(3, 3), (2, 3), (3, 2), (2, 2)], [8, 2, 2, 1])[0]
        outputs = rng.choices(["0e", "0e1o", "0e1o2e", "0e1o2e3o"], [2, 5, 3, 1])[0]
        if l_max == 2 and outputs == "0e1o2e3o":
            outputs = "0e1o2e"
        if dtype == "bf16":
            l_max = nu = 3
        if dtype == "f64" and outputs == "0e1o2e3o":
            outputs = "0e1o2e"
        usual = (l_max, nu) == (3, 3)
        channels = rng.choice([64, 72, 96, 128, 128, 192, 256])
        if kind == "serve":
            # within the scratch that the library keeps for these calls
            if outputs == "0e1o2e3o" or dtype == "f64":
                channels = min(channels, 128)
            if dtype == "f64":
                outputs = "0e1o" if outputs == "0e1o2e" else outputs
            hi = 2_000 if usual else 500
        else:
            hi = 200_000 if usual else 5_000
            if outputs == "0e1o2e3o" or dtype == "f64":
                hi = min(hi, 20_000)
            elif outputs == "0e1o2e" or kind == "sc_force":
                hi = min(hi, 50_000)
            hi = hi * 128 // max(channels, 128)
        grouped = kind != "serve" and rng.random() < 0.15
        component_major = kind != "serve" and usual and dtype != "bf16" and rng.random() < 0.15
        return _drawn(_sc("", kind, _log_size(rng, 1 if kind == "serve" else 40, hi), channels, l_max, nu, outputs, dtype,
                          grouped, component_major))
    if kind in ("tp_step", "tp_force"):
        dtype = rng.choices(["f32", "f64"], [4, 1])[0]
        l = rng.choices([3, 2], [3, 1])[0]
        l_h = rng.choices([0, 1, 2], [2, 3, 2])[0]
        channels = rng.choice([64, 96, 128, 128, 256])
        usual = l == 3 and l_h < 2 and channels != 96
        hi = (20_000 if usual else 3_000) * 64 // channels // (1 if dtype == "f32" else 2)
        return _drawn(_tp("", kind, _log_size(rng, 40, hi), channels, l, l_h, l, dtype))
    if kind == "linear":
        k_in, k_out = rng.choice([(64, 64), (128, 128), (128, 128), (256, 256), (128, 256), (256, 128), (96, 96),
                                  (192, 128), (100, 128)])
        dtype = rng.choices(["f32", "f64"], [4, 1])[0]
        hi = 24_000 * 128 * 128 // (k_in * k_out) if k_in % 64 == 0 and dtype == "f32" else 4_000
        return _drawn(_linear("", _log_size(rng, 40, hi), k_in, k_out, rng.choices([3, 2, 1], [3, 1, 1])[0], dtype))
    k_in, channels = rng.choice([(128, 128), (128, 128), (64, 128), (256, 256), (96, 96)])
    hi = 20_000 * 128 * 128 // (k_in * channels) if k_in % 64 == 0 else 4_000
    return _drawn(_fused("", _log_size(rng, 40, hi), k_in, channels,
                         rng.choice(["0e1o", "0e1o", "0e1o2e"]), rng.choices(["f32", "f64"], [4, 1])[0]))


# ---------------------------------------------------------------------------------------------
# inputs


def _normal(gen, shape, dtype, scale=1.0):
    """N(0, scale^2) on the device; scale is a number or a tensor that broadcasts."""
    x = torch.randn(shape, generator=gen, device="cuda", dtype=torch.float64 if dtype == torch.float64 else torch.float32)
    if not isinstance(scale, float) or scale != 1.0:
        x = x.mul_(scale)
    return x.to(dtype)


def _element_indices(gen, nodes, grouped):
    p = torch.as_tensor(workloads.element_probabilities(ELEMENTS, "skewed"), dtype=torch.float64, device="cuda")
    z = torch.multinomial(p, nodes, replacement=True, generator=gen)
    if grouped:
        z = torch.sort(z).values
    return z.to(torch.int32)


def _contraction_weights(gen, plan, channels, dtype):
    """W ~ N(0,1) / sqrt(number of paths of the same correlation order and output irrep)."""
    paths = sc.sc_plan_paths(plan)
    _, group, count = np.unique(paths[:, :2], axis=0, return_inverse=True, return_counts=True)
    scale = torch.as_tensor(1.0 / np.sqrt(count[group.reshape(-1)]), dtype=dtype, device="cuda")[None, :, None]
    return _normal(gen, (ELEMENTS, len(paths), channels), dtype, scale)


def _prepare_contraction(case, gen):
    rows, weights = ROW_TYPE[case["dtype"]], WEIGHT_TYPE[case["dtype"]]
    n, K = case["nodes"], case["channels"]
    plan = sc.sc_plan_create(K, case["l_max"], case["nu"], ELEMENTS, OUTPUTS[case["outputs"]],
                             PLAN_TYPE[case["dtype"]], torch.cuda.current_device())
    info = sc.sc_plan_info(plan)
    cm = case.get("component_major", False)

    def shape(components):
        return (n, components, K) if cm else (n, K, components)
    s = {"plan": plan, "n": n, "z": _element_indices(gen, n, case.get("grouped", False)),
         "W": _contraction_weights(gen, plan, K, weights)}
    s["flags"] = (sc.SC_Z_GROUPED if case.get("grouped", False) else 0) | (sc.SC_COMPONENT_MAJOR if cm else 0)
    s["B"] = torch.empty(shape(info.n_LM), dtype=rows, device="cuda")
    if case["kind"] != "fused":
        s["A"] = _normal(gen, shape(info.n_lm), rows)
    if case["kind"] == "serve":
        return s
    s["dB"] = _normal(gen, shape(info.n_LM), rows)
    s["dW"] = torch.empty_like(s["W"])
    if case["kind"] == "fused":
        k_in = case["k_in"]
        s["k_in"] = k_in
        s["X"] = _normal(gen, (n, k_in, info.n_lm), rows)
        s["W_lin"] = _normal(gen, (case["l_max"] + 1, k_in, K), rows, 1.0 / math.sqrt(k_in))
        s["dX"], s["dW_lin"] = torch.empty_like(s["X"]), torch.empty_like(s["W_lin"])
        s["bytes"] = max(el.el_sc_workspace_bytes(plan, k_in, n), el.el_sc_backward_workspace_bytes(plan, k_in, n))
    else:
        s["dA"] = torch.empty_like(s["A"])
        s["bytes"] = sc.sc_workspace_bytes(plan, n)
    if case["kind"] == "sc_force":
        s["H"] = _normal(gen, shape(info.n_lm), rows)
        s["ddB"], s["dA2"], s["dW2"] = torch.empty_like(s["B"]), torch.empty_like(s["A"]), torch.empty_like(s["W"])
    s["ws"] = torch.empty(s["bytes"], dtype=torch.uint8, device="cuda")
    return s


def _num_edges(nodes):
    """Edges of a graph of that many atoms: what the generator draws on average."""
    return int(0.99 * MEAN_DEGREE * nodes)


def _graph(wl, rng):
    """A graph of the workloads' distribution with a set number of edges, so that the sizes of the
    tensors follow from the case: edges chosen at random are left out or taken twice."""
    sender, receiver = workloads.make_tp_graph(wl, rng)
    E = _num_edges(wl.num_nodes)
    if len(sender) >= E:
        keep = np.sort(rng.permutation(len(sender))[:E])
    else:
        keep = np.sort(np.concatenate([np.arange(len(sender)), rng.integers(0, len(sender), E - len(sender))]))
    return sender[keep], receiver[keep]


def _prepare_messages(case, gen, seed):
    t, n, K = ROW_TYPE[case["dtype"]], case["nodes"], case["channels"]
    wl = workloads.TPWorkload("messages", n, MEAN_DEGREE, K, case["l_Y"], case["l_h"], case["L_max"], case["dtype"], 0)
    sender, receiver = _graph(wl, np.random.default_rng(seed))
    row_ptr, send_ptr, send_edge = workloads.graph_indices(sender, receiver, n)
    plan = tp.tp_plan_create(K, case["l_Y"], case["l_h"], case["L_max"], PLAN_TYPE[case["dtype"]],
                             torch.cuda.current_device())
    paths = tp.tp_plan_paths(plan)
    per_l3 = np.bincount(paths[:, 2], minlength=case["L_max"] + 1)
    scale = torch.as_tensor(1.0 / np.sqrt(MEAN_DEGREE * per_l3[paths[:, 2]]), dtype=t, device="cuda")[None, :, None]
    E, P = len(sender), len(paths)
    s = {"plan": plan, "n": n, "E": E}
    for name, index in (("sender", sender), ("row_ptr", row_ptr), ("send_ptr", send_ptr), ("send_edge", send_edge)):
        s[name] = torch.as_tensor(index, dtype=torch.int32).cuda()
    s["Y"] = _normal(gen, (E, wl.n_Y), t)
    s["h"] = _normal(gen, (n, K, wl.n_h), t)
    s["R"] = _normal(gen, (E, P, K), t, scale)
    s["dA"] = _normal(gen, (n, K, wl.n_out), t)
    s["A"] = torch.empty_like(s["dA"])
    for out, like in (("dY", "Y"), ("dh", "h"), ("dR", "R")):
        s[out] = torch.empty_like(s[like])
    if case["kind"] == "tp_force":
        s["HY"], s["Hh"], s["HR"] = (_normal(gen, tuple(s[k].shape), t) for k in ("Y", "h", "R"))
        s["ddA"] = torch.empty_like(s["dA"])
        for out, like in (("d2Y", "Y"), ("d2h", "h"), ("d2R", "R")):
            s[out] = torch.empty_like(s[like])
    s["bytes"] = tp.tp_workspace_bytes(plan, E)
    s["ws"] = torch.empty(s["bytes"], dtype=torch.uint8, device="cuda")
    return s


def _prepare_linear(case, gen):
    t, n, k_in, k_out, l_max = ROW_TYPE[case["dtype"]], case["nodes"], case["k_in"], case["k_out"], case["l_max"]
    nc = (l_max + 1) ** 2
    cfg = el.make_config(k_in, k_out, l_max, PLAN_TYPE[case["dtype"]], torch.cuda.current_device())
    s = {"cfg": cfg, "n": n}
    s["X"] = _normal(gen, (n, k_in, nc), t)
    s["W"] = _normal(gen, (l_max + 1, k_in, k_out), t, 1.0 / math.sqrt(k_in))
    s["dY"] = _normal(gen, (n, k_out, nc), t)
    s["Y"], s["dX"], s["dW"] = torch.empty_like(s["dY"]), torch.empty_like(s["X"]), torch.empty_like(s["W"])
    s["bytes"] = el.el_workspace_bytes(cfg, n)
    s["ws"] = torch.empty(s["bytes"], dtype=torch.uint8, device="cuda")
    return s


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    kind = case["kind"]
    if kind == "linear":
        s = _prepare_linear(case, gen)
    elif kind in ("tp_step", "tp_force"):
        s = _prepare_messages(case, gen, seed)
    else:
        s = _prepare_contraction(case, gen)
    s["kind"] = kind
    return s


# ---------------------------------------------------------------------------------------------
# one pass


def _run_contraction(s):
    plan, n, z, W, ws, nb, flags = s["plan"], s["n"], s["z"], s["W"], s["ws"], s["bytes"], s["flags"]
    sc.sc_forward(plan, n, s["A"], z, W, s["B"], ws, nb, flags)
    flags |= sc.SC_REUSE_GROUPING | sc.SC_REUSE_WEIGHTS
    sc.sc_backward(plan, n, s["A"], z, W, s["dB"], s["dA"], s["dW"], ws, nb, flags)
    out = {"B": s["B"], "dA": s["dA"], "dW": s["dW"]}
    if s["kind"] == "sc_force":
        sc.sc_double_backward(plan, n, s["A"], z, W, s["dB"], s["H"], s["ddB"], s["dA2"], s["dW2"], ws, nb, flags)
        out.update(ddB=s["ddB"], dA2=s["dA2"], dW2=s["dW2"])
    return out


def _run_messages(s):
    plan, n, E = s["plan"], s["n"], s["E"]
    edges = (s["sender"], s["row_ptr"], s["send_ptr"], s["send_edge"])
    tp.tp_forward(plan, n, n, E, s["Y"], s["h"], s["R"], s["sender"], s["row_ptr"], s["A"])
    tp.tp_backward(plan, n, n, E, s["Y"], s["h"], s["R"], *edges, s["dA"], s["dY"], s["dh"], s["dR"], s["ws"], s["bytes"])
    out = {k: s[k] for k in ("A", "dY", "dh", "dR")}
    if s["kind"] == "tp_force":
        tp.tp_double_backward(plan, n, n, E, s["Y"], s["h"], s["R"], *edges, s["dA"], s["HY"], s["Hh"], s["HR"],
                              s["ddA"], s["d2Y"], s["d2h"], s["d2R"], s["ws"], s["bytes"])
        out.update({k: s[k] for k in ("ddA", "d2Y", "d2h", "d2R")})
    return out


def run(state):
    s = state
    kind = s["kind"]
    if kind == "serve":
        sc.sc_forward_noalloc(s["plan"], s["n"], s["A"], s["z"], s["W"], s["B"])
        return s["B"]
    if kind in ("sc_step", "sc_force"):
        return _run_contraction(s)
    if kind in ("tp_step", "tp_force"):
        return _run_messages(s)
    if kind == "linear":
        el.el_forward(s["cfg"], s["n"], s["X"], s["W"], s["Y"])
        el.el_backward(s["cfg"], s["n"], s["X"], s["W"], s["dY"], s["dX"], s["dW"], s["ws"], s["bytes"])
        return {"Y": s["Y"], "dX": s["dX"], "dW": s["dW"]}
    el.el_sc_forward(s["plan"], s["k_in"], s["n"], s["X"], s["W_lin"], s["z"], s["W"], s["B"], s["ws"], s["bytes"])
    el.el_sc_backward(s["plan"], s["k_in"], s["n"], s["X"], s["W_lin"], s["z"], s["W"], s["dB"], s["dX"], s["dW_lin"],
                      s["dW"], s["ws"], s["bytes"])
    return {"B": s["B"], "dX": s["dX"], "dW_lin": s["dW_lin"], "dW": s["dW"]}


# ---------------------------------------------------------------------------------------------
# what a pass cannot do without: every call reads each of its inputs once and writes each of its
# outputs once


def _num_paths(case):
    plan = sc.sc_plan_create(case["channels"], case["l_max"], case["nu"], ELEMENTS, OUTPUTS[case["outputs"]],
                             sc.SC_F64, 0, sc.SC_PLAN_HOST_ONLY)
    return sc.sc_plan_info(plan).num_paths


def _contraction_work(case):
    n, K = case["nodes"], case["channels"]
    a, b = (case["l_max"] + 1) ** 2, sum(2 * L + 1 for L, _ in OUTPUTS[case["outputs"]])
    row = n * K * ELEMENT_BYTES[case["dtype"]]
    w = ELEMENTS * _num_paths(case) * K * (8 if case["dtype"] == "f64" else 4)
    # Horner's rule: per order one multiply-add for every pair of a component of A and one of B;
    # a reverse pass costs twice as much, the second-order pass twice that
    horner = 2 * case["nu"] * a * b * n * K
    nbytes, flops = row * (a + b) + 4 * n + w, horner
    if case["kind"] in ("sc_step", "sc_force", "fused"):
        nbytes += row * (2 * a + b) + 2 * w
        flops += 2 * horner
    if case["kind"] == "sc_force":
        nbytes += row * (3 * a + 2 * b) + 2 * w
        flops += 4 * horner
    return nbytes, flops


def work(case):
    kind, n = case["kind"], case["nodes"]
    if kind in ("serve", "sc_step", "sc_force"):
        nbytes, flops = _contraction_work(case)
        return {"bytes": nbytes, "flops": flops}
    e = ELEMENT_BYTES[case["dtype"]]
    if kind in ("linear", "fused"):
        k_in, k_out, c, L = case["k_in"], case.get("k_out", case.get("channels")), (case["l_max"] + 1) ** 2, case["l_max"] + 1
        x, y, w = n * k_in * c * e, n * k_out * c * e, L * k_in * k_out * e
        flops = 3 * 2 * n * k_in * k_out * c
        if kind == "linear":
            return {"bytes": (x + w + y) + (x + w + y) + (x + w), "flops": flops}
        # behind one call the mixed features need not pass through memory
        b2, f2 = _contraction_work(case)
        return {"bytes": b2 - n * k_out * 3 * c * e + 3 * x + 3 * w, "flops": flops + f2}
    K, E = case["channels"], _num_edges(n)
    ny, nh, no = ((case[k] + 1) ** 2 for k in ("l_Y", "l_h", "L_max"))
    triples = [(a, b, c) for a in range(case["l_Y"] + 1) for b in range(case["l_h"] + 1)
               for c in range(abs(a - b), min(a + b, case["L_max"]) + 1) if (a + b + c) % 2 == 0]
    R, Y, h, A = E * len(triples) * K * e, E * ny * e, n * nh * K * e, n * no * K * e
    # per path one multiply-add for every pair of a component of h and one of A
    pairs = 2 * sum((2 * b + 1) * (2 * c + 1) for _, b, c in triples) * E * K
    nbytes, flops = (R + Y + h + A + 4 * E), pairs
    nbytes += 2 * (R + Y + h) + A + 8 * E
    flops += 3 * pairs
    if kind == "tp_force":
        nbytes += 3 * (R + Y + h) + 2 * A + 8 * E
        flops += 6 * pairs
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # About four times the differences seen between these paths and the same paths in 64 bits
    # (64-bit cases: between the generated and the table-driven kernels).
    kind, dtype = case["kind"], case["dtype"]
    if dtype == "f64":
        return {"rel": 1e-14}     # seen: up to 1e-15
    if dtype == "bf16":
        return {"rel": 7e-3}      # seen: 1.7e-3, one rounding of a row element
    if kind in ("linear", "fused"):
        return {"rel": 4e-6}      # seen: 2e-7 (Y, dX), 4e-7 (dW over 10 000 atoms; grows with them)
    return {"rel": 7e-7}          # seen: 0.9e-7 to 1.6e-7
