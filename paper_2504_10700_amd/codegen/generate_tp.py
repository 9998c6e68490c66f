"""Generator of the straight-line device code of the channelwise tensor product kernels.

    python -m paper_2504_10700_amd.codegen.generate_tp            # rewrite csrc/generated/tp_gen_*.inc
    python -m paper_2504_10700_amd.codegen.generate_tp --check    # fail if a file would change

Per (edge, channel) Algorithm 1 of arXiv 2504.10700 is a sum over paths (l1,l2,l3) of
R[p] * C(l1,l2,l3) Y_l1 h_l2.  Two programs are emitted per configuration, each a set of
bilinear couplings through the same sparse tensors with a different free index:

  forward   acc[l3] += C . Y_l1 . (R[p] h_l2)
  backward  q[l1]    = C . h_l2 . g_l3 ;  dR[p] = Y_l1 . q ;  dY_l1 += R[p] q
            s[l2]    = C . Y_l1 . g_l3 ;  dh_l2 += R[p] s      (the edge's share of its sender's dh)

A third program, the second-order pass, adds the message's derivative along the cotangents
(hy, hh, hr) of (dY, dh, dR) to ddA and writes the derivatives d2Y, d2h and d2R of
sum(g * that derivative).  All programs go path by path.

The sparse terms come from the library's host tables (tp_plan_terms on a host-only plan);
every coupling tensor is divided by its most frequent |coefficient| (the factor is folded
into the one multiplication by R[p]) so that most terms need no constant.  The programs are
checked in fp64 against the terms before anything is written.  Deterministic.
"""
from __future__ import annotations

import argparse
import ctypes as C
import os
import sys
from typing import Dict, List, Optional, Tuple

import numpy as np

from .program import Program
from .scheme import couple_into
from .tables import HOST_LIB

_HERE = os.path.dirname(os.path.abspath(__file__))
OUT_DIR = os.path.join(os.path.dirname(_HERE), "csrc", "generated")

# tag -> (l_Y, l_h, L_max): the messages of a model whose atomic basis goes up to L_max = l_Y, for sender
# features up to any order l_h <= L_max (0: the first layer; the outputs of the product basis afterwards)
SPECS = {f"y{l}h{lh}o{l}": (l, lh, l) for l in (3, 2, 1) for lh in range(l + 1)}


class _Config(C.Structure):
    _fields_ = [("struct_size", C.c_int32), ("num_channels", C.c_int32), ("l_Y", C.c_int32), ("l_h", C.c_int32),
                ("L_max", C.c_int32), ("dtype", C.c_int32), ("device", C.c_int32), ("flags", C.c_uint32)]


class TPTables:
    """Paths and dense per-path coupling tensors from the library's host-side table builder."""

    def __init__(self, lib_path: str, l_Y: int, l_h: int, L_max: int):
        lib = C.CDLL(lib_path)
        lib.sc_last_error.restype = C.c_char_p
        cfg = _Config()
        cfg.struct_size = C.sizeof(_Config)
        cfg.num_channels, cfg.l_Y, cfg.l_h, cfg.L_max = 64, l_Y, l_h, L_max
        cfg.dtype, cfg.device, cfg.flags = 1, 0, 1 | 2      # f64, host only, generic
        plan = C.c_void_p()

        def check(st):
            if st != 0:
                raise RuntimeError(lib.sc_last_error().decode())
        check(lib.tp_plan_create(C.byref(cfg), C.byref(plan)))
        info = (C.c_int32 * 11)()
        check(lib.tp_plan_info(plan, info))
        self.n_Y, self.n_h, self.n_out, self.P = info[0], info[1], info[2], info[3]
        paths = np.zeros((self.P, 3), dtype=np.int32)
        ip = C.POINTER(C.c_int32)
        check(lib.tp_plan_paths(plan, paths.ctypes.data_as(ip)))
        self.paths = [tuple(int(x) for x in r) for r in paths]
        n = C.c_int32()
        check(lib.tp_plan_terms(plan, 0, C.byref(n), None, None, None, None, None))
        arr = [np.zeros(n.value, dtype=np.int32) for _ in range(4)]
        coef = np.zeros(n.value)
        check(lib.tp_plan_terms(plan, n.value, C.byref(n), *[x.ctypes.data_as(ip) for x in arr],
                                coef.ctypes.data_as(C.POINTER(C.c_double))))
        self.terms = (*arr, coef)
        # dense C[p][m1][m2][m3] of every path
        self.C: List[np.ndarray] = []
        for p, (l1, l2, l3) in enumerate(self.paths):
            D = np.zeros((2 * l1 + 1, 2 * l2 + 1, 2 * l3 + 1))
            sel = arr[0] == p
            D[arr[1][sel] - l1 * l1, arr[2][sel] - l2 * l2, arr[3][sel] - l3 * l3] = coef[sel]
            self.C.append(D)
        check(lib.tp_plan_destroy(plan))


def split_scale(Cp: np.ndarray) -> Tuple[np.ndarray, float]:
    """Cp = kappa * Cs with the most frequent |entry| of Cs exactly 1."""
    nz = np.abs(Cp[Cp != 0.0])
    vals, counts = np.unique(np.round(nz, 12), return_counts=True)
    mode = vals[np.argmax(counts)]
    kappa = float(nz[np.abs(nz - mode) < 1e-11][0])
    Cs = Cp / kappa
    unit = np.abs(np.abs(Cs) - 1.0) < 1e-13
    Cs[unit] = np.sign(Cs[unit])
    return Cs, kappa


def sl(l: int) -> slice:
    return slice(l * l, (l + 1) * (l + 1))


def couple_directly(P: Program, C: np.ndarray, x, v, acc: List[Optional[int]]) -> None:
    """acc[c] += sum_ab C[a,b,c] x[a] v[b] with a fused multiply-add straight into acc for every term of unit magnitude.
    Terms of another magnitude: v scaled by it once, or the terms of a component summed and then scaled, whichever takes
    fewer operations.

    More roundings at the size of acc than by sums of equal magnitude (couple_into): in fp64, twenty edges, l_h = 2, the error of the
    sum is 5.5e-16 for 4.3e-16 of its 2-norm, 6.8e-16 for 4.3e-16 in the second-order pass.  So for fp32 rows in fp64 arithmetic, whose results
    are rounded to 6e-8 and whose kernels are bound by the instructions: l_h = 2, forward 404 -> 350 operations, 3001 atoms,
    128 channels 140 -> 130 us; second-order pass 1725 -> 1679, 1500 atoms 316 -> 305 us; l = 2, l_h = 2, 2500 atoms, 64 channels,
    forward 33.4 -> 32.0."""
    by_mag: Dict[float, Dict[int, List[Tuple[int, int, float]]]] = {}
    for a, b, c in zip(*np.nonzero(C)):
        by_mag.setdefault(round(abs(float(C[a, b, c])), 11), {}).setdefault(int(c), []).append((int(a), int(b), float(C[a, b, c])))
    for mag, targets in sorted(by_mag.items(), key=lambda kv: (abs(kv[0] - 1.0) > 1e-9, kv[0])):
        factors = {b for lst in targets.values() for _, b, _ in lst}
        unit = abs(mag - 1.0) < 1e-9
        if unit or len(factors) <= len(targets):
            exact = 1.0 if unit else abs(next(iter(targets.values()))[0][2])
            scaled = {b: P.cmul(v[b], exact) for b in sorted(factors)}
            for c, lst in targets.items():
                for a, b, coef in lst:
                    if acc[c] is None:
                        acc[c] = P.cmul(P.mul(x[a], scaled[b]), 1.0 if coef > 0 else -1.0)
                    else:
                        acc[c] = P.fma(x[a], scaled[b], acc[c]) if coef > 0 else P.fnma(x[a], scaled[b], acc[c])
            continue
        for c, lst in targets.items():
            q = P.mul(x[lst[0][0]], v[lst[0][1]])
            for a, b, coef in lst[1:]:
                q = P.fma(x[a], v[b], q) if (coef > 0) == (lst[0][2] > 0) else P.fnma(x[a], v[b], q)
            acc[c] = P.cfma(q, lst[0][2], acc[c])


def in_fp32(tab: TPTables) -> bool:
    """Shapes whose fp32 rows are computed in fp32."""
    return tab.n_Y == 16 and tab.n_out == 16 and tab.n_h <= 4


def build_forward(tab: TPTables, couple) -> Program:
    """acc[c] += sum C[a,b,c] y[a] (kappa r[p] h[b]), by couple_into or couple_directly."""
    scaled = [split_scale(Cp) for Cp in tab.C]
    F = Program()
    y = [F.inp(f"y[{a}]") for a in range(tab.n_Y)]
    h = [F.inp(f"h[{b}]") for b in range(tab.n_h)]
    acc: List[Optional[int]] = [F.inp(f"acc[{c}]") for c in range(tab.n_out)]
    for p, (l1, l2, l3) in enumerate(tab.paths):
        Cs, kappa = scaled[p]
        rk = F.cmul(F.load(f"r[{p}]"), kappa)
        u = [F.mul(rk, hb) for hb in h[sl(l2)]]
        part = acc[sl(l3)]
        couple(F, Cs, y[sl(l1)], u, part)
        acc[sl(l3)] = part
        if tab.n_h >= 9:   # many paths: without a boundary all of r is converted to fp64 in front of them
            F.fence(part)
    for c in range(tab.n_out):
        F.out(f"acc[{c}]", acc[c])
    return F


def build_backward(tab: TPTables) -> Program:
    """Backward of one edge."""
    Bq = Program()
    y = [Bq.inp(f"y[{a}]") for a in range(tab.n_Y)]
    h = [Bq.inp(f"h[{b}]") for b in range(tab.n_h)]
    g = [Bq.inp(f"g[{c}]") for c in range(tab.n_out)]
    # path by path, so that only the sums over the paths stay live from one path to the next
    dy: List[Optional[int]] = [None] * tab.n_Y
    # the gradient of the sender's features: sums in fp32 take the edge's share at once, the others term by term (or from
    # zero, where the kernel adds the share: see the header of the function)
    dh_in = [Bq.inp(f"dh[{b}]") for b in range(tab.n_h)]
    dh: List[Optional[int]] = [None] * tab.n_h if in_fp32(tab) else list(dh_in)
    for p, (l1, l2, l3) in enumerate(tab.paths):
        terms, kappa = scaled_terms(Bq, tab.C[p], g[sl(l3)])
        rk = Bq.cmul(Bq.load(f"r[{p}]"), kappa)
        s = couple_terms(Bq, terms, y[sl(l1)], "b", [None] * (2 * l2 + 1))      # s[b] = sum C[a,b,c] y[a] g[c]
        u = [Bq.mul(rk, x) for x in h[sl(l2)]]
        dy[sl(l1)] = couple_terms(Bq, terms, u, "a", dy[sl(l1)])                # dy[a] += sum C[a,b,c] u[b] g[c]
        Bq.out(f"dr[{p}]", scaled_dot(Bq, h[sl(l2)], s, kappa))
        add_scaled(Bq, rk, s, dh, l2)
        out_when_complete(Bq, "dy", dy, tab.paths, p)
        Bq.fence(dy[sl(l1)] + dh[sl(l2)])
    for b in range(tab.n_h):
        Bq.out(f"dh[{b}]", Bq.add(dh[b], dh_in[b]) if in_fp32(tab) else dh[b])
    return Bq


def out_when_complete(P: Program, name: str, v, paths, p: int) -> None:
    """The components of order l1 of `v` leave with the last path that has this l1 (paths are ordered by l1)."""
    l1 = paths[p][0]
    if p + 1 == len(paths) or paths[p + 1][0] != l1:
        for a in range(l1 * l1, (l1 + 1) * (l1 + 1)):
            P.out(f"{name}[{a}]", v[a])


def scaled_terms(P: Program, Cp: np.ndarray, g):
    """The terms of a path as (a, b, sign, |C[a,b,c]| / kappa * g[c]): g scaled once per magnitude and
    shared by every coupling that contracts with g."""
    Cs, kappa = split_scale(Cp)
    return [(int(a), int(b), Cs[a, b, c] > 0, P.cmul(g[c], round_unit(abs(float(Cs[a, b, c])))))
            for a, b, c in zip(*np.nonzero(Cs))], kappa


def round_unit(c: float) -> float:
    return 1.0 if abs(c - 1.0) < 1e-13 else c


def couple_terms(P: Program, terms, x, free: str, acc: List[Optional[int]]) -> List[Optional[int]]:
    """acc[free index] += sum over the terms of sign * x[the other index] * scaled g."""
    acc = list(acc)
    for a, b, plus, gs in terms:
        i, xi = (a, x[b]) if free == "a" else (b, x[a])
        if acc[i] is None:
            t = P.mul(xi, gs)
            acc[i] = t if plus else P.cmul(t, -1.0)
        else:
            acc[i] = P.fma(xi, gs, acc[i]) if plus else P.fnma(xi, gs, acc[i])
    return acc


def scaled_dot(P: Program, x, v, kappa: float) -> Optional[int]:
    """kappa * sum_i x[i] v[i]; entries of v that do not occur are None."""
    dot = None
    for xi, vi in zip(x, v):
        if vi is not None:
            dot = P.fma(xi, vi, dot)
    return None if dot is None else P.cmul(dot, kappa)


def add_scaled(P: Program, f: int, v, acc: List[Optional[int]], l: int) -> None:
    """acc[components of order l] += f * v."""
    for i, vi in enumerate(v):
        if vi is not None:
            acc[l * l + i] = P.fma(f, vi, acc[l * l + i])


def build_double_backward(tab: TPTables, couple) -> Program:
    """psi = sum_c g[c] * (derivative of the edge's message along (hy, hh, hr)):
    dda += that derivative; d2y, d2h, d2r = d psi / d (y, h, r) (overwritten).

    The message is linear in each of y, h and r, so every path needs five couplings through its
    tensor, and nothing of one path is needed by another (k = kappa):
      u = k r h,  v = k (hr h + r hh)
      dda += C.y.v + C.hy.u,   d2y += C.v.g
      s = C.y.g,  s' = C.hy.g:   d2r = k (h.s' + hh.s),   d2h += k (hr s + r s')
    (Differentiating the forward program mechanically gives the same sums in an order in which the
    intermediates of all paths are live at once: 6 KB of scratch per lane for l_h = 2 in fp64.)"""
    P = Program()
    y = [P.inp(f"y[{a}]") for a in range(tab.n_Y)]
    hy = [P.inp(f"hy[{a}]") for a in range(tab.n_Y)]
    h = [P.inp(f"h[{b}]") for b in range(tab.n_h)]
    hh = [P.inp(f"hh[{b}]") for b in range(tab.n_h)]
    g = [P.inp(f"g[{c}]") for c in range(tab.n_out)]
    dda: List[Optional[int]] = [P.inp(f"dda[{c}]") for c in range(tab.n_out)]
    d2y: List[Optional[int]] = [None] * tab.n_Y
    d2h: List[Optional[int]] = [None] * tab.n_h
    for p, (l1, l2, l3) in enumerate(tab.paths):
        Cs, kappa = split_scale(tab.C[p])
        rk, hrk = P.cmul(P.load(f"r[{p}]"), kappa), P.cmul(P.load(f"hr[{p}]"), kappa)
        u = [P.mul(rk, x) for x in h[sl(l2)]]
        v = [P.fma(hrk, x, P.mul(rk, hx)) for x, hx in zip(h[sl(l2)], hh[sl(l2)])]
        part = dda[sl(l3)]
        couple(P, stack_pairs(Cs), y[sl(l1)] + hy[sl(l1)], v + u, part)
        dda[sl(l3)] = part
        terms, _ = scaled_terms(P, tab.C[p], g[sl(l3)])
        d2y[sl(l1)] = couple_terms(P, terms, v, "a", d2y[sl(l1)])
        s = couple_terms(P, terms, y[sl(l1)], "b", [None] * (2 * l2 + 1))
        sh = couple_terms(P, terms, hy[sl(l1)], "b", [None] * (2 * l2 + 1))
        P.out(f"d2r[{p}]", scaled_dot(P, h[sl(l2)] + hh[sl(l2)], sh + s, kappa))
        add_scaled(P, hrk, s, d2h, l2)
        add_scaled(P, rk, sh, d2h, l2)
        out_when_complete(P, "d2y", d2y, tab.paths, p)
        P.fence(dda[sl(l3)] + d2y[sl(l1)] + d2h[sl(l2)])
    for c in range(tab.n_out):
        P.out(f"dda[{c}]", dda[c])
    for b in range(tab.n_h):
        P.out(f"d2h[{b}]", d2h[b])
    return P


def stack_pairs(C: np.ndarray) -> np.ndarray:
    """The tensor of C.x.v + C.x'.v' as one coupling of (x, x') with (v, v')."""
    Z = np.zeros_like(C)
    return np.concatenate([np.concatenate([C, Z], 1), np.concatenate([Z, C], 1)], 0)


def self_check_double(tab: TPTables, D: Program, dtype=np.float64) -> Dict[str, float]:
    rng = np.random.default_rng(1357)
    n = 1500
    shapes = {"y": tab.n_Y, "hy": tab.n_Y, "h": tab.n_h, "hh": tab.n_h, "r": tab.P, "hr": tab.P, "g": tab.n_out}
    v = {k: rng.standard_normal((n, m)).astype(dtype).astype(np.float64) for k, m in shapes.items()}
    p, a, b, c, coef = tab.terms
    dda = np.zeros((n, tab.n_out))
    d2r = np.zeros((n, tab.P))
    d2y = np.zeros((n, tab.n_Y))
    d2h = np.zeros((n, tab.n_h))
    for t in range(len(coef)):
        Y, HY, X, HX, R, HR, G = (v["y"][:, a[t]], v["hy"][:, a[t]], v["h"][:, b[t]], v["hh"][:, b[t]],
                                  v["r"][:, p[t]], v["hr"][:, p[t]], v["g"][:, c[t]])
        dda[:, c[t]] += coef[t] * (HR * Y * X + R * HY * X + R * Y * HX)
        d2r[:, p[t]] += coef[t] * G * (HY * X + Y * HX)
        d2y[:, a[t]] += coef[t] * G * (HR * X + R * HX)
        d2h[:, b[t]] += coef[t] * G * (HR * Y + R * HY)
    inputs = {f"{k}[{i}]": v[k][:, i] for k, m in shapes.items() for i in range(m)}
    inputs.update({f"dda[{i}]": np.zeros(n) for i in range(tab.n_out)})
    inputs["T(0)"] = np.zeros(n)
    res = D.evaluate(inputs, dtype)

    def col(x):
        return np.zeros(n) if x is None else x.astype(np.float64)

    def err(x, ref):
        return float(np.abs(x - ref).max() / np.sqrt((ref ** 2).mean()))
    return {
        "ddA": err(np.stack([col(res[f"dda[{i}]"]) for i in range(tab.n_out)], 1), dda),
        "d2R": err(np.stack([col(res[f"d2r[{i}]"]) for i in range(tab.P)], 1), d2r),
        "d2Y": err(np.stack([col(res[f"d2y[{i}]"]) for i in range(tab.n_Y)], 1), d2y),
        "d2h": err(np.stack([col(res[f"d2h[{i}]"]) for i in range(tab.n_h)], 1), d2h),
    }


def self_check(tab: TPTables, F: Program, Bq: Program, dtype=np.float64) -> Dict[str, float]:
    rng = np.random.default_rng(2468)
    n = 1500
    y = rng.standard_normal((n, tab.n_Y))
    h = rng.standard_normal((n, tab.n_h))
    r = rng.standard_normal((n, tab.P))
    g = rng.standard_normal((n, tab.n_out))
    y, h, r, g = (x.astype(dtype).astype(np.float64) for x in (y, h, r, g))
    p, a, b, c, coef = tab.terms
    msg = np.zeros((n, tab.n_out))
    dr = np.zeros((n, tab.P))
    dy = np.zeros((n, tab.n_Y))
    dh = np.zeros((n, tab.n_h))
    for t in range(len(coef)):
        msg[:, c[t]] += coef[t] * r[:, p[t]] * y[:, a[t]] * h[:, b[t]]
        dr[:, p[t]] += coef[t] * y[:, a[t]] * h[:, b[t]] * g[:, c[t]]
        dy[:, a[t]] += coef[t] * r[:, p[t]] * h[:, b[t]] * g[:, c[t]]
        dh[:, b[t]] += coef[t] * r[:, p[t]] * y[:, a[t]] * g[:, c[t]]
    inputs = {f"y[{i}]": y[:, i] for i in range(tab.n_Y)}
    inputs.update({f"h[{i}]": h[:, i] for i in range(tab.n_h)})
    inputs.update({f"r[{i}]": r[:, i] for i in range(tab.P)})
    inputs.update({f"g[{i}]": g[:, i] for i in range(tab.n_out)})
    inputs.update({f"acc[{i}]": np.zeros(n) for i in range(tab.n_out)})
    inputs.update({f"dh[{i}]": np.zeros(n) for i in range(tab.n_h)})

    def col(v):
        return np.zeros(n) if v is None else v.astype(np.float64)

    def err(x, ref):
        return float(np.abs(x - ref).max() / np.sqrt((ref ** 2).mean()))
    rf, rq = F.evaluate(inputs, dtype), Bq.evaluate(inputs, dtype)
    return {
        "msg": err(np.stack([col(rf[f"acc[{i}]"]) for i in range(tab.n_out)], 1), msg),
        "dR": err(np.stack([col(rq[f"dr[{i}]"]) for i in range(tab.P)], 1), dr),
        "dY": err(np.stack([col(rq[f"dy[{i}]"]) for i in range(tab.n_Y)], 1), dy),
        "dh": err(np.stack([col(rq[f"dh[{i}]"]) for i in range(tab.n_h)], 1), dh),
    }


def flops(c: Dict[str, int]) -> int:
    return 2 * (c.get("fma", 0) + c.get("fnma", 0) + c.get("cfma", 0)) + sum(c.get(k, 0) for k in ("mul", "add", "sub", "cmul"))


def emit_either(L: List[str], direct: Program, by_magnitude: Program) -> None:
    """The body of a function whose first template parameter is kDirect (one program where both are the same)."""
    if direct is by_magnitude:
        L.append(direct.emit("T", "    "))
        return
    L.append("    if constexpr (kDirect) {")
    L.append(direct.emit("T", "      "))
    L.append("    } else {")
    L.append(by_magnitude.emit("T", "      "))
    L.append("    }")


def emit_inc(tag: str, spec, tab: TPTables, F, Bq: Program, D) -> str:
    """F, D: (term by term, by magnitude)."""
    l_Y, l_h, L_max = spec
    cs = [F[0].count(), Bq.count(), D[0].count()]
    cs_by_magnitude = [F[1].count(), Bq.count(), D[1].count()]
    L = []
    L.append(f"// GENERATED by paper_2504_10700_amd/codegen/generate_tp.py for l_Y={l_Y}, l_h={l_h}, L_max={L_max}.  Do not edit.")
    L.append("//")
    L.append("// Straight-line evaluation of Algorithm 1 of arXiv 2504.10700 per (edge, channel) and of its")
    L.append("// derivatives; paths (index of r): " + " ".join(f"{i}:({a},{b},{c})" for i, (a, b, c) in enumerate(tab.paths)))
    L.append(f"struct GenTP_{tag} {{")
    L.append(f"  static constexpr int kLY = {l_Y}, kLh = {l_h}, kLout = {L_max};")
    L.append(f"  static constexpr int kNY = {tab.n_Y}, kNh = {tab.n_h}, kNout = {tab.n_out}, kP = {tab.P};")
    L.append("  // vector instructions / flops (a fused multiply-add counts twice) per (edge, channel):")
    L.append("  // forward, backward, second-order pass; of the programs without and with kDirect")
    L.append("  static constexpr int kOps[2][3] = {" + ", ".join(
        "{" + ", ".join(str(c["total"]) for c in x) + "}" for x in (cs_by_magnitude, cs)) + "};")
    L.append("  static constexpr int kFlops[2][3] = {" + ", ".join(
        "{" + ", ".join(str(flops(c)) for c in x) + "}" for x in (cs_by_magnitude, cs)) + "};")
    L.append("  // does backward add the terms of dh to the sum one by one (or the edge's share at once)?")
    L.append(f"  static constexpr bool kDhByTerms = {'false' if in_fp32(tab) else 'true'};")
    L.append("")
    L.append("  // kDirect: the terms of a coupling go into the sum over the edges one by one, and not as sums of equal magnitude: fewer")
    L.append("  // operations, more roundings at the size of that sum." + ("  (Not for this shape.)" if in_fp32(tab) else ""))
    L.append("  // R: r[p] as T.  DR, DY: element p or a is assigned once, where the last path that contributes ends.")
    L.append("  // acc += message of one edge")
    L.append("  template <bool kDirect, typename T, typename R>")
    L.append("  static __device__ __forceinline__ void forward(const T (&y)[kNY], const T (&h)[kNh], const R& r, T (&acc)[kNout]) {")
    emit_either(L, *F)
    L.append("  }")
    L.append("")
    L.append("  // g = dA of the receiver; overwritten: dr and dy (this channel's share of the edge's dY); dh += the edge's")
    L.append("  // share of the gradient of its sender's features")
    L.append("  template <typename T, typename R, typename DR, typename DY>")
    L.append("  static __device__ __forceinline__ void backward(const T (&y)[kNY], const T (&h)[kNh], const R& r,")
    L.append("                                                  const T (&g)[kNout], DR& dr, DY& dy, T (&dh)[kNh]) {")
    L.append(Bq.emit("T", "    "))
    L.append("  }")
    L.append("")
    L.append("  // Second-order pass of one edge.  hy, hh, hr: cotangents of (dY, dh, dR); g = dA of the receiver.")
    L.append("  // dda += derivative of the edge's message along (hy, hh, hr); with psi = sum(g * that derivative):")
    L.append("  // d2r = d psi / d r, d2y = this channel's share of d psi / d y, d2h = the edge's share of d psi / d h")
    L.append("  // (all three overwritten).")
    L.append("  template <bool kDirect, typename T, typename R, typename DR, typename DY>")
    L.append("  static __device__ __forceinline__ void double_backward(const T (&y)[kNY], const T (&hy)[kNY], const T (&h)[kNh],")
    L.append("                                                         const T (&hh)[kNh], const R& r, const R& hr,")
    L.append("                                                         const T (&g)[kNout], T (&dda)[kNout], DR& d2r, DY& d2y,")
    L.append("                                                         T (&d2h)[kNh]) {")
    emit_either(L, *D)
    L.append("  }")
    L.append("};")
    return "\n".join(L) + "\n"


def generate(tag: str, lib_path: str = HOST_LIB, verbose: bool = True) -> str:
    spec = SPECS[tag]
    tab = TPTables(lib_path, *spec)
    Bq = build_backward(tab)
    F, D = [], []
    for couple in (couple_into,) if in_fp32(tab) else (couple_directly, couple_into):
        F.append(build_forward(tab, couple))
        D.append(build_double_backward(tab, couple))
        e64 = self_check(tab, F[-1], Bq, np.float64)
        assert max(e64.values()) < 1e-12, e64
        d64 = self_check_double(tab, D[-1], np.float64)
        assert max(d64.values()) < 1e-12, d64
        if verbose:
            e32 = self_check(tab, F[-1], Bq, np.float32)
            d32 = self_check_double(tab, D[-1], np.float32)
            print(f"[tp {tag}] {couple.__name__}: P={tab.P} terms={len(tab.terms[4])} ops fwd={F[-1].count()['total']} "
                  f"bwd={Bq.count()['total']} second-order={D[-1].count()['total']}")
            print(f"[tp {tag}] fp64 self-check max|err|/rms: {e64} {d64}")
            print(f"[tp {tag}] fp32 emulation  max|err|/rms: {e32} {d32}")
    return emit_inc(tag, spec, tab, (F[0], F[-1]), Bq, (D[0], D[-1]))


def main(argv=None) -> int:
    ap = argparse.ArgumentParser()
    ap.add_argument("--check", action="store_true")
    ap.add_argument("--lib", default=HOST_LIB)
    args = ap.parse_args(argv)
    os.makedirs(OUT_DIR, exist_ok=True)
    rc = 0
    for tag in SPECS:
        text = generate(tag, args.lib, verbose=not args.check)
        path = os.path.join(OUT_DIR, f"tp_gen_{tag}.inc")
        old = open(path).read() if os.path.exists(path) else None
        if args.check:
            if old != text:
                print(f"{path} is out of date", file=sys.stderr)
                rc = 1
        elif old != text:
            with open(path, "w") as f:
                f.write(text)
            print("wrote", path)
    return rc


if __name__ == "__main__":
    sys.exit(main())
