#!/usr/bin/env python3
"""Generate recon_gen.h: the linear parts of the HWENO reconstruction.

Derived here with exact rational arithmetic (sympy) from the moment
conditions of the paper:
  * 1D q_2, q_3, q_4 (eq. q): square systems on the cells i-1, i, i+1.
  * 2D q_2, q_3, q_4 (eqs. 2D-q2 .. 2D-q4): the centre cell average is kept
    exactly and every other condition is fitted in the unweighted
    least-squares sense (KKT system, solved exactly).
  * smoothness-indicator quadratic forms of eq. (beta) / (2D-beta) in the
    cell's reference coordinates (kappa = 2, 3, 5; every multi-index once).
  * evaluation of a polynomial at the Gauss-Lobatto points of eq. (F)
    (nodes +-1/2, +-sqrt(5)/10; tensor grid in 2D).
  * the first-moment modification of eq. (p0)/(vi).

The 2D stencil is symmetric under x -> -x and y -> -y, so the maps
decouple by the parity class (a mod 2, b mod 2) of the monomial xi^a eta^b
once the stencil data are combined into even/odd sums and differences, and
the (even, even) class once more under the exchange of x and y.  The
generator applies these changes of variables exactly and emits only the
non-zero entries, which roughly halves the arithmetic.  The coefficients are
kept in twice the cell's reference coordinates, where the outer
Gauss-Lobatto nodes are +-1 and the inner ones +-1/sqrt(5): the evaluation
then needs two constants and is factored axis by axis.

Output: straight-line FP64 device code with each constant written as an
exact hexadecimal literal of the correctly rounded double.

Run:  python gen_recon.py > recon_gen.h
"""
from __future__ import annotations

import itertools
import re
import sys
from fractions import Fraction

import sympy as sp

R = sp.Rational


# ------------------------------------------------------------ helpers
import struct

# FP64 constants that an instruction cannot encode directly (their low 32
# bits are not zero) are collected into one table: on the device the table
# is copied into LDS once per work group and read with broadcast LDS loads,
# instead of being rebuilt in scalar registers at every use.
_KTAB = []
_KIDX = {}


def _encodable(f: float) -> bool:
    return (struct.unpack("<Q", struct.pack("<d", f))[0] & 0xFFFFFFFF) == 0


def lit(x) -> str:
    x = sp.nsimplify(x)
    if x.is_Rational:
        f = float(Fraction(int(x.p), int(x.q)))   # correctly rounded
    else:
        f = float(sp.N(x, 60))
    if f == 0.0:
        return "0.0"
    if _encodable(f):
        return f.hex()
    a = abs(f)
    if a not in _KIDX:
        _KIDX[a] = len(_KTAB)
        _KTAB.append(a)
    return ("-" if f < 0 else "") + f"MR_KT({_KIDX[a]})"


def mono_avg(n, d):
    a, b = R(d) - R(1, 2), R(d) + R(1, 2)
    return (b ** (n + 1) - a ** (n + 1)) / (n + 1)


def mono_mom(n, d):
    return mono_avg(n + 1, d) - d * mono_avg(n, d)


def dot_code(terms, indent="  "):
    """terms: list of (coef (Rational), expr str) -> C expression string."""
    terms = [(c, e) for c, e in terms if c != 0]
    if not terms:
        return "0.0"
    parts = []
    for c, e in terms:
        if c == 1:
            parts.append(f"{e}")
        elif c == -1:
            parts.append(f"-{e}")
        else:
            parts.append(f"{lit(c)} * {e}")
    s = " + ".join(parts)
    return s.replace("+ -", "- ")


# ================================================================== 1D
def maps_1d():
    """q_l coefficient maps over data (um, u0, up, vm, v0, vp)."""
    data = sp.symbols("um u0 up vm v0 vp")
    conds = {2: [(0, -1), (0, 0), (0, 1)],
             3: [(0, -1), (0, 0), (0, 1), (1, 0)],
             4: [(0, -1), (0, 0), (0, 1), (1, -1), (1, 0), (1, 1)]}
    didx = {(0, -1): 0, (0, 0): 1, (0, 1): 2, (1, -1): 3, (1, 0): 4, (1, 1): 5}
    deg = {2: 2, 3: 3, 4: 5}
    out = {}
    for l, cl in conds.items():
        n = deg[l] + 1
        A = sp.Matrix([[mono_avg(p, d) if t == 0 else mono_mom(p, d) for p in range(n)] for t, d in cl])
        b = sp.Matrix([data[didx[c]] for c in cl])
        sol = A.LUsolve(b)
        out[l] = [sp.Poly(sp.expand(s), *data) for s in sol]
    return data, out


def gram_1d(kappa, n):
    G = sp.zeros(n, n)
    for a in range(1, kappa + 1):
        for p in range(a, n):
            for s in range(a, n):
                fp = sp.ff(p, a)
                fs = sp.ff(s, a)
                G[p, s] += fp * fs * mono_avg(p + s - 2 * a, 0)
    return G


def quad_form_code(name, G, idx, var, lines, acc):
    """Emit acc = sum_{p,s in idx} G[p,s] var[p] var[s] with symmetric
    folding: t_p = G_pp v_p + 2 sum_{s>p} G_ps v_s; acc += t_p v_p."""
    first = True
    for a, p in enumerate(idx):
        terms = [(G[p, p], f"{var}[{p}]")]
        for s in idx[a + 1:]:
            terms.append((2 * G[p, s], f"{var}[{s}]"))
        terms = [(c, e) for c, e in terms if c != 0]
        if not terms:
            continue
        lines.append(f"  {{ const double t = {dot_code(terms)};")
        if first:
            lines.append(f"    {acc} = t * {var}[{p}]; }}")
            first = False
        else:
            lines.append(f"    {acc} = fma(t, {var}[{p}], {acc}); }}")
    if first:
        lines.append(f"  {acc} = 0.0;")


def emit_1d(lines):
    data, maps = maps_1d()
    names = ["um", "u0", "up", "vm", "v0", "vp"]
    lines.append("/* ---- 1D: q_2 (3 coefs), q_3 (4), q_4 (6) of eq. (q) ---- */")
    lines.append("MR_DEV inline void mr1_maps(double um, double u0, double up, double vm, double v0, double vp,")
    lines.append("                            double q2[3], double q3[4], double q4[6]) {")
    # parity combos
    lines.append("  const double su = um + up, du = up - um, sv = vm + vp, dv = vp - vm;")
    sym = {"su": None}
    for l, arr in ((2, "q2"), (3, "q3"), (4, "q4")):
        for k, poly in enumerate(maps[l]):
            expr = poly.as_expr()
            # rewrite in terms of (u0, su, du, v0, sv, dv)
            um, u0, up, vm, v0, vp = data
            su, du, sv, dv = sp.symbols("su du sv dv")
            e = sp.expand(expr.subs({um: (su - du) / 2, up: (su + du) / 2, vm: (sv - dv) / 2, vp: (sv + dv) / 2}))
            pe = sp.Poly(e, u0, su, du, v0, sv, dv)
            terms = []
            for sname, s in (("u0", u0), ("su", su), ("du", du), ("v0", v0), ("sv", sv), ("dv", dv)):
                terms.append((pe.coeff_monomial(s), sname))
            lines.append(f"  {arr}[{k}] = {dot_code(terms)};")
    lines.append("}")
    # beta forms
    for kappa, n, nm in ((2, 3, "mr1_beta_k2"), (3, 4, "mr1_beta_k3"), (5, 6, "mr1_beta_k5")):
        G = gram_1d(kappa, n)
        lines.append(f"MR_DEV inline double {nm}(const double c[{n}]) {{")
        lines.append("  double b;")
        quad_form_code(nm, G, list(range(1, n)), "c", lines, "b")
        lines.append("  return b;")
        lines.append("}")
    # evaluation at the 4 GL nodes, parity split
    lines.append("/* values at xi = -1/2, -sqrt(5)/10, sqrt(5)/10, 1/2 of a quintic */")
    lines.append("MR_DEV inline void mr1_eval(const double c[6], double out[4]) {")
    s5 = sp.sqrt(5) / 10
    for nm_, x in (("a", R(1, 2)), ("b", s5)):
        ev = [(sp.nsimplify(x ** k), f"c[{k}]") for k in (0, 2, 4)]
        od = [(sp.nsimplify(x ** k), f"c[{k}]") for k in (1, 3, 5)]
        lines.append(f"  const double e{nm_} = {dot_code(ev)};")
        lines.append(f"  const double o{nm_} = {dot_code(od)};")
    lines.append("  out[0] = ea - oa; out[1] = eb - ob; out[2] = eb + ob; out[3] = ea + oa;")
    lines.append("}")


# ================================================================== 2D
def monos(deg):
    out = []
    for d in range(deg + 1):
        for a in range(d, -1, -1):
            out.append((a, d - a))
    return out


MON = monos(5)   # 21 monomials; P2 = first 6, P3 = first 10


def lab_off(lab):
    return (lab - 1) % 3 - 1, (lab - 1) // 3 - 1


def cond_row(t, lab, a, b):
    dx, dy = lab_off(lab)
    if t == 0:
        return mono_avg(a, dx) * mono_avg(b, dy)
    if t == 1:
        return mono_mom(a, dx) * mono_avg(b, dy)
    return mono_avg(a, dx) * mono_mom(b, dy)


def lsq_map_2d(ncoef, conds):
    """Exact constrained least-squares map: coefficient = M @ data, data are
    the condition values in the order of conds; centre average exact."""
    rows = [[cond_row(t, lab, *MON[p]) for p in range(ncoef)] for t, lab in conds]
    ctr = conds.index((0, 5))
    n = ncoef + 1
    K = sp.zeros(n, n)
    Rhs = sp.zeros(n, len(conds))
    for r, (t, lab) in enumerate(conds):
        if r == ctr:
            for p in range(ncoef):
                K[ncoef, p] = rows[r][p]
                K[p, ncoef] = rows[r][p]
            Rhs[ncoef, r] = 1
            continue
        for p in range(ncoef):
            for s in range(ncoef):
                K[p, s] += rows[r][p] * rows[r][s]
            Rhs[p, r] += rows[r][p]
    sol = K.LUsolve(Rhs)
    return sol[:ncoef, :]


# stencil data symbols: u1..u9, v1..v9, w1..w9 (labels)
U = sp.symbols("u1:10")
V = sp.symbols("v1:10")
W = sp.symbols("w1:10")


def parity_vars():
    """Even/odd combinations of the 3x3 data.  Returns (defs, subs) where
    defs are C definitions and subs maps each raw symbol to an expression in
    the combination symbols."""
    defs = []
    subs = {}
    # averages: a(dx, dy) at label 1 + (dx+1) + 3(dy+1)
    def lab(dx, dy):
        return 1 + (dx + 1) + 3 * (dy + 1)
    combos = {}
    # x-stage for each row dy: e = a(-1)+a(1), o = a(1)-a(-1), c = a(0)
    # y-stage: f_even = f(-1)+f(1), f_odd = f(1)-f(-1), f_mid = f(0)
    # u: classes by (x part, y part)
    syms = {}
    for base, arr in (("u", U),):
        for xp in ("c", "e", "o"):
            for yp in ("m", "s", "d"):
                syms[f"{base}{xp}{yp}"] = sp.Symbol(f"{base}{xp}{yp}")
    # inverse relations: a(dx,dy) in terms of combos
    # x: a(-1) = (e - o)/2, a(1) = (e + o)/2, a(0) = c
    # y: f(-1) = (s - d)/2, f(1) = (s + d)/2, f(0) = m
    def xy_inv(base, dx, dy, xparts=("c", "e", "o")):
        if dy == 0:
            ypart = lambda xp: syms[f"{base}{xp}m"]
        elif dy == -1:
            ypart = lambda xp: (syms[f"{base}{xp}s"] - syms[f"{base}{xp}d"]) / 2
        else:
            ypart = lambda xp: (syms[f"{base}{xp}s"] + syms[f"{base}{xp}d"]) / 2
        if dx == 0:
            return ypart("c")
        if dx == -1:
            return (ypart("e") - ypart("o")) / 2
        return (ypart("e") + ypart("o")) / 2
    for dx in (-1, 0, 1):
        for dy in (-1, 0, 1):
            subs[U[lab(dx, dy) - 1]] = xy_inv("u", dx, dy)
    return syms, subs


def emit_2d(lines):
    nco = {2: 6, 3: 10, 4: 21}
    vl = [1, 3, 4, 5, 6, 7, 9]
    wl = [1, 2, 3, 5, 7, 8, 9]
    conds = {2: [(0, l) for l in range(1, 10)],
             3: [(0, l) for l in range(1, 10)] + [(1, 5), (2, 5)],
             4: [(0, l) for l in range(1, 10)] + [(1, l) for l in vl] + [(2, l) for l in wl]}

    def dsym(t, lab):
        return (U, V, W)[t][lab - 1]

    # ---- change of variables to even/odd combinations ----
    # averages
    def lab(dx, dy):
        return 1 + (dx + 1) + 3 * (dy + 1)
    cdefs = []
    cvars = {}
    raw = {}
    def add(name, expr_c, sym_expr):
        cvars[name] = sp.Symbol(name)
        cdefs.append((name, expr_c))
        raw[name] = sym_expr
    def u_(dx, dy):
        return f"u[{lab(dx, dy) - 1}]"
    def v_(dx, dy):
        return f"v[{lab(dx, dy) - 1}]"
    def w_(dx, dy):
        return f"w[{lab(dx, dy) - 1}]"
    # averages: rows (dy) -> e, o, c
    for dy, tag in ((-1, "b"), (0, "m"), (1, "t")):
        add(f"ue{tag}", f"{u_(-1, dy)} + {u_(1, dy)}", U[lab(-1, dy) - 1] + U[lab(1, dy) - 1])
        add(f"uo{tag}", f"{u_(1, dy)} - {u_(-1, dy)}", U[lab(1, dy) - 1] - U[lab(-1, dy) - 1])
    add("usm", f"{u_(0, -1)} + {u_(0, 1)}", U[lab(0, -1) - 1] + U[lab(0, 1) - 1])
    U5 = U[4]
    final_u = {
        "a00": (f"{u_(0, 0)}", U5),
        "a01": ("usm + uem", raw["usm"] + raw["uem"]),
        "a02": ("usm - uem", raw["usm"] - raw["uem"]),
        "a03": ("ueb + uet", raw["ueb"] + raw["uet"]),
        "a10": ("uom", raw["uom"]),
        "a11": ("uob + uot", raw["uob"] + raw["uot"]),
        "a20": (f"{u_(0, 1)} - {u_(0, -1)}", U[lab(0, 1) - 1] - U[lab(0, -1) - 1]),
        "a21": ("uet - ueb", raw["uet"] - raw["ueb"]),
        "a30": ("uot - uob", raw["uot"] - raw["uob"]),
    }
    # classes: a0x -> (0,0), a1x -> (1,0), a2x -> (0,1), a3x -> (1,1)
    # vtilde: available at (+-1, dy) and (0, 0)
    for dy, tag in ((-1, "b"), (0, "m"), (1, "t")):
        add(f"vs{tag}", f"{v_(1, dy)} + {v_(-1, dy)}", V[lab(1, dy) - 1] + V[lab(-1, dy) - 1])
        add(f"vd{tag}", f"{v_(1, dy)} - {v_(-1, dy)}", V[lab(1, dy) - 1] - V[lab(-1, dy) - 1])
    final_v = {
        "b10": ("vsm", raw["vsm"]),                         # (1,0)
        "b11": ("vsb + vst", raw["vsb"] + raw["vst"]),      # (1,0)
        "b12": (f"{v_(0, 0)}", V[4]),                       # (1,0)
        "b20": ("vdt - vdb", raw["vdt"] - raw["vdb"]),      # (0,1)
        "b30": ("vst - vsb", raw["vst"] - raw["vsb"]),      # (1,1)
    }
    # wtilde: available at (dx, +-1) and (0, 0); mirror of vtilde
    for dx, tag in ((-1, "l"), (0, "m"), (1, "r")):
        add(f"ws{tag}", f"{w_(dx, 1)} + {w_(dx, -1)}", W[lab(dx, 1) - 1] + W[lab(dx, -1) - 1])
        add(f"wd{tag}", f"{w_(dx, 1)} - {w_(dx, -1)}", W[lab(dx, 1) - 1] - W[lab(dx, -1) - 1])
    final_w = {
        "c20": ("wsm", raw["wsm"]),                         # (0,1)
        "c21": ("wsl + wsr", raw["wsl"] + raw["wsr"]),      # (0,1)
        "c22": (f"{w_(0, 0)}", W[4]),                       # (0,1)
        "c10": ("wdr - wdl", raw["wdr"] - raw["wdl"]),      # (1,0)
        "c30": ("wsr - wsl", raw["wsr"] - raw["wsl"]),      # (1,1)
    }
    # (0,0) from both: sums and differences under the exchange of x and y
    add("vds", "vdb + vdt", raw["vdb"] + raw["vdt"])
    add("wds", "wdl + wdr", raw["wdl"] + raw["wdr"])
    final_w.update({
        "b00": ("vdm + wdm", raw["vdm"] + raw["wdm"]),
        "b01": ("vds + wds", raw["vds"] + raw["wds"]),
        "c00": ("vdm - wdm", raw["vdm"] - raw["wdm"]),
        "c01": ("vds - wds", raw["vds"] - raw["wds"]),
    })
    finals = {}
    finals.update(final_u)
    finals.update(final_v)
    finals.update(final_w)
    # express the raw data in terms of the final combination variables:
    # solve the linear system raw -> finals (exact)
    fin_names = list(finals.keys())
    fin_syms = sp.symbols(" ".join(fin_names))
    used_raw = list(U) + [V[l - 1] for l in vl] + [W[l - 1] for l in wl]
    eqs = [sp.Eq(fs, finals[n][1]) for n, fs in zip(fin_names, fin_syms)]
    sol = sp.solve(eqs, used_raw, dict=True)[0]

    lines.append("/* ---- 2D: q_2 (6 coefs), q_3 (10), q_4 (21) of eqs. (2D-q2)-(2D-q4),")
    lines.append("   centre average exact, other conditions in the least-squares sense.")
    lines.append("   Monomial order: degree by degree, xi power descending:")
    lines.append("   " + ", ".join(f"x^{a}y^{b}" for a, b in MON) + ".")
    lines.append("   With c the monomial coefficients, entry (a, b) holds 2^(1-a-b) c_ab (the")
    lines.append("   coefficients in X = 2 xi, Y = 2 eta, twice over, so that the outer nodes are")
    lines.append("   +-1); entries 3 and 5 hold the sum and 2/5 of the difference of the x^2 and")
    lines.append("   y^2 coefficients, entries 10 and 14 the sum and 12/25 of the difference of")
    lines.append("   the x^4 and y^4 ones (the exchange x <-> y decouples them) */")
    lines.append("MR_DEV inline void mr2_maps(const double u[9], const double v[9], const double w[9],")
    lines.append("                            double q2[6], double q3[10], double q4[21]) {")
    for name, cexpr in cdefs:
        lines.append(f"  const double {name} = {cexpr};")
    for n in fin_names:
        cexpr = finals[n][0]
        lines.append(f"  const double {n} = {cexpr};")
    # basis of the coefficients: z = B c
    B = sp.zeros(21, 21)
    for p, (a, b) in enumerate(MON):
        B[p, p] = R(2) ** (1 - a - b)
    for p, q, f in ((3, 5, R(2, 5)), (10, 14, R(12, 25))):
        sp_, sq_ = B[p, p], B[q, q]
        B[p, q] = sq_
        B[q, p], B[q, q] = f * sp_, -f * sq_
    Bi = B.inv()
    zcls = {p: (MON[p][0] % 2, MON[p][1] % 2, 1 if p in (5, 14) else 0) for p in range(21)}
    total_terms = 0
    rows2 = None
    for l, arr in ((2, "q2"), (3, "q3"), (4, "q4")):
        M = B[:nco[l], :nco[l]] * lsq_map_2d(nco[l], conds[l])
        # q_2 and q_3 share these entries (the evaluation takes q_3's)
        if l == 2:
            rows2 = M
        elif l == 3:
            assert all(M[p, :9] == rows2[p, :9] and not any(M[p, 9:]) for p in (0, 3, 4, 5))
        datas = [dsym(t, lb) for t, lb in conds[l]]
        for p in range(nco[l]):
            expr = sum(M[p, k] * datas[k] for k in range(len(datas)))
            e = sp.expand(expr.subs(sol))
            terms = [(e.coeff(fs), n) for n, fs in zip(fin_names, fin_syms)]
            # sanity: nothing left over
            rest = sp.expand(e - sum(c * fs for c, (nn, fs) in zip([t[0] for t in terms], zip(fin_names, fin_syms))))
            assert rest == 0, rest
            total_terms += sum(1 for c, _ in terms if c != 0)
            lines.append(f"  {arr}[{p}] = {dot_code(terms)};")
    lines.append(f"  /* {total_terms} non-zero map entries after the parity split */")
    lines.append("}")

    # ---- how far q_l may be from the centre average at a face point ----
    # q_l - u_5 is a sum over the stencil data; per group of data that the
    # symmetries exchange, the largest coefficient at any face point
    nodes = [-0.5, -0.2236067977499790, 0.2236067977499790, 0.5]

    def group(t, lb):
        dx, dy = lab_off(lb)
        if t == 0:
            return "UE" if dx == 0 or dy == 0 else "UC"
        return "M0" if dx == 0 and dy == 0 else ("ME" if dx == 0 or dy == 0 else "MC")
    lines.append("/* largest |coefficient| of a datum in q_l - u_5 at the face points (rounded up):")
    lines.append("   UE, UC: averages of the edge and corner neighbours minus u_5; M0, ME, MC:")
    lines.append("   first moments of the cell, its edge and its corner neighbours */")
    for l in (2, 3, 4):
        Mn = [[float(z) for z in row] for row in lsq_map_2d(nco[l], conds[l]).tolist()]
        big = dict(UE=0.0, UC=0.0, M0=0.0, ME=0.0, MC=0.0)
        for i, x in enumerate(nodes):
            for j, y in enumerate(nodes):
                if i not in (0, 3) and j not in (0, 3):
                    continue
                ev = [x ** a * y ** b for a, b in MON[:nco[l]]]
                for k, (t, lb) in enumerate(conds[l]):
                    if (t, lb) != (0, 5):
                        g = group(t, lb)
                        big[g] = max(big[g], abs(sum(e * Mn[p][k] for p, e in enumerate(ev))))
        for g, v in big.items():
            lines.append(f"#define MR_BND_Q{l}_{g} {v * 1.0001:.5f}")

    # ---- beta quadratic forms, blocks by parity class ----
    def gram2(kappa, n):
        G = sp.zeros(n, n)
        for ax in range(0, kappa + 1):
            for ay in range(0, kappa + 1 - ax):
                if ax + ay == 0:
                    continue
                for p in range(n):
                    a1, b1 = MON[p]
                    if a1 < ax or b1 < ay:
                        continue
                    for s in range(n):
                        a2, b2 = MON[s]
                        if a2 < ax or b2 < ay:
                            continue
                        G[p, s] += (sp.ff(a1, ax) * sp.ff(a2, ax) * sp.ff(b1, ay) * sp.ff(b2, ay)
                                    * mono_avg(a1 + a2 - 2 * ax, 0) * mono_avg(b1 + b2 - 2 * ay, 0))
        return G
    for kappa, n, nm in ((2, 6, "mr2_beta_k2"), (3, 10, "mr2_beta_k3"), (5, 21, "mr2_beta_k5")):
        G = Bi[:n, :n].T * gram2(kappa, n) * Bi[:n, :n]
        lines.append(f"MR_DEV inline double {nm}(const double c[{n}]) {{")
        lines.append("  double b = 0.0, part;")
        for cls in ((0, 0, 0), (0, 0, 1), (1, 0, 0), (0, 1, 0), (1, 1, 0)):
            idx = [p for p in range(1, n) if zcls[p] == cls]
            # check block structure
            for p in idx:
                for s in range(1, n):
                    if s not in idx:
                        assert G[p, s] == 0
            if not idx:
                continue
            quad_form_code(nm, G, idx, "c", lines, "part")
            lines.append("  b += part;")
        lines.append("  return b;")
        lines.append("}")

    # ---- evaluation at the 4x4 Gauss-Lobatto grid ----
    # nodes X = -1, -sigma, sigma, 1 with sigma = 1/sqrt(5), t = sigma^2 = 1/5
    t, sg = R(1, 5), 1 / sp.sqrt(5)
    T, S = lit(t), lit(sg)
    E = []
    # even-even class at (|X|, |Y|) = (1, 1), (1, s), (s, 1), (s, s)
    E += ["h = c[10] + c[12]", "e00 = c[0] + (c[3] + h)", f"e11 = c[0] + {T} * (c[3] + {T} * h)",
          f"em = c[0] + {lit((1 + t) / 2)} * c[3] + {lit((1 + t * t) / 2)} * c[10] + {T} * c[12]",
          "ed = c[5] + c[14]", "e01 = em + ed", "e10 = em - ed"]
    # odd classes without the factors X, Y, X Y: x<i><j> at |X|_i, |Y|_j
    for n_, (k1, k3, k12, k5, k32, k14) in (("x", (1, 6, 8, 15, 17, 19)), ("y", (2, 9, 7, 20, 18, 16))):
        E += [f"{n_}a = c[{k1}] + c[{k3}] + c[{k5}]", f"{n_}b = c[{k1}] + {T} * (c[{k3}] + {T} * c[{k5}])",
              f"{n_}c = c[{k12}] + c[{k32}]", f"{n_}d = c[{k12}] + {T} * c[{k32}]"]
        # own axis at 1 / s (first index), the other axis at 1 / s (second)
        E += [f"{n_}00 = {n_}a + ({n_}c + c[{k14}])", f"{n_}01 = {n_}a + {T} * ({n_}c + {T} * c[{k14}])",
              f"{n_}10 = {n_}b + ({n_}d + c[{k14}])", f"{n_}11 = {n_}b + {T} * ({n_}d + {T} * c[{k14}])"]
    E += ["g = c[11] + c[13]", "r00 = c[4] + g", f"r11 = c[4] + {T} * g", f"r01 = c[4] + c[11] + {T} * c[13]",
          f"r10 = c[4] + c[13] + {T} * c[11]"]
    lines.append("/* values of the polynomial (2D basis above; half the sum of the entries times")
    lines.append("   the monomials in X, Y: the factor 1/2 belongs to the caller's weights) at")
    lines.append("   (xi_k, eta_l), out[k + 4 l], xi, eta in {-1/2, -sqrt(5)/10, sqrt(5)/10, 1/2} */")
    lines.append("MR_DEV inline void mr2_eval(const double c[21], double out[16]) {")
    for e in E:
        lines.append(f"  const double {e};")
    O = []
    for ix in (0, 1):
        for iy in (0, 1):
            q, x, y, r = f"e{ix}{iy}", f"x{ix}{iy}", f"y{iy}{ix}", f"r{ix}{iy}"
            f = {(0, 0): "1", (0, 1): S, (1, 0): S, (1, 1): T}[(ix, iy)]
            if f == "1":
                O += [f"s1_{ix}{iy} = {q} + {r}", f"d1_{ix}{iy} = {q} - {r}"]
            else:
                O += [f"s1_{ix}{iy} = fma({f}, {r}, {q})", f"d1_{ix}{iy} = fma(-{f}, {r}, {q})"]
            if ix == iy:
                O += [f"s2_{ix}{iy} = {x} + {y}", f"d2_{ix}{iy} = {x} - {y}"]
            elif iy == 1:
                O += [f"s2_{ix}{iy} = fma({S}, {y}, {x})", f"d2_{ix}{iy} = fma(-{S}, {y}, {x})"]
            else:
                O += [f"s2_{ix}{iy} = fma({S}, {x}, {y})", f"d2_{ix}{iy} = fma({S}, {x}, -{y})"]
            kp, km = (3, 0) if ix == 0 else (2, 1)
            lp, lm = (3, 0) if iy == 0 else (2, 1)
            w = "" if ix == 0 or iy == 0 else S
            for k, l, a, sgn, b in ((km, lm, "s1", "-", "s2"), (kp, lm, "d1", "+", "d2"), (km, lp, "d1", "-", "d2"),
                                    (kp, lp, "s1", "+", "s2")):
                if w:
                    O += [f"out[{k + 4 * l}] = fma({'-' if sgn == '-' else ''}{w}, {b}_{ix}{iy}, {a}_{ix}{iy})"]
                else:
                    O += [f"out[{k + 4 * l}] = {a}_{ix}{iy} {sgn} {b}_{ix}{iy}"]
    for o in O:
        lines.append(f"  {'' if o.startswith('out') else 'const double '}{o};")
    lines.append("}")
    check_eval(E, O, B)


def check_eval(E, O, B):
    """The emitted evaluation statements against the monomials (60 digits)."""
    ns = {"MR_KT": lambda i: sp.Float(_KTAB[i], 60), "fma": lambda a, b, c: a * b + c, "c": [], "out": [None] * 16}
    coef = [sp.Rational(3 * p * p - 7 * p + 5, 11 + p) for p in range(21)]
    ns["c"] = list(B * sp.Matrix(coef))
    for st in E + O:
        name, ex = st.split(" = ", 1)
        ex = re.sub(r"-?0x1\.[0-9a-f]+p[+-][0-9]+", lambda m: repr(float.fromhex(m.group(0))), ex)
        if name.startswith("out["):
            ns["out"][int(name[4:-1])] = eval(ex, {}, ns)
        else:
            ns[name] = eval(ex, {}, ns)
    nd = [-R(1, 2), -sp.sqrt(5) / 10, sp.sqrt(5) / 10, R(1, 2)]
    for l in range(4):
        for k in range(4):
            want = sum(c * nd[k] ** a * nd[l] ** b for c, (a, b) in zip(coef, MON))
            assert abs(sp.N(ns["out"][k + 4 * l] / 2 - want, 40)) < 1e-13, (k, l)


def emit_mod(lines):
    """Step 2.2, eqs. (p0)/(vi): first moment of the quartic p_0."""
    c = sp.symbols("p0:5")
    conds = [(0, -1), (0, 0), (0, 1), (1, -1), (1, 1)]
    A = sp.Matrix([[mono_avg(p, d) if t == 0 else mono_mom(p, d) for p in range(5)] for t, d in conds])
    um, u0, up, vm, vp = sp.symbols("um u0 up vm vp")
    sol = A.LUsolve(sp.Matrix([um, u0, up, vm, vp]))
    vnew = sp.expand(sum(sol[p] * mono_mom(p, 0) for p in range(5)))
    cu = vnew.coeff(up)
    cv = vnew.coeff(vm)
    assert vnew.coeff(um) == -cu and vnew.coeff(vp) == cv and vnew.coeff(u0) == 0
    lines.append(f"/* modified first moment: {cu} (u_+ - u_-) + ({cv}) (v_- + v_+) */")
    lines.append("MR_DEV inline double mr_modified_moment(double um, double up, double vm, double vp) {")
    lines.append(f"  return {lit(cu)} * (up - um) + {lit(cv)} * (vm + vp);")
    lines.append("}")


def main():
    body = []
    emit_mod(body)
    emit_1d(body)
    emit_2d(body)
    lines = ["/* Generated by gen_recon.py -- do not edit. */",
             "#pragma once",
             "#ifndef MR_DEV",
             "#define MR_DEV __host__ __device__ __attribute__((always_inline))",
             "#endif",
             f"#define MR_NKT {len(_KTAB)}",
             "/* constants the instructions cannot encode; MR_KT(i) reads entry i",
             "   (the including file defines MR_KT and the table storage) */",
             "#define MR_KT_VALUES \\"]
    for k in range(0, len(_KTAB), 4):
        lines.append("  " + ", ".join(v.hex() for v in _KTAB[k:k + 4]) + ", \\")
    lines.append("  0.0")
    lines.append("MR_KT_DECLARE")
    lines.append("")
    lines.extend(body)
    sys.stdout.write("\n".join(lines) + "\n")


if __name__ == "__main__":
    main()
