#!/usr/bin/env python3
"""Emit expansions_gen.h: straight-line Cartesian expansion code for p = 0..4.

Build step of the HIP library (run by the package build; the output is also
committed).  For each order P it writes a specialisation of
``sfmm::Exp<P>`` with these device functions, fully unrolled so every
coefficient lives in a register:

  p2m_add  Q_a += m b^a / a!                      (Sect. 2.1, Eq. massmom)
  m2m_add  Q_a += sum_{b<=a} Qc_b g^(a-b)/(a-b)!  (Appendix A.1, Eq. massmomtrans)
  m2l_add  local += M2L(r = s_src - s_tgt, Q)     (Sect. 2.2, Eq. dmkdeffmm; M_k)
  m2l_h    the same M2L in reduced components, and what goes with it (below)
  l2l      local re-centred by h                  (Appendix A.2, Eq. gravmtranslat)
  l2p      field and potential polynomials at a  (Sect. 2.2)

Notation: multi-indices a = (ax, ay, az) in graded order (degree, then ax
descending, then ay descending); Q~_a = sum m b^a / a!; D_a = d^a (1/|r|).
The local expansion of a node holds
  H_g = (-1)^(|g|+1) sum_{|a| <= P+1-|g|} D_(a+g) Q~_a   for 1 <= |g| <= P+1
  P_b = (-1)^|b|     sum_{|a| <= P-|b|}   D_(a+b) Q~_a   for |b| <= P
stored as local[0 .. NH-2] = H (slots 1..NH-1) followed by local[NH-1 ..] = P.
The field at offset a from the centre is F_c = sum_b H_(b+e_c) a^b/b! and the
potential sum_b P_b a^b/b!; the caller multiplies both by -G.

The reduced form (the shared far field in FP64).  1/|r| is harmonic, so every
degree of D is trace-free, D_(g+2x) + D_(g+2y) + D_(g+2z) = 0, and so are the
sums over a whole degree of Q~ that make up a local expansion.  A degree n has
2n + 1 independent components, here those with z exponent 0 or 1:
  reduce   Qr from Q~: a moment with z exponent >= 2 is taken off its two
           partners, Qr_(a-2z+2x) -= Q~_a and Qr_(a-2z+2y) -= Q~_a
  m2l_h    S_g += sum_{|a| <= P-|g|} D_(a+g) Qr_a    for |g| <= P
           X_g += sum_{|a| = P+1-|g|} D_(a+g) Qr_a   for 1 <= |g| <= P+1
           over the independent components of g and a
  expand   H_g = (-1)^(|g|+1) (S_g + X_g), P_g = (-1)^|g| S_g, the other
           components from the traces
At P = 3 that is 146 multiply-adds and 40 sums a node pair where the full
components take 175, 54 additions and 54 sums.  m2l_h takes D from
  R^m_0 = (-1)^m (2m-1)!! / r,  D_a = R^0_a,
  R^m_(a+e) = (r_e / r^2) R^(m+1)_a + (a_e / r^2) R^(m+1)_(a-e),
one multiply-add or two a component, instead of the recurrence in |r|^2.  A
component R^m_a is of the size of r^-(|a|+1): nothing leaves the range of FP64
before D does (with the powers of 1/r^2 in R instead, r^-(2P+3) did, at P = 4
for |r| beyond 1e28).
With ok false m2l_h and m2l_add_f32 add nothing (1/r = 0, so every D is 0), nor
does m2l_h where |r|^2 overflows (1/r from the hardware's estimate would be NaN): a
lane without an entry then needs no branch, behind which the compiler would
hold every sum twice.

D_a otherwise comes from the Laplace-kernel recurrence written for D itself:
  n |r|^2 D_a = -(2n-1) sum_c a_c r_c D_(a-e_c) - (n-1) sum_c a_c (a_c-1) D_(a-2e_c).
For |g| <= P the potential sum of P_g is a prefix of the field sum of H_g, so
both come out of one pass over a.
"""
import math
import os
import sys

PMAX = 4
# multiply-adds between two scheduling barriers of m2l_h
SCHED_EVERY = 12


def multi(n_max):
    out = []
    for n in range(n_max + 1):
        for a in range(n, -1, -1):
            for b in range(n - a, -1, -1):
                out.append((a, b, n - a - b))
    return out


def ncoef(p):
    return (p + 1) * (p + 2) * (p + 3) // 6


def fac(a):
    return math.factorial(a[0]) * math.factorial(a[1]) * math.factorial(a[2])


def add(a, b):
    return (a[0] + b[0], a[1] + b[1], a[2] + b[2])


def sub(a, b):
    return (a[0] - b[0], a[1] - b[1], a[2] - b[2])


def lit(v):
    r = repr(float(v))
    return r


class Counter:
    def __init__(self):
        self.fma = 0
        self.mul = 0
        self.add = 0

    def flops(self):
        return 2 * self.fma + self.mul + self.add


def monomial_code(name, vec, deg, idx, lines, cnt, over_fact=True):
    """name[k] = vec^a / a! (or vec^a) for |a| <= deg, in graded order."""
    ms = multi(deg)
    lines.append(f"    double {name}[{len(ms)}];")
    lines.append(f"    {name}[0] = 1.0;")
    for k, a in enumerate(ms[1:], start=1):
        # build from the predecessor with the first positive component lowered
        c = 0 if a[0] > 0 else (1 if a[1] > 0 else 2)
        prev = list(a); prev[c] -= 1
        pk = idx[tuple(prev)]
        if over_fact and a[c] > 1:
            lines.append(f"    {name}[{k}] = {name}[{pk}] * ({vec}[{c}] * {lit(1.0 / a[c])});")
            cnt.mul += 2
        else:
            lines.append(f"    {name}[{k}] = {name}[{pk}] * {vec}[{c}];")
            cnt.mul += 1


def reduced(n_max, n_min=0):
    """The independent components, graded order: z exponent 0 or 1."""
    return [a for a in multi(n_max) if a[2] <= 1 and sum(a) >= n_min]


def gen_reduced(P):
    """reduce, m2l_h and expand (see the docstring)."""
    ms = multi(P + 1)
    idx = {a: k for k, a in enumerate(ms)}
    NH, NQ = ncoef(P + 1), ncoef(P)
    rq = reduced(P)                 # moments and S
    rx = reduced(P + 1, 1)          # X
    qi = {a: k for k, a in enumerate(rq)}
    si = qi
    xi = {a: len(rq) + k for k, a in enumerate(rx)}
    out = [f"  static constexpr int NQR = {len(rq)};   // independent moments",
           f"  static constexpr int NLR = {len(rq) + len(rx)};  // S then X"]
    # reduce: from the largest z exponent down
    L = ["  __device__ __forceinline__ static void reduce(const double* Q, double* Qr) {"]
    var = {a: f"Q[{idx[a]}]" for a in multi(P)}
    terms = {a: [(1, a)] for a in multi(P)}  # kept: signed sums of full moments
    for a in sorted(multi(P), key=lambda t: -t[2]):
        if a[2] < 2:
            continue
        for e in ((2, 0, -2), (0, 2, -2)):
            b = add(a, e)
            terms[b] = terms[b] + [(-s, t) for s, t in terms[a]]
        terms[a] = []
    for a in rq:
        merged = {}
        for sg, t in terms[a]:
            merged[t] = merged.get(t, 0) + sg
        expr = ""
        for t, cf in merged.items():
            if cf == 0:
                continue
            body = var[t] if abs(cf) == 1 else f"{lit(abs(cf))} * {var[t]}"
            expr += (" + " if cf > 0 else " - ") + body if expr else ("" if cf > 0 else "-") + body
        L.append(f"    Qr[{qi[a]}] = {expr};")
    L.append("  }")
    out += L
    # m2l_h
    c = Counter()
    L = ["  __device__ __forceinline__ static void m2l_h(const double* r, const double* Qr, double* lr, bool ok) {",
         "    const double r2 = fma(r[0], r[0], fma(r[1], r[1], r[2] * r[2]));",
         "    const double ri = rsqrt_refined(r2);",
         "    const double rinv = ok && r2 < __builtin_inf() ? ri : 0.0;",
         "    const double s = rinv * rinv;",
         "    const double w[3] = {r[0] * s, r[1] * s, r[2] * s};",
         "    const double R0_000 = rinv;"]
    c.fma += 2; c.mul += 5
    f = 1
    for m in range(1, P + 2):
        f *= -(2 * m - 1)
        L.append(f"    const double R{m}_000 = {lit(f)} * rinv;")
        c.mul += 1
    done = {(m, (0, 0, 0)) for m in range(P + 2)}
    over = set()  # T = R / r^2

    def name(m, a):
        return f"R{m}_{a[0]}{a[1]}{a[2]}"

    def need(m, a):
        if (m, a) in done:
            return
        if m == 0 and a[2] >= 2:  # trace (z exponent 2)
            b1, b2 = add(a, (2, 0, -2)), add(a, (0, 2, -2))
            need(0, b1); need(0, b2)
            L.append(f"    const double {name(0, a)} = -({name(0, b1)} + {name(0, b2)});")
            c.add += 1
            done.add((m, a))
            return
        e = 2 if a[2] > 0 else (0 if a[0] >= a[1] else 1)
        b = list(a); b[e] -= 1; b = tuple(b)
        need(m + 1, b)
        if b[e] == 0:
            L.append(f"    const double {name(m, a)} = w[{e}] * {name(m + 1, b)};")
            c.mul += 1
        else:
            d = list(b); d[e] -= 1; d = tuple(d)
            need(m + 1, d)
            t = "T" + name(m + 1, d)[1:]
            if t not in over:
                L.append(f"    const double {t} = s * {name(m + 1, d)};")
                c.mul += 1
                over.add(t)
            if b[e] == 1:
                L.append(f"    const double {name(m, a)} = fma(w[{e}], {name(m + 1, b)}, {t});")
                c.fma += 1
            else:
                L.append(f"    const double {name(m, a)} = fma(w[{e}], {name(m + 1, b)}, {lit(b[e])} * {t});")
                c.fma += 1; c.mul += 1
        done.add((m, a))

    # one component of D after the other, each used as soon as it is known and
    # the compiler kept from moving code across every few of them: what is held
    # at once then fits three waves per SIMD at P = 3
    todo = 0
    for n in range(P + 2):
        for d in [t for t in ms if sum(t) == n and t[2] <= 2]:
            if todo >= SCHED_EVERY:
                L.append("    __builtin_amdgcn_sched_barrier(0);")
                todo = 0
            need(0, d)
            for g in reduced(P + 1):
                a = sub(d, g)
                if min(a) < 0 or a[2] > 1 or sum(a) > P:
                    continue
                k = si[g] if n <= P else xi[g]
                L.append(f"    lr[{k}] = fma({name(0, d)}, Qr[{qi[a]}], lr[{k}]);")
                c.fma += 1
                todo += 1
    L.append("  }")
    out += L
    out.append(f"  static constexpr int FLOPS_M2L_H = {c.flops()};  // + one refined rsqrt")
    # expand
    L = ["  __device__ __forceinline__ static void expand(const double* lr, double* local) {",
         f"    double t[{NH}];"]
    for which in ("P", "H"):
        for g in ms:
            ng = sum(g)
            if (which == "P" and ng > P) or (which == "H" and ng == 0):
                continue
            if g[2] <= 1:
                if which == "P":
                    v = f"lr[{si[g]}]"
                else:
                    v = f"lr[{xi[g]}]" if ng > P else f"(lr[{si[g]}] + lr[{xi[g]}])"
                sign = ng % 2 if which == "P" else (ng + 1) % 2
                L.append(f"    t[{idx[g]}] = {'-' if sign else ''}{v};")
            else:
                b1, b2 = add(g, (2, 0, -2)), add(g, (0, 2, -2))
                L.append(f"    t[{idx[g]}] = -(t[{idx[b1]}] + t[{idx[b2]}]);")
            L.append(f"    local[{(NH - 1 + idx[g]) if which == 'P' else idx[g] - 1}] = t[{idx[g]}];")
    L.append("  }")
    out += L
    return out


def gen(P):
    NQ = ncoef(P)
    NH = ncoef(P + 1)
    NL = (NH - 1) + NQ
    ms = multi(P + 1)
    idx = {a: k for k, a in enumerate(ms)}
    out = []
    out.append(f"template <> struct Exp<{P}> {{")
    out.append(f"  static constexpr int P = {P};")
    out.append(f"  static constexpr int NQ = {NQ};   // mass moments, |a| <= P")
    out.append(f"  static constexpr int NL = {NL};   // local coefficients: H then P")

    # ---- P2M
    c = Counter()
    L = []
    L.append("  __device__ __forceinline__ static void p2m_add(const double* b, double m, double* Q) {")
    monomial_code("mb", "b", P, idx, L, c)
    for k in range(NQ):
        L.append(f"    Q[{k}] = fma(m, mb[{k}], Q[{k}]);")
        c.fma += 1
    L.append("  }")
    out += L
    out.append(f"  static constexpr int FLOPS_P2M = {c.flops()};")

    # ---- M2M
    c = Counter()
    L = ["  __device__ __forceinline__ static void m2m_add(const double* g, const double* Qc, double* Q) {"]
    monomial_code("mg", "g", P, idx, L, c)
    mq = multi(P)
    for k, a in enumerate(mq):
        terms = []
        for kb, b in enumerate(mq):
            d = sub(a, b)
            if min(d) < 0:
                continue
            terms.append((kb, idx[d]))
        expr = f"Q[{k}]"
        for kb, kd in terms:
            if kd == 0:
                expr = f"({expr} + Qc[{kb}])"
                c.add += 1
            else:
                expr = f"fma(Qc[{kb}], mg[{kd}], {expr})"
                c.fma += 1
        L.append(f"    Q[{k}] = {expr};")
    L.append("  }")
    out += L
    out.append(f"  static constexpr int FLOPS_M2M = {c.flops()};")

    # ---- M2L
    c = Counter()
    L = ["  __device__ __forceinline__ static void m2l_add(const double* r, const double* Q, double* local) {"]
    L.append("    const double r2 = r[0] * r[0] + r[1] * r[1] + r[2] * r[2];")
    c.mul += 3; c.add += 2
    L.append("    const double rinv = rsqrt(r2);")
    L.append("    const double rinv2 = rinv * rinv;")
    c.mul += 1
    L.append(f"    double D[{NH}];")
    L.append("    D[0] = rinv;")
    for n in range(1, P + 2):
        L.append(f"    const double sn{n} = rinv2 * {lit(-1.0 / n)};")
        c.mul += 1
    for k, a in enumerate(ms[1:], start=1):
        n = sum(a)
        terms = []
        for cc in range(3):
            if a[cc] >= 1:
                b = list(a); b[cc] -= 1
                coef = (2 * n - 1) * a[cc]
                terms.append(f"{lit(coef)} * r[{cc}] * D[{idx[tuple(b)]}]")
                c.mul += 2
            if a[cc] >= 2:
                b = list(a); b[cc] -= 2
                coef = (n - 1) * a[cc] * (a[cc] - 1)
                terms.append(f"{lit(coef)} * D[{idx[tuple(b)]}]")
                c.mul += 1
        c.add += len(terms) - 1
        c.mul += 1
        L.append(f"    D[{k}] = ({' + '.join(terms)}) * sn{n};")
    # contractions
    for kg, g in enumerate(ms[1:], start=1):
        ng = sum(g)
        hslot = kg - 1
        # sum over a in graded order with |a| <= P+1-ng (a within mass-moment range)
        alist = [a for a in multi(P + 1 - ng)]
        acc = None
        lines_g = []
        first = True
        pdone = False
        for a in alist:
            na = sum(a)
            if ng <= P and not pdone and na > P - ng:
                # potential prefix complete
                lines_g.append(f"      local[{NH - 1 + kg}] {'+' if ng % 2 == 0 else '-'}= s;")
                c.add += 1
                pdone = True
            term_d = idx[add(a, g)]
            term_q = idx[a]
            if first:
                lines_g.append(f"      double s = D[{term_d}] * Q[{term_q}];")
                c.mul += 1
                first = False
            else:
                lines_g.append(f"      s = fma(D[{term_d}], Q[{term_q}], s);")
                c.fma += 1
        if ng <= P and not pdone:
            lines_g.append(f"      local[{NH - 1 + kg}] {'+' if ng % 2 == 0 else '-'}= s;")
            c.add += 1
        sign_h = '+' if (ng + 1) % 2 == 0 else '-'
        lines_g.append(f"      local[{hslot}] {sign_h}= s;")
        c.add += 1
        L.append("    {")
        L += lines_g
        L.append("    }")
    # P_0
    L.append("    {")
    first = True
    for a in multi(P):
        if first:
            L.append(f"      double s = D[{idx[a]}] * Q[{idx[a]}];")
            c.mul += 1
            first = False
        else:
            L.append(f"      s = fma(D[{idx[a]}], Q[{idx[a]}], s);")
            c.fma += 1
    L.append(f"      local[{NH - 1}] += s;")
    c.add += 1
    L.append("    }")
    L.append("  }")
    out += L
    out.append(f"  static constexpr int FLOPS_M2L = {c.flops()};  // + one rsqrt")
    # same contraction in FP32 (r and Q rounded to FP32), each term added to
    # the FP64 local expansion
    Lm = []
    for line in L:
        line = line.replace("static void m2l_add(const double* r, const double* Q, double* local)",
                            "static void m2l_add_f32(const float* r, const float* Q, double* local, bool ok = true)")
        if line == "    {":  # (bounds the registers: two waves per SIMD)
            Lm.append("    __builtin_amdgcn_sched_barrier(0);")
        line = line.replace("const double ", "const float ").replace("double D[", "float D[")
        line = line.replace("double s = ", "float s = ")
        line = line.replace("rsqrt(r2)", "ok ? __frsqrt_rn(r2) : 0.0f")
        line = line.replace("fma(", "fmaf(")
        import re as _re
        line = _re.sub(r"(-?\d+\.\d+(e-?\d+)?)", r"\1f", line) if ("D[" in line and "=" in line and "local" not in line) or "sn" in line else line
        line = line.replace("local[", "local[").replace("] += s;", "] += (double)s;").replace("] -= s;", "] -= (double)s;")
        Lm.append(line)
    out += Lm

    # ---- the reduced form
    out += gen_reduced(P)

    # ---- M2L of one node pair in both directions (the one-sided symmetric
    # form): D(r) once for r = s_S - s_T; the target side as m2l_add; the
    # source side with D(-r) = (-1)^|k| D(r): with QTs the target's moments
    # with odd degrees negated (the caller's), H_g -= s and P_b += s, added to
    # outS atomically
    c = Counter()
    L = ["  __device__ __forceinline__ static void m2l_pair(const double* r, const double* QS,",
         "                                                    const double* QTs, double* local,",
         "                                                    double* outS) {"]
    body = []
    capture = False
    for line in out[out.index("  __device__ __forceinline__ static void m2l_add(const double* r, const double* Q, double* local) {") + 1:]:
        if line.startswith("    {") and not capture:
            capture = True
        if capture:
            break
        body.append(line)
    L += body  # r2, rinv, D recurrence
    # flops of the derivative part, from the same counts as m2l_add
    c.mul += 4; c.add += 2
    for k, a in enumerate(ms[1:], start=1):
        n = sum(a)
        nt = sum(1 for cc in range(3) if a[cc] >= 1) + sum(1 for cc in range(3) if a[cc] >= 2)
        c.mul += 2 * sum(1 for cc in range(3) if a[cc] >= 1) + sum(1 for cc in range(3) if a[cc] >= 2) + 1
        c.add += nt - 1
    c.mul += P + 1
    for side in ("T", "S"):
        Q = "QS" if side == "T" else "QTs"
        for kg, g in enumerate(ms[1:], start=1):
            ng = sum(g)
            hslot = kg - 1
            alist = [a for a in multi(P + 1 - ng)]
            lines_g = []
            first = True
            pdone = False
            def put(slot, sign):
                if side == "T":
                    return f"      local[{slot}] {sign}= s;"
                return f"      unsafeAtomicAdd(&outS[{slot}], {'-' if sign == '-' else ''}s);"
            for a in alist:
                na = sum(a)
                if ng <= P and not pdone and na > P - ng:
                    lines_g.append(put(NH - 1 + kg, ('+' if ng % 2 == 0 else '-') if side == "T" else '+'))
                    c.add += 1
                    pdone = True
                if first:
                    lines_g.append(f"      double s = D[{idx[add(a, g)]}] * {Q}[{idx[a]}];")
                    c.mul += 1
                    first = False
                else:
                    lines_g.append(f"      s = fma(D[{idx[add(a, g)]}], {Q}[{idx[a]}], s);")
                    c.fma += 1
            if ng <= P and not pdone:
                lines_g.append(put(NH - 1 + kg, ('+' if ng % 2 == 0 else '-') if side == "T" else '+'))
                c.add += 1
            lines_g.append(put(hslot, ('+' if (ng + 1) % 2 == 0 else '-') if side == "T" else '-'))
            c.add += 1
            L.append("    {")
            L += lines_g
            L.append("    }")
        L.append("    {")
        first = True
        for a in multi(P):
            if first:
                L.append(f"      double s = D[{idx[a]}] * {Q}[{idx[a]}];")
                c.mul += 1
                first = False
            else:
                L.append(f"      s = fma(D[{idx[a]}], {Q}[{idx[a]}], s);")
                c.fma += 1
        L.append(f"      local[{NH - 1}] += s;" if side == "T" else f"      unsafeAtomicAdd(&outS[{NH - 1}], s);")
        c.add += 1
        L.append("    }")
    L.append("  }")
    out += L
    out.append(f"  static constexpr int FLOPS_M2L_PAIR = {c.flops()};  // both directions, + one rsqrt")

    # ---- L2L (in place)
    c = Counter()
    L = ["  __device__ __forceinline__ static void l2l(const double* h, double* local) {"]
    monomial_code("mh", "h", P, idx, L, c)
    for kg, g in enumerate(ms[1:], start=1):
        ng = sum(g)
        expr = f"local[{kg - 1}]"
        for kd, d in enumerate(multi(P + 1 - ng)):
            if kd == 0:
                continue
            e = add(g, d)
            expr = f"fma(local[{idx[e] - 1}], mh[{kd}], {expr})"
            c.fma += 1
        L.append(f"    local[{kg - 1}] = {expr};")
    for kb, b in enumerate(multi(P)):
        nb = sum(b)
        expr = f"local[{NH - 1 + kb}]"
        for kd, d in enumerate(multi(P - nb)):
            if kd == 0:
                continue
            e = add(b, d)
            expr = f"fma(local[{NH - 1 + idx[e]}], mh[{kd}], {expr})"
            c.fma += 1
        L.append(f"    local[{NH - 1 + kb}] = {expr};")
    L.append("  }")
    out += L
    out.append(f"  static constexpr int FLOPS_L2L = {c.flops()};")

    # ---- L2P
    c = Counter()
    L = ["  __device__ __forceinline__ static void l2p(const double* a, const double* local, double* f, double& phi) {"]
    monomial_code("ma", "a", P, idx, L, c)
    for cc in range(3):
        e = [0, 0, 0]; e[cc] = 1
        expr = None
        for kb, b in enumerate(multi(P)):
            hk = idx[add(b, tuple(e))] - 1
            if expr is None:
                expr = f"local[{hk}]"
            else:
                expr = f"fma(local[{hk}], ma[{kb}], {expr})"
                c.fma += 1
        L.append(f"    f[{cc}] += {expr};")
        c.add += 1
    expr = None
    for kb, b in enumerate(multi(P)):
        if expr is None:
            expr = f"local[{NH - 1}]"
        else:
            expr = f"fma(local[{NH - 1 + kb}], ma[{kb}], {expr})"
            c.fma += 1
    L.append(f"    phi += {expr};")
    c.add += 1
    L.append("  }")
    out += L
    out.append(f"  static constexpr int FLOPS_L2P = {c.flops()};")
    out.append("};")
    return "\n".join(out)


def main(path):
    parts = [
        "// Generated by gen_expansions.py -- do not edit.",
        "// Cartesian expansion kernels for orders 0..%d (see the generator's docstring)." % PMAX,
        "#pragma once",
        "#include \"softening.h\"",
        "namespace sfmm {",
        "template <int P> struct Exp;",
    ]
    for P in range(PMAX + 1):
        parts.append(gen(P))
    parts.append("}  // namespace sfmm")
    text = "\n".join(parts) + "\n"
    old = open(path).read() if os.path.exists(path) else None
    if old != text:
        with open(path, "w") as f:
            f.write(text)


if __name__ == "__main__":
    main(sys.argv[1] if len(sys.argv) > 1 else
         os.path.join(os.path.dirname(os.path.abspath(__file__)), "expansions_gen.h"))
