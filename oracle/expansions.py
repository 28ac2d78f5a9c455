"""The truncated FMM sums of a given tree in extended precision -- TEST INFRASTRUCTURE ONLY.

Only the tests may import this module.  It shares no code with the GPU
library.  For a quad-tree (numpy arrays as oracle.tree gives them) it evaluates
what the FMM of order p stands for, truncation included, so that a comparison
shows the kernels' own errors:

  * outside a box with centre c and w = (x - c)/alpha = rho e^{i theta}:
    phi(x) = sum_{|n| <= p} M_n K_n(rho) e^{i n theta}, where a charge q at w
    gives M_n = q I_n(rho) e^{-i n theta} and a dipole D = d (n_x + i n_y) its
    derivative, (conj(D) F_{n-1} + D F_{n+1})/(2 alpha) with F_n = I_n(rho)
    e^{-i n theta};
  * inside: phi(x) = sum_{|m| <= p} L_m I_m(rho) e^{i m theta}, L_m = q K_m(rho)
    e^{-i m theta} for a charge, -(conj(D) G_{m-1} + D G_{m+1})/(2 alpha) with
    G_m = K_m(rho) e^{-i m theta} for a dipole;
  * the shifts by e: M'_k = sum_n M_n I_{k-n}(|e|) e^{-i (k-n) phi} to the parent,
    L'_k = sum_m L_m I_{m-k}(|e|) e^{i (m-k) phi} to a child, and from source to
    target centre, d apart, L_m = (-1)^m sum_n M_n K_{n-m}(|d|) e^{i (n-m) phi}
    (Graf's addition theorem), all sums over |n|, |m| <= p.

Beside each value stands the sum of the absolute values of what enters it, from
which a bound on rounding errors is a multiple.
"""
from __future__ import annotations

import numpy as np

from .tree import compact

LD = np.longdouble
CLD = np.clongdouble
R2 = np.sqrt(LD(2))


def bessel_i(x, nmax):
    """I_0 .. I_nmax, [nmax + 1, ...]: two series, then the recurrence downwards."""
    x = np.asarray(x, dtype=LD)
    y = x * x / 4
    F = np.empty((nmax + 1,) + x.shape, dtype=LD)   # I_n n! / (x/2)^n
    terms = 40 + int(2 * np.max(x, initial=0))
    for n in (nmax, nmax - 1) if nmax > 0 else (0,):
        t = np.ones_like(x)
        s = t.copy()
        for k in range(1, terms):
            t = t * y / (LD(k) * (n + k))
            s += t
        F[n] = s
    for n in range(nmax - 1, 0, -1):
        F[n - 1] = F[n] + y / (LD(n) * (n + 1)) * F[n + 1]
    f = np.ones_like(x)
    for n in range(nmax + 1):
        F[n] *= f
        f = f * x / (2 * LD(n + 1))
    return F


def bessel_k01(x):
    """K_0, K_1 by the trapezoidal rule for int_0^inf exp(-x cosh t) cosh(nu t) dt.
    The integrand is analytic in |Im t| < pi/2 and there at most e^{x (1 - cos Im
    t)} times its values on the axis, so that the rule's relative error at spacing
    h is about exp(-pi^2 / h), or exp(-2 pi^2 / (x h^2)) for large x."""
    x = np.asarray(x, dtype=LD)
    if x.size == 0:
        return x, x
    h = LD(min(0.15, 0.6 / np.sqrt(float(np.max(x)))))
    k0, k1 = 0.5 * np.ones_like(x), 0.5 * np.ones_like(x)   # (times exp(-x))
    top = float(np.arccosh(1 + 60 / float(np.min(x))))
    for j in range(1, int(top / float(h)) + 2):
        c = np.cosh(j * h)
        e = np.exp(-x * (c - 1))
        k0 += e
        k1 += e * c
    s = h * np.exp(-x)
    return k0 * s, k1 * s


def bessel_k(x, nmax):
    """K_0 .. K_nmax, the recurrence upwards."""
    x = np.asarray(x, dtype=LD)
    K = np.empty((max(nmax, 1) + 1,) + x.shape, dtype=LD)
    K[0], K[1] = bessel_k01(x)
    for n in range(1, nmax):
        K[n + 1] = K[n - 1] + 2 * n / x * K[n]
    return K[:nmax + 1]


def _waves(theta, nmax, sign):
    """e^{sign i n theta}, n = 0 .. nmax."""
    n = np.arange(nmax + 1, dtype=LD).reshape((-1,) + (1,) * np.ndim(theta))
    return np.cos(n * theta) + sign * 1j * np.sin(n * theta)


def _full(a):
    """Coefficients -p .. p of a real field from 0 .. p."""
    return np.concatenate([np.conj(a[:0:-1]), a])


class Sums:
    """tree: dict with square, leaf_level, lmin, level_begin, box_code, parent, leaf_range, perm, ulist_off, ulist,
    vlist; for an adaptive one also leaf_box, box_level and the W and X lists.  Charges q at xy (set 0), dipoles d at
    bxy with normals nrm (set 1)."""

    def __init__(self, tree, alpha, p, xy, q, bxy=None, nrm=None, d=None):
        self.t, self.alpha, self.p = tree, LD(alpha), p
        n0 = len(xy)
        n1 = 0 if bxy is None else len(bxy)
        perm = np.asarray(tree["perm"], dtype=np.int64)
        self.n0 = n0
        self.xy = np.concatenate([np.asarray(xy)[perm[:n0]]] + ([np.asarray(bxy)[perm[n0:n0 + n1]]] if n1 else [])).astype(LD)
        self.q = np.zeros(n0 + n1, dtype=LD)
        self.q[:n0] = np.asarray(q)[perm[:n0]]
        self.D = np.zeros(n0 + n1, dtype=CLD)
        if n1:
            nr = np.asarray(nrm)[perm[n0:n0 + n1]].astype(LD)
            self.D[n0:] = np.asarray(d)[perm[n0:n0 + n1]].astype(LD) * (nr[:, 0] + 1j * nr[:, 1])
        nb = len(tree["box_code"])
        self.adaptive = "leaf_box" in tree
        lb = np.asarray(tree["level_begin"])
        self.level = (np.asarray(tree["box_level"]).astype(int) if self.adaptive
                      else np.repeat(np.arange(len(lb) - 1), np.diff(lb)))
        self.leaf_box = (np.asarray(tree["leaf_box"]) if self.adaptive else np.arange(lb[-2], lb[-1]))
        x0, y0, size = (LD(v) for v in tree["square"])
        code = np.asarray(tree["box_code"]).astype(np.uint64)
        self.side = size / LD(2) ** self.level.astype(LD)
        self.ix, self.iy = compact(code).astype(np.int64), compact(code >> np.uint64(1)).astype(np.int64)
        self.c = np.stack([x0 + (self.ix + LD(0.5)) * self.side, y0 + (self.iy + LD(0.5)) * self.side], 1)
        # roundings of a position, in sides: the coordinates' size over the box's
        self.pos = (size + max(abs(x0), abs(y0))) / self.side
        par = np.asarray(tree["parent"])
        lmin = tree["lmin"]
        # leaf multipoles, their absolute sums, then the shifts upwards
        self.M = np.zeros((nb, p + 1), dtype=CLD)
        self.Q = np.zeros((nb, 2), dtype=LD)   # sums of |q| and of |d|
        lr = np.asarray(tree["leaf_range"])
        rank = np.full(len(self.xy), -1)
        for k in range(len(self.leaf_box)):
            for s in (0, 1):
                rank[lr[k, 2 * s]:lr[k, 2 * s + 1]] = k
        self.leaf_of = rank
        box = self.leaf_box[rank]
        self._p2m(box)
        np.add.at(self.Q[:, 0], box, np.abs(self.q))
        np.add.at(self.Q[:, 1], box, np.abs(self.D))
        for l in range(int(self.level.max()), 0, -1):
            for b in np.flatnonzero(self.level == l):
                self.Q[par[b]] += self.Q[b]
            if l <= lmin:
                continue
            for pos in range(4):
                ch = np.flatnonzero((self.level == l) & ((self.ix & 1) + 2 * (self.iy & 1) == pos))
                if len(ch) == 0:
                    continue
                e = (self.c[ch[0]] - self.c[par[ch[0]]]) / self.alpha
                S = self._shift(e, -1)
                full = np.concatenate([np.conj(self.M[ch][:, :0:-1]), self.M[ch]], 1)
                self.M[par[ch]] += full @ S.T
        self.vl, self.ops = np.asarray(tree["vlist"]), {}
        self.at = {(int(l), int(i), int(j)): b for b, (l, i, j) in enumerate(zip(self.level, self.ix, self.iy))}

    def _shift(self, e, sign):
        """[k][n] = I_{k-n}(|e|) e^{sign i (k-n) phi}, k = 0 .. p, n = -p .. p (parents for sign -1; the conjugate
        index difference, m - k, for +1)."""
        p = self.p
        I = bessel_i(np.hypot(e[0], e[1]), 2 * p)
        w = _waves(np.arctan2(e[1], e[0]), 2 * p, 1)
        k, n = np.arange(p + 1)[:, None], np.arange(-p, p + 1)[None, :]
        m = k - n if sign < 0 else n - k
        v = I[abs(m)] * np.where(m >= 0, w[abs(m)], np.conj(w[abs(m)]))
        return np.conj(v) if sign < 0 else v

    def _p2m(self, box):
        p = self.p
        step = 20000
        for a in range(0, len(self.xy), step):
            s = slice(a, a + step)
            w = (self.xy[s] - self.c[box[s]]) / self.alpha
            F = bessel_i(np.hypot(w[:, 0], w[:, 1]), p + 1) * _waves(np.arctan2(w[:, 1], w[:, 0]), p + 1, -1)
            lo = np.concatenate([np.conj(F[1:2]), F[:p]])   # F_{n-1}, n = 0 .. p
            m = self.q[s] * F[:p + 1] + (np.conj(self.D[s]) * lo + self.D[s] * F[1:]) / (2 * self.alpha)
            np.add.at(self.M, box[s], m.T)

    def _sources(self, leaves):
        lr = np.asarray(self.t["leaf_range"])
        return np.concatenate([np.arange(lr[k, 2 * s], lr[k, 2 * s + 1]) for k in leaves for s in (0, 1)]).astype(np.int64)

    def _direct(self, x, src):
        """Sum over the sources at point x (coincident ones skipped) and its absolute value."""
        dx = x - self.xy[src]
        r = np.hypot(dx[:, 0], dx[:, 1])
        keep = r > 0
        dx, r, src = dx[keep], r[keep], src[keep]
        if len(r) == 0:
            return LD(0), LD(0)
        K0, K1 = bessel_k01(r / self.alpha)
        D = self.D[src]
        v = self.q[src] * K0 + (D.real * dx[:, 0] + D.imag * dx[:, 1]) * K1 / (self.alpha * r)
        return np.sum(v), np.sum(np.abs(self.q[src]) * K0 + np.abs(D) * K1 / self.alpha)

    def _point_sum(self, q, d, rho):
        """Absolute value of an expansion's terms at argument rho (> 0): charges' and dipoles' sums times K_0, K_1."""
        K0, K1 = bessel_k01(rho)
        return q * K0 + d * K1 / self.alpha

    def at_sorted(self, j, group_side=4.0):
        """(value, sum of absolute values, the same weighted by what a rounding of a position changes) at sorted
        point j.  Levels of sides up to group_side alpha count the sources of all the box's siblings' V lists (their
        terms are mixed there)."""
        p, al, t = self.p, self.alpha, self.t
        x, leaf = self.xy[j], int(self.leaf_of[j])
        uo, ul = t["ulist_off"], t["ulist"]
        val, mag = self._direct(x, self._sources(ul[uo[leaf]:uo[leaf + 1]]))
        pos = LD(0)
        path, b = [], int(self.leaf_box[leaf])
        while b >= 0 and self.level[b] >= t["lmin"]:
            path.append(b)
            b = int(t["parent"][b])
        L = np.zeros(p + 1, dtype=CLD)
        xs = {int(b): k for k, b in enumerate(t["xbox"])} if self.adaptive else {}
        for b in reversed(path):
            l, s = int(self.level[b]), self.side[b]
            par = int(t["parent"][b])
            if b != path[-1]:
                L = self._shift((self.c[b] - self.c[par]) / al, 1) @ _full(L)
            for src in self.vl[b]:
                if src >= 0:
                    L = L + self._m2l(l, b, src) @ _full(self.M[src])
            if s <= group_side * al:
                near = [self.at.get((l, 2 * (int(self.ix[par]) + i) + a, 2 * (int(self.iy[par]) + k) + c))
                        for i in (-1, 0, 1) for k in (-1, 0, 1) if (i, k) != (0, 0) for a in (0, 1) for c in (0, 1)]
            else:
                near = [int(v) for v in self.vl[b] if v >= 0]
            Q = sum((self.Q[v] for v in near if v is not None), np.zeros(2, dtype=LD))
            m = self._point_sum(Q[0], Q[1], (2 - R2) * s / al)
            mag += m
            pos += m * self.pos[b] * (1 + s / al)
            if b in xs:
                k = xs[b]
                src = self._sources(t["xlist"][t["xlist_off"][k]:t["xlist_off"][k + 1]])
                w = (self.xy[src] - self.c[b]) / al
                rho = np.hypot(w[:, 0], w[:, 1])
                G = bessel_k(rho, p + 1) * _waves(np.arctan2(w[:, 1], w[:, 0]), p + 1, -1)
                lo = np.concatenate([np.conj(G[1:2]), G[:p]])
                D = self.D[src]
                L = L + np.sum(self.q[src] * G[:p + 1] - (np.conj(D) * lo + D * G[1:]) / (2 * al), axis=1)
                m = np.sum(self._point_sum(np.abs(self.q[src]), np.abs(D), rho - s / (R2 * al)))
                mag += m
                pos += m * self.pos[b] * (1 + s / al)
        if path:
            w = (x - self.c[path[0]]) / al
            F = bessel_i(np.hypot(w[0], w[1]), p) * _waves(np.arctan2(w[1], w[0]), p, 1)
            val += np.real(L[0] * F[0] + 2 * np.sum(L[1:] * F[1:]))
        if self.adaptive:
            for b in t["wlist"][t["wlist_off"][leaf]:t["wlist_off"][leaf + 1]]:
                w = (x - self.c[b]) / al
                rho = np.hypot(w[0], w[1])
                F = bessel_k(rho, p) * _waves(np.arctan2(w[1], w[0]), p, 1)
                val += np.real(self.M[b][0] * F[0] + 2 * np.sum(self.M[b][1:] * F[1:]))
                s = self.side[b]
                m = self._point_sum(self.Q[b][0], self.Q[b][1], rho - s / (R2 * al))
                mag += m
                pos += m * self.pos[b] * (1 + s / al)
        two_pi = 2 * np.arccos(LD(-1))
        return val / two_pi, mag / two_pi, pos / two_pi

    def _m2l(self, l, b, src):
        p = self.p
        key = (l, int(self.ix[b] - self.ix[src]), int(self.iy[b] - self.iy[src]))
        if key not in self.ops:
            dv = np.array(key[1:], dtype=LD) * self.side[b] / self.alpha
            K = bessel_k(np.hypot(dv[0], dv[1]), 2 * p)
            w = _waves(np.arctan2(dv[1], dv[0]), 2 * p, 1)
            m, n = np.arange(p + 1)[:, None], np.arange(-p, p + 1)[None, :]
            k = n - m
            self.ops[key] = K[abs(k)] * np.where(k >= 0, w[abs(k)], np.conj(w[abs(k)])) * np.where(m % 2, -1, 1)
        return self.ops[key]
