"""Generate the Lobatto rules of the kernel tables' set-up sweep.

On one table interval (x in [-1, 1]) a function is held by its values at the K
Chebyshev-Lobatto nodes x_k = -cos(pi k / (K - 1)).  The sweep needs
    Q[k][m] = int_{-1}^{x_k} l_m(x) dx     (l_m the Lagrange basis),
whose last row holds the weights of the whole interval, and the FP64 tables
    A[n][k]: node values -> Chebyshev coefficients,
    T[n][j]: Chebyshev -> monomial coefficients (integers).
Everything is computed at 50 digits (mpmath).

    python paper_1910_12007_amd/csrc/gen_pbrule.py   # rewrites swim_pbrule.h
"""
import os

import mpmath as mp

HERE = os.path.dirname(os.path.abspath(__file__))
mp.mp.dps = 50


def nodes(K):
    return [-mp.cos(mp.pi * k / (K - 1)) for k in range(K)]


def lagrange(x, m):
    """Monomial coefficients (ascending) of the m-th Lagrange polynomial."""
    c = [mp.mpf(1)]
    for j, xj in enumerate(x):
        if j != m:
            d = x[m] - xj
            c = [(c[i - 1] if i else mp.mpf(0)) / d - (xj * c[i] / d if i < len(c) else 0) for i in range(len(c) + 1)]
    return c


def integral(c, a, b):
    return mp.fsum(ci * (b ** (i + 1) - a ** (i + 1)) / (i + 1) for i, ci in enumerate(c))


def cheb_monomials(n):
    T = [[1], [0, 1]]
    while len(T) <= n:
        a, b = T[-1], T[-2]
        T.append([(2 * a[j - 1] if j else 0) - (b[j] if j < len(b) else 0) for j in range(len(a) + 1)])
    return T[:n + 1]


def num(v):
    v = mp.nstr(v, 20) if abs(v) > mp.mpf(10) ** -40 else "0.0"
    return v if "." in v or "e" in v else v + ".0"


def array(name, rows):
    dims = "[%d]" % len(rows) if not isinstance(rows[0], list) else "[%d][%d]" % (len(rows), len(rows[0]))
    if not isinstance(rows[0], list):
        return "static constexpr double %s%s = {%s};" % (name, dims, ", ".join(num(v) for v in rows))
    body = ",\n    ".join("{%s}" % ", ".join(num(v) for v in r) for r in rows)
    return "static constexpr double %s%s = {\n    %s};" % (name, dims, body)


def main():
    out = ["// generated by gen_pbrule.py: Chebyshev-Lobatto rules of the kernel tables' sweep",
           "#pragma once", "", "namespace swim {"]
    for K in (7, 9):
        x = nodes(K)
        L = [lagrange(x, m) for m in range(K)]
        out.append("// xi = (1 + x) / 2 at the %d nodes; integrals from -1 to each node" % K)
        out.append(array("LOB%d_XI" % K, [(1 + v) / 2 for v in x]))
        out.append(array("LOB%d_Q" % K, [[integral(L[m], mp.mpf(-1), x[k]) for m in range(K)] for k in range(K)]))
    K, N = 9, 8
    A = [[mp.mpf(2) / N * (mp.mpf(1) / 2 if n in (0, N) else 1) * (mp.mpf(1) / 2 if k in (0, N) else 1) *
          mp.cos(n * mp.pi * (N - k) / N) for k in range(K)] for n in range(K)]
    T = [[mp.mpf(v) for v in r] + [mp.mpf(0)] * (K - len(r)) for r in cheb_monomials(N)]
    out.append("// node values -> Chebyshev coefficients; Chebyshev -> monomial")
    out.append(array("LOB9_A", A))
    out.append(array("LOB9_T", T))
    out.append("}  // namespace swim")
    with open(os.path.join(HERE, "swim_pbrule.h"), "w") as f:
        f.write("\n".join(out) + "\n")


if __name__ == "__main__":
    main()
