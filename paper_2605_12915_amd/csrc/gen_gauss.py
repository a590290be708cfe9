"""Generate af_gauss.h: Gauss-Legendre nodes and weights on [0, 1] for the quadrature
of the foot-centred exact update (32 points per angular piece), with cos(pi x) and
sin(pi x) of the nodes.

Nodes are the roots of the Legendre polynomial P_n, found by Newton's method in
40-digit arithmetic (mpmath) from the Chebyshev-like initial guesses
cos(pi (k - 1/4) / (n + 1/2)); weights 2 / ((1 - x^2) P_n'(x)^2); both mapped from
[-1, 1] to [0, 1] and rounded once to double.

    python gen_gauss.py            # rewrites af_gauss.h next to this file
"""
import os

import mpmath as mp

mp.mp.dps = 40


def legendre_and_derivative(n, x):
    p0, p1 = mp.mpf(1), x
    for k in range(2, n + 1):
        p0, p1 = p1, ((2 * k - 1) * x * p1 - (k - 1) * p0) / k
    dp = n * (x * p1 - p0) / (x * x - 1)
    return p1, dp


def rule(n):
    xs, ws = [], []
    for k in range(1, n + 1):
        x = mp.cos(mp.pi * (k - mp.mpf(1) / 4) / (n + mp.mpf(1) / 2))
        for _ in range(100):
            p, dp = legendre_and_derivative(n, x)
            dx = p / dp
            x -= dx
            if abs(dx) < mp.mpf(10) ** -38:
                break
        _, dp = legendre_and_derivative(n, x)
        xs.append((1 - x) / 2)                     # ascending on [0, 1]
        ws.append(1 / ((1 - x * x) * dp * dp))     # 2 / (...) halved by the map
    return xs, ws


def main():
    here = os.path.dirname(os.path.abspath(__file__))
    lines = ["// Generated by gen_gauss.py -- do not edit.",
             "// Gauss-Legendre nodes and weights on [0, 1] (ascending nodes; weights sum to 1).",
             "#pragma once", "namespace af {"]
    for n in (32,):
        xs, ws = rule(n)
        assert abs(sum(ws) - 1) < mp.mpf(10) ** -35
        lines.append(f"constexpr double kGaussW{n}[{n}] = {{")
        lines += [f"    {mp.nstr(w, 20, min_fixed=-1, max_fixed=1)}," for w in ws]
        lines.append("};")
        # cos and sin of pi x, the clustering map of an angular piece
        for name, f in (("Cos", lambda x: mp.cos(mp.pi * x)), ("Sin", lambda x: mp.sin(mp.pi * x))):
            lines.append(f"constexpr double kGauss{name}{n}[{n}] = {{")
            lines += [f"    {mp.nstr(f(x), 20, min_fixed=-1, max_fixed=1)}," for x in xs]
            lines.append("};")
    lines.append("}  // namespace af")
    text = "\n".join(lines) + "\n"
    path = os.path.join(here, "af_gauss.h")
    old = open(path).read() if os.path.exists(path) else None
    if old != text:
        with open(path, "w") as fh:
            fh.write(text)


if __name__ == "__main__":
    main()
