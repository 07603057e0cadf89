"""Generate screening.h: polynomial coefficients for erfcx on the P2P range.

The near-field kernel needs C(x) = erfc(x) + (2/sqrt(pi)) x e^{-x^2} for 0 <= x <= XMAX
(x = xi r < xi r_c).  Writing erfc(x) = e^{-x^2} erfcx(x), the library evaluates erfcx(x)
as a polynomial in t = (x - K)/(x + K) (the Moebius map of [0, inf) onto [-1, 1) used by
Weideman, SIAM J. Numer. Anal. 31 (1994), for the complex error function).  The polynomial is
the Chebyshev interpolant of erfcx in u, where u maps t in [-1, t(XMAX)] affinely onto
[-1, 1] (computed with mpmath at 50 digits and truncated to the printed degree).

FP64 kernels take it in the monomial basis of t, divided by its leading coefficient
(kScreenLead*): Horner then starts with an addition, t + m[deg-1], and the kernel forms
t = 1 - 2K/(x + K) with one FMA from the reciprocal.  The FP32 kernel takes the monomial basis
of u (kScreenC32, kScreenA, kScreenB).

It also prints the polynomials of 2^s on |s| <= 1/2 for the reduced-cost exponentials
(e^{-y} = 2^z with z = -y log2(e) = n + s, n = rint(z)): Chebyshev interpolants of the printed
degrees at 50 digits, in the monomial basis of s, divided by their leading coefficients
(kExpLead*).

The reduced-cost FP64 pairs take erfcx(x) + (2/sqrt(pi)) x itself as a polynomial (kScreenV*), in
X = x sqrt(log2 e) (so that e^{-x^2} = 2^{-X^2}), divided by its leading coefficient: the minimax
polynomial under the weight e^{-x^2} that multiplies it (Remez exchange at 50 digits), which needs no
reciprocal.  Run: python gen_screening.py > screening.h
"""
import mpmath as mp

mp.mp.dps = 50
K = 3
XMAX = mp.mpf(13) / 2
# "64": FP64 plans with tol < 1e-10; "64s": FP64 plans with 1e-10 <= tol < 1e-8; "64f": FP64
# plans with tol >= 1e-8; "32": FP32 bulk
DEGREES = {"64": 16, "64s": 12, "64f": 10, "32": 11}
# degree of the polynomial of 2^s, |s| <= 1/2: "1" for 1e-10 <= tol < 1e-8, "2" for tol >= 1e-8
EXP_DEGREES = {"1": 8, "2": 7}
# degrees of the weighted polynomials, by the same levels: V, which the kernels take, and W, one degree
# lower, which no kernel takes.  W's largest error is below that of the Moebius form (64s, 64f), but it is as
# large over the whole range where that one falls: the root of the integral of dC^2, which is what enters a
# sum over uniform pairs, is 1.9 (level 1) and 1.7 times (level 2) as large.  V's is half as large.
WEIGHTED_DEGREES = {"W1": 18, "W2": 15, "V1": 19, "V2": 16}


def weighted_remez(fun, weight, deg, xmax):
    """Monomial coefficients of the degree-deg polynomial p that minimises the maximum of
    weight (p - fun) on [0, xmax], by Remez exchange on a grid of 3001 points."""
    n = deg + 2
    # first reference: Chebyshev points of the range where the weight leaves something to fit
    xe = min(xmax, mp.sqrt(mp.mpf(deg)) * mp.mpf("1.05") + mp.mpf("0.6"))
    pts = [xe * (1 - mp.cos(mp.pi * k / (n - 1))) / 2 for k in range(n)]
    grid = [xmax * mp.mpf(k) / 3000 for k in range(3001)]
    ref = [fun(x) for x in grid]
    for _ in range(30):
        a, b = mp.matrix(n, n), mp.matrix(n, 1)
        for i, x in enumerate(pts):
            wx = weight(x)
            for j in range(deg + 1):
                a[i, j] = wx * x ** j
            a[i, deg + 1] = (-1) ** i
            b[i] = wx * fun(x)
        s = mp.lu_solve(a, b)
        c = [s[j] for j in range(deg + 1)]
        err = [weight(x) * (mp.polyval(c[::-1], x) - r) for x, r in zip(grid, ref)]
        ext, cur = [], 0  # the largest error of each run of one sign
        for k in range(1, len(grid)):
            if (err[k] > 0) != (err[cur] > 0):
                ext.append(cur)
                cur = k
            elif abs(err[k]) > abs(err[cur]):
                cur = k
        ext.append(cur)
        if max(abs(e) for e in err) < abs(s[deg + 1]) * mp.mpf("1.02"):
            return c
        while len(ext) > n:
            ext.pop(0 if abs(err[ext[0]]) < abs(err[ext[-1]]) else -1)
        pts = [grid[k] for k in ext]
    raise RuntimeError("no convergence at degree %d" % deg)


def cheb_coeffs(fun, n):
    """Chebyshev coefficients of the degree n-1 interpolant of fun on [-1, 1] (first kind nodes)."""
    nodes = [mp.cos(mp.pi * (k + mp.mpf(1) / 2) / n) for k in range(n)]
    vals = [fun(v) for v in nodes]
    return [(2 if j else 1) * mp.fsum(vals[k] * mp.cos(mp.pi * j * (k + mp.mpf(1) / 2) / n) for k in range(n)) / n
            for j in range(n)]


def cheb_to_mono(c):
    """Monomial coefficients of sum_j c[j] T_j(v)."""
    deg = len(c) - 1
    tk = [[mp.mpf(1)], [mp.mpf(0), mp.mpf(1)]]
    for k in range(2, deg + 1):
        nxt = [mp.mpf(0)] + [2 * v for v in tk[k - 1]]
        for i, v in enumerate(tk[k - 2]):
            nxt[i] -= v
        tk.append(nxt)
    out = [mp.mpf(0)] * (deg + 1)
    for j in range(deg + 1):
        for i, v in enumerate(tk[j]):
            out[i] += c[j] * v
    return out


def affine_substitute(c, A, B):
    """Monomial coefficients in t of sum_j c[j] (A t + B)^j."""
    out = [mp.mpf(0)] * len(c)
    for j, cj in enumerate(c):
        for k in range(j + 1):
            out[k] += cj * mp.binomial(j, k) * A ** k * B ** (j - k)
    return out


def arr(name, vals):
    return "constexpr double %s[%d] = {%s};" % (name, len(vals), ", ".join("%.17g" % float(v) for v in vals))


def main():
    t0, t1 = mp.mpf(-1), (XMAX - K) / (XMAX + K)
    A = 2 / (t1 - t0)
    B = -1 - t0 * A

    def erfcx_of_u(u):
        t = t0 + (u + 1) * (t1 - t0) / 2
        x = K * (1 + t) / (1 - t)
        return mp.erfc(x) * mp.exp(x * x)

    cheb = cheb_coeffs(erfcx_of_u, 96)
    print("// Generated by gen_screening.py -- do not edit.")
    print("// erfcx(x) for 0 <= x <= %s: FP64 in t = (x - K)/(x + K), monomials divided by the" % mp.nstr(XMAX, 3))
    print("// leading coefficient (kScreenLead*; kScreenM*[k], k < deg, the leading 1 implicit);")
    print("// FP32 in u = A t + B (kScreenC32).  2^s for |s| <= 1/2: kExpLead* x monic kExpM*.")
    print("// erfcx(x) + 2x/sqrt(pi), minimax under the weight e^{-x^2}, in X = x sqrt(log2 e):")
    print("// kScreenLeadV* x monic kScreenV* (W: one degree lower, not taken by any kernel).")
    print("#pragma once")
    print("namespace ewald {")
    print("constexpr double kScreenK = %d;" % K)
    print("constexpr double kScreenXmax = %.17g;" % float(XMAX))
    print("constexpr double kScreenA = %.17g;" % float(A))
    print("constexpr double kScreenB = %.17g;" % float(B))
    for tag, deg in DEGREES.items():
        mono_u = cheb_to_mono(cheb[: deg + 1])
        print("constexpr int kScreenDeg%s = %d;" % (tag, deg))
        if tag == "32":
            print(arr("kScreenC32", mono_u))
            continue
        mono_t = affine_substitute(mono_u, A, B)
        lead = mono_t[deg]
        print("constexpr double kScreenLead%s = %.17g;" % (tag, float(lead)))
        print(arr("kScreenM%s" % tag, [v / lead for v in mono_t[:deg]]))
    # 2^s = e^{s ln 2} on |s| <= 1/2, s = v / 2
    echeb = cheb_coeffs(lambda v: mp.exp(v * mp.log(2) / 2), 64)
    for tag, deg in EXP_DEGREES.items():
        mono_v = cheb_to_mono(echeb[: deg + 1])
        mono_s = [c * 2 ** i for i, c in enumerate(mono_v)]
        lead = mono_s[deg]
        print("constexpr int kExpDeg%s = %d;" % (tag, deg))
        print("constexpr double kExpLead%s = %.17g;" % (tag, float(lead)))
        print(arr("kExpM%s" % tag, [v / lead for v in mono_s[:deg]]))
    scale = mp.sqrt(1 / mp.log(2))  # X = x sqrt(log2 e)
    for tag, deg in WEIGHTED_DEGREES.items():
        c = weighted_remez(lambda x: mp.erfc(x) * mp.exp(x * x) + 2 * x / mp.sqrt(mp.pi),
                           lambda x: mp.exp(-x * x), deg, XMAX)
        c = [v / scale ** k for k, v in enumerate(c)]
        lead = c[deg]
        print("constexpr int kScreenDeg%s = %d;" % (tag, deg))
        print("constexpr double kScreenLead%s = %.17g;" % (tag, float(lead)))
        print(arr("kScreen%s" % tag, [v / lead for v in c[:deg]]))
    print("}  // namespace ewald")


if __name__ == "__main__":
    main()
