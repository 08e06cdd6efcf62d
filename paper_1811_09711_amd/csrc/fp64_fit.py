"""Coefficients of the FP64 special functions of the channel maps in
mcv_device.h (erfcinv_group, m_tan, m_exp2) and of the far tail of the
FP32 erfcinv (erfcinv_far).

erfcinv: as in erfcinv_fit.py, with w = -log2(y (2 - y)), erfcinv(y) =
(1 - y) P(w); P is a polynomial in t on [-1, 1], t linear in w up to W1 and in
sqrt(w) on the pieces beyond.  Each polynomial interpolates P at Chebyshev
nodes in 40-digit arithmetic and is cut at the stated degree (the dropped
Chebyshev coefficients bound the error), then written in the power basis for
Horner's rule.  log2(1 + f) = s (L0 + z L(z)), s = f / (2 + f), z = s^2, L0 =
2 / ln 2; sin(a) = a S(z), cos(a) = C(z), z = a^2, |a| <=
pi / 4; 2^f on [-1/2, 1/2].

    python fp64_fit.py
"""
import mpmath as mp

W1 = 11
PIECES = ((11, 36), (36, 144), (144, 1089))  # w beyond W1: sqrt(w) in [3.3, 6], [6, 12], [12, 33]
DEG_CENTRAL, DEG_PIECE = 25, 23
FAR = (26, 151)          # the FP32 far tail: y from 7.5e-9 down to the smallest denormal
DEG_FAR = 10
DEG_LOG, DEG_SIN, DEG_COS, DEG_EXP2 = 8, 6, 7, 11


def p_of_w(w):
    """erfinv(x) / x at 1 - x^2 = 2^-w."""
    q = mp.mpf(2) ** (-w)
    x = mp.sqrt(1 - q)
    if x < mp.mpf(10) ** -12:
        return mp.sqrt(mp.pi) / 2 * (1 + mp.pi / 12 * x * x)
    y = q / (1 + x)  # 1 - x
    if y > mp.mpf(1) / 2:
        return mp.erfinv(x) / x
    z = mp.sqrt(-mp.log(y))
    for _ in range(60):
        u = (mp.erfc(z) - y) / (-2 / mp.sqrt(mp.pi) * mp.exp(-z * z))
        step = u / (1 + z * u)
        z -= step
        if abs(step) < mp.mpf(10) ** -35 * z:
            break
    return z / x


def cheb(f, a, b, deg):
    """Power-basis coefficients in t = (2 v - a - b) / (b - a), highest first,
    and the size of what was cut, relative to f's largest value."""
    a, b = mp.mpf(a), mp.mpf(b)
    n = deg + 9
    xs = [mp.cos(mp.pi * (k + mp.mpf(1) / 2) / n) for k in range(n)]
    fs = [f(a + (b - a) * (x + 1) / 2) for x in xs]
    c = [2 * mp.fsum(fs[k] * mp.cos(mp.pi * j * (k + mp.mpf(1) / 2) / n) for k in range(n)) / n
         for j in range(n)]
    c[0] /= 2
    cut = mp.fsum(abs(v) for v in c[deg + 1:]) / min(abs(v) for v in fs)
    t0, t1 = [mp.mpf(1)], [mp.mpf(0), mp.mpf(1)]  # power bases of T_0, T_1
    out = [mp.mpf(0)] * (deg + 1)
    for j in range(deg + 1):
        for i, v in enumerate(t0):
            out[i] += c[j] * v
        nxt = [mp.mpf(0)] + [2 * v for v in t1]
        for i, v in enumerate(t0):
            nxt[i] -= v
        t0, t1 = t1, nxt
    return out[::-1], float(cut)


def unscaled(f, b, deg):
    """Power-basis coefficients in v on [0, b], highest first."""
    p, cut = cheb(f, 0, b, deg)
    b = mp.mpf(b)
    q = [mp.mpf(0)]
    for c in p:  # q(v) <- q(v) (2 v / b - 1) + c
        r = [mp.mpf(0)] * (len(q) + 1)
        for i, v in enumerate(q):
            r[i] -= v
            r[i + 1] += 2 * v / b
        r[0] += c
        q = r
    return q[:deg + 1][::-1], cut


def fits():
    mp.mp.dps = 40
    out = {"central": cheb(p_of_w, 0, W1, DEG_CENTRAL)}
    for i, (a, b) in enumerate(PIECES):
        out["piece%d" % i] = cheb(lambda s: p_of_w(s * s), mp.sqrt(a), mp.sqrt(b), DEG_PIECE)
    out["far"] = cheb(lambda s: p_of_w(s * s), mp.sqrt(FAR[0]), mp.sqrt(FAR[1]), DEG_FAR)
    zmax = ((mp.sqrt(2) - 1) / (mp.sqrt(2) + 1)) ** 2

    def log_rest(z):  # (2 atanh(s) / (s ln 2) - 2 / ln 2) / z
        if z < mp.mpf(10) ** -12:
            return 2 / mp.log(2) * (mp.mpf(1) / 3 + z / 5)
        s = mp.sqrt(z)
        return (2 * mp.atanh(s) / (s * mp.log(2)) - 2 / mp.log(2)) / z

    out["log"] = unscaled(log_rest, zmax * mp.mpf("1.001"), DEG_LOG)
    q = (mp.pi / 4) ** 2 * mp.mpf("1.001")
    out["sin"] = unscaled(lambda z: mp.sin(mp.sqrt(z)) / mp.sqrt(z) if z > 0 else mp.mpf(1), q, DEG_SIN)
    out["cos"] = unscaled(lambda z: mp.cos(mp.sqrt(z)), q, DEG_COS)

    # 2^f on [-1/2, 1/2]: t = 2 f, rescaled to f
    c, cut = cheb(lambda f: mp.mpf(2) ** f, -mp.mpf(1) / 2, mp.mpf(1) / 2, DEG_EXP2)
    out["exp2"] = ([v * 2 ** (DEG_EXP2 - i) for i, v in enumerate(c)], cut)
    return out


if __name__ == "__main__":
    for name, (c, cut) in fits().items():
        print("// %s: cut %.2g" % (name, cut))
        fmt = "%.9ef" if name == "far" else "%.17g"
        print("{" + ", ".join(fmt % float(v) for v in c) + "}")
    for a, b in PIECES + (FAR,):
        s, e = mp.sqrt(a), mp.sqrt(b)
        print("// t = (sqrt(w) - %.17g) * %.17g" % (float((s + e) / 2), float(2 / (e - s))))
