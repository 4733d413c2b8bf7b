"""Writes series_tables.h: the float64 tables of the control stage's
table-driven exp2 and log2 (Tang's method; P. T. P. Tang, "Table-driven
implementation of the exponential function in IEEE floating-point
arithmetic", ACM TOMS 15(2), 1989, and its logarithm counterpart, ACM TOMS
16(4), 1990), every entry correctly rounded from 60-digit decimal arithmetic:

  EXP2_T[j]      = 2^(j / 256),          j = 0 .. 255
  LOG2_T[j + 76] = log2(1 + j / 256),    j = -76 .. 107
  INV_C[j + 76]  = 1 / (1 + j / 256),    j = -76 .. 107

(the log2 reduction takes m in [1/sqrt 2, sqrt 2), so j = rint(256 (m - 1))
lies in -75 .. 106).

and sine_table.h, the quarter wave of the adjoint's table-driven sine and
cosine (the same reduction with the addition theorems):

  SIN_T[j]       = sin(2 pi j / 256),    j = 0 .. 64

Run from this directory: python gen_series_tables.py.
"""
from decimal import Decimal, getcontext
import os

getcontext().prec = 60
LN2 = Decimal(2).ln()
LOG_J0, LOG_J1 = -76, 107          # table points 1 + j/256 of the log2 reduction


def hexd(x: Decimal) -> str:
    return float(x).hex()


def tables():
    exp2 = [(Decimal(j) / 256 * LN2).exp() for j in range(256)]
    log2 = [(1 + Decimal(j) / 256).ln() / LN2 for j in range(LOG_J0, LOG_J1 + 1)]
    invc = [1 / (1 + Decimal(j) / 256) for j in range(LOG_J0, LOG_J1 + 1)]
    return exp2, log2, invc


def sine_table():
    # pi by Machin's formula, sin by its Taylor series, both in 60 digits
    def atan_inv(n):
        t, k, tot = Decimal(1) / n, 1, Decimal(0)
        while abs(t) > Decimal(10) ** -58:
            tot += t / k if k % 4 == 1 else -t / k
            t /= n * n
            k += 2
        return tot
    pi = 4 * (4 * atan_inv(5) - atan_inv(239))

    def sin(x):
        t, k, tot = x, 1, Decimal(0)
        while abs(t) > Decimal(10) ** -58:
            tot += t
            t = -t * x * x / ((k + 1) * (k + 2))
            k += 2
        return tot
    return [sin(2 * pi * j / 256) for j in range(65)]


def main(path=None):
    path = path or os.path.join(os.path.dirname(os.path.abspath(__file__)), "series_tables.h")
    exp2, log2, invc = tables()

    def arr(name, vals):
        body = ",\n".join("    " + ", ".join(hexd(v) for v in vals[i:i + 4])
                          for i in range(0, len(vals), 4))
        return f"static __device__ double {name}[{len(vals)}] = {{\n{body}}};\n"
    txt = ("// Generated by gen_series_tables.py: tables of the table-driven float64\n"
           "// exp2 and log2 (2^(j/256) for j = 0..255; log2(1 + j/256) and 1/(1 + j/256)\n"
           "// for j = -76..107), correctly rounded.\n"
           "// Device memory the compiler does not fold: the kernels read them with\n"
           "// vector loads (lane-varying j).\n"
           "#pragma once\n\nnamespace synth {\nnamespace voice {\n\n"
           + f"constexpr int kLogJ0 = {-LOG_J0};   // kLog2T[j + kLogJ0] = log2(1 + j/256)\n\n"
           + arr("kExp2T", exp2) + "\n" + arr("kLog2T", log2) + "\n" + arr("kInvC", invc)
           + "\n}  // namespace voice\n}  // namespace synth\n")
    with open(path, "w") as f:
        f.write(txt)
    return path


def main_sine(path=None):
    path = path or os.path.join(os.path.dirname(os.path.abspath(__file__)), "sine_table.h")
    vals = [hexd(v) for v in sine_table()]
    body = ",\n".join("    " + ", ".join(vals[i:i + 4]) for i in range(0, len(vals), 4))
    with open(path, "w") as f:
        f.write("// Generated by gen_series_tables.py: sin(2 pi j / 256), j = 0 .. 64, correctly\n"
                "// rounded.\n#pragma once\n\nnamespace synth {\nnamespace voice {\n\n"
                f"static __device__ double kSinT[{len(vals)}] = {{\n{body}}};\n"
                "\n}  // namespace voice\n}  // namespace synth\n")
    return path


if __name__ == "__main__":
    print(main())
    print(main_sine())
