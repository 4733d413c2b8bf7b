"""The adjoint's table-driven float64 sine and cosine and its 64-point exp2, the
device's reductions and terms evaluated in numpy float64 against numpy's
functions.  Bounds: the joined sine has five roundings of terms of at most 1
(6e-16 with the table's); exp2's series six, relative."""

import importlib.util
import os

import numpy as np

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2104_12922_amd", "csrc")


def _gen():
    spec = importlib.util.spec_from_file_location("gen", os.path.join(CSRC, "gen_series_tables.py"))
    m = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(m)
    return m


def test_header_holds_the_generated_table():
    m = _gen()
    txt = open(os.path.join(CSRC, "sine_table.h")).read()
    vals = [m.hexd(v) for v in m.sine_table()]
    assert len(vals) == 65
    body = txt[txt.index("= {") + 3:txt.index("};")]
    assert [v.strip() for v in body.split(",")] == vals
    ref = np.sin(2 * np.pi * np.arange(65) / 256)
    assert np.abs(np.array([float.fromhex(v) for v in vals]) - ref).max() <= 2.3e-16


def test_sincos_table():
    q = np.array([float(v) for v in _gen().sine_table()])
    j = np.arange(256)
    r, o = j & 63, j >> 6
    a, b = q[r], q[64 - r]
    S = np.choose(o, [a, b, -a, -b])
    C = np.choose(o, [b, -a, -b, a])
    rng = np.random.default_rng(0)
    th = np.concatenate([rng.uniform(0.0, 4.0, 200000), np.arange(1025) / 256, [0.0, 0.5, 0.25]])
    n = np.rint(256.0 * th)
    x = (th - n / 256.0) * (2 * np.pi)
    x2 = x * x
    sa = x + x * x2 * (-1.0 / 6.0 + x2 / 120.0)
    ca = x2 * (-0.5 + x2 * (1.0 / 24.0 - x2 / 720.0))
    k = n.astype(np.int64) & 255
    s, c = S[k] + (S[k] * ca + C[k] * sa), C[k] + (C[k] * ca - S[k] * sa)
    ref = np.longdouble(2) * np.longdouble("3.14159265358979323846264338327950288") * th
    assert np.abs(s - np.sin(ref)).max() <= 6e-16 and np.abs(c - np.cos(ref)).max() <= 6e-16


def test_exp2_64_points():
    rng = np.random.default_rng(1)
    y = -np.concatenate([rng.uniform(0.0, 60.0, 100000), rng.uniform(0.0, 1000.0, 10000), [0.0]])
    n = np.rint(64.0 * y)
    z = (y - n / 64.0) * np.log(2.0)
    p = 1 + z * (1 + z * (0.5 + z * (1 / 6 + z * (1 / 24 + z / 120))))
    k = n.astype(np.int64)
    got = np.ldexp(2.0 ** ((k & 63) / 64.0) * p, k >> 6)
    assert np.abs(got / np.exp2(y) - 1).max() <= 7e-16
