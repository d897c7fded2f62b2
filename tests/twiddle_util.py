"""The twiddle tables of a plan's Green's buffer, made anew from their definition.

Radix plans are read from the kernels' source; everything else is computed here:
for each radix plan of a pencil of length L, forward order then reversed, stage
s >= 1 with radix R and span NS holds w^(p k), p = 1, 2, 4, 8, 16, 3, for
k < NS, w = exp(-2 pi i / (NS R)).  Rows (L = n2) add exp(-i pi k / n2), k <= n2;
axis 0 (L = 2 n0) adds every power w^(r k), 1 <= r < R; axis 1 has L = 2 n1.
Each plan's tables start at a multiple of 256 bytes.
"""
from __future__ import annotations

import os
import re

import numpy as np

_SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2405_02603_amd", "csrc",
                    "fft_core.hpp")


def radix_plans():
    """[{L: radices}] of plan 0 and plan 1."""
    text = open(_SRC).read()
    text = text[text.index("constexpr RadixPlan radix_plan("):]
    text = text[:text.index("plan_len(")]
    one, zero = text.split("switch (L) {")[1:3]
    case = re.compile(r"case (\d+): return \{(\d), \{([\d, ]+)\}\};")
    return [{int(L): [int(r) for r in rs.split(",")][:int(k)] for L, k, rs in case.findall(t)} for t in (zero, one)]


def _cis(t, d):
    """exp(-2 pi i t / d), t and d whole numbers."""
    t = np.asarray(t, dtype=np.int64) % d
    a = 2 * np.arctan2(np.longdouble(0), np.longdouble(-1)) * t.astype(np.longdouble) / np.longdouble(d)
    return np.stack([np.cos(a), -np.sin(a)], axis=-1)


def _stages(radices):
    for order in (radices, radices[::-1]):
        span = 1
        for s, R in enumerate(order):
            if s:
                yield span, R
            span *= R


def tables(n, real):
    """(values, byte offset) of every table of a plan on n = (n0, n1, n2), and their total bytes."""
    out, at = [], 0
    for role, length in (("row", n[2]), ("axis1", 2 * n[1]), ("axis0", 2 * n[0])):
        for plans in radix_plans():
            parts = [_cis(np.multiply.outer(np.arange(ns), [1, 2, 4, 8, 16, 3]).ravel(), ns * R)
                     for ns, R in _stages(plans[length])]
            if role == "row":
                parts.append(_cis(np.arange(n[2] + 1), 2 * n[2]))
            if role == "axis0":
                parts += [_cis(np.multiply.outer(np.arange(ns), np.arange(1, R)).ravel(), ns * R)
                          for ns, R in _stages(plans[length])]
            values = np.concatenate(parts) if parts else np.zeros((0, 2), np.longdouble)
            out.append((values, at))
            at += -(-values.size * np.dtype(real).itemsize // 256) * 256
    return out, at
