"""The bound on the fitted tip height (run_fit_err) over everything the library accepts: sides to
65536, runs of every level and start, suns from below the horizon to near the zenith, bodies from
10 km up, and the long runs of a 16384^2 polar tile.  Only rays that the descent fits count: origins
within 5% of the radius whose path moves 0.95 to 1.09 texels per nominal texel of travel."""
import math
import os
import subprocess

import numpy as np
import pytest
from test_tip_fit import CSRC, DRIVER, exact_tip, f32, fit, fma, quartic


def rays(rng, W, H, texel, R, Lz, hd, n):
    """sp, cp, c, 1/rho (float32) of n rays of the tile that a descent would fit."""
    X, Y = (rng.uniform(-0.5, 0.5, n) * s * texel / R for s in (W, H))
    k = rng.integers(0, 4, n)  # corners among them, where the bound is tightest
    corner = rng.random(n) < 0.2
    X = np.where(corner, np.where(k & 1, 0.5, -0.5) * W * texel / R, X)
    Y = np.where(corner, np.where(k & 2, 0.5, -0.5) * H * texel / R, Y)
    az, Lxy = rng.uniform(0, 2 * math.pi), math.sqrt(1 - Lz * Lz)
    Lx, Ly = Lxy * math.cos(az), Lxy * math.sin(az)
    g = np.sqrt(1 + X * X + Y * Y)
    r1 = 1 + rng.uniform(-0.0499, 0.0499, n) * rng.choice([0.01, 1.0], n)
    Kx, Ky = ((l - q * Lz) * g / (r1 * texel) for l, q in ((Lx, X), (Ly, Y)))
    k2 = (Kx * Kx + Ky * Ky) * 4.0 * hd * hd
    ok = (k2 > 0.9) & (k2 < 1.2)
    sp = (X * Lx + Y * Ly + Lz) / g
    cp = np.sqrt(np.maximum(0, 1 - sp * sp))
    return [v[ok].astype(f32) for v in (sp, cp, Lz * g / r1 / R, 1 / (R * r1))]


def test_bound_over_the_accepted_range(tmp_path):
    src, exe = tmp_path / "d.cpp", str(tmp_path / "d")
    src.write_text(DRIVER)
    r = subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                        "-I" + CSRC, str(src), "-o", exe], capture_output=True, text=True)
    if r.returncode != 0 and "hip_runtime.h" in r.stderr:
        pytest.skip("no HIP headers")
    assert r.returncode == 0, r.stderr
    rng = np.random.default_rng(7)
    cases = []

    def case(W, H, texel, R, e, a0, m):
        cases.append((W, H, texel, 1.0 / R, math.sin(e), 0.5 * texel / math.cos(e), a0, m))

    for _ in range(6000):
        W, H = (int(2 ** rng.uniform(0, 16)) for _ in range(2))
        R = 1737400.0 if rng.random() < 0.5 else 10 ** rng.uniform(4, 8)
        e = rng.choice([rng.uniform(-0.02, 0.07), rng.uniform(-0.3, 1.5)])
        case(W, H, 10 ** rng.uniform(-1, 3), R, e, int(2 ** rng.uniform(0, 18)), int(rng.integers(1, 17)))
    # the 16384^2 polar tile at 2 m: rays of 60 km, runs of 5, 6, 7, ... levels; and no cap
    for deg in (1.5, 0.5, 3.0, 6.0):
        a0, j = 0, 0
        while a0 < 2 * 32768:
            m = min(4 + j, 14)
            case(16384, 16384, 2.0, 1737400.0, math.radians(deg), a0, m)
            a0, j = a0 + (2 << m), j + 1
    out = subprocess.run([exe], input="\n".join(" ".join(map(repr, c)) for c in cases),
                         capture_output=True, text=True).stdout.split("\n")
    used = deep = lows = 0
    for (W, H, texel, invR, Lz, hd, a0, m), line in zip(cases, out):
        if line == "none":
            continue
        top, low = map(float, line.split())
        R = 1.0 / float(f32(invR))
        sp, cp, c, ir = rays(rng, W, H, texel, R, Lz, hd, 200)
        if not len(sp):
            continue
        used += 1
        deep += a0 > 2 ** 14 or max(W, H) > 2 ** 14
        t0, t1 = (a0 + 1) * hd, (a0 + (2 << m) + 1) * hd
        u0 = (t0 / (1 + np.float64(c) * t0)).astype(f32)
        u1 = (t1 / (1 + np.float64(c) * t1)).astype(f32)
        a = quartic(sp, cp, c, ir)
        n = len(sp)
        for bound, part in ((top, 1.0), (low, 1.5 / 8)):
            if part < 1.0 and m < 7:  # taken again in runs of level 7 and up
                continue
            lows += part < 1.0
            d = (u1 - u0) * f32(part)
            lo = u0 + (u1 - u0 - d) * rng.uniform(0, 1, n).astype(f32)
            hi = lo + d
            k0, k1, k2 = fit(sp, a, lo, hi)
            for f in (np.zeros(n), np.ones(n), rng.uniform(0, 1, n)):
                u = np.clip(lo + (hi - lo) * f.astype(f32), lo, hi)
                off = np.abs(np.float64(fma(u, fma(u, k2, k1), k0)) -
                             np.float64(exact_tip(sp, c, ir, u, rng)))
                assert 2.0 * off.max() <= bound, (W, H, texel, R, Lz, a0, m, part, off.max(), bound)
    assert used > 1000 and deep > 300 and lows > 400, (used, deep, lows)
