"""The bound on the fitted tip height (run_fit_err) against the kernels' exact FP32 tip
height, both evaluated in float32 with the kernels' operations (a fused multiply-add
rounds once; reciprocal and root are off by up to one ulp): the difference stays below the
bound over body radii, suns below and above the horizon, tile extents and run positions."""
import math
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2005_06671_amd", "csrc")

DRIVER = r"""
#include <stdio.h>
#include "common.h"
int main() {
  int W, H, a0, m;
  double texel, invR, Lz, hd;
  while (scanf("%d %d %lf %lf %lf %lf %d %d", &W, &H, &texel, &invR, &Lz, &hd, &a0, &m) == 8) {
    const unsigned e = run_fit_err(W, H, (float)texel, (float)invR, (float)Lz, hd, run_pack(a0, m));
    float top, low;
    const unsigned t = e & 0xffff0000u, l = e << 16;
    memcpy(&top, &t, 4);
    memcpy(&low, &l, 4);
    if (e == SS_FIT_NONE) printf("none\n");
    else printf("%.9g %.9g\n", top, low);
  }
}
"""

f32 = np.float32


def fma(a, b, c):
    return (np.float64(a) * np.float64(b) + np.float64(c)).astype(f32)


def ulp_off(x, rng):
    return np.nextafter(x, x + f32(1.0) * np.abs(x) * rng.choice([-1, 0, 1], size=x.shape).astype(f32))


def exact_tip(sp, c, ir, u, rng):
    A = fma(-c, u, f32(1.0))
    v = u * ir
    P = fma(f32(2.0) * sp, A, v)
    S = ulp_off(np.sqrt(fma(A, A, v * P)), rng)
    return (u * P) * ulp_off(f32(1.0) / ((S + A) * A), rng)


def quartic(sp, cp, c, ir):
    k = cp * cp * ir
    b2, b3 = f32(0.5) * k, f32(-0.5) * sp * k * ir
    b4 = k * (f32(5.0) * sp * sp - f32(1.0)) * f32(0.125) * ir * ir
    a2 = fma(sp, c, b2)
    a3 = fma(c, fma(sp, c, f32(2.0) * b2), b3)
    a4 = fma(c, fma(c, fma(sp, c, f32(3.0) * b2), f32(3.0) * b3), b4)
    return a2, a3, a4


def fit(sp, a, u0, u1):
    a2, a3, a4 = a
    uc = f32(0.5) * (u0 + u1)
    w = uc * uc
    k2 = fma(uc, fma(f32(6.0) * a4, uc, f32(3.0) * a3), a2)
    k1 = fma(-w, fma(f32(8.0) * a4, uc, f32(3.0) * a3), sp)
    k0 = (w * uc) * fma(f32(3.0) * a4, uc, a3)
    return k0, k1, k2


def test_fit_error_bound(tmp_path):
    src = tmp_path / "d.cpp"
    src.write_text(DRIVER)
    exe = str(tmp_path / "d")
    r = subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                        "-I" + CSRC, str(src), "-o", exe], capture_output=True, text=True)
    if r.returncode != 0 and "hip_runtime.h" in r.stderr:
        pytest.skip("no HIP headers")
    assert r.returncode == 0, r.stderr
    rng = np.random.default_rng(11)
    cases = []
    for _ in range(3000):
        W, H = (int(2 ** rng.uniform(4, 14)) for _ in range(2))
        texel = 10 ** rng.uniform(-0.3, 2.3)
        R = MOON = 1737400.0
        if rng.random() < 0.5:
            R = 10 ** rng.uniform(4, 7.5)
        e = rng.choice([rng.uniform(-0.02, 0.07), rng.uniform(-0.3, 1.4)])
        m = int(rng.integers(1, 14))
        a0 = int(2 ** rng.uniform(0, 14))
        cases.append((W, H, texel, 1.0 / R, math.sin(e), 0.5 * texel / math.cos(e), a0, m))
    out = subprocess.run([exe], input="\n".join(" ".join(map(repr, c)) for c in cases),
                         capture_output=True, text=True).stdout.split("\n")
    used = tops = lows = 0
    for (W, H, texel, invR, Lz, hd, a0, m), line in zip(cases, out):
        if line == "none":
            continue
        used += 1
        top, low = map(float, line.split())
        R, n = 1.0 / float(f32(invR)), 300
        ext = 0.5 * math.hypot(W, H) * texel
        q = ext * np.sqrt(rng.uniform(0, 1, n))
        th, az = rng.uniform(0, 2 * math.pi, n), rng.uniform(0, 2 * math.pi)
        X, Y = q * np.cos(th) / R, q * np.sin(th) / R
        Lxy = math.sqrt(1 - Lz * Lz)
        Lx, Ly = Lxy * math.cos(az), Lxy * math.sin(az)
        g = np.sqrt(1 + X * X + Y * Y)
        r1 = 1 + rng.uniform(-0.05, 0.05, n) * rng.choice([0.01, 1.0])
        sp = ((X * Lx + Y * Ly + Lz) / g).astype(f32)
        cp = np.sqrt(np.maximum(0, 1 - np.float64(sp) ** 2)).astype(f32)
        c, ir = (Lz * g / r1 / R).astype(f32), (1 / (R * r1)).astype(f32)
        t0, t1 = (a0 + 1) * hd, (a0 + (2 << m) + 1) * hd
        u0 = (t0 / (1 + np.float64(c) * t0)).astype(f32)
        u1 = (t1 / (1 + np.float64(c) * t1)).astype(f32)
        a = quartic(sp, cp, c, ir)
        for bound, lo, hi in ((top, u0, u1), (low, None, None)):
            if lo is None:
                # a stretch of 1.5 texels of the level SS_REFIT (3) below, anywhere in the run
                if m < 7:
                    continue
                d = (u1 - u0) * f32(1.5 / 8)
                lo = u0 + (u1 - u0 - d) * rng.uniform(0, 1, n).astype(f32)
                hi = lo + d
                lows += 1
            else:
                tops += 1
            k0, k1, k2 = fit(sp, a, lo, hi)
            for f in (0.0, 1.0, rng.uniform(0, 1, n)):
                u = np.clip((lo + (hi - lo) * f32(f) if np.isscalar(f) else lo + (hi - lo) * f.astype(f32)), lo, hi)
                near = fma(u, fma(u, k2, k1), k0)
                off = np.abs(np.float64(near) - np.float64(exact_tip(sp, c, ir, u, rng)))
                assert 2.0 * off.max() <= bound, (W, H, texel, R, Lz, a0, m, off.max(), bound)
    assert used > 500 and tops > 500 and lows > 200
