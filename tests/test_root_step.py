"""The general edge cost's root by a Newton step from the reciprocal root.

On the CPU: the step itself, over every float of [1, 4) and of both ends of the
range (tests/native/sqrt_rsq_check.cpp).  On the GPU: every float of [1, 4), and of
four more ranges a power of 4 away, as the argument of an edge cost of the
transform.  A correctly rounded root has one result, so the tolerance is zero."""
import os
import re
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
NATIVE = os.path.join(ROOT, "tests", "native")
CSRC = os.path.join(ROOT, "paper_2208_00001_amd", "csrc")

# x (as its float in [1, 4)) and the distance of y from the float nearest to 1 / sqrt(x)
# where the step does not round to the nearest: four mantissas, five pairs
OFF = {(0x3ffc114a, 1), (0x404d142a, -1), (0x405ae03b, -1), (0x406e9372, -1), (0x406e9372, 1)}


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_newton_step_over_all_mantissas(tmp_path):
    exe = str(tmp_path / "sqrt_rsq_check")
    subprocess.run(["g++", "-O2", "-mfma", "-ffp-contract=off", "-I", CSRC, "-o", exe,
                    os.path.join(NATIVE, "sqrt_rsq_check.cpp"), "-lm"], check=True)
    out = subprocess.run([exe], capture_output=True, text=True, check=True).stdout
    for r in range(3):
        off = {(int(x, 16), int(k)) for x, k in re.findall(rf"off range {r} x (0x[0-9a-f]+) y ([+-]1)", out)}
        assert off == OFF, f"range {r}: {off}"
    assert "wrong with the nearest y: 0" in out


@pytest.mark.gpu
@pytest.mark.parametrize("e", [-47, -20, 0, 20, 58])
def test_every_mantissa_through_the_passes(e):
    """Arguments x 4^e for every float x of [1, 4).  On an image whose even rows are 0
    and seeds, an odd row's distance is the root of lambda d^2 + (1 - lambda) s^2
    for its value d, the nearest of its neighbours; with lambda 0.5 and (1 - lambda)
    s^2 = A, every float of [A, 1.2 A] is reached by some d, since steps of d move
    lambda d^2 by less than a unit in the last place of the sum."""
    import torch

    from gpu_util import DEV
    from paper_2208_00001_amd import binding as B
    lam, scale, Wd = 0.5, 2.0 ** e, 1024
    s = np.float32(np.sqrt(2.0)) - np.float32(2e-7)
    first, end = 0x3f800000, 0x40800000  # 1.0, 4.0
    done = 0
    while first < end:
        A = float(np.float32(0.5 * float(s) * float(s)))  # the library's constant for this spacing
        assert A <= float(np.uint32(first).view(np.float32))
        last = min(end, int(np.float32(1.2 * A).view(np.uint32)))
        n = last - first
        x = torch.arange(first, last, dtype=torch.int32, device=DEV).view(torch.float32)
        d0 = ((x.double() - A) / lam).sqrt().float()
        d, found = torch.zeros_like(x), torch.zeros_like(x, dtype=torch.bool)
        for k in range(-4, 5):
            t = (d0.view(torch.int32) + k).view(torch.float32)
            hit = ((t * t).double() * lam + A).float() == x
            d, found = torch.where(hit & ~found, t, d), found | hit
        assert bool(found.all()), f"{int((~found).sum())} arguments not reached from A = {A}"
        rows = -(-n // Wd)
        img, mask = torch.zeros((2 * rows + 1, Wd), device=DEV), torch.zeros((2 * rows + 1, Wd), device=DEV)
        img[1::2] = torch.nn.functional.pad(d, (0, rows * Wd - n)).view(rows, Wd) * scale
        mask[1::2] = 1.0
        out = B.ggdt2d(img, mask, (float(s) * scale, 3.0 * float(s) * scale), 1e30, lam, 1, check=True)
        got, ref = out[1::2].reshape(-1)[:n], (x.double().sqrt() * scale).float()
        bad = int((got != ref).sum())
        assert bad == 0, f"{bad} roots differ, the first at {float(x[(got != ref)][0])}"
        done += n
        first, s = last, np.float32(np.sqrt(2.0 * 1.1999 * A))
    assert done == 1 << 24
