"""The general edge cost's root on the GPU against the oracle's, bit for bit.

On an image of two rows, the first constant and a seed everywhere (D = 0), the
second row's distance after one pass is the smallest of three roots, and with
equal first-row values that is the root of fmaf(lambda, g, A) for the straight
offset, so the arguments can be chosen.  A correctly rounded root has one
result, so the tolerance is zero.
"""
import numpy as np
import pytest

import oracle
from gpu_util import DEV, to_dev, to_host

pytestmark = pytest.mark.gpu

# The mantissas for which one Newton step from a reciprocal root one float off
# would round the wrong way, in [1, 4); scaled by powers of 4.
HARD = [np.uint32(b).view(np.float32) for b in (0x3ffc114a, 0x404d142a, 0x405ae03b, 0x406e9372)]


def run_both(img, lam, spacing, v=1e30):
    from paper_2208_00001_amd import binding as B
    C, H, W = img.shape
    mask = np.ones((H, W), np.float32)
    mask[0] = 0.0
    ws = B.new_workspace((H, W), C, DEV)
    got = to_host(B.ggdt2d(to_dev(img), to_dev(mask), spacing, v, lam, 1, workspace=ws))
    assert B.workspace_status(ws) == 0
    ref = oracle.ggdt(img, mask, spacing, v, lam, 1, "f32")
    assert np.array_equal(got.view(np.uint32), ref.view(np.uint32)), (
        f"{int((got.view(np.uint32) != ref.view(np.uint32)).sum())} values differ")
    return got


def hits(x, lam, A):
    """Differences d with float32(lam * float32(d * d) + A) == x (one rounding)."""
    d0 = np.float32(np.sqrt((float(x) - float(A)) / lam))
    d = (d0.view(np.uint32) + np.arange(-400, 401)).astype(np.uint32).view(np.float32)
    dd = (d * d).astype(np.float64)
    return d[(lam * dd + float(A)).astype(np.float32) == x]


@pytest.mark.parametrize("C", [1, 2])
def test_root_at_the_hard_mantissas(C):
    for x in HARD:
        for k in (-20, -2, 0, 2, 20):
            xs = np.float32(float(x) * 4.0 ** k)
            lam = 0.5 if C == 1 else 1.0
            for part in np.linspace(0.5, 0.75, 60):  # split x until a difference reaches it
                if C == 1:
                    s, d0 = float(np.float32(np.sqrt(float(xs) * part / 0.5))), np.float32(0)
                    A = np.float32(0.5 * (s * s))
                else:  # lambda 1: the argument is d0^2 + d1^2
                    s, d0 = 1.0, np.float32(np.sqrt(float(xs) * part))
                    A = d0 * d0
                d = hits(xs, lam, A)
                if d.size:
                    break
            assert d.size > 0, f"no difference reaches {xs}"
            img = np.zeros((C, 2, d.size), np.float32)
            img[0, 1] = d0
            img[C - 1, 1] = d
            run_both(img, lam, (s, 3.0 * s))


@pytest.mark.parametrize("C,lam,spacing", [(1, 0.5, (1.0, 4.0)), (1, 0.999, (2.0 ** -30, 1.0)), (3, 1.0, (1.0, 1.0)),
                                           (2, 0.3, (1e-3, 1.0))])
def test_root_over_dense_arguments(C, lam, spacing):
    rng = np.random.default_rng(3)
    img = np.zeros((C, 2, 1 << 18), np.float32)
    img[:, 1] = np.exp2(rng.uniform(-12, 12, size=img[:, 1].shape)) * (rng.random(img[:, 1].shape) < 0.8)
    run_both(img, lam, spacing)


@pytest.mark.parametrize("C,lam,spacing", [(1, 0.5, (1e-30, 1e-30)), (2, 0.5, (1e-30, 1e-30)), (1, 0.25, (3e20, 3e20)),
                                           (1, 0.5, (1e18, 2e19)), (2, 1.0, (1.0, 1.0))])
def test_root_at_the_ends_of_the_range(C, lam, spacing):
    """Edge constants that underflow to 0 or overflow, and equal pixels: the
    argument is 0, tiny or infinite, where the short form must not run."""
    rng = np.random.default_rng(4)
    img = np.zeros((C, 2, 300), np.float32)
    img[:, 1, 100:] = np.exp2(rng.uniform(-60, 20, size=(C, 200)))
    img[:, 1, 200:250] = 1.0
    run_both(img, lam, spacing)
