"""Branches that a call's sizes choose, at sizes that reach them, against the
oracle or against the route that other tests hold to it.  The kernels run the
oracle's FP32 operations in its order, so the tolerance is zero."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from gpu_util import DEV, to_dev, to_host
from paper_2208_00001_amd import synth

pytestmark = pytest.mark.gpu


def same(got, ref, what):
    got, ref = np.asarray(got), np.asarray(ref).reshape(got.shape)
    assert np.array_equal(got, ref), f"{what}: {int((got != ref).sum())} values differ"


def round256(n):
    return -(-n // 256) * 256


# voxels per plane step just above what sends the reverse of a volume to one launch
# a pass: about 12300 at lambda 0 and 1, 15000 between
@pytest.mark.parametrize("shape,lam", [((200, 201, 203), 0.0), ((200, 201, 203), 1.0), ((256, 236, 200), 0.7)], ids=str)
def test_reverse_of_large_volumes(shape, lam):
    from paper_2208_00001_amd import binding as B
    lib, dims, N = B.load_library(), (ctypes.c_int * 3)(*shape), int(np.prod(shape))
    least = lib.ggdt_backward_workspace_min_bytes(3, dims, 1)
    full = lib.ggdt_backward_workspace_bytes(3, dims, 1)
    assert full - least == 4 * round256(4 * N) + 2 * round256(N), "the workspace does not ask for one launch a pass"
    c = synth.small_case(shape, C=1, seed=110, lam=lam, iterations=1, soft=True, v=10.0)
    W = np.random.default_rng(111).standard_normal(shape).astype(np.float32)
    args = (c["spacing"], c["v"], c["lam"], 1)
    img = to_dev(c["image"])
    _, rec = B.ggdt_forward_rec(img, to_dev(c["mask"]), *args, check=True)
    grads = []
    # one launch a pass; scan and edges on copies, and in place (one launch in place at lambda 0)
    for n in (full, least + 2 * round256(4 * N) + round256(N), least):
        print(f"case {c['name']} lam={lam} workspace {n}", flush=True)
        ws = torch.empty(n, dtype=torch.uint8, device=DEV)
        grads.append([to_host(t) for t in B.ggdt_backward(img, rec, to_dev(W), *args, workspace=ws, check=True)])
    for gi, gm in grads[1:]:
        same(gm, grads[0][1], "dL/dM of two routes")
        same(gi, grads[0][0], "dL/dI of two routes")
    if lam == 1.0:
        rgi, rgm = oracle.backward(c["image"], to_host(rec), W, *args, "f32")
        same(grads[0][1], rgm, "dL/dM")
        same(grads[0][0], rgi, "dL/dI")
