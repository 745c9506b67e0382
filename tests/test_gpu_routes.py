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


def batch_of(shapes, lam, iterations=1, seed=120):
    cs = [synth.small_case(s, C=1, seed=seed + i, lam=lam, iterations=iterations) for i, s in enumerate(shapes)]
    return cs, [dict(image=to_dev(c["image"]), softmask=to_dev(c["mask"]), spacing=c["spacing"], v=c["v"], lam=c["lam"],
                     iterations=iterations) for c in cs]


# 24 x 24 tiles where the passes have several tiles a workgroup for most of their
# planes, and not where only the few planes of a short axis have
@pytest.mark.parametrize("shape,n,lam,wide", [((400, 400, 8), 2, 1.0, False), ((400, 400, 8), 2, 0.5, False),
                                              ((64, 200, 200), 4, 0.5, False), ((64, 200, 200), 4, 1.0, False),
                                              ((150, 150, 150), 6, 0.5, True), ((40, 410, 410), 4, 1.0, True)], ids=str)
def test_batch_takes_wide_tiles(shape, n, lam, wide):
    from paper_2208_00001_amd.batched import BatchedPlan
    img, m = torch.rand(shape, device=DEV), torch.ones(shape, device=DEV)
    inst = [dict(image=img, softmask=m, spacing=(1.0, 1.0, 1.0), v=1e10, lam=lam, iterations=1) for _ in range(n)]
    size = {}
    for name, tuning in (("own", None), ("16", dict(tile_p=16)), ("24", dict(tile_p=24))):
        plan = BatchedPlan(inst, tuning)
        size[name] = plan.workspace.numel()
        plan.close()
    assert size["16"] != size["24"], "the exchange words do not tell the tiles apart"
    assert size["own"] == size["24" if wide else "16"]


# batches that the plan gives 16 x 16, 24 x 24, 8 x 16 and 8 x 8 tiles, some with images
@pytest.mark.parametrize("shapes", [[(20, 40, 44)] * 30, [(20, 40, 44)] * 56 + [(70, 300), (33, 40)] * 2,
                                    [(30, 31, 29)] * 24 + [(140, 50)], [(30, 29, 31)] * 6 + [(9, 30, 1)]],
                         ids=["16x16", "24x24", "8x16", "8x8"])
@pytest.mark.parametrize("lam", [0.5, 1.0])
def test_batch_classes(shapes, lam):
    from paper_2208_00001_amd.batched import BatchedPlan
    cs, inst = batch_of(shapes, lam)
    plan = BatchedPlan(inst)
    plan.run()
    plan.check()
    for c, d in zip(cs, plan.inst):
        ref = oracle.ggdt(c["image"], c["mask"], c["spacing"], c["v"], c["lam"], 1, "f32")
        same(to_host(d["out"]), ref, c["name"])
    plan.close()


def sides_of(kind, shape):
    """Transforms that a composed operation runs side by side, from the workspace it asks for."""
    from paper_2208_00001_amd import binding as B
    lib, dims, vol = B.load_library(), (ctypes.c_int * 3)(*shape), round256(4 * int(np.prod(shape)))
    n = (lib.ggdt_signed_workspace_bytes if kind == "signed" else lib.ggdt_gsf_workspace_bytes)(3, dims, 1)
    words = lib.ggdt_workspace_min_bytes(3, dims, 1) - 256  # exchange words of one transform
    found = [s for s in (2, 4) if n == round256(256 + s * words) + (7 if kind == "gsf" else 2) * vol + (s + 1) * vol]
    return found[0] if found else 1


# the filter's four transforms in pairs, whose masks take turns on one set of
# copies; and four together whose tiles outnumber the chip's workgroups on an axis
# of several chunks
@pytest.mark.parametrize("shape,sides", [((84, 86, 161), 2), ((26, 140, 150), 4)], ids=str)
@pytest.mark.parametrize("lam", [0.6, 1.0])
def test_filter_side_by_side(shape, sides, lam):
    from paper_2208_00001_amd import binding as B
    assert sides_of("gsf", shape) == sides and sides_of("signed", shape) == 2
    c = synth.small_case(shape, C=1, seed=160, lam=lam, iterations=1)
    m = (c["mask"] > 0).astype(np.float32)
    m[tuple(slice(s // 4, s // 2) for s in shape)] = 0.0
    img, md = to_dev(c["image"]), to_dev(m)
    print(f"case {c['name']} lam={lam} sides={sides}", flush=True)
    got = B.ggdt_gsf(img, md, 0.3, 0.2, c["spacing"], c["v"], c["lam"], 1, check=True)
    same(to_host(got), oracle.gsf(c["image"], m, 0.3, 0.2, c["spacing"], c["v"], c["lam"], 1), "filter")


@pytest.mark.parametrize("shapes", [[(20, 33, 40), (9, 50, 41)], [(20, 33, 40), (70, 65)], [(130, 70)]], ids=str)
@pytest.mark.parametrize("lam", [0.0, 0.6, 1.0])
def test_records_beyond_the_offsets(shapes, lam):
    """Record bytes that name no offset (records of another schedule) index nothing and
    end a voxel's path, in the batched reverses as in the plain one (the image
    gradient is then unspecified).  Bytes from 16 run too, with no value asserted."""
    from paper_2208_00001_amd import binding as B
    from paper_2208_00001_amd.batched import BatchedPlan
    rng = np.random.default_rng(170)
    cs = [synth.small_case(s, C=1, seed=170 + i, lam=lam, iterations=1, soft=True, v=10.0) for i, s in enumerate(shapes)]
    W = [to_dev(rng.standard_normal(s).astype(np.float32)) for s in shapes]
    plan = BatchedPlan([dict(image=to_dev(c["image"]), softmask=to_dev(c["mask"]), spacing=c["spacing"], v=c["v"],
                             lam=c["lam"], iterations=1, records=True, grad_out=w) for c, w in zip(cs, W)])
    plan.run()
    plan.check()
    for top in (256, 16):
        for rec in plan.records:
            other = rng.integers(10, top, size=tuple(rec.shape)).astype(np.uint8)
            rec.copy_(torch.where(to_dev(rng.random(tuple(rec.shape)) < 0.2), to_dev(other), torch.clamp(rec, max=9)))
        grads = plan.backward()
        plan.check()
    for c, d, w, (gi, gm) in zip(cs, plan.inst, W, grads):
        _, pm = B.ggdt_backward(d["image"], d["records"], w, c["spacing"], c["v"], c["lam"], 1, check=True)
        same(to_host(gm), to_host(pm), "dL/dM")
    plan.close()
