"""Tile geometries of the 3D passes and their reverse, against the oracle bit
for bit: planes at the edges of each tile size's range (8 x 8 while at most 256
tiles cover the plane, then 8 x 16, then 16 x 16), ragged tiles, chunk
remainders, one to three channels, and planes with more tiles than workgroups.
The kernels run the oracle's FP32 operations in its order, so the tolerance is
zero."""
import numpy as np
import pytest

import oracle
from gpu_util import DEV, to_dev, to_host
from paper_2208_00001_amd import synth

pytestmark = pytest.mark.gpu

# axis 0 scans a plane of H x W: 256 tiles of 8 x 8; one row more; 256 of 8 x 16; one row more
PLANES = [(9, 128, 128), (10, 129, 127), (17, 128, 256), (9, 136, 257)]


def same(got, ref, what):
    got, ref = np.asarray(got), np.asarray(ref).reshape(got.shape)
    assert np.array_equal(got, ref), f"{what}: {int((got != ref).sum())} values differ"


@pytest.mark.parametrize("shape", PLANES, ids=str)
@pytest.mark.parametrize("C,lam", [(1, 0.5), (1, 1.0), (1, 0.0), (2, 0.5), (3, 1.0), (2, 0.0)])
def test_forward_records_and_backward(shape, C, lam):
    from paper_2208_00001_amd import binding as B
    c = synth.small_case(shape, C=C, seed=40 + C, lam=lam, iterations=1, soft=True, v=10.0)
    W = np.random.default_rng(41).standard_normal(shape).astype(np.float32)
    args = (c["spacing"], c["v"], c["lam"], 1)
    ref, rrec = oracle.ggdt(c["image"], c["mask"], *args, "f32", records=True)
    rgi, rgm = oracle.backward(c["image"], rrec, W, *args, "f32")
    img, m = to_dev(c["image"]), to_dev(c["mask"])
    print(f"case {c['name']} lam={lam}", flush=True)
    for minimal in (False, True):  # last axis on scan-major copies, and in place
        ws = B.new_workspace(shape, C, DEV, minimal=minimal)
        same(to_host(B.ggdt3d(img, m, *args, workspace=ws, check=True)), ref, "forward")
        out, rec = B.ggdt_forward_rec(img, m, *args, workspace=ws, check=True)
        same(to_host(out), ref, "forward with records")
        same(to_host(rec), rrec, "records")
    gi, gm = B.ggdt_backward(img, rec, to_dev(W), *args, check=True)
    same(to_host(gm), rgm, "dL/dM")
    same(to_host(gi), rgi, "dL/dI")


@pytest.mark.parametrize("C", [1, 2])
def test_more_tiles_than_workgroups(C):
    from paper_2208_00001_amd import binding as B
    shape = (4, 620, 500)  # axis 0: 39 x 32 tiles of 16 x 16
    c = synth.small_case(shape, C=C, seed=50, lam=0.6, iterations=1, soft=True, v=10.0)
    W = np.random.default_rng(51).standard_normal(shape).astype(np.float32)
    args = (c["spacing"], c["v"], c["lam"], 1)
    ref, rrec = oracle.ggdt(c["image"], c["mask"], *args, "f32", records=True)
    rgi, rgm = oracle.backward(c["image"], rrec, W, *args, "f32")
    img, m = to_dev(c["image"]), to_dev(c["mask"])
    out, rec = B.ggdt_forward_rec(img, m, *args, check=True)
    same(to_host(out), ref, "forward")
    gi, gm = B.ggdt_backward(img, rec, to_dev(W), *args, check=True)
    same(to_host(gm), rgm, "dL/dM")
    same(to_host(gi), rgi, "dL/dI")


@pytest.mark.parametrize("C,lam,scale", [(2, 0.0, 2.0 ** 61), (2, 0.5, 2.0 ** 61), (3, 1.0, 2.0 ** -30)])
def test_multichannel_fallback_cost(C, lam, scale):
    """Huge or small image values: the general cost with the full root."""
    from paper_2208_00001_amd import binding as B
    shape = (11, 30, 21)
    c = synth.small_case(shape, C=C, seed=60, lam=lam, iterations=2)
    image = (c["image"] * np.float32(scale)).astype(np.float32)
    ref = oracle.ggdt(image, c["mask"], c["spacing"], c["v"], c["lam"], 2, "f32")
    got = B.ggdt3d(to_dev(image), to_dev(c["mask"]), c["spacing"], c["v"], c["lam"], 2, check=True)
    same(to_host(got), ref, "forward")


@pytest.mark.parametrize("shape,C", [((17, 33), 1), ((18, 32), 2), ((34, 31), 3), ((70, 65), 4), ((1, 40), 1),
                                     ((40, 1), 3), ((2, 2), 8)], ids=str)
@pytest.mark.parametrize("lam", [0.0, 0.6, 1.0])
def test_image_backward(shape, C, lam):
    """The reverse of 2D passes at the edges of its 32-cell tiles and 16-row chunks."""
    from paper_2208_00001_amd import binding as B
    c = synth.small_case(shape, C=C, seed=70 + C, lam=lam, iterations=2, soft=True, v=10.0)
    W = np.random.default_rng(71).standard_normal(shape).astype(np.float32)
    args = (c["spacing"], c["v"], c["lam"], 2)
    _, rrec = oracle.ggdt(c["image"], c["mask"], *args, "f32", records=True)
    rgi, rgm = oracle.backward(c["image"], rrec, W, *args, "f32")
    gi, gm = B.ggdt_backward(to_dev(c["image"]), to_dev(rrec), to_dev(W), *args, check=True)
    same(to_host(gm), rgm, "dL/dM")
    same(to_host(gi), rgi, "dL/dI")


# volumes whose tiles make the plan take each of its tile sizes (8 x 8, 8 x 16,
# 16 x 16, 24 x 24), with images of one and of several groups of four tiles, and
# a volume whose last axis has one element
BATCHES = [[(9, 100, 100), (33, 70), (9, 30, 1)], [(9, 130, 200), (18, 129)], [(9, 160, 200), (10, 159, 190), (200, 17)],
           [(9, 160, 200), (9, 150, 210), (10, 159, 200), (9, 170, 200), (60, 300), (9, 1, 20)]]


@pytest.mark.parametrize("records", [False, True])
@pytest.mark.parametrize("batch", range(len(BATCHES)))
@pytest.mark.parametrize("lam", [0.0, 0.5, 1.0])
def test_batched_tile_sizes(batch, lam, records):
    from paper_2208_00001_amd.batched import BatchedPlan
    cs = [synth.small_case(s, C=1, seed=80 + i, lam=lam, iterations=1) for i, s in enumerate(BATCHES[batch])]
    inst = [dict(image=to_dev(c["image"]), softmask=to_dev(c["mask"]), spacing=c["spacing"], v=c["v"], lam=c["lam"],
                 iterations=1, **({"records": True} if records else {})) for c in cs]
    plan = BatchedPlan(inst)
    plan.run()
    plan.check()
    for c, d in zip(cs, plan.inst):
        ref, rrec = oracle.ggdt(c["image"], c["mask"], c["spacing"], c["v"], c["lam"], 1, "f32", records=True)
        same(to_host(d["out"]), ref, c["name"])
        if records:
            same(to_host(d["records"]), rrec, c["name"] + " records")
    plan.close()


@pytest.mark.parametrize("shape,C", [((70, 65), 2), ((33, 40), 4), ((20, 33, 40), 1), ((9, 130, 200), 1), ((12, 21, 17), 3),
                                     ((9, 20, 1), 1), ((11, 14, 13), 4)], ids=str)
@pytest.mark.parametrize("lam", [0.0, 0.6, 1.0])
def test_signed_and_filter_side_by_side(shape, C, lam):
    """The composed operations with the workspace asked for, and with the smaller
    one that holds one transform at a time."""
    from paper_2208_00001_amd import binding as B
    import torch
    c = synth.small_case(shape, C=C, seed=90 + C, lam=lam, iterations=2)
    m = (c["mask"] > 0).astype(np.float32)
    m[tuple(slice(0, max(1, s // 3)) for s in shape)] = 0.0
    img, md, nd = to_dev(c["image"]), to_dev(m), len(shape)
    td, te = 0.3, 0.2
    rs = oracle.signed(c["image"], m, c["spacing"], c["v"], c["lam"], 2)
    rg = oracle.gsf(c["image"], m, td, te, c["spacing"], c["v"], c["lam"], 2)
    lib = B.load_library()
    dims = (3 * __import__("ctypes").c_int)(*shape, *([1] * (3 - nd)))
    buf = -(-int(np.prod(shape)) * 4 // 256) * 256
    alone = -(-lib.ggdt_workspace_min_bytes(nd, dims, C) // 256) * 256
    for ws2, ws4 in ((None, None), *(((torch.empty(alone + n * buf, dtype=torch.uint8, device=DEV)) for n in (2, 4)),)):
        same(to_host(B.ggdt_signed(img, md, c["spacing"], c["v"], c["lam"], 2, workspace=ws2)), rs, "signed")
        same(to_host(B.ggdt_gsf(img, md, td, te, c["spacing"], c["v"], c["lam"], 2, workspace=ws4)), rg, "filter")


@pytest.mark.parametrize("shape", [(3, 4, w) for w in (1, 2, 3, 4, 5, 7, 9)] + [(1, 1, 4), (9, 70, 6), (2, 300, 11)] +
                         [(5, w) for w in (2, 3, 4, 6)] + [(270, 5), (513, 33)], ids=str)
@pytest.mark.parametrize("C,lam", [(1, 1.0), (2, 0.5)])
def test_toivanen_row_ends(shape, C, lam):
    """Rows shorter and longer than the four elements moved at a time, first and
    last rows of the array, several blocks and sweeps."""
    from paper_2208_00001_amd import binding as B
    c = synth.small_case(shape, C=C, seed=95, lam=lam, iterations=2)
    args = (c["spacing"], c["v"], c["lam"], 2)
    ref = oracle.toivanen(c["image"], c["mask"], *args, "f32")
    same(to_host(B.ggdt_toivanen(to_dev(c["image"]), to_dev(c["mask"]), *args, check=True)), ref, c["name"])


@pytest.mark.parametrize("shapes", [[(9, 70, 60), (12, 33, 41)], [(9, 130, 190)], [(9, 160, 200), (10, 150, 180)]], ids=str)
@pytest.mark.parametrize("lam", [0.0, 0.7, 1.0])
def test_batched_reverse_tile_sizes(shapes, lam):
    """Batches of volumes whose reverse takes 8 x 8, 8 x 16 and 16 x 16 tiles."""
    from paper_2208_00001_amd.batched import BatchedPlan
    cs = [synth.small_case(s, C=1, seed=85 + i, lam=lam, iterations=1, soft=True, v=10.0) for i, s in enumerate(shapes)]
    W = [np.random.default_rng(86 + i).standard_normal(s).astype(np.float32) for i, s in enumerate(shapes)]
    plan = BatchedPlan([dict(image=to_dev(c["image"]), softmask=to_dev(c["mask"]), spacing=c["spacing"], v=c["v"],
                             lam=c["lam"], iterations=1, records=True, grad_out=to_dev(w)) for c, w in zip(cs, W)])
    plan.run()
    grads = plan.backward()
    plan.check()
    for c, w, (gi, gm) in zip(cs, W, grads):
        _, rrec = oracle.ggdt(c["image"], c["mask"], c["spacing"], c["v"], c["lam"], 1, "f32", records=True)
        rgi, rgm = oracle.backward(c["image"], rrec, w, c["spacing"], c["v"], c["lam"], 1, "f32")
        same(to_host(gm), rgm, "dL/dM")
        same(to_host(gi), rgi, "dL/dI")
    plan.close()
