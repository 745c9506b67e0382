"""Every bounded wait of the single-instance and batched launches gives up under a
spin limit of one poll, forced from the host (each kernel still exits normally):
the status query reports the watchdog, and with the limit restored the same
workspace gives the oracle's result.  One case for each kernel that waits: teams
(images), thread-per-cell passes by tile and channels, tile passes (more than 3
channels), both scans of the reverse, and the batched reverse."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import to_dev, to_host
from paper_2208_00001_amd import synth

pytestmark = pytest.mark.gpu

GGDT_ERR_WATCHDOG = -6


@pytest.fixture(autouse=True)
def default_spin_limit():
    from paper_2208_00001_amd import binding as B
    B.load_library()
    yield
    B.set_spin_limit(0)


def expires(call, status, what):
    """call() under a limit of one poll until a wait has given up, then the default again."""
    from paper_2208_00001_amd import binding as B
    B.set_spin_limit(1)
    codes = set()
    for attempt in range(3):
        print(f"attempt {attempt}: {what} with a spin limit of one poll", flush=True)
        call()
        codes.add(status())
        if GGDT_ERR_WATCHDOG in codes:
            break
    B.set_spin_limit(0)
    assert codes <= {0, GGDT_ERR_WATCHDOG} and GGDT_ERR_WATCHDOG in codes, f"{what}: status {codes}"


@pytest.mark.parametrize("shape,C,lam", [((300, 280), 1, 1.0), ((280, 300), 3, 0.5), ((200, 250), 1, 0.0),
                                         ((300, 700), 4, 0.5), ((60, 70, 50), 1, 0.5), ((40, 150, 130), 1, 1.0),
                                         ((40, 200, 210), 1, 0.5), ((40, 60, 70), 3, 0.5), ((40, 60, 70), 4, 0.5)], ids=str)
def test_forward(shape, C, lam):
    from paper_2208_00001_amd import binding as B
    c = synth.small_case(shape, C=C, seed=130, lam=lam, iterations=1)
    img, m = to_dev(c["image"]), to_dev(c["mask"])
    ws = B.new_workspace(shape, C, img.device)
    fn = B.ggdt2d if len(shape) == 2 else B.ggdt3d

    def call():
        return fn(img, m, c["spacing"], c["v"], c["lam"], 1, workspace=ws)

    expires(call, lambda: B.workspace_status(ws), c["name"])
    out = call()
    assert B.workspace_status(ws) == 0
    assert np.array_equal(to_host(out), oracle.ggdt(c["image"], c["mask"], c["spacing"], c["v"], c["lam"], 1, "f32"))


@pytest.mark.parametrize("shape,C", [((300, 280), 1), ((280, 300), 4), ((60, 70, 50), 1), ((40, 60, 70), 2),
                                     ((40, 150, 130), 1), ((30, 200, 210), 1)], ids=str)
def test_reverse(shape, C):
    from paper_2208_00001_amd import binding as B
    c = synth.small_case(shape, C=C, seed=140, lam=0.5, iterations=1, soft=True, v=10.0)
    W = np.random.default_rng(141).standard_normal(shape).astype(np.float32)
    args = (c["spacing"], c["v"], c["lam"], 1)
    _, rec = oracle.ggdt(c["image"], c["mask"], *args, "f32", records=True)
    img, r, w = to_dev(c["image"]), to_dev(rec), to_dev(W)
    lib = B.load_library()
    n = lib.ggdt_backward_workspace_bytes(len(shape), B._dims(shape), C)
    ws = torch.empty(n, dtype=torch.uint8, device=img.device)

    def call():
        return B.ggdt_backward(img, r, w, *args, workspace=ws)

    expires(call, lambda: B.workspace_status(ws), c["name"])
    gi, gm = call()
    assert B.workspace_status(ws) == 0
    rgi, rgm = oracle.backward(c["image"], rec, W, *args, "f32")
    assert np.array_equal(to_host(gm), rgm.reshape(shape))
    assert np.array_equal(to_host(gi).reshape(rgi.shape), rgi)


@pytest.mark.parametrize("kind", ["volumes", "images", "both"])
def test_batched_reverse(kind):
    from paper_2208_00001_amd import binding as B
    from paper_2208_00001_amd.batched import BatchedPlan
    shapes = [(40, 70, 60), (50, 33, 41)] if kind != "images" else []
    shapes += [(300, 280), (150, 400)] if kind != "volumes" else []
    cs = [synth.small_case(s, C=1, seed=150 + i, lam=0.7, iterations=1, soft=True, v=10.0) for i, s in enumerate(shapes)]
    W = [np.random.default_rng(151 + i).standard_normal(s).astype(np.float32) for i, s in enumerate(shapes)]
    plan = BatchedPlan([dict(image=to_dev(c["image"]), softmask=to_dev(c["mask"]), spacing=c["spacing"], v=c["v"],
                             lam=c["lam"], iterations=1, records=True, grad_out=to_dev(w)) for c, w in zip(cs, W)])
    plan.run()
    plan.check()
    expires(plan.backward, plan.status, f"batched reverse of {kind}")
    grads = plan.backward()
    plan.check()
    for c, w, (gi, gm) in zip(cs, W, grads):
        _, rec = oracle.ggdt(c["image"], c["mask"], c["spacing"], c["v"], c["lam"], 1, "f32", records=True)
        rgi, rgm = oracle.backward(c["image"], rec, w, c["spacing"], c["v"], c["lam"], 1, "f32")
        assert np.array_equal(to_host(gm), rgm.reshape(gm.shape))
        assert np.array_equal(to_host(gi).reshape(rgi.shape), rgi)
    plan.close()
