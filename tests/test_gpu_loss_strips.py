"""GPU tests of the loss at the sizes where large images are cut into strips
(64 columns, 34 rows): strips that end with one column or row, with all of
them, several views, and the narrow views that stay with tiles."""
import numpy as np
import pytest
import torch

import wsr_synth as ws
from oracle import train as T
from paper_2410_18931_amd.train import Loss
from tests.gpu_helpers import log
from tests.test_gpu_train import DL_TOL, LOSS_RTOL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [[(961, 511)], [(1024, 442)], [(703, 341), (65, 35), (705, 308)], [(639, 705)],
                                   [(640, 703)], [(65, 7000)], [(300, 100)] * 17, [(17, 26500)]])
def test_loss_of_large_images(sizes):
    log(f"case: loss {sizes}")
    rng = np.random.default_rng(len(sizes))
    imgs = [rng.random((h, w, 3)).astype(np.float32) for w, h in sizes]
    tgts = [np.clip(a + rng.normal(0, 0.1, a.shape), 0, 1).astype(np.float32) for a in imgs]
    flat = lambda xs: torch.from_numpy(np.concatenate([x.reshape(-1, 3) for x in xs])).cuda()  # noqa: E731
    loss = Loss([ws.look_at_camera((0.0, 0.0, -4.0), w, h) for w, h in sizes])
    value, dL = loss(flat(imgs), flat(tgts))
    torch.cuda.synchronize()
    ref, ref_g = T.loss_views(imgs, tgts)
    assert abs(value.item() - ref) <= LOSS_RTOL * abs(ref)
    # each view against its own largest gradient (their scales differ with their sizes)
    got, at = dL.cpu().numpy().astype(np.float64), 0
    for (w, h), g in zip(sizes, ref_g):
        err = np.abs(got[at:at + w * h] - g.reshape(-1, 3)).max()
        at += w * h
        assert err <= DL_TOL * np.abs(g).max(), (w, h, err)
