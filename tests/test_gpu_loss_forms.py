"""GPU tests of the loss where its form changes: strips (64 columns, 34 rows)
that end with one column or row, or with all of them, launches of 16 views of
which some take strips and some tiles in one workspace."""
import numpy as np
import pytest
import torch

import wsr_synth as ws
from oracle import train as T
from paper_2410_18931_amd.train import Loss
from tests import plan_lib
from tests.gpu_helpers import log
from tests.test_gpu_train import DL_TOL, LOSS_RTOL

pytestmark = pytest.mark.gpu


def _cams(sizes):
    return [ws.look_at_camera((0.0, 0.0, -4.0), w, h) for w, h in sizes]


@pytest.mark.parametrize("sizes,forms", [
    ([(1025, 647)], ["strips"]), ([(1024, 680)], ["strips"]), ([(703, 341), (65, 35), (705, 477)], ["strips"]),
    ([(961, 511)], ["strips"]), ([(300, 100)] * 17, ["strips", "tiles"]),
    ([(60, 50)] * 16 + [(1025, 647)], ["tiles", "strips"]),
    ([(700, 500)] * 2 + [(64, 40)] * 14 + [(33, 17)] * 16 + [(1100, 680)], ["strips", "tiles", "strips"])])
def test_loss_of_each_form(sizes, forms):
    log(f"case: loss {sizes}")
    assert plan_lib.loss_forms(sizes) == forms
    rng = np.random.default_rng(len(sizes))
    imgs = [rng.random((h, w, 3)).astype(np.float32) for w, h in sizes]
    tgts = [np.clip(a + rng.normal(0, 0.1, a.shape), 0, 1).astype(np.float32) for a in imgs]
    flat = lambda xs: torch.from_numpy(np.concatenate([x.reshape(-1, 3) for x in xs])).cuda()  # noqa: E731
    value, dL = Loss(_cams(sizes))(flat(imgs), flat(tgts))
    torch.cuda.synchronize()
    ref, ref_g = T.loss_views(imgs, tgts)
    assert abs(value.item() - ref) <= LOSS_RTOL * abs(ref)
    # each view against its own largest gradient (their scales differ with their sizes)
    got, at = dL.cpu().numpy().astype(np.float64), 0
    for (w, h), g in zip(sizes, ref_g):
        err = np.abs(got[at:at + w * h] - g.reshape(-1, 3)).max()
        at += w * h
        assert err <= DL_TOL * np.abs(g).max(), (w, h, err)


@pytest.mark.parametrize("size,copies", [((800, 600), 2), ((703, 341), 4), ((130, 777), 8), ((64, 1020), 8)])
def test_strips_give_the_tiles_bits(size, copies):
    """A view alone takes tiles, a power of two of copies of it strips: each
    copy's gradient is the view's, divided by their number, to the bit."""
    w, h = size
    log(f"case: loss bits {size} x {copies}")
    assert plan_lib.loss_forms([size]) == ["tiles"] and plan_lib.loss_forms([size] * copies) == ["strips"]
    rng = np.random.default_rng(w)
    img = rng.random((h, w, 3)).astype(np.float32)
    tgt = np.clip(img + rng.normal(0, 0.1, img.shape), 0, 1).astype(np.float32)
    img[: h // 4] = tgt[: h // 4]           # equal, dark and bright parts
    img[h // 4: h // 3, : w // 2] = tgt[h // 4: h // 3, : w // 2] = 0.0
    img[h // 2: h // 2 + 40] *= 30.0
    a, b = (torch.from_numpy(x.reshape(-1, 3)).cuda() for x in (img, tgt))
    one, dL_one = Loss(_cams([size]))(a, b)
    many, dL = Loss(_cams([size] * copies))(a.repeat(copies, 1), b.repeat(copies, 1))
    torch.cuda.synchronize()
    for k in range(copies):
        assert torch.equal(copies * dL[k * w * h:(k + 1) * w * h], dL_one), k
    # the shares are summed in FP64 in another order
    assert abs(many.item() - one.item()) <= 2.0 ** -22 * abs(one.item())
