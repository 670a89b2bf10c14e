"""GPU tests of the binning's forms against each other: a view's lists do not
depend on the block and band sizes, which follow all views of the call."""
import numpy as np
import pytest
import torch

import oracle
import wsr_synth as ws
from paper_2410_18931_amd import WSRContext, globals_tensor, scene_to_device
from tests import plan_lib
from tests.gpu_helpers import amb_kw, compare_image, gpu_forward, log, to_views

pytestmark = pytest.mark.gpu


def _plan(n, sizes, tile):
    """(Gaussians per block, tiles of the largest band, bands of the tallest view)."""
    plan = plan_lib.load()
    t = [((w + tile - 1) // tile, (h + tile - 1) // tile) for w, h in sizes]
    rows = [min(plan.bin_rows(tx, max(ty for _, ty in t)), ty) for tx, ty in t]
    return (plan.bin_chunk(n, len(t), sum(x * y for x, y in t), max(x * y for x, y in t)),
            max(r * tx for r, (tx, _) in zip(rows, t)), max((ty + r - 1) // r for r, (_, ty) in zip(rows, t)))


def _entries(sc, cams, st):
    n = sc["means"].shape[1]
    ctx = WSRContext(n, cams, st)
    ctx.project(scene_to_device(sc), globals_tensor(st))
    ctx.bin(grow=True)
    torch.cuda.synchronize()
    # pair buffer: 40 bytes per pair of gradients, then the (id, slot) list entries
    ent = ctx.pairs[40 * ctx.capacity: 40 * ctx.capacity + 8 * ctx.last_pairs]
    return ent.view(torch.int32).reshape(-1, 2).cpu().numpy()


@pytest.mark.parametrize("n,size,tile,other,alone,both", [
    # bands of 1, 31, 32, 33 and two rows of 16 tiles: bit by bit up to 32
    (300, (8, 8), 8, (320, 200), (256, 1, 1), (256, 200, 5)),
    (3000, (248, 48), 8, (320, 200), (256, 31, 6), (256, 200, 5)),
    (3000, (256, 48), 8, (320, 200), (256, 32, 6), (256, 200, 5)),
    (3000, (264, 48), 8, (320, 200), (256, 33, 6), (256, 200, 5)),
    (3000, (256, 180), 16, (640, 400), (256, 32, 6), (256, 200, 5)),
    # one row of tiles: a single band; a width whose tags need a pitch of their own
    (3000, (1024, 8), 8, (1024, 1024), (256, 128, 1), (256, 2816, 6)),
    # blocks of 256 and 2,048, of 1,024 and 4,096 Gaussians; bands that LDS cuts to a few rows
    (20_000, (128, 128), 8, (2560, 1440), (256, 48, 6), (2048, 4800, 12)),
    (200_000, (128, 128), 8, (3840, 2160), (1024, 48, 6), (4096, 4800, 27)),
    (90_000, (1280, 300), 8, (16384, 64), (1024, 1120, 6), (2048, 4096, 6)),
])
def test_lists_do_not_depend_on_the_other_views(n, size, tile, other, alone, both):
    sc, _, st = ws.make_scene("c1", n=n)
    st = st.copy(tile=tile)
    log(f"case: bands n={n} {size} beside {other}, tile {tile}")
    assert _plan(n, [size], tile) == alone and _plan(n, [size, other], tile) == both
    assert plan_lib.load().few_tiles() == 32
    cam, cam2 = ws.look_at_camera((0.0, 0.0, -4.0), *size), ws.look_at_camera((0.5, 0.0, -5.0), *other)
    one, two = _entries(sc, [cam], st), _entries(sc, [cam, cam2], st)
    assert len(one) > 0
    np.testing.assert_array_equal(one, two[:len(one)])
    # every slot once, a Gaussian's in a row, Gaussians in order
    order = np.argsort(one[:, 1], kind="stable")
    np.testing.assert_array_equal(one[order, 1], np.arange(len(one)))
    assert (np.diff(one[order, 0]) >= 0).all()


@pytest.mark.parametrize("n,size,tile", [(300, (8, 8), 8), (1500, (248, 48), 8), (1500, (256, 48), 8), (1500, (264, 48), 8),
                                         (1500, (256, 180), 16)])
def test_images_of_few_tiles_a_band(n, size, tile):
    sc, _, st = ws.make_scene("c1", n=n)
    st = st.copy(tile=tile)
    cams = [ws.look_at_camera((0.0, 0.0, -4.0), *size)]
    log(f"case: few tiles n={n} {size} tile {tile}")
    ctx, dev, g, (rgb, den) = gpu_forward(sc, cams, st)
    compare_image(to_views(ctx, rgb)[0], oracle.render(sc, cams[0], st, **amb_kw(st)), label=f"n={n} {size}")
