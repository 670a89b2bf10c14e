"""GPU tests of the tile lists at the sizes where their kernels change form:
the binning's block sizes and bands, and the per-tile depth sort."""
import threading

import numpy as np
import pytest
import torch

import oracle
import wsr_synth as ws
from paper_2410_18931_amd import WSRContext, globals_tensor, scene_to_device
from tests.gpu_helpers import amb_kw, compare_image, gpu_forward, log, to_views

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,sizes,tile", [
    (1, [(17, 9)], 8), (63, [(64, 64)], 16), (256, [(100, 52)], 8), (257, [(70, 45), (33, 81)], 16),
    (1025, [(200, 120)], 32), (22000, [(32767, 20)], 8), (70000, [(1280, 300)], 8)])
def test_images_across_binning_block_sizes(n, sizes, tile):
    """Blocks of 256 (up to the last one's single Gaussian), 512 and 1,024
    Gaussians, views whose rows of tiles are all one band or (4,096 tiles
    wide) one row a band."""
    sc, _, st = ws.make_scene("c1", n=n)
    st = st.copy(tile=tile)
    cams = [ws.look_at_camera((0.0, 0.0, -4.0 - k), w, h) for k, (w, h) in enumerate(sizes)]
    log(f"case: binning n={n} {sizes} tile {tile}")
    ctx, dev, g, (rgb, den) = gpu_forward(sc, cams, st)
    for v, cam in enumerate(cams):
        w, h = cam["width"], cam["height"]
        crop = (0, 0, w, h) if w < 1000 else (w // 2 - 60, 0, w // 2 + 68, min(h, 64))
        x0, y0, x1, y1 = crop
        compare_image(to_views(ctx, rgb)[v][y0:y1, x0:x1], oracle.render(sc, cam, st, crop=crop, **amb_kw(st)),
                      label=f"n={n} view {v}")


@pytest.mark.parametrize("length", [1, 2, 63, 64, 65, 256, 257, 2047, 2048, 2049, 4097, 8192, 8193, 16384])
@pytest.mark.parametrize("depths", ["spread", "clumped", "equal"])
def test_sorted_list_order(length, depths):
    """One tile that every splat reaches: the list is in depth order, equal
    depths in id order, and every entry keeps its slot.  Distinct depths lie
    further apart than their float32 rounding."""
    rng = np.random.default_rng(length)
    sc, _, st = ws.make_scene("c1", n=length)
    st = st.copy(weight_kind="dir", tile=16)
    z = rng.permutation(length) * (2.0 / length)
    if depths == "clumped":      # half of them within a thousandth of the range
        z = np.where(z < 1.0, 1.0 + z * 2e-3, z)
        z = np.round(z * 2.0 ** 20) / 2.0 ** 20
    elif depths == "equal":
        z = np.full(length, 0.5)
    sc["means"] = np.stack([np.zeros(length), np.zeros(length), z]).astype(np.float32)
    sc["log_scales"] = np.full((3, length), -1.0, np.float32)
    cams = [ws.look_at_camera((0.0, 0.0, -4.0), 16, 16)]
    log(f"case: sort length={length} {depths}")
    ctx = WSRContext(length, cams, st)
    g = globals_tensor(st)
    ctx.project(scene_to_device(sc), g)
    ctx.bin(grow=True)
    assert ctx.last_pairs == length
    ctx.render_sorted(g)
    torch.cuda.synchronize()
    ctx.check()
    # pair buffer: 40 bytes per pair of gradients, then the (id, slot) list entries
    ent = ctx.pairs[40 * ctx.capacity: 48 * ctx.capacity].view(torch.int32).cpu().numpy().reshape(-1, 2)[:length]
    depth = sc["means"][2] + np.float32(4.0)
    np.testing.assert_array_equal(ent[:, 0], np.argsort(depth, kind="stable"))
    np.testing.assert_array_equal(ent[:, 1], ent[:, 0])


def test_pair_counts_read_back_by_several_threads():
    """Each thread reads the pair count of its own context on its own stream,
    and gets that of the same scene binned alone."""
    def count(n, repeat):
        sc, cams, st = ws.make_scene("c1", n=n)
        ctx = WSRContext(n, cams, st)
        dev, g = scene_to_device(sc), globals_tensor(st)
        torch.cuda.current_stream().synchronize()
        got = set()
        for _ in range(repeat):
            ctx.project(dev, g)
            ctx.bin(grow=True)
            got.add(ctx.last_pairs)
        return got

    sizes = [500, 1000, 2000, 4000]
    alone = [count(n, 1) for n in sizes]
    found = [None] * len(sizes)

    def work(k):
        with torch.cuda.stream(torch.cuda.Stream()):
            found[k] = count(sizes[k], 20)

    log("case: pair counts from four threads")
    threads = [threading.Thread(target=work, args=(k,)) for k in range(len(sizes))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert found == alone
