"""GPU test of calls whose pair capacity is smaller than the binning's: every
stage stays within the buffer that it is given."""
import ctypes as C

import pytest
import torch

import wsr_synth as ws
from paper_2410_18931_amd import WSRContext, _lib, globals_tensor, scene_to_device
from tests.gpu_helpers import log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", [8, 16, 32])
@pytest.mark.parametrize("sorted_path", [False, True])
def test_stages_without_a_pair_buffer_after_a_full_binning(tile, sorted_path):
    """Lists are binned with room for every pair; the later stages are then
    called with capacity 0 and no buffer: they see empty lists, so the image is
    the background and the per-Gaussian gradients are zero."""
    n = 1500
    sc, cams, st = ws.make_scene("c1", n=n)
    st = st.copy(tile=tile, weight_kind="dir" if sorted_path else st.weight_kind)
    log(f"case: capacity 0, tile {tile}, sorted {sorted_path}")
    ctx = WSRContext(n, cams, st)
    dev, g = scene_to_device(sc), globals_tensor(st)
    ctx.project(dev, g)
    ctx.bin(grow=True)
    # no list is split, so no partial sums are kept in the pair buffer
    assert 0 < ctx.last_pairs <= ctx.capacity and n <= 2048
    null, P = C.c_void_p(None), ctx.total_pixels
    p = lambda t: C.c_void_p(t.data_ptr())  # noqa: E731
    stream = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    rgb = torch.full((P, 3), float("nan"), device="cuda")
    den = torch.full((P,), float("nan"), device="cuda")
    views = (ctx.cams_c, ctx.nv, C.byref(ctx.params), n)
    if sorted_path:
        _lib.check("wsr_sort_tiles", ctx.lib.wsr_sort_tiles(*views, p(ctx.ws), ctx.ws_bytes, null, 0, stream))
        blend = _lib.WsrBlend(0.99, 0.0, 0.0, 0)
        _lib.check("wsr_render_sorted", ctx.lib.wsr_render_sorted(*views, p(g), C.byref(blend), p(ctx.ws), ctx.ws_bytes,
                                                                  null, 0, p(rgb), p(den), stream))
        assert torch.equal(den, torch.ones_like(den))
    else:
        _lib.check("wsr_render_fwd", ctx.lib.wsr_render_fwd(*views, p(g), p(ctx.ws), ctx.ws_bytes, null, 0, p(rgb),
                                                            p(den), null, stream))
        assert torch.equal(den, g[2].expand(P))
        grads = ctx.alloc_grads(dev)
        gs, scene = ctx.grads_struct(grads), ctx.scene_struct(dev)
        dL = torch.ones_like(rgb)
        _lib.check("wsr_render_bwd", ctx.lib.wsr_render_bwd(
            C.byref(scene), *views[:3], p(g), p(ctx.ws), ctx.ws_bytes, null, 0, p(dL), p(rgb), p(den), C.byref(gs),
            null, stream))
        for k in ("means", "log_scales", "quats", "sh", "opacity_logit"):
            assert torch.equal(grads[k], torch.zeros_like(grads[k])), k
    torch.testing.assert_close(rgb, g[3:].expand(P, 3), rtol=1e-6, atol=0)
