"""GPU tests of threads that end beside other work of the process."""
import os
import threading
import time

import pytest
import torch

import wsr_synth as ws
from paper_2410_18931_amd import WSRContext, globals_tensor, scene_to_device
from paper_2410_18931_amd.graph import GraphStep
from tests.gpu_helpers import log

pytestmark = pytest.mark.gpu


def test_a_thread_that_read_a_pair_count_ends_during_a_capture():
    """A capture in the strictest mode (any thread's unsafe call breaks it) goes
    on over the end of a thread that has read status words, and its replays
    give the eager results."""
    log("case: thread end during capture")
    sc, cams, st = ws.make_scene("c1", n=700)
    dev, g = scene_to_device(sc), globals_tensor(st)
    ready, leave, count = threading.Event(), threading.Event(), []

    def reader():
        ctx = WSRContext(700, cams, st)
        with torch.cuda.stream(torch.cuda.Stream()):
            ctx.project(dev, g)
            ctx.bin(grow=True)
        count.append(ctx.last_pairs)
        ready.set()
        leave.wait(60)

    t = threading.Thread(target=reader)
    t.start()
    assert ready.wait(60)

    class Step(GraphStep):
        runs = 0

        def _enqueue(self):
            super()._enqueue()
            self.runs += 1
            if self.runs == 2:  # under capture: the other thread ends now, its thread-local objects included
                leave.set()
                t.join(60)
                for _ in range(1000):
                    if not os.path.exists(f"/proc/self/task/{t.native_id}"):
                        break
                    time.sleep(0.01)
                assert not os.path.exists(f"/proc/self/task/{t.native_id}")

    ctx = WSRContext(700, cams, st)
    r = torch.from_numpy(ws.upstream_grad(cams, seed=0)[0].reshape(-1, 3)).cuda()
    step = Step(ctx, dev, g, dL=r)
    assert step.runs == 2
    eager = WSRContext(700, cams, st)
    rgb, den = eager.forward(dev, g)
    grads = eager.render_bwd(dev, g, r, rgb, den)
    assert count == [eager.last_pairs]
    for _ in range(3):
        step.rgb.fill_(float("nan"))
        step.replay()
        torch.cuda.synchronize()
        step.check()
        assert torch.equal(step.rgb, rgb)
        for k in ("means", "sh", "globals"):
            assert torch.equal(step.grads[k], grads[k]), k
