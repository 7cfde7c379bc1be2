"""The deterministic backward of a small render, whose entry count the host has
not waited for: it is enqueued behind the render without a wait, and gives the
gradients that it gives after the count has been read."""
import numpy as np
import pytest

from paper_2506_12787_amd import synth

pytestmark = pytest.mark.gpu


def test_deterministic_backward_returns_after_enqueueing():
    import torch
    from paper_2506_12787_amd import binding as B
    n, H, W, nb = 60, 48, 64, 4  # 12 tiles: 2880 entries at most
    ctx = B.Context(0)
    sid = ctx.upload_scene(synth.gaussians(n, H, W, seed=5, scale_range=(0.5, 12.0)), H, W)
    go = torch.from_numpy(np.random.default_rng(1).standard_normal((nb, H, W)).astype(np.float32)).cuda()
    a = torch.randn((8192, 8192), device="cuda")
    b = torch.empty_like(a)
    torch.mm(a, a, out=b)
    aux = torch.empty(8 * nb * H * W, dtype=torch.uint8, device="cuda")
    out = torch.empty((nb, H, W), device="cuda")
    stream, done = torch.cuda.Stream(), torch.cuda.Event()
    grads = [{k: torch.zeros(n, device="cuda") for k in B.PARAMS[:7]} for _ in range(3)]

    def step(gr, behind=0, count=False):
        with torch.cuda.stream(stream):
            ctx.render(sid, None, flags=B.NO_DEFORM | B.KEEP_AUX, batch=nb, out=out, aux=aux)
            if count:
                assert ctx.device_status()["list_entries"] > 0
            for _ in range(behind):  # 7 ms each
                torch.mm(a, a, out=b)
            done.record()
            ctx.render_backward(sid, None, B.NO_DEFORM | B.DETERMINISTIC, go, aux, gr)
            return done.query()

    torch.cuda.synchronize()
    step(grads[0])  # sizes the workspace (an allocation waits)
    torch.cuda.synchronize()
    waited = step(grads[1], behind=20)
    assert not waited, "the call waited for work queued before it"
    torch.cuda.synchronize()
    step(grads[2], count=True)
    torch.cuda.synchronize()
    for k in B.PARAMS[:7]:
        assert torch.count_nonzero(grads[0][k]) > 0, k
        for g in grads[1:]:
            assert torch.equal(grads[0][k], g[k]), k
    ctx.release_scene(sid)
    ctx.close()
