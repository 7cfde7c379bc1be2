"""Device memory that the MLP backward takes: its rows of gradients and the
slices of the launches that it runs, not those of other forms of it."""
import numpy as np
import pytest

from paper_2506_12787_amd import synth

pytestmark = pytest.mark.gpu


def _step(ctx, n, nb, H=90, W=360):
    """Bytes that the first backward of this context allocates."""
    import torch
    from paper_2506_12787_amd import binding as B
    r = np.random.default_rng(3)
    dims = [89, 256, 256, 7]
    Ws = [(0.05 * r.standard_normal((o, i))).astype(np.float32) for i, o in zip(dims, dims[1:])]
    bs = [np.zeros(o, np.float32) for o in dims[1:]]
    sid = ctx.upload_scene(synth.gaussians(n, H, W, seed=4, scale_range=(0.5, 2.0)), H, W, mlp=(Ws, bs))
    tx = torch.from_numpy(synth.tx_positions(nb, seed=2)).cuda()
    out, aux = ctx.render(sid, tx, flags=B.MLP_BF16 | B.KEEP_AUX)
    gr = {k: torch.empty(n, device="cuda") for k in B.PARAMS[:7]}
    gr["weight"] = [torch.empty(w.shape, device="cuda") for w in Ws]
    gr["bias"] = [torch.empty(b.shape, device="cuda") for b in bs]
    go = torch.ones_like(out)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    ctx.render_backward(sid, tx, B.MLP_BF16, go, aux, gr)
    torch.cuda.synchronize()
    used = free - torch.cuda.mem_get_info()[0]
    assert all(bool(torch.isfinite(g).all()) for g in gr["weight"])
    ctx.release_scene(sid)
    return used


def test_bf16_backward_scratch():
    from paper_2506_12787_amd import binding as B
    n, nb = 200_000, 32
    P = n * nb
    small, ctx = B.Context(0), B.Context(0)
    try:
        _step(small, 100, 2)  # the kernels are loaded before the memory is looked at
        used = _step(ctx, n, nb)
        # gradient rows of two layers, 22 words of gradients and 3 bits' words (of 32 rows) per pair, the sums per
        # Gaussian, and the slices of the weight gradient; each buffer is a quarter larger than what was asked for
        need = 2 * 512 * P + 4 * (8 + 7 + 7) * P + 4 * 3 * P // 32 + 1024 * n + 256 * 258 * 1024
        print("scratch", used, "needed", need, flush=True)
        assert used <= 1.25 * need + (64 << 20)
    finally:
        small.close()
        ctx.close()
