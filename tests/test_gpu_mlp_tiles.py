"""The BF16 MLP's tile shapes against one another (bitwise: every shape forms the
same products and sums). Batches around the sizes where the shape changes: few
Gaussians per query cut as flat rows (several queries per tile), batches of one
and of two rounds over the compute units;
residuals against the tiling that never straddles two queries, and the stored
activations of a batch against those of its queries alone. Likewise the FP32
MLP's blocks."""
import numpy as np
import pytest

from paper_2506_12787_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pair():
    from paper_2506_12787_amd import binding
    a, b = binding.Context(0), binding.Context(0, mlp_pairs_per_wave=32)
    yield a, b
    a.close()
    b.close()


SHAPES = [(1, 1), (1, 300), (3, 33), (6, 70), (7, 70), (19, 41), (43, 9), (50, 1), (50, 1024), (63, 5), (64, 1),
          (65, 256), (100, 77), (383, 3), (384, 2), (385, 300), (16384, 1), (16385, 1), (20011, 5), (98304, 1),
          (98305, 1), (100_000, 1), (33_000, 7)]


@pytest.mark.parametrize("n,nb", SHAPES)
@pytest.mark.parametrize("hidden_layers", [4, 1])
def test_residuals_do_not_depend_on_the_tiles(pair, n, nb, hidden_layers):
    import torch
    from paper_2506_12787_amd import binding as B
    g = synth.gaussians(n, 90, 360, seed=n)
    mlp = synth.mlp_weights(seed=n + 1, n_hidden=hidden_layers, out_scale=1.0)
    tx = torch.from_numpy(synth.tx_positions(nb, seed=n + 2)).cuda()
    out = []
    for c in pair:
        sid = c.upload_scene(g, 90, 360, mlp=mlp)
        out.append(c.debug_deform(sid, tx, B.MLP_BF16))
        torch.cuda.synchronize()
        c.release_scene(sid)
    assert torch.equal(out[0], out[1])


@pytest.mark.parametrize("n,nb", [(50, 9), (385, 3), (20011, 5)])
def test_stored_activations_do_not_depend_on_the_batch(pair, n, nb):
    import torch
    from paper_2506_12787_amd import binding as B
    from paper_2506_12787_amd.autograd import Renderer
    lib = pair[0]
    m = Renderer(synth.gaussians(n, 32, 48, seed=n), 32, 48, mlp=synth.mlp_weights(seed=n + 1), lib=lib)
    tx = torch.from_numpy(synth.tx_positions(nb, seed=n + 2)).cuda()

    def pattern(t):
        out = m(t, flags=B.MLP_BF16)
        torch.autograd.grad(out, list(m.parameters()), torch.ones_like(out))
        return lib.debug_relu_pattern(t.shape[0], n, 4)

    whole = pattern(tx)
    for q in range(nb):
        np.testing.assert_array_equal(whole[q], pattern(tx[q:q + 1].contiguous())[0])


@pytest.mark.parametrize("n,nb", [(1, 1), (15, 2), (16, 3), (17, 5), (64, 2), (8192, 2), (8193, 2), (12_305, 4),
                                  (16_384, 3), (16_385, 2), (24_577, 3)])
@pytest.mark.parametrize("hidden_layers", [1, 4, 7])
def test_fp32_residuals_do_not_depend_on_the_blocks(pair, n, nb, hidden_layers):
    """64- and 16-pair blocks form the same sums: a batch's residuals are those of its queries alone, whose pairs
    fall into other blocks (the kinds change at 512 groups of 16 pairs and at whole rounds of 1024)."""
    import torch
    from paper_2506_12787_amd import binding as B
    lib = pair[0]
    mlp = synth.mlp_weights(seed=n + 1, n_hidden=hidden_layers, out_scale=1.0)
    sid = lib.upload_scene(synth.gaussians(n, 90, 360, seed=n), 90, 360, mlp=mlp)
    tx = torch.from_numpy(synth.tx_positions(nb, seed=n + 2)).cuda()
    whole = lib.debug_deform(sid, tx, B.MLP_FP32)
    for q in range(nb):
        assert torch.equal(whole[q], lib.debug_deform(sid, tx[q:q + 1].contiguous(), B.MLP_FP32)[0]), q
    lib.release_scene(sid)
