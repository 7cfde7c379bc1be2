"""The MLP backward takes only the pairs with a gradient, in groups of 32 rows:
a zero upstream gradient gives exact zeros, and a batch's gradient is the sum of
its queries' gradients taken alone (whose groups cut the rows elsewhere), at pair
counts around the groups, the 64-row blocks, the 256-row blocks of the counting
pass and the 1024 groups of a listing block."""
import numpy as np
import pytest

from paper_2506_12787_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    from paper_2506_12787_amd import binding
    c = binding.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("mlp", ["bf16", "fp32"])
@pytest.mark.parametrize("n,layers", [(1, 4), (31, 4), (33, 2), (64, 4), (127, 3), (255, 4), (1000, 4), (12_000, 4),
                                      (50, 1)])
def test_batch_gradient_is_the_sum_of_its_queries(lib, n, layers, mlp):
    import torch
    from paper_2506_12787_amd import binding as B
    from paper_2506_12787_amd.autograd import Renderer
    H, W, nb = 33, 49, 3
    flags = (B.MLP_BF16 if mlp == "bf16" else B.MLP_FP32) | B.DETERMINISTIC
    m = Renderer(synth.gaussians(n, H, W, seed=n), H, W, mlp=synth.mlp_weights(seed=n + 1, n_hidden=layers), lib=lib)
    tx = torch.from_numpy(synth.tx_positions(nb, seed=n + 2)).cuda()
    up = torch.from_numpy(np.random.default_rng(n).normal(size=(nb, H, W)).astype(np.float32)).cuda()
    up[:, :, :20] = 0.0  # pairs seen only there have no gradient

    def grads(t, u):
        out = m(t, flags=flags)
        return [g.double() for g in torch.autograd.grad(out, list(m.parameters()), u)]

    assert all(bool((g == 0).all()) for g in grads(tx, torch.zeros_like(up)))
    whole = grads(tx, up)
    alone = [grads(tx[q:q + 1].contiguous(), up[q:q + 1].contiguous()) for q in range(nb)]
    for k, g in enumerate(whole):
        parts = torch.stack([a[k] for a in alone])
        # the same terms added in other orders: FP32 sums of at most 3 n rows
        bound = 4 * (3 * n) ** 0.5 * 2.0 ** -24 * 64 * float(parts.abs().max())
        assert float((g - parts.sum(0)).abs().max()) <= bound + 1e-30, k
