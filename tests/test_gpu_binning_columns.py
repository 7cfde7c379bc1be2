"""Column prefixes of the tile lists where a thread takes more than 32 rows of
its column (summed, then read again and rewritten in place): the lists against
the full 64-bit sort of the same records, bitwise, on both forms of the kernel."""
import numpy as np
import pytest

from paper_2506_12787_amd import synth

pytestmark = pytest.mark.gpu

# n, H, W, batch: 547 blocks of 256 pairs over 16 threads per column (35 rows each); 132 blocks of 2048 pairs over
# four threads per column (33 rows each: 8 queries of 2112 columns are past the 16-thread form's 16,384)
CASES = [(140_000, 90, 360, 1), (270_000, 360, 1440, 8)]


@pytest.mark.parametrize("n,H,W,nb", CASES)
@pytest.mark.parametrize("wrap", [False, True])
def test_lists_equal_the_full_sort(n, H, W, nb, wrap):
    from paper_2506_12787_amd import binding as B
    ctx = B.Context(0)
    try:
        tiles = -(-H // 16) * -(-W // 16)
        sid = ctx.upload_scene(synth.gaussians(n, H, W, seed=n, scale_range=(0.5, 2.0)), H, W)
        flags = B.NO_DEFORM | (B.WRAP_AZIMUTH if wrap else 0)
        out, keys = [], []
        for f in (flags, flags | B.FULL_SORT):
            out.append(ctx.render(sid, None, flags=f, batch=nb).cpu().numpy())
            keys.append(ctx.debug_keys(nb, n, tiles))
            print("rendered", f, flush=True)
        for k in ("counts", "keys", "values", "ranges"):
            np.testing.assert_array_equal(keys[0][k], keys[1][k], err_msg=k)
        np.testing.assert_array_equal(out[0], out[1])
    finally:
        ctx.close()
