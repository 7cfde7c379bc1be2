"""Per-tile lists by binning against the full 64-bit sort of the same records
(bitwise): every form of grid the binning takes, around the sizes at which its
blocks, waves and lists change (64-pair chunks, 256- to 2048-pair blocks, rows
dealt over 1 to 12 waves, segments of 8 columns), with a periodic azimuth and
with 8 x 8 tiles; and the culled-pair counts of both paths."""
import numpy as np
import pytest

from paper_2506_12787_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2506_12787_amd import binding
    c = binding.Context(0)
    yield c
    c.close()


# n, H, W, batch, largest log-scale (pixels)
CASES = [
    (1, 16, 16, 1, 4.0), (50, 16, 16, 3, 4.0), (63, 16, 17, 2, 4.0), (65, 7, 200, 1, 12.0), (256, 33, 130, 2, 12.0),
    (257, 128, 129, 1, 12.0), (1025, 90, 360, 2, 12.0), (700, 90, 360, 600, 6.0), (4097, 180, 720, 1, 20.0),
    (9001, 360, 1440, 2, 60.0), (2049, 4096, 256, 1, 200.0), (3000, 144, 1824, 150, 30.0),
    (10, 16, 16, 300, 4.0), (5, 16, 16, 128, 4.0), (5, 16, 16, 129, 4.0), (9, 30, 50, 130, 9.0), (40_000, 90, 360, 1, 6.0), (33_000, 60, 100, 3, 6.0),
]


@pytest.mark.parametrize("n,H,W,nb,smax", CASES)
@pytest.mark.parametrize("mode", ["plane", "wrap", "tile8"])
def test_lists_equal_the_full_sort(ctx, n, H, W, nb, smax, mode):
    from paper_2506_12787_amd import binding as B
    tile = 8 if mode == "tile8" else 16
    tiles = -(-H // tile) * -(-W // tile)
    if tiles > 4096:
        pytest.skip("beyond the binning path's tiles per query")
    g = synth.gaussians(n, H, W, seed=41 + n, scale_range=(0.5, smax))
    r = np.random.default_rng(n)
    off = r.uniform(size=n) < 0.1
    g["mean_y"] = np.where(off, -5000.0, g["mean_y"]).astype(np.float32)
    g["log_scale_x"] = np.where(r.uniform(size=n) < 0.05, np.nan, g["log_scale_x"]).astype(np.float32)
    flags = B.NO_DEFORM | {"plane": 0, "wrap": B.WRAP_AZIMUTH, "tile8": B.TILE8}[mode]
    sid = ctx.upload_scene(g, H, W)
    got = []
    for f in (flags, flags | B.FULL_SORT):
        out = ctx.render(sid, None, flags=f, batch=nb).cpu().numpy()
        got.append((out, ctx.debug_keys(nb, n, tiles), ctx.device_status()))
    ctx.release_scene(sid)
    (a, ka, sa), (b, kb, sb) = got
    for k in ("counts", "keys", "values", "ranges"):
        np.testing.assert_array_equal(ka[k], kb[k], err_msg=k)
    np.testing.assert_array_equal(a, b)
    # (a render whose lists outgrow the context's buffers runs twice: flags and rerenders may differ)
    for k in ("pairs", "culled_nonfinite", "culled_offgrid", "list_entries"):
        assert sa[k] == sb[k], k
    assert sa["pairs"] == n * nb
