"""Entry counts of the tile lists beyond 32 bits: the call is refused, and
nothing is placed."""
import numpy as np
import pytest

from paper_2506_12787_amd import synth

pytestmark = pytest.mark.gpu


def test_more_than_2_to_the_32_entries_are_refused():
    """2^26 Gaussians that cover the 64 tiles of a 128 x 128 grid have 2^32 list
    entries, one more than positions of 32 bits number (a sum of the tiles'
    counts in 32 bits is 0). Both ways of sizing the lists have to see it: from
    the count, and at the capacity that an earlier render left."""
    from paper_2506_12787_amd import binding as B
    n, H, W = 1 << 26, 128, 128
    zero = np.zeros(n, np.float32)
    g = {k: zero for k in B.PARAMS}
    g["mean_x"] = g["mean_y"] = np.full(n, 64.0, np.float32)
    g["log_scale_x"] = g["log_scale_y"] = np.full(n, 5.0, np.float32)  # three sigma: 445 pixels
    ctx = B.Context(0)
    try:
        big = ctx.upload_scene(g, H, W)
        print("uploaded", flush=True)
        with pytest.raises(B.SwfError, match="more list entries"):
            ctx.render(big, None, flags=B.NO_DEFORM, batch=1)
        print("refused by its count", flush=True)
        small = synth.gaussians(5000, H, W, seed=3, scale_range=(0.5, 12.0))
        sid = ctx.upload_scene(small, H, W)
        want = ctx.render(sid, None, flags=B.NO_DEFORM, batch=1).cpu().numpy()
        assert ctx.device_status()["list_entries"] > 4096
        with pytest.raises(B.SwfError, match="more list entries"):
            ctx.render(big, None, flags=B.NO_DEFORM, batch=1)
        print("refused at the earlier capacity", flush=True)
        np.testing.assert_array_equal(ctx.render(sid, None, flags=B.NO_DEFORM, batch=1).cpu().numpy(), want)
    finally:
        ctx.close()


def test_the_list_limit_is_on_the_entries_not_on_the_buffer():
    """A list buffer is a quarter larger than what it was sized for, so after a
    render near the context's limit it holds more than that: the next render of
    the same query, sized by the buffer, has as many entries as the first."""
    from paper_2506_12787_amd import binding as B
    n, H, W = 3000, 90, 360  # 138 tiles: past the 2^18 entries up to which no count is waited for
    g = synth.gaussians(n, H, W, seed=8, scale_range=(0.5, 12.0))
    free = B.Context(0)
    sid = free.upload_scene(g, H, W)
    want = free.render(sid, None, flags=B.NO_DEFORM, batch=1).cpu().numpy()
    entries = free.device_status()["list_entries"]
    free.close()
    assert entries > 4096
    tight = B.Context(0, max_list_entries=entries)
    sid = tight.upload_scene(g, H, W)
    for _ in range(3):
        np.testing.assert_array_equal(tight.render(sid, None, flags=B.NO_DEFORM, batch=1).cpu().numpy(), want)
    tight.close()
    short = B.Context(0, max_list_entries=entries - 1)
    sid = short.upload_scene(g, H, W)
    for _ in range(2):
        with pytest.raises(B.SwfError, match="more list entries"):
            short.render(sid, None, flags=B.NO_DEFORM, batch=1)
    short.close()
