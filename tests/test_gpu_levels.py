"""Tile runs that leave the event rounds (too many events, full lists, subbins
above 60,000), against the oracle, byte for byte: chains wound through every
tile, so that a run has many points and levels to raise, one bin in falling
order, and both mixed with tiles of small subbins; every repair scheduler, tile
shape and sweep order, and the batch call."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

BARRIER = 100.0  # in a bin of its own at a bound of 10


@pytest.fixture(scope="module")
def P():
    import paper_2603_26968_amd as P
    return P


def wound(blocks, rows, cols, every=2):
    """A chain wound through `blocks` blocks of rows x cols, laid side by side:
    along row 0, down one column, back along row `every`, and so on, then into
    the next block; its values fall along it, the rest lies in another bin."""
    order = []
    for b in range(blocks):
        x0, right = b * cols, True
        used = list(range(0, rows, every))
        used = used[:len(used) - (len(used) + 1) % 2]  # an odd number: out on the right
        down = b % 2 == 0
        for n, y in enumerate(used):
            yy = y if down else used[-1] - y
            xs = range(x0, x0 + cols - 1) if right else range(x0 + cols - 2, x0 - 1, -1)
            order += [(yy, x) for x in xs]
            if n + 1 < len(used):
                x = x0 + cols - 2 if right else x0
                step = 1 if down else -1
                order += [(yy + step * k, x) for k in range(1, every)]
            right = not right
        order += [(order[-1][0], x0 + cols - 1)]  # the way into the next block
    f = np.full((rows, blocks * cols), BARRIER)
    y, x = np.array(order).T
    f[y, x] = np.arange(len(order), 0, -1) / 2.0 ** 19
    return f


def fields():
    rng = np.random.default_rng(12)
    w = wound(3, 31, 64)
    yield "wound 2D", w, 0
    yield "wound 2D, 16 rows", wound(4, 15, 128), 0
    # more than 255 levels in a tile of either shape, entered from outside
    assert (w[:31, :64] < BARRIER).sum() > 500
    yield "falling 2D", -np.arange(70 * 150).reshape(70, 150) / 2.0 ** 19, 0
    yield "falling 3D", -np.arange(9 * 30 * 70).reshape(9, 30, 70) / 2.0 ** 19, 0
    yield "random 2D", rng.permutation(200 * 300).reshape(200, 300) / 2.0 ** 19, 0
    big = wound(160, 31, 64)
    big[big < BARRIER] -= 4  # leave room below for points of small subbins
    small = rng.random(big.shape) < 0.1
    mixed = np.where((big == BARRIER) & small, 90.0 + rng.random(big.shape), big)
    yield "wound 2D, above 60,000", mixed, 60000
    # a thin 2D field, both ways round: rows (columns) above each other in one bin
    yield "3 x 70000", -np.arange(3 * 70000).reshape(3, 70000) / 2.0 ** 19, 60000
    yield "70000 x 3", -np.arange(3 * 70000).reshape(70000, 3) / 2.0 ** 19, 60000
    # planes of the wound field above each other: every neighbour direction
    deep = np.repeat(wound(170, 31, 64)[None], 2, axis=0)
    deep[1] -= deep[1] < BARRIER
    yield "wound 3D, above 60,000", deep, 60000


@pytest.mark.parametrize("dt", [np.float32, np.float64], ids=["f32", "f64"])
def test_runs_over_whole_tiles(P, ref, dt):
    from paper_2603_26968_amd import lopc
    for name, f, above in fields():
        x = np.ascontiguousarray(f.astype(dt))
        want = ref.compress(x, 10.0, ref.ABS)
        top = int(ref.decode_codes(want)[1].max())
        print("[case]", name, x.shape, dt.__name__, "highest subbin", top, flush=True)
        assert top > above
        t = torch.from_numpy(x).cuda()
        three = x.ndim == 3
        for tile in range(3 if three else 2):
            for mode, order in ((lopc.LOPC_REPAIR_SWEEPS, 1), (lopc.LOPC_REPAIR_SWEEPS, 2),
                                (lopc.LOPC_REPAIR_HYBRID, 0), (lopc.LOPC_REPAIR_QUEUE, 0),
                                (lopc.LOPC_REPAIR_AUTO, 0)):
                if above and max(x.shape) == 70000 and mode != lopc.LOPC_REPAIR_AUTO:
                    continue  # thousands of tiles in a row
                ctx = lopc.lopc_ctx_create(0)
                try:
                    lopc.lopc_ctx_set_option(ctx, lopc.LOPC_OPT_TILE_3D if three else
                                             lopc.LOPC_OPT_TILE_2D, tile)
                    lopc.lopc_ctx_set_option(ctx, lopc.LOPC_OPT_REPAIR, mode)
                    lopc.lopc_ctx_set_option(ctx, lopc.LOPC_OPT_SWEEP_ORDER, order)
                    got = P.compress(t, 10.0, "abs", ctx=ctx).cpu().numpy().tobytes()
                finally:
                    lopc.lopc_ctx_destroy(ctx)
                assert got == want, (name, tile, mode, order)
        for pct in (0, 100):
            ctx = lopc.lopc_ctx_create(0)
            try:
                lopc.lopc_ctx_set_option(ctx, lopc.LOPC_OPT_PERSIST_PCT, pct)
                ss = P.compress_batch([t, t], 10.0, "abs", ctx=ctx)
            finally:
                lopc.lopc_ctx_destroy(ctx)
            assert all(s.cpu().numpy().tobytes() == want for s in ss), (name, "batch", pct)
