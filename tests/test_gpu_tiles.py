"""Tile runs of the repair against the oracle, byte for byte, at the sizes and
values where their parts meet: shapes one point around the tile edges, fields
of few levels (ties), one bin for the whole field (long event rounds, full
event lists), float64 bins around 2^30 from the tile's first bin, every repair
scheduler, tile shape and sweep order."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ref():
    import oracle
    return oracle


@pytest.fixture(scope="module")
def P():
    import paper_2603_26968_amd as P
    return P


def streams(P, x, eb):
    """The field's stream under every repair scheduler with both sweep orders
    and every tile shape of its kind."""
    import torch
    d = torch.from_numpy(np.ascontiguousarray(x)).cuda()
    three = x.ndim == 3 and x.shape[0] > 1
    for tile in range(3 if three else 2):
        for repair in (P.LOPC_REPAIR_SWEEPS, P.LOPC_REPAIR_HYBRID, P.LOPC_REPAIR_QUEUE):
            for order in (1, 2) if repair == P.LOPC_REPAIR_SWEEPS else (0,):
                ctx = P.lopc_ctx_create(0)
                try:
                    P.lopc_ctx_set_option(ctx, P.LOPC_OPT_TILE_3D if three else P.LOPC_OPT_TILE_2D,
                                          tile)
                    P.lopc_ctx_set_option(ctx, P.LOPC_OPT_REPAIR, repair)
                    P.lopc_ctx_set_option(ctx, P.LOPC_OPT_SWEEP_ORDER, order)
                    yield (tile, repair, order), P.compress(d, eb, "abs",
                                                            ctx=ctx).cpu().numpy().tobytes()
                finally:
                    P.lopc_ctx_destroy(ctx)


def check(P, ref, x, eb, what):
    print("[case]", what, x.shape, x.dtype, eb, flush=True)
    want = ref.compress(x, eb, ref.ABS)
    for how, got in streams(P, x, eb):
        assert got == want, f"{what}: stream differs with (tile, repair, order) = {how}"
    ss, hs = P.compress_batch([_dev(x)] * 2, eb, "abs", headers=True)
    assert all(s.cpu().numpy().tobytes() == want for s in ss), f"{what}: batch stream differs"


def _dev(x):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


SHAPES = [(1, 1), (31, 63), (32, 64), (33, 65), (97, 130), (15, 127), (17, 129),
          (1, 1, 1), (3, 7, 31), (4, 8, 32), (5, 9, 33), (9, 17, 17), (13, 33, 70), (2, 40, 97)]


@pytest.mark.parametrize("dt", [np.float32, np.float64], ids=["f32", "f64"])
@pytest.mark.parametrize("shape", SHAPES, ids=[str(s) for s in SHAPES])
def test_tile_edges(P, ref, shape, dt):
    rng = np.random.default_rng(sum(shape) * 7 + len(shape))
    ties = rng.integers(0, 4, shape).astype(dt)  # few levels: equal values everywhere
    check(P, ref, ties, 1.6, "few levels")
    walk = np.cumsum(rng.standard_normal(shape), axis=-1).astype(dt)  # runs in one bin
    check(P, ref, walk, 2.0, "walk")


@pytest.mark.parametrize("shape", [(70, 150), (11, 30, 70)], ids=["2d", "3d"])
def test_one_bin_for_the_whole_field(P, ref, shape):
    idx = np.indices(shape).sum(axis=0)
    rng = np.random.default_rng(3)
    # a plane falling with the index: every step raises the subbin, whole
    # tiles rise from one corner; and the same in random order
    check(P, ref, (-1e-6 * idx).astype(np.float64), 1.0, "falling plane")
    check(P, ref, (1e-6 * rng.permutation(idx.size).reshape(shape)).astype(np.float64), 1.0,
          "random order")


@pytest.mark.parametrize("shape", [(40, 70), (6, 10, 40)], ids=["2d", "3d"])
def test_float64_bins_far_from_the_first(P, ref, shape):
    rng = np.random.default_rng(11)
    b = 2 ** 30
    far = np.array([0, b - 1, b, b + 1, -b, -b - 1, -b + 1, 2 * b - 1, 2 * b, 4 * b, 4 * b + 1])
    for levels in (far[:2], far[[0, 1, 4]], far[[0, 2]], far[[0, 5]], far):
        # bins of width 1 and values a quarter off their centres: neighbours
        # in the same bin in both orders, and equal low halves of the bins
        x = rng.choice(levels, shape) + rng.choice([-0.25, 0.0, 0.25], shape)
        check(P, ref, x.astype(np.float64), 1.0, f"bins {levels.tolist()}")


def test_more_marked_tiles_than_resident_workgroups(P, ref):
    # sweeps that hand several tiles to a workgroup: 3,780 tiles (2,100 of a
    # colour) for at most 1,536 workgroups, few levels so that every sweep of
    # several marks tiles all over the field
    rng = np.random.default_rng(21)
    z, y, x = np.meshgrid(np.arange(28), np.arange(477), np.arange(259), indexing="ij")
    f = np.sin(z / 9.0) + np.sin(y / 23.0) * np.cos(x / 31.0) + rng.normal(0, 0.02, z.shape)
    check(P, ref, f.astype(np.float32), 0.25, "many tiles")
