"""Sweeps over few marked tiles, which the resident workgroups look for and run
in turn: fields of more than eight tiles to such a workgroup (thin ones, so of
few points), whose late sweeps mark few tiles; call after call on one context,
as it goes by the marks of the call before, and between fields whose marks
differ, against the oracle, byte for byte."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def fields():
    rng = np.random.default_rng(30)
    # 13,000 tiles of 4 x 8 x 1 points, and of 32 x 1 and 1 x 64 points
    for shape in ((130, 3200, 1), (13000 * 32, 1), (1, 13000 * 64)):
        noise = rng.integers(0, 3, shape).astype(np.float64)
        yield "few levels", noise
        chain = np.full(shape, 0.0)
        flat = chain.reshape(-1)
        flat[:] = rng.integers(0, 2, flat.size) * 100.0
        # some long runs in one bin, falling, through a few tiles
        for at in rng.integers(0, flat.size - 3000, 6):
            flat[at:at + 900] = -np.arange(900) / 1024.0
        yield "a few chains", chain


@pytest.mark.parametrize("order", [1, 2])
def test_late_sweeps_of_many_tiles(ref, order):
    import paper_2603_26968_amd as P
    from paper_2603_26968_amd import lopc
    ctx = lopc.lopc_ctx_create(0)
    try:
        lopc.lopc_ctx_set_option(ctx, lopc.LOPC_OPT_REPAIR, lopc.LOPC_REPAIR_SWEEPS)
        lopc.lopc_ctx_set_option(ctx, lopc.LOPC_OPT_SWEEP_ORDER, order)
        last = None
        for name, x in fields():
            x = x.astype(np.float32)
            print("[case]", name, x.shape, "order", order, flush=True)
            now = (torch.from_numpy(x).cuda(), ref.compress(x, 10.0, ref.ABS))
            for t, want in [now] * 3 + ([last, now] if last else []):
                s, st = P.compress(t, 10.0, "abs", stats=True, ctx=ctx)
                assert s.cpu().numpy().tobytes() == want, (name, x.shape)
            print("  sweeps", st["repair_sweeps"], "tile runs", st["active_tiles_total"], flush=True)
            last = now
    finally:
        lopc.lopc_ctx_destroy(ctx)
