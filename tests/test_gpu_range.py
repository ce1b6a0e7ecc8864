"""Fields with values past the bin range or infinite, of either sign and at
every corner of the grid: every repair scheduler, the enqueued call and the
batch call return the code, and the context goes on working."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_2603_26968_amd as P
    return P


def fields(dt):
    rng = np.random.default_rng(4)
    big = 3e9 if dt == np.float32 else 1e19
    for shape in ((3, 70), (40, 3), (2, 9, 33), (5, 3, 2)):
        for v, code in ((-big, -4), (big, -4), (-np.inf, -2), (np.inf, -2)):
            for at in (0, -1, shape[-1] - 1, None):  # None: everywhere
                x = rng.standard_normal(shape).astype(dt)
                if at is None:
                    x[:] = v
                else:
                    x.flat[at] = v
                yield x, code, (shape, v, at)


@pytest.mark.parametrize("dt", [np.float32, np.float64], ids=["f32", "f64"])
def test_codes_under_every_scheduler(P, ref, dt):
    from paper_2603_26968_amd import lopc
    ctx = lopc.lopc_ctx_create(0)
    ok = torch.from_numpy(np.cumsum(np.ones((40, 70), dt), axis=1)).cuda()
    want = ref.compress(ok.cpu().numpy(), 3.0, ref.ABS)
    try:
        for mode in (lopc.LOPC_REPAIR_SWEEPS, lopc.LOPC_REPAIR_HYBRID, lopc.LOPC_REPAIR_QUEUE,
                     lopc.LOPC_REPAIR_POINTS, lopc.LOPC_REPAIR_AUTO):
            lopc.lopc_ctx_set_option(ctx, lopc.LOPC_OPT_REPAIR, mode)
            print("[case]", dt.__name__, "scheduler", mode, flush=True)
            for x, code, what in fields(dt):
                t = torch.from_numpy(x).cuda()
                with pytest.raises(lopc.LopcError) as e:
                    P.compress(t, 1.0, "abs", ctx=ctx)
                assert e.value.code == code, (mode, what)
                if mode in (lopc.LOPC_REPAIR_HYBRID, lopc.LOPC_REPAIR_QUEUE, lopc.LOPC_REPAIR_AUTO):
                    _, size, status = P.compress_enqueue(t, 1.0, "abs", ctx=ctx)
                    torch.cuda.synchronize()
                    assert (status.item(), size.item()) == (code, 0), (mode, what)
            assert P.compress(ok, 3.0, "abs", ctx=ctx).cpu().numpy().tobytes() == want
        print("[case]", dt.__name__, "batch", flush=True)
        xs = [(torch.from_numpy(x).cuda(), code) for x, code, _ in fields(dt)]
        ss, st = P.compress_batch([ok] + [x for x, _ in xs], 1.0, "abs",
                                  stats=True, ctx=ctx, raise_on_error=False)
        assert st["status"] == [0] + [code for _, code in xs]
        assert ss[0].cpu().numpy().tobytes() == ref.compress(ok.cpu().numpy(), 1.0, ref.ABS)
    finally:
        lopc.lopc_ctx_destroy(ctx)
