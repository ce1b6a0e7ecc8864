"""The chunk decoder against the oracle, bit for bit, where its paths meet:
bin ranges of a chunk around the edge table's size, bins 2^30 and 2^31 from the
chunk's first, bins without values and edges next to ties, ragged chunks, and
fields that only keep their elements' alignment."""
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


def check(P, ref, x, eb, what):
    import torch
    print("[case]", what, x.shape, x.dtype, eb, flush=True)
    stream = ref.compress(x, eb, ref.ABS)
    want = ref.decompress(stream).view(np.uint8)
    s = torch.frombuffer(bytearray(stream), dtype=torch.uint8).cuda()
    assert np.array_equal(P.decompress(s).cpu().numpy().view(np.uint8), want), what
    # one element past an allocation: 4 or 8 bytes off a 16-byte boundary
    dt = torch.float32 if x.dtype == np.float32 else torch.float64
    y = torch.full((x.size + 2,), 7.0, dtype=dt, device="cuda")
    P.decompress(s, out=y[1:-1].view(x.shape))
    h = y.cpu().numpy()
    assert np.array_equal(h[1:-1].reshape(x.shape).view(np.uint8), want), what + ", unaligned"
    assert h[0] == 7.0 and h[-1] == 7.0, what + ": wrote outside the field"
    b = P.decompress_batch([s, s])
    assert all(np.array_equal(v.cpu().numpy().view(np.uint8), want) for v in b), what + ", batch"


SPANS = {np.float32: (1, 4093, 4094, 4095, 4096, 5000, 2 ** 30 - 1, 2 ** 30, 2 ** 31 - 3),
         np.float64: (1, 2045, 2046, 2047, 2048, 3000, 2 ** 30 - 1, 2 ** 30, 2 ** 31, 2 ** 40,
                      2 ** 52)}


@pytest.mark.parametrize("dt", [np.float32, np.float64], ids=["f32", "f64"])
def test_bin_ranges_of_a_chunk(P, ref, dt):
    rng = np.random.default_rng(5)
    for span in SPANS[dt]:
        lo = -(span // 2)
        x = rng.integers(lo, lo + span + 1, (3, 31, 101)).astype(np.float64)
        x.flat[[0, 5]] = lo, lo + span  # both ends in the first chunk
        x += rng.choice([0.0, 0.25, -0.25], x.shape)
        x = np.clip(x, lo - 0.25, lo + span + 0.25).astype(dt)
        check(P, ref, x, 1.0, f"span {span}")


@pytest.mark.parametrize("dt", [np.float32, np.float64], ids=["f32", "f64"])
def test_edges_next_to_ties_and_empty_bins(P, ref, dt):
    rng = np.random.default_rng(9)
    half = rng.integers(-900, 900, (40, 120)) + 0.5
    # products with inv that are half-integers, and the values next to them
    for eb in (1.0, 0.25, 2.0 ** -20, 0.1, 1 / 3):
        x = (half * eb).astype(dt)
        x = np.where(rng.random(x.shape) < 0.3, np.nextafter(x, dt(np.inf)), x)
        x = np.where(rng.random(x.shape) < 0.3, np.nextafter(x, dt(-np.inf)), x)
        check(P, ref, x, eb, f"half-integers times {eb}")
    # bins narrower than the spacing of the values: most hold none
    big = (dt(2.0 ** 22 if dt == np.float32 else 2.0 ** 51) + rng.integers(0, 60, (30, 70))).astype(dt)
    check(P, ref, big, 0.05, "empty bins")
    tiny = np.finfo(dt).smallest_subnormal
    check(P, ref, (rng.integers(-40, 40, (30, 70)) * tiny).astype(dt), float(3 * tiny) if dt ==
          np.float32 else 1e-305, "subnormal values")


@pytest.mark.parametrize("dt", [np.float32, np.float64], ids=["f32", "f64"])
@pytest.mark.parametrize("n", [1, 7, 63, 64, 65, 1000, 2047, 2048, 2049, 4095, 4096, 4097, 4160,
                               5000])
def test_ragged_chunks(P, ref, dt, n):
    rng = np.random.default_rng(n)
    check(P, ref, np.cumsum(rng.standard_normal((1, n)), axis=1).astype(dt), 0.3, f"{n} points")
