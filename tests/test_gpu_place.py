"""Placement of a single field's records: with a wave per record up to 4,096
chunks, with scanned offsets above.  Batches place theirs in the encoder, so the
two have to agree byte for byte."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [1, 2, 3, 4, 5, 1023, 4095, 4096, 4097])
def test_single_and_batch_streams_agree(rows):
    import torch
    import paper_2603_26968_amd as P
    print("[case]", rows, "chunks", flush=True)
    g = torch.Generator(device="cuda").manual_seed(rows)
    # rows of one chunk each
    x = torch.cumsum(torch.randn((rows, 4096), device="cuda", generator=g), 1)
    x[::3] *= 0.01  # records of different sizes
    one = P.compress(x, 0.05, "abs")
    both = P.compress_batch([x], 0.05, "abs")[0]
    assert torch.equal(one, both)
