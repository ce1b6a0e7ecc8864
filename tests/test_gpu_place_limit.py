"""Placement of a single field's records around the chunk count above which
their offsets come from a scan: batches place theirs in the encoder, so the two
have to agree byte for byte."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [8191, 16383, 16384, 16385])
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
