"""Rows of 8 (mod 16) bytes are permuted two at a time: against the index formula at the smallest such
row, odd and even sequence lengths, several outer indices, a device count that does not divide the
pairs, and a destination that is only 8-byte aligned (which takes the row-at-a-time kernel)."""
import pytest
import torch

from paper_2311_09431_amd import binding as sa

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("outer,n_seq,units,N", [
    (1, 2, 5, 1), (3, 6, 5, 3), (2, 30, 7, 15), (5, 35, 25, 5), (2, 4096, 25, 8), (3, 1026, 63, 2), (1, 64, 301, 4),
])
def test_rows_of_an_odd_number_of_units(outer, n_seq, units, N, offset):
    x = torch.arange(outer * n_seq * units, dtype=torch.int64, device="cuda").view(outer, 1, n_seq, units)
    buf = torch.zeros(2, x.numel() + 2, dtype=torch.int64, device="cuda")
    y, z = (b[offset:offset + x.numel()].view_as(x) for b in buf)
    sa.sa_stripe_permute(x, y, N)
    sa.sa_unstripe_permute(y, z, N)
    want = x.view(outer, 1, n_seq // N, N, units).transpose(2, 3).reshape_as(x)
    assert torch.equal(y, want) and torch.equal(z, x)
    assert int(buf[0, -1 - (1 - offset)]) == 0 and (offset == 0 or int(buf[0, 0]) == 0)
