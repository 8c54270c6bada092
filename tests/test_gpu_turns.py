"""The short segments of large batches, whose sweep is taken in parts by
whichever wavefront is next: every segment is summed, bit for bit as by the
single sweep without a workspace, at sizes around the rule (32 windows a part,
8 parts) and with chains taking some of the workgroups."""
import pytest
import torch

from paper_2010_13100_amd import tc

pytestmark = pytest.mark.gpu

DIM, BAGS = 256, 512  # the widest row of one segment per wavefront: the fewest segments
PARTED = 8 * 32


@pytest.mark.parametrize("windows,chains", [(PARTED - 1, 0), (PARTED, 0), (PARTED + 7, 3)])
def test_parts_cover_every_segment(windows, chains):
    waves = torch.cuda.get_device_properties(0).multi_processor_count * 8 * 4
    num = windows * waves - 5
    gen = torch.Generator(device="cuda").manual_seed(windows)
    dev = dict(dtype=torch.int32, device="cuda")
    lengths = torch.randint(1, 3, (num,), generator=gen, **dev)
    if chains:  # below the length from which sums are taken in pieces
        lengths[:: num // chains] = 600
    seg = torch.zeros(num + 1, **dev)
    seg[1:] = torch.cumsum(lengths, 0)
    n = int(seg[-1])
    ids = torch.randint(0, BAGS // 2, (n,), generator=gen, **dev)
    first = torch.repeat_interleave(seg[:-1], lengths.long())
    # non-decreasing within a segment, as the cast leaves them
    ids = torch.where((torch.arange(n, **dev) > first), ids % 16 + BAGS // 2, ids)
    ids = torch.where(torch.repeat_interleave(lengths > 2, lengths.long()),
                      torch.clamp((torch.arange(n, **dev) - first) // 2, max=BAGS - 1), ids)
    grad = torch.randn(BAGS, DIM, generator=gen, device="cuda")
    nu = torch.tensor([num], **dev)
    print(f"\n{num} segments, {n} pairs", flush=True)
    ws = torch.empty(tc.tc_backward_workspace_bytes(n, DIM), dtype=torch.uint8, device="cuda")
    out = [torch.full((num, DIM), float("nan"), device="cuda") for _ in range(2)]
    tc.tc_embed_backward(grad, seg, ids, nu, num, out[0], ws)
    tc.tc_embed_backward(grad, seg, ids, nu, num, out[1], None)
    torch.cuda.synchronize()
    assert torch.equal(out[0], out[1])
