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


# lane groups narrower than a wavefront, rows of two chunks a lane, and the
# optimizer: a segment taken twice would be updated twice
@pytest.mark.parametrize("dim,optimizer,chains", [
    (16, tc.TC_OPT_SGD, 0), (64, tc.TC_OPT_ADAGRAD, 900), (128, tc.TC_OPT_SGD, 5),
    (256, tc.TC_OPT_SGD, 40), (512, tc.TC_OPT_SGD, 0), (512, tc.TC_OPT_SGD, 900)])
def test_parts_update_every_row_once(dim, optimizer, chains):
    groups = 256 // min(64, max(1, dim // 4))  # segments of a workgroup's window
    window = torch.cuda.get_device_properties(0).multi_processor_count * 8 * groups
    num = PARTED * window + 3 * window // 2 + 1
    gen = torch.Generator(device="cuda").manual_seed(dim + chains)
    dev = dict(dtype=torch.int32, device="cuda")
    lengths = torch.ones(num, **dev)
    lengths[num // 3] = 2
    if chains:
        lengths[:: num // chains] = 600
    seg = torch.zeros(num + 1, **dev)
    torch.cumsum(lengths, 0, out=seg[1:])
    n = int(seg[-1])
    ids = torch.randint(0, BAGS, (n,), generator=gen, **dev)
    for k in torch.nonzero(lengths > 1).flatten().tolist():  # non-decreasing within a segment
        a, b = int(seg[k]), int(seg[k + 1])
        ids[a:b] = torch.sort(ids[a:b]).values
    grad = torch.randn(BAGS, dim, generator=gen, device="cuda")
    nu = torch.tensor([num], **dev)
    rows = torch.arange(num - 1, -1, -1, **dev)
    print(f"\n[d{dim}] {num} segments, {n} pairs", flush=True)
    ws = torch.empty(tc.tc_backward_workspace_bytes(n, dim), dtype=torch.uint8, device="cuda")
    W = torch.randn(num, dim, generator=gen, device="cuda")
    A = None if optimizer == tc.TC_OPT_SGD else torch.rand(num, dim, generator=gen, device="cuda")
    got, ref = (W.clone(), A.clone() if A is not None else None), (W, A)
    for (w, a), space in ((got, ws), (ref, None)):
        tc.tc_embed_backward_update(grad, seg, ids, rows, nu, num, w, a, optimizer, 0.1, 1e-8,
                                    workspace=space)
    torch.cuda.synchronize()
    assert torch.equal(got[0], ref[0])
    assert A is None or torch.equal(got[1], ref[1])


def test_room_for_parts_and_a_short_batch():
    # the launch has workgroups for the later parts, the batch no use for them
    waves = torch.cuda.get_device_properties(0).multi_processor_count * 8 * 4
    cap, num = PARTED * waves, 1000
    dev = dict(dtype=torch.int32, device="cuda")
    lengths = torch.ones(num, **dev)
    lengths[::90] = 200
    seg = torch.zeros(num + 1, **dev)
    seg[1:] = torch.cumsum(lengths, 0)
    n = int(seg[-1])
    ids = torch.arange(n, **dev) * BAGS // n
    grad = torch.randn(BAGS, DIM, device="cuda")
    nu = torch.tensor([num], **dev)
    ws = torch.empty(tc.tc_backward_workspace_bytes(cap, DIM), dtype=torch.uint8, device="cuda")
    out = [torch.full((cap, DIM), float("nan"), device="cuda") for _ in range(2)]
    tc.tc_embed_backward(grad, seg, ids, nu, cap, out[0], ws)
    tc.tc_embed_backward(grad, seg, ids, nu, cap, out[1], None)
    torch.cuda.synchronize()
    assert torch.equal(out[0][:num], out[1][:num]) and bool(out[0][num:].isnan().all())
