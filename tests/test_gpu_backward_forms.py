"""Forms of the backward's arguments that the trainer does not make: segments
without pairs (more of them than the workspace covers pairs), and seg_offsets
of this batch's size beside coalesced rows for many more, and long segments
whose rows lie further apart than a buffer window reaches. Against the call
without a workspace, bit for bit (the segments are shorter than those summed
in pieces), and the fused update against the two calls."""
import pytest
import torch

from paper_2010_13100_amd import tc

pytestmark = pytest.mark.gpu


def segments(lens, dim, seed, bags=300):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    lens = torch.tensor(lens, dtype=torch.int32, device="cuda")
    seg = torch.zeros(len(lens) + 1, dtype=torch.int32, device="cuda")
    seg[1:] = torch.cumsum(lens, 0)
    n = int(seg[-1])
    ids = torch.randint(0, bags, (n,), generator=gen, dtype=torch.int64, device="cuda")
    owner = torch.repeat_interleave(torch.arange(len(lens), device="cuda"), lens.long())
    ids = (torch.sort(owner * bags + ids).values % bags).to(torch.int32)
    grad = torch.randn(bags, dim, generator=gen, device="cuda")
    nu = torch.tensor([len(lens)], dtype=torch.int32, device="cuda")
    return seg, ids, grad, nu, n


def run_both(lens, dim, room, seed, bags=300):
    seg, ids, grad, nu, n = segments(lens, dim, seed, bags)
    num, cap = len(lens), len(lens) + room
    print(f"\n{num} segments, {n} pairs, room for {cap}", flush=True)
    ws = torch.empty(tc.tc_backward_workspace_bytes(n, dim), dtype=torch.uint8, device="cuda")
    out = [torch.full((cap, dim), float("nan"), device="cuda") for _ in range(2)]
    tc.tc_embed_backward(grad, seg, ids, nu, cap, out[0], ws)
    tc.tc_embed_backward(grad, seg, ids, nu, cap, out[1], None)
    torch.cuda.synchronize()
    assert torch.equal(out[0][:num], out[1][:num])
    assert bool(out[0][num:].isnan().all())
    rows = torch.randperm(num, device="cuda").to(torch.int32)
    W = torch.randn(num, dim, device="cuda")
    got, ref = W.clone(), W
    tc.tc_embed_backward_update(grad, seg, ids, rows, nu, cap, got, None, tc.TC_OPT_SGD, 0.1,
                                0.0, workspace=ws)
    tc.tc_sparse_update(ref, None, rows, out[1], nu, cap, tc.TC_OPT_SGD, 0.1, 0.0)
    torch.cuda.synchronize()
    assert torch.equal(got, ref)


@pytest.mark.parametrize("dim", [16, 64, 260])
def test_segments_without_pairs(dim):
    lens = [0] * 9000 + [1, 0, 600, 47, 0, 48, 0, 0, 49, 1999] + [0] * 2000 + [100, 2, 0]
    run_both(lens, dim, 0, dim)


@pytest.mark.parametrize("room", [1, 1000, 250_000, 300_000])
def test_offsets_of_the_batch_beside_room_for_more(room):
    run_both([3, 1, 60, 1, 700, 2] * 150, 64, room, room)


def test_rows_beyond_a_buffer_window():
    # 2.4 GB of gradients: 64-bit addresses, 32 rows at a time
    run_both([48, 49, 63, 64, 65, 1, 79, 80, 95, 96, 97, 128, 511, 512, 513, 700, 2047] * 9, 1024,
             0, 5, bags=600_000)
