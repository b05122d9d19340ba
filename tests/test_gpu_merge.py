"""Items cut over several stream-K ranges and merged in the launch: the numbers
of parts at which the merge changes form (one batch of records, two, groups of
8, 16 and 32), whatever the workspace holds beforehand, and a recorded launch
replayed."""
import numpy as np
import pytest
import torch

from paper_2504_09345_amd import binding as pb
from paper_2504_09345_amd import workloads as W

from parity_util import announce, assert_parity, run_oracle, upload

pytestmark = pytest.mark.gpu


def _run(b, dev, ws):
    out = torch.full_like(dev["q"], float("nan"))
    dims = pb.make_dims(dev["q"], dev["k"], dev["bt"], int(b.context_lens.max()))
    pb.paged_attn(dev["q"], dev["k"], dev["v"], dev["bt"], dev["cl"], b.scale, out, dims, workspace=ws)
    torch.cuda.synchronize()
    return out.float().cpu().numpy()


# one sequence of as many pages as its item has parts (one unit per range, up
# to the grid: 208 workgroups with 8 KV heads, more ranges with fewer)
@pytest.mark.parametrize("dtype,D", [("bf16", 128), ("bf16", 64), ("fp32", 128)])
@pytest.mark.parametrize("H_kv,s,pages", [
    (8, 4, 2), (8, 6, 8), (8, 8, 9), (8, 4, 16), (8, 1, 17), (8, 4, 64), (8, 2, 65), (8, 4, 208), (8, 4, 500),
    (1, 4, 256), (1, 8, 257), (2, 6, 500), (4, 1, 1000)])
def test_parts(dtype, D, H_kv, s, pages):
    announce(f"merge {dtype} D={D} H_kv={H_kv} s={s} pages={pages}")
    b = W.generate("tiny", seed=pages, dtype=dtype, overrides=dict(
        H_q=s * H_kv, H_kv=H_kv, D=D, ctx=("list", [16 * pages - 3]), pool=("factor", 1.2)))
    dev = upload(b)
    n = pb.pa_workspace_size(pb.make_dims(dev["q"], dev["k"], dev["bt"], 16 * pages))
    ws = torch.zeros(n, dtype=torch.uint8, device="cuda")
    got = _run(b, dev, ws)
    # (sums of up to 8,000 fp32 terms: the tolerance is that of the strict floor
    # only for short contexts)
    assert_parity(got, run_oracle(b), strict=False, what=f"{pages} parts")
    again = _run(b, dev, ws)  # the counters as the first call left them
    assert np.array_equal(got.view(np.uint32), again.view(np.uint32))
    for fill in (0xFF, 0x01, None):  # NaN, small counts, random bytes
        ws = (torch.randint(0, 256, (n,), dtype=torch.uint8, device="cuda") if fill is None
              else torch.full((n,), fill, dtype=torch.uint8, device="cuda"))
        again = _run(b, dev, ws)
        assert np.array_equal(got.view(np.uint32), again.view(np.uint32)), fill


@pytest.mark.parametrize("first,step", [(83, 5), (20, 4)])
def test_two_cut_items_per_range_and_head_blocks(first, step):
    """Ranges of four or five units, and of two or three, that end one item and
    start the next, with two head blocks per page: both records of a range
    counted at its end."""
    announce(f"two cut items per range, contexts from {first}")
    b = W.generate("tiny", seed=3, overrides=dict(H_q=64, H_kv=16, D=128,
                                                  ctx=("list", [first + step * i for i in range(40)]),
                                                  pool=("factor", 1.2)))
    units = 2 * int(((b.context_lens + 15) // 16).sum())
    assert (4 if first == 83 else 2) <= units / 208 <= (5 if first == 83 else 3)
    dev = upload(b)
    ws = torch.randint(0, 256, (pb.pa_workspace_size(pb.make_dims(dev["q"], dev["k"], dev["bt"], int(b.context_lens.max()))),),
                       dtype=torch.uint8, device="cuda")
    got = _run(b, dev, ws)
    assert_parity(got, run_oracle(b), what="two cut items")
    for _ in range(8):
        assert np.array_equal(got.view(np.uint32), _run(b, dev, ws).view(np.uint32))


def test_recorded_launch_replays():
    """A captured call replayed several times, with and without other calls
    between the replays, gives the eager result each time."""
    announce("graph replay")
    b = W.generate("tiny", seed=4, overrides=dict(H_q=32, H_kv=8, D=128, ctx=("list", [300, 2000, 45, 16]),
                                                  pool=("factor", 1.2)))
    dev = upload(b)
    qsl = torch.arange(b.num_seqs + 1, dtype=torch.int32, device="cuda")
    dims = pb.make_dims(dev["q"], dev["k"], dev["bt"], 2000, num_q_rows=b.num_seqs, max_q_len=1)
    out = torch.zeros_like(dev["q"])

    def call():
        pb.paged_attn_varlen_noalloc(dev["q"], dev["k"], dev["v"], dev["bt"], dev["cl"], qsl, b.scale, out, dims)

    call()
    torch.cuda.synchronize()
    ref = out.clone()
    assert_parity(ref.float().cpu().numpy(), run_oracle(b), what="eager")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for i in range(6):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref), f"replay {i}"
        if i % 2:
            out.zero_()
            call()
            torch.cuda.synchronize()
            assert torch.equal(out, ref), f"eager after replay {i}"


# with one range per workgroup, and (past 8,000 units) several of at least 4 units
@pytest.mark.parametrize("dtype,D", [("bf16", 128), ("bf16", 64), ("fp32", 128)])
@pytest.mark.parametrize("H_kv,s,pages,parts", [(1, 4, 2064, 0), (1, 8, 8200, 1024), (2, 1, 8100, 1024)])
def test_parts_in_groups_of_32(dtype, D, H_kv, s, pages, parts):
    """More than 256 parts.  What the call wrote shows the form of its merge: a
    record per part, and a counter left at 0 for the item and for each group of
    more than one part.  (parts: their number, 0 where it follows from how many
    workgroups fit a CU.)"""
    announce(f"merge in groups of 32: {dtype} D={D} H_kv={H_kv} s={s} pages={pages}")
    b = W.generate("tiny", seed=pages, dtype=dtype, overrides=dict(
        H_q=s * H_kv, H_kv=H_kv, D=D, ctx=("list", [16 * pages - 3]), pool=("factor", 1.1)))
    dev = upload(b)
    n = pb.pa_workspace_size(pb.make_dims(dev["q"], dev["k"], dev["bt"], 16 * pages))
    record = H_kv * s * (D + 2) * 4 // 8  # words of a part's record, all its waves
    got = None
    for fill in (0xFF, 0x01, 0xFF):
        ws = torch.full((n,), fill, dtype=torch.uint8, device="cuda")
        before = ws.view(torch.int64)[0].item()
        out = _run(b, dev, ws)
        counters = int((ws.view(torch.int64) == 0).sum())
        n_parts, rest = divmod(int((ws.view(torch.int64) != before).sum()) - counters, record)
        if dtype == "fp32" and H_kv == 2:  # one range per workgroup at any size
            assert n_parts > 64
        else:
            assert rest == 0 and n_parts > 256 and n_parts in (parts or n_parts,)
            assert counters == n_parts // 32 + (n_parts % 32 > 1) + 1
        if got is None:
            got = out
            assert_parity(got, run_oracle(b), strict=False, what=f"{pages} pages")
        assert np.array_equal(got.view(np.uint32), out.view(np.uint32)), fill
    for _ in range(2):  # the counters as that call left them
        assert np.array_equal(got.view(np.uint32), _run(b, dev, ws).view(np.uint32))


@pytest.mark.parametrize("pages,low", [(13, 0x3F80), (13, 5), (2, 1), (64, 0x3F80), (64, 7), (208, 5)])
def test_workspace_partly_written_over(pages, low):
    """The low two bytes of every 8-byte word of the workspace written over
    between calls (a bf16 column, small counts): the same bits each time."""
    announce(f"merge after low bytes {low:#x} pages={pages}")
    b = W.generate("tiny", seed=pages, overrides=dict(H_q=32, H_kv=8, D=128, ctx=("list", [16 * pages - 3]),
                                                      pool=("factor", 1.2)))
    dev = upload(b)
    n = pb.pa_workspace_size(pb.make_dims(dev["q"], dev["k"], dev["bt"], 16 * pages))
    ws = torch.zeros(n, dtype=torch.uint8, device="cuda")
    got = _run(b, dev, ws)
    assert_parity(got, run_oracle(b), strict=False, what=f"{pages} parts")
    for _ in range(3):
        ws.view(torch.int16)[::4] = low
        for _ in range(2):
            assert np.array_equal(got.view(np.uint32), _run(b, dev, ws).view(np.uint32))


@pytest.mark.parametrize("H_kv,dtype,D", [(1, "bf16", 128), (2, "bf16", 64), (4, "fp32", 128), (3, "bf16", 128)])
@pytest.mark.parametrize("pages", [None, 1000])
def test_teams_of_fewer_heads(H_kv, dtype, D, pages):
    """Fewer than 8 KV heads: several ranges per workgroup, which end at
    different units (contexts of 0 to 40 pages, some teams without a range);
    with a declared bound of 1,000 pages for each of 600 sequences, past the
    teams' unit tables, one range per workgroup."""
    announce(f"teams H_kv={H_kv} {dtype} D={D} bound={pages}")
    rng = np.random.default_rng(H_kv)
    ctx = [int(x) for x in rng.integers(0, 640, size=600 if pages else 37)]
    b = W.generate("tiny", seed=H_kv, dtype=dtype, overrides=dict(H_q=4 * H_kv, H_kv=H_kv, D=D, ctx=("list", ctx),
                                                                  pool=("factor", 1.2)))
    ref = run_oracle(b)
    if pages:
        table = np.zeros((b.num_seqs, pages), np.int32)
        table[:, :b.block_table.shape[1]] = b.block_table
        b = W.Batch(**{**b.__dict__, "block_table": table})
    dev = upload(b)
    out = torch.full_like(dev["q"], float("nan"))
    dims = pb.make_dims(dev["q"], dev["k"], dev["bt"], 16 * pages if pages else int(b.context_lens.max()))
    for _ in range(3):
        pb.paged_attn(dev["q"], dev["k"], dev["v"], dev["bt"], dev["cl"], b.scale, out, dims)
    torch.cuda.synchronize()
    assert_parity(out.float().cpu().numpy(), ref, strict=False, what="teams")
