"""Varlen calls whose dims do not match query_start_loc, outside the contract
but answered before the kernels were routed by those dims: a chunk longer than a
max_q_len of 1, a single row where every sequence should have max_q_len rows,
and at head_dim 64 fewer rows than query_start_loc says (chunk rows past
num_q_rows are not written) and chunks longer than their context (rows that see
a key are computed, the others NaN).  All buffers hold every row that query_start_loc
names."""
import numpy as np
import pytest
import torch

from paper_2504_09345_amd import binding as pb
from paper_2504_09345_amd import workloads as W

from parity_util import announce, assert_parity, run_oracle, upload

pytestmark = pytest.mark.gpu


def _batch(rows, ctx, s, H_kv, D, seed):
    b = W.generate("tiny", seed=seed, overrides=dict(H_q=s * H_kv, H_kv=H_kv, D=D, ctx=("list", ctx), pool=("factor", 1.3)))
    q = W._fill_normal((sum(rows), s * H_kv, D), seed, "q", 1.0, "bf16", 1)
    return W.Batch(**{**b.__dict__, "q": q, "query_start_loc": np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)})


def _call(b, dev, num_q_rows, max_q_len, trace=None):
    out = torch.full_like(dev["q"], float("nan"))
    dims = pb.make_dims(dev["q"], dev["k"], dev["bt"], int(b.context_lens.max()), num_q_rows=num_q_rows, max_q_len=max_q_len)
    args = (dev["q"], dev["k"], dev["v"], dev["bt"], dev["cl"])
    if trace is None:
        pb.paged_attn_varlen(*args, dev["qsl"], b.scale, out, dims)
    else:
        pb.pa_gather_trace(*args, b.scale, out, dims, trace, query_start_loc=dev["qsl"])
    torch.cuda.synchronize()
    return out.float().cpu().numpy()


@pytest.mark.parametrize("s,H_kv", [(1, 8), (4, 8), (8, 16), (4, 1), (6, 2), (2, 4)])
def test_longer_chunk_in_a_decode_only_call(s, H_kv):
    announce(f"max_q_len 1 with longer chunks s={s} H_kv={H_kv}")
    rows, ctx = [1, 3, 0, 1, 0, 17, 0] + [0] * 20 + [1], [300, 40, 0, 77, 0, 517, 0] + [0] * 20 + [16]
    b = _batch(rows, ctx, s, H_kv, 128, s)
    dev = upload(b)
    ref = run_oracle(b)
    assert_parity(_call(b, dev, sum(rows), 1), ref, strict=False, what="longer chunks")
    trace = torch.empty((H_kv, len(ctx), b.block_table.shape[1] * 16), dtype=torch.int64, device="cuda")
    assert_parity(_call(b, dev, sum(rows), 1, trace), ref, strict=False, what="longer chunks, traced")
    got = trace.cpu().numpy()
    for i, C in enumerate(ctx):
        t = np.arange(C)
        for g in range(H_kv):
            want = np.full(got.shape[2], -1)
            want[:C] = (b.block_table[i, t // 16].astype(np.int64) * H_kv + g) * 16 + t % 16
            assert np.array_equal(got[g, i], want)


@pytest.mark.parametrize("D", [64, 128])
def test_single_row_where_every_sequence_should_have_two(D):
    announce(f"single row beside longer chunks D={D}")
    b = _batch([1, 3, 2, 1, 3], [50, 70, 2, 1, 400], 4, 8, D, D)
    assert_parity(_call(b, upload(b), 10, 2), run_oracle(b), strict=False, what="single rows")


@pytest.mark.parametrize("cut", [1, 30, 300])
def test_rows_past_num_q_rows_are_not_written(cut):
    announce(f"rows past num_q_rows cut={cut}")
    rows = [1, 40, 5, 280]
    b = _batch(rows, [L + 33 for L in rows], 4, 8, 64, cut)
    n = sum(rows) - cut
    got = _call(b, upload(b), n, 280)
    assert np.isnan(got[n:]).all()
    assert_parity(got[:n], run_oracle(b)[:n], strict=False, what="rows of the call")


def test_query_start_loc_far_past_the_rows():
    """The last entry near 2^30 (the first chunk in order, the second of which
    one row is the call's): the work is bounded by the call's rows."""
    announce("query_start_loc far past the rows")
    rows = [40, 60]
    b = _batch(rows, [70, 60], 4, 8, 64, 3)
    dev = upload(b)
    dev["qsl"][2] = 1 << 30
    got = _call(b, dev, 41, 40)
    assert_parity(got[:40], run_oracle(b)[:40], strict=False, what="rows of the first chunk")
    assert np.isnan(got[40:]).all()  # (a chunk longer than its context, its row 40 without a key; the others not written)


def test_chunk_longer_than_its_context():
    announce("D=64 chunk longer than its context")
    rows, ctx = [9, 20, 2], [5, 120, 1]
    b = _batch(rows, ctx, 4, 2, 64, 5)
    got = _call(b, upload(b), sum(rows), 20)
    keep = np.r_[4:9, 9:29, 30:31]
    sub = W.Batch(**{**b.__dict__, "q": b.q[keep], "query_start_loc": np.array([0, 5, 25, 26], np.int32)})
    assert_parity(got[keep], run_oracle(sub), strict=False, what="rows with keys")
    assert np.isnan(np.delete(got, keep, axis=0)).all()
