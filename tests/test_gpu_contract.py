"""Varlen calls whose dims do not match query_start_loc, outside the contract
but answered before the kernels were routed by those dims: a chunk longer than a
max_q_len of 1, and a single row where every sequence should have max_q_len
rows.  All buffers hold every row that query_start_loc names."""
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
