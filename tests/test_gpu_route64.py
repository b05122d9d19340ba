"""bf16 head_dim 64 chunks on either side of the rule that sends few rows on long
contexts to the split-K kernel: the results against the oracle, with decode rows
beside them (on the stream kernel) and without, a row of one where every chunk
should have max_q_len rows, through the workspace and the no-allocation entry
and through the gather trace."""
import numpy as np
import pytest
import torch

from paper_2504_09345_amd import binding as pb
from paper_2504_09345_amd import workloads as W

from parity_util import announce, assert_parity, run_oracle, upload
from route_util import takes_split

pytestmark = pytest.mark.gpu


def _batch(chunks, s, H_kv, seed):
    """Chunks as (rows, prior tokens)."""
    rows, ctx = [L for L, _ in chunks], [L + p for L, p in chunks]
    b = W.generate("tiny", seed=seed, poison=True, overrides=dict(H_q=s * H_kv, H_kv=H_kv, D=64, ctx=("list", ctx),
                                                                  pool=("factor", 1.3)))
    q = W._fill_normal((sum(rows), s * H_kv, 64), seed, "q", 1.0, "bf16", 1)
    return W.Batch(**{**b.__dict__, "q": q, "query_start_loc": np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)})


@pytest.mark.parametrize("s,H_kv,chunks,split", [
    (4, 8, [(2, 6000), (3, 2047)], True),
    (4, 8, [(2, 6000), (1, 300), (3, 2047), (1, 5000), (1, 1)], True),  # decode rows
    (1, 2, [(17, 2040), (16, 0), (1, 40)], True),
    (8, 1, [(64, 4096), (64, 33)], True),
    (6, 2, [(9, 9000)], True),
    (2, 8, [(5, 3000), (5, 10), (10, 700), (1, 16), (4, 100)], True),  # rows = num_seqs * 5, one of them single
    (4, 8, [(300, 2500), (1, 3000), (90, 0)], False),
    (8, 8, [(20, 100), (1, 90), (2, 0)], False),
    (1, 8, [(400, 900)], False),
])
def test_either_route(s, H_kv, chunks, split):
    announce(f"D=64 route s={s} H_kv={H_kv} {chunks}")
    b = _batch(chunks, s, H_kv, s + H_kv)
    max_q = 5 if (5, 10) in chunks else int(b.q_lens.max())
    assert takes_split(b, torch.cuda.get_device_properties(0).multi_processor_count) == split
    dev, ref = upload(b), run_oracle(b)
    dims = pb.make_dims(dev["q"], dev["k"], dev["bt"], int(b.context_lens.max()), num_q_rows=b.num_q_rows, max_q_len=max_q)
    args = (dev["q"], dev["k"], dev["v"], dev["bt"], dev["cl"])
    outs = [torch.full_like(dev["q"], float("nan")) for _ in range(3)]
    trace = torch.empty((H_kv, b.num_seqs, b.block_table.shape[1] * 16), dtype=torch.int64, device="cuda")
    pb.paged_attn_varlen(*args, dev["qsl"], b.scale, outs[0], dims)
    pb.paged_attn_varlen_noalloc(*args, dev["qsl"], b.scale, outs[1], dims)
    pb.pa_gather_trace(*args, b.scale, outs[2], dims, trace, query_start_loc=dev["qsl"])
    torch.cuda.synchronize()
    for o in outs:
        assert_parity(o.float().cpu().numpy(), ref, strict=False, what="route")
    got = trace.cpu().numpy()
    for i, C in enumerate(b.context_lens):
        t = np.arange(C)
        for g in range(H_kv):
            want = np.full(got.shape[2], -1)
            want[:C] = (b.block_table[i, t // 16].astype(np.int64) * H_kv + g) * 16 + t % 16
            assert np.array_equal(got[g, i], want)
