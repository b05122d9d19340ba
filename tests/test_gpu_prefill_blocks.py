"""Chunk rows on either side of the line between items of 128 and of 256 query
rows (on 256 CUs: 8 KV heads with 4,096 query rows each), with chunks at the
edges of an item, against the oracle for every group size and head dim."""
import numpy as np
import pytest

from paper_2504_09345_amd import workloads as W

from parity_util import announce, assert_parity, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("s", [1, 2, 4, 6, 8])
@pytest.mark.parametrize("item", [128, 256])
def test_item_edges(item, s, D):
    announce(f"prefill items of {item} rows s={s} D={D}")
    pb = item // s  # positions per item
    chunks = [(2, 0), (pb - 1, 0), (pb, 1), (pb + 1, 15), (3, 61), (17, 63), (2 * pb + 5, 33)]  # (rows, prior tokens)
    p1, n = 128 // s, len(chunks) + 1
    total = 33 * p1 - 1 - n * (p1 - 1) + (item == 256)  # the most rows that n chunks may have in 32 items; one more
    chunks.append((total - sum(L for L, _ in chunks), 7))
    H_kv = 8
    b = W.generate("tiny", seed=item + s, poison=True, overrides=dict(
        H_q=s * H_kv, H_kv=H_kv, D=D, ctx=("list", [L + p for L, p in chunks]), pool=("factor", 1.3)))
    q = W._fill_normal((total, s * H_kv, D), s, "q", 1.0, "bf16", 1)
    qsl = np.concatenate([[0], np.cumsum([L for L, _ in chunks])]).astype(np.int32)
    b = W.Batch(**{**b.__dict__, "q": q, "query_start_loc": qsl})
    assert_parity(run_gpu(b), run_oracle(b), strict=False, what=f"items of {item} rows s={s} D={D}")
