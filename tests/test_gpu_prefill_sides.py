"""The prefill kernel's rarer passes on both of its item sizes (128 and 256 query
rows): items computed again for V outside fp16's range (head_dim 128) or for
rows that are not finite (head_dim 64), V of large and tiny scale, and a
block-table window that slides past 2,048 pages.  Short chunks pad a batch until
its bound on items is past the CUs, where the kernel takes 256 rows; each test
states which side its batch is on, and that the prefill kernel takes it."""
import numpy as np
import pytest
import torch

from paper_2504_09345_amd import workloads as W

from parity_util import announce, assert_parity, run_gpu, run_oracle
from route_util import takes_blocks, takes_split

pytestmark = pytest.mark.gpu


def _batch(chunks, s, H_kv, D, seed, blocks, poison=False):
    """Chunks as (rows, prior tokens), padded with chunks of two rows on no
    prior context to the side of `blocks` 16-row blocks per wave."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    chunks = list(chunks)
    if blocks == 2:
        chunks += [(2, 0)] * (cus // H_kv + 1)
    rows, ctx = [L for L, _ in chunks], [L + p for L, p in chunks]
    b = W.generate("tiny", seed=seed, poison=poison, overrides=dict(H_q=s * H_kv, H_kv=H_kv, D=D, ctx=("list", ctx),
                                                                    pool=("factor", 1.1)))
    q = W._fill_normal((sum(rows), s * H_kv, D), seed, "q", 1.0, "bf16", 1)
    b = W.Batch(**{**b.__dict__, "q": q, "query_start_loc": np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)})
    assert takes_blocks(b, cus) == blocks
    assert D == 128 or not takes_split(b, cus)
    return b


@pytest.mark.parametrize("blocks", [1, 2])
@pytest.mark.parametrize("s", [1, 4, 6, 8])
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
def test_nonfinite_v_at_head_dim_64(value, s, blocks):
    """One key of each long chunk: inside the chunk (the rows before it do not
    see it), before it (every row does), and in its last page."""
    announce(f"D=64 V = {value} s={s} blocks={blocks}")
    n = 256 // s
    chunks = [(n + 40, 30), (2 * n + 3, 0), (n // 2 + 20, 65)]
    b = _batch(chunks, s, 8, 64, s, blocks)
    bits = W.f32_to_bf16_bits(np.array([value], np.float32))[0]
    v = b.v_pages.copy()
    for i, (t, g, d) in enumerate(((30 + n // 3, 0, 5), (1, 3, slice(None)), (n // 2 + 84, 7, 63))):
        v[b.block_table[i, t // 16], g, t % 16, d] = bits
    b = W.Batch(**{**b.__dict__, "v_pages": v})
    got, ref = run_gpu(b), run_oracle(b)
    assert np.isfinite(ref[0]).all() and not np.isfinite(ref).all()
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    assert np.array_equal(np.isposinf(got), np.isposinf(ref)) and np.array_equal(np.isneginf(got), np.isneginf(ref))
    ok = np.isfinite(ref).all(axis=-1)
    assert_parity(got[ok], ref[ok], strict=False, what="finite rows")


@pytest.mark.parametrize("blocks", [1, 2])
@pytest.mark.parametrize("s", [1, 6, 8])
@pytest.mark.parametrize("D,exp", [(64, -60), (64, 60), (128, -30), (128, 17)])
def test_v_scales(D, exp, s, blocks):
    """At head_dim 128 both scales leave fp16's range: the bf16 pass."""
    announce(f"D={D} V scaled 2^{exp} s={s} blocks={blocks}")
    b = _batch([(256 // s + (400 if s == 1 else 20), 30), (70, 300)], s, 8, D, 7 + s, blocks)
    v = W.bf16_bits_to_f32(b.v_pages) * np.float32(2.0) ** exp
    b = W.Batch(**{**b.__dict__, "v_pages": W.f32_to_bf16_bits(v)})
    got, ref = run_gpu(b) * 2.0 ** -exp, run_oracle(b) * 2.0 ** -exp  # (powers of two: exact)
    assert_parity(got, ref, strict=False, what=f"V scale 2^{exp}")


@pytest.mark.parametrize("blocks", [1, 2])
@pytest.mark.parametrize("D,scale", [(64, 1.0), (128, 1.0), (128, 2.0 ** 17)])
def test_window_past_2048_pages(D, scale, blocks):
    """600 rows on 32,700 tokens, with V beyond fp16 at head_dim 128 also the
    second pass, which starts from the first window again; the first and the
    last rows against the oracle (a chunk's row sees what it would see in a
    chunk of fewer rows)."""
    announce(f"window slide D={D} scale={scale} blocks={blocks}")
    L, prior, s = 600, 32700, 8
    b = _batch([(L, prior)], s, 1, D, 3, blocks)
    if scale != 1.0:
        v = W.bf16_bits_to_f32(b.v_pages) * np.float32(scale)
        b = W.Batch(**{**b.__dict__, "v_pages": W.f32_to_bf16_bits(v)})
    got = run_gpu(b) / scale
    for lo, hi in ((0, 20), (L - 20, L)):
        sub = W.Batch(**{**b.__dict__, "q": b.q[lo:hi], "block_table": b.block_table[:1],
                         "context_lens": np.array([prior + hi], np.int32), "query_start_loc": np.array([0, hi - lo], np.int32)})
        assert_parity(got[lo:hi], run_oracle(sub) / scale, strict=False, what=f"rows {lo}..{hi}")
    if blocks == 2:
        rest = W.Batch(**{**b.__dict__, "q": b.q[L:], "block_table": b.block_table[1:], "context_lens": b.context_lens[1:],
                          "query_start_loc": (b.query_start_loc[1:] - L).astype(np.int32)})
        assert_parity(got[L:], run_oracle(rest) / scale, strict=False, what="short chunks")
