"""Chunk rows at head_dim 64 on the matrix cores (bf16 V, P as bf16 high and
low parts; four pages per step): block, step and page edges for every group
size against the oracle, large and tiny V, and V that is infinite or NaN at
keys that some rows of a block do not see (those rows stay finite, as in the
per-row kernel)."""
import numpy as np
import pytest

from paper_2504_09345_amd import workloads as W

from parity_util import announce, assert_parity, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


def _batch(chunks, s, H_kv, seed, poison=True):
    """Chunks as (rows, prior tokens)."""
    ctx = [L + p for L, p in chunks]
    b = W.generate("tiny", seed=seed, poison=poison, overrides=dict(H_q=s * H_kv, H_kv=H_kv, D=64, ctx=("list", ctx),
                                                                    pool=("factor", 1.3)))
    rows = [L for L, _ in chunks]
    q = W._fill_normal((sum(rows), s * H_kv, 64), seed, "q", 1.0, "bf16", 1)
    qsl = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    return W.Batch(**{**b.__dict__, "q": q, "query_start_loc": qsl})


@pytest.mark.parametrize("s", [1, 2, 4, 6, 8])
def test_edges(s):
    announce(f"prefill D=64 edges s={s}")
    pb = 256 // s  # positions per block
    chunks = [(2, 0), (pb - 1, 0), (pb, 1), (pb + 1, 15), (3, 61), (2, 62), (17, 63), (64, 64), (1, 40), (65, 200), (2 * pb + 5, 33)]
    b = _batch(chunks, s, 2, 100 + s)
    assert_parity(run_gpu(b), run_oracle(b), strict=False, what=f"D=64 s={s}")


def test_beyond_the_block_table_window():
    announce("prefill D=64 past 2,048 pages")
    b = _batch([(9, 33000), (40, 32750)], 2, 1, 7, poison=False)
    assert_parity(run_gpu(b), run_oracle(b), strict=False, what="D=64 long")


@pytest.mark.parametrize("exp", [-60, -20, 20, 60])
def test_v_scales(exp):
    announce(f"prefill D=64 V scaled 2^{exp}")
    b = _batch([(70, 30), (33, 500)], 4, 2, 9, poison=False)
    v = W.bf16_bits_to_f32(b.v_pages) * np.float32(2.0) ** exp
    b = W.Batch(**{**b.__dict__, "v_pages": W.f32_to_bf16_bits(v)})
    got, ref = run_gpu(b) * 2.0 ** -exp, run_oracle(b) * 2.0 ** -exp  # (powers of two: exact)
    assert_parity(got, ref, strict=False, what=f"V scale 2^{exp}")


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
def test_nonfinite_v(value):
    """Keys 20 (seen by all rows of sequence 1), and 90 (the chunk of sequence
    0 starts at 40: rows before position 90 do not see it)."""
    announce(f"prefill D=64 V = {value}")
    b = _batch([(100, 40), (30, 50)], 4, 2, 11, poison=False)
    bits = W.f32_to_bf16_bits(np.array([value], np.float32))[0]
    v = b.v_pages.copy()
    v[b.block_table[0, 90 // 16], 0, 90 % 16, 5] = bits
    v[b.block_table[1, 20 // 16], 1, 20 % 16, :] = bits
    b = W.Batch(**{**b.__dict__, "v_pages": v})
    got, ref = run_gpu(b), run_oracle(b)
    assert np.array_equal(np.isfinite(got), np.isfinite(ref))
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    assert np.isfinite(ref[:50]).all() and not np.isfinite(ref[50:100, :4, 5]).any()
    ok = np.isfinite(ref).all(axis=-1)
    assert_parity(got[ok], ref[ok], strict=False, what="finite rows")
