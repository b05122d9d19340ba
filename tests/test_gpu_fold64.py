"""The matrix-core folds at head_dim 64 hold what the VALU fold held: softmax
weights in fp32.  Shown by the share of bf16 outputs that are not the float64
result correctly rounded: an output whose fp32 value is off by a relative r
lands on another bf16 value where a rounding boundary lies in between, in at
most 2^8 r of the cases.  Weights of 24 bits leave the error of the fp32 sums
(r about 1e-6: measured 1e-4 to 5e-4 of the outputs, as with the VALU fold),
weights of 16 bits add 2^-17 each (r about 1e-5: measured 1.3e-3 to 2.5e-3).
The line is between the two."""
import numpy as np
import pytest

from paper_2504_09345_amd import workloads as W

from parity_util import announce, assert_parity, run_gpu, run_oracle

pytestmark = pytest.mark.gpu

MISROUNDED = 1e-3


def _exact(b):
    """float64 attention, row by row."""
    f = W.bf16_bits_to_f32
    q, k, v = f(b.q).astype(np.float64), f(b.k_pages), f(b.v_pages)
    T, H_q, D = q.shape
    H_kv = k.shape[1]
    s = H_q // H_kv
    qsl = np.arange(T + 1) if b.query_start_loc is None else b.query_start_loc
    out = np.empty(q.shape)
    for i, C in enumerate(b.context_lens):
        pages = b.block_table[i, :(C + 15) // 16]
        L = qsl[i + 1] - qsl[i]
        kd = k[pages].transpose(1, 0, 2, 3).reshape(H_kv, -1, D)[:, :C].astype(np.float64)
        vd = v[pages].transpose(1, 0, 2, 3).reshape(H_kv, -1, D)[:, :C].astype(np.float64)
        hidden = np.arange(C)[None, :] > np.arange(C - L, C)[:, None]
        for h in range(H_q):
            x = q[qsl[i]:qsl[i + 1], h] @ kd[h // s].T * b.scale
            x[hidden] = -np.inf
            p = np.exp(x - x.max(axis=1, keepdims=True))
            out[qsl[i]:qsl[i + 1], h] = (p / p.sum(axis=1, keepdims=True)) @ vd[h // s]
    return out


def _misrounded(b):
    got, ref = run_gpu(b), _exact(b)
    assert_parity(got, ref, strict=False, what="float64")
    rounded = W.bf16_bits_to_f32(W.f32_to_bf16_bits(ref.astype(np.float32)))
    return float((got != rounded).mean())


def _batch(s, H_kv, ctx, rows, seed):
    b = W.generate("tiny", seed=seed, overrides=dict(H_q=s * H_kv, H_kv=H_kv, D=64, ctx=("list", ctx),
                                                     pool=("factor", 1.2)))
    if rows is None:
        return b
    q = W._fill_normal((sum(rows), s * H_kv, 64), seed, "q", 1.0, "bf16", 1)
    return W.Batch(**{**b.__dict__, "q": q, "query_start_loc": np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)})


@pytest.mark.parametrize("s,H_kv", [(1, 8), (4, 8), (6, 2), (8, 1)])
def test_decode_weights_keep_24_bits(s, H_kv):
    announce(f"D=64 decode precision s={s} H_kv={H_kv}")
    ctx = [int(x) for x in np.random.default_rng(s).integers(200, 1500, size=2048 // (s * H_kv))]
    assert _misrounded(_batch(s, H_kv, ctx, None, 50 + s)) <= MISROUNDED


@pytest.mark.parametrize("s,H_kv,rows,prior", [(4, 2, [400, 333], [0, 700]), (1, 8, [300], [300]), (8, 1, [150] * 3, [40] * 3),
                                               (6, 8, [1500], [0])])
def test_chunk_weights_keep_24_bits(s, H_kv, rows, prior):
    announce(f"D=64 chunk precision s={s} H_kv={H_kv} rows={rows}")
    b = _batch(s, H_kv, [L + p for L, p in zip(rows, prior)], rows, 60 + s)
    assert _misrounded(b) <= MISROUNDED


# (sequences' contexts: items of many parts, of two parts and whole ones, with
# one range per workgroup and with several)
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("s,H_kv,ctx", [(4, 8, [2000, 500, 33, 16, 700]), (8, 8, [90 + 3 * i for i in range(120)]),
                                        (1, 2, [40 + 7 * i for i in range(60)]), (6, 1, [1500, 31])])
def test_decode_nonfinite_v(s, H_kv, ctx, value):
    """One element of V at one key per sequence (first, last and inner keys):
    rows are infinite or NaN where the oracle's are, and nowhere else."""
    announce(f"D=64 decode V = {value} s={s} H_kv={H_kv}")
    b = W.generate("tiny", seed=s, poison=False, overrides=dict(H_q=s * H_kv, H_kv=H_kv, D=64, ctx=("list", ctx),
                                                                pool=("factor", 1.2)))
    bits = W.f32_to_bf16_bits(np.array([value], np.float32))[0]
    v = b.v_pages.copy()
    for i, C in enumerate(ctx):
        if i % 3 != 2:
            t = (0, C - 1, C // 2, C // 3)[i % 4]
            v[b.block_table[i, t // 16], i % H_kv, t % 16, (7 * i) % 64] = bits
    b = W.Batch(**{**b.__dict__, "v_pages": v})
    got, ref = run_gpu(b), run_oracle(b)
    assert np.isinf(ref).any() != np.isnan(value) and not np.isfinite(ref).all()
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    assert np.array_equal(np.isposinf(got), np.isposinf(ref)) and np.array_equal(np.isneginf(got), np.isneginf(ref))
    ok = np.isfinite(ref).all(axis=-1)
    assert_parity(got[ok], ref[ok], strict=False, what="finite rows")


def test_decode_huge_v():
    """Scores that rise by less than the lazy base's slack (weights near 2^7.8
    against the first page's) over V near 2^115: the weighted sum against that
    base is beyond fp32, that against the maximum is not.  (200 sequences of 13
    pages over 256 ranges: most ranges hold a first page and others.)"""
    announce("D=64 decode huge V")
    b = W.generate("tiny", seed=2, poison=False, overrides=dict(H_q=16, H_kv=8, D=64, ctx=("list", [200] * 200),
                                                                pool=("factor", 1.2)))
    q = W.f32_to_bf16_bits(np.ones(b.q.shape, np.float32))
    k = np.full(b.k_pages.shape, 5.4 / 64 / b.scale, np.float32)
    k[b.block_table[:, 0]] = 0.0
    v = W.bf16_bits_to_f32(b.v_pages) * 0.25 + 1.0
    b = W.Batch(**{**b.__dict__, "q": q, "k_pages": W.f32_to_bf16_bits(k),
                   "v_pages": W.f32_to_bf16_bits(v * np.float32(2.0) ** 115)})
    got, ref = run_gpu(b) * 2.0 ** -115, run_oracle(b) * 2.0 ** -115  # (powers of two: exact)
    assert np.isfinite(ref).all()
    assert_parity(got, ref, strict=False, what="huge V")
