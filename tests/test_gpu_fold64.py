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
