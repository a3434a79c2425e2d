"""Groups whose query heads are swept in parts by the wavefronts of one workgroup (bf16: 5 to 8 heads, f32: 3 to 8), heads with
short windows that share a block of 32 rows, and 32-bit products formed from bf16 parts."""
import dataclasses

import numpy as np
import pytest

from oracle import lava_oracle as O
from paper_2509_09754_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def lava():
    from paper_2509_09754_amd import lava as L
    yield L
    L.set_tuning()


def scores_of(lava, shapes, layers, sweep_shape="auto", lse=None):
    s = shapes[0]
    desc = lava.LayerDesc.make(s.n_q_heads, s.n_kv_heads, s.head_dim, s.window, s.dtype)
    q, k, v = (torch.cat([lava.to_device(x[i], s.dtype).reshape(-1) for x in layers]) for i in range(3))
    lava.set_tuning(sweep_shape=sweep_shape)
    out = lava.lava_window_scores(desc, [x.n for x in shapes], q, k, v, lse=lse)
    torch.cuda.synchronize()
    lava.set_tuning()
    return [x.cpu().numpy().astype(np.float64) for x in out]


def check(shapes, refs, out, tol=1e-5):
    """fp32 sums (over d_h products, then over the keys of a row) of values exact to 2^-24: a few 1e-6 of a score."""
    at = 0
    for b, (s, want) in enumerate(zip(shapes, refs)):
        got = out[0][at: at + s.n_kv_heads * s.n].reshape(s.n_kv_heads, s.n)
        at += s.n_kv_heads * s.n
        mask = want > 1e-30 * want.max()
        assert np.max(np.abs(got[:, : s.n_prefix][mask] - want[mask]) / want[mask]) < tol
        assert np.all(got[:, : s.n_prefix][want == 0] == 0)
        assert np.all(np.isposinf(got[:, s.n_prefix:]))
        e = O.layer_entropy(want)
        assert abs(out[2][b] - e) <= 1e-4 * abs(e) + 2e-5 / want.size


def shape_of(dtype, d, G, w, n):
    return dataclasses.replace(synth.config(1, n=n, budget=0, heavy_count=4), n_q_heads=2 * G, n_kv_heads=2, head_dim=d,
                               window=w, dtype=dtype)


# every number of heads per part and of parts, a part with heads missing, windows of two row blocks, two and four heads in a
# block, blocks with heads missing; one tile per wavefront, several, ragged ends; and the shape of two workgroups per
# compute unit
@pytest.mark.parametrize("sweep_shape", ["wide", "narrow"])
@pytest.mark.parametrize("dtype,d,G,w", [("bf16", 128, 5, 32), ("bf16", 128, 8, 7), ("bf16", 64, 6, 16), ("bf16", 128, 3, 33),
                                         ("bf16", 128, 9, 32), ("f32", 64, 1, 8), ("f32", 64, 2, 8), ("f32", 64, 4, 32),
                                         ("f32", 64, 5, 8), ("f32", 64, 3, 40), ("f32", 128, 1, 32), ("f32", 128, 4, 32),
                                         ("f32", 128, 6, 20), ("f32", 128, 3, 40), ("f32", 128, 9, 8),
                                         ("bf16", 128, 2, 8), ("bf16", 128, 2, 16), ("bf16", 128, 4, 8), ("bf16", 64, 3, 9),
                                         ("bf16", 128, 16, 8), ("bf16", 64, 16, 16), ("f32", 128, 7, 5), ("f32", 64, 16, 1)])
def test_groups_in_parts(lava, dtype, d, G, w, sweep_shape):
    lengths = [w + 1, 333, 2085] if sweep_shape == "wide" else [2085, 333]
    print(f"groups in parts {dtype} d{d} G{G} w{w} {sweep_shape} {lengths}", flush=True)
    shapes = [shape_of(dtype, d, G, w, n) for n in lengths]
    inps = [synth.gen_layer(s, 3 + i) for i, s in enumerate(shapes)]
    refs = [O.lava_scores(*i.f64(), s.window, s.pool_kernel)[0] for s, i in zip(shapes, inps)]
    check(shapes, refs, scores_of(lava, shapes, [(i.q_win, i.k, i.v) for i in inps], sweep_shape))


@pytest.mark.parametrize("d,G", [(64, 4), (128, 4), (128, 1)])
def test_32_bit_products_of_any_values(lava, d, G):
    """Values over many magnitudes, the largest there are (no part may overflow) and infinities (a key that minus
    infinity takes out of every softmax, in a tile of its own way through the kernel)."""
    print(f"32-bit products of any values d{d} G{G}", flush=True)
    s = shape_of("f32", d, G, 32, 700)
    i = synth.gen_layer(s, 5)
    q, k, v = (np.array(x, dtype=np.float32) for x in (i.q_win, i.k, i.v))
    rng = np.random.Generator(np.random.PCG64(3))
    k *= np.exp2(rng.integers(-20, 2, size=k.shape)).astype(np.float32)
    q[..., 0] = np.abs(q[..., 0]) + 0.1
    q[..., 1] = 0.0
    k[0, 40, 0] = -np.inf
    k[1, 300, 0] = -np.inf
    k[:, 77, 1] = np.finfo(np.float32).max
    k[:, 78, 1] = -np.finfo(np.float32).max
    want = O.lava_scores(q.astype(np.float64), k.astype(np.float64), v.astype(np.float64), s.window, s.pool_kernel)[0]
    assert np.isfinite(want).all()
    check([s], [want], scores_of(lava, [s], [(q, k, v)]))


@pytest.mark.parametrize("dtype,d,G,w", [("bf16", 128, 4, 8), ("bf16", 64, 3, 16), ("f32", 64, 5, 7), ("f32", 128, 2, 12)])
def test_heads_sharing_a_block_take_the_callers_log_sum_exp(lava, dtype, d, G, w):
    print(f"heads sharing a block, caller's log-sum-exp, {dtype} d{d} G{G} w{w}", flush=True)
    s = shape_of(dtype, d, G, w, 900)
    i = synth.gen_layer(s, 8)
    q, k, v = i.f64()
    x = np.einsum("gtrd,gnd->gtrn", q.reshape(2, G, w, d), k) / np.sqrt(d)
    x[..., s.n - w:][..., np.arange(w)[None, :] > np.arange(w)[:, None]] = -np.inf
    m = x.max(-1, keepdims=True)
    lse = (m + np.log(np.exp(x - m).sum(-1, keepdims=True))).reshape(2 * G, w)
    want = O.lava_scores(q, k, v, s.window, s.pool_kernel)[0]
    # the log-sum-exp is handed over in 32 bits: 6e-8 of a value around 10 is 6e-7 of a score
    check([s], [want], scores_of(lava, [s], [(i.q_win, i.k, i.v)], lse=torch.from_numpy(lse.astype(np.float32)).cuda()))


@pytest.mark.parametrize("big_q", [1.0, 2.0**10, 2.0**25, 2.0**70])
@pytest.mark.parametrize("d,G,w", [(64, 4, 32), (128, 4, 32), (128, 1, 7)])
def test_32_bit_products_that_overflow(lava, d, G, w, big_q):
    """Keys masked by the type's lowest value (or near it) against queries of any size: the product is the lowest value or
    minus infinity, the key's weight zero and the other keys' weights what they are without it.  No part of a value and no
    product of parts may overflow to the other side."""
    print(f"32-bit products that overflow d{d} G{G} w{w} query {big_q}", flush=True)
    s = shape_of("f32", d, G, w, 700)
    i = synth.gen_layer(s, 6)
    q, k, v = (np.array(x, dtype=np.float32) for x in (i.q_win, i.k, i.v))
    top = np.finfo(np.float32).max
    q[..., 1] = np.float32(big_q)
    k[..., 1] = 0.0
    for row, x in ((40, -top), (77, -top * np.float32(0.5020)), (300, -top * np.float32(0.9980))):
        k[:, row, 1] = x
    want = O.lava_scores(q.astype(np.float64), k.astype(np.float64), v.astype(np.float64), s.window, s.pool_kernel)[0]
    assert np.isfinite(want).all()
    check([s], [want], scores_of(lava, [s], [(q, k, v)]))


def test_32_bit_queries_of_the_largest_value(lava):
    """A query row with the largest value, put together again from its parts for the 32-bit instructions."""
    print("32-bit queries of the largest value", flush=True)
    s = shape_of("f32", 128, 2, 32, 700)
    i = synth.gen_layer(s, 7)
    q, k, v = (np.array(x, dtype=np.float32) for x in (i.q_win, i.k, i.v))
    q[..., 1] = np.finfo(np.float32).max
    k[..., 1] = 0.0
    k[:, 5, 1] = 2.0**-128                                       # times the query: 1 - 2^-24
    want = O.lava_scores(q.astype(np.float64), k.astype(np.float64), v.astype(np.float64), s.window, s.pool_kernel)[0]
    check([s], [want], scores_of(lava, [s], [(q, k, v)]))


@pytest.mark.parametrize("d", [64, 128])
def test_32_bit_products_of_one_channel(lava, d):
    """Rows whose logit is one product (an outlier channel), with mantissas that make the left-out products of parts as
    large as they get, of one sign.  Against a key whose product has one digit and no error, a logit is off by at most
    0.99 * 2^-24 of it for what is left out and 2^-24 for the rounding of the sum; 0.25 * 2^-24 for the exponential and the
    score (half a unit each in 32 bits, of a logit of about 256)."""
    print(f"32-bit products of one channel d{d}", flush=True)
    heads, n = 16, 1201
    rng = np.random.Generator(np.random.PCG64(9))
    q, k, v = np.zeros((heads, 1, d), np.float32), np.zeros((heads, n, d), np.float32), np.ones((heads, n, d), np.float32)
    for h, bits in enumerate([0x3f80fe80, 0x3f807f40, 0x3f803f40, 0x3f817f40] * (heads // 4)):
        x = np.uint32(bits).view(np.float32)
        at = int(rng.integers(d))
        q[h, 0, at] = 16 * x
        k[h, :, at] = 16 + 16 * rng.random(n) / 128
        k[h, 100:400, at] = 16 * x
        k[h, 0, at] = 16.0
    desc = lava.LayerDesc.make(heads, heads, d, 1, "f32", pool_kernel=1, softmax_scale=1.0)
    scores, _, _ = lava.lava_window_scores(desc, [n], *(lava.to_device(x, "f32") for x in (q, k, v)))
    torch.cuda.synchronize()
    got = scores.cpu().numpy().reshape(heads, n)[:, : n - 1].astype(np.float64)
    logits = (q.astype(np.float64) @ k.astype(np.float64).transpose(0, 2, 1))[:, 0, : n - 1]
    err = np.log(got / got[:, :1]) - (logits - logits[:, :1])
    worst = float(np.max(np.abs(err) / logits)) * 2.0**24
    print(f"   worst {worst:.2f} * 2^-24 of the logit", flush=True)
    assert worst < 0.99 + 1.0 + 0.25


@pytest.mark.parametrize("what", ["nan key", "inf key", "inf query", "nan window"])
@pytest.mark.parametrize("dtype,d,G,w", [("bf16", 128, 2, 16), ("bf16", 64, 2, 9), ("f32", 64, 2, 16), ("f32", 128, 2, 5), ("bf16", 128, 4, 8),
                                         ("f32", 64, 3, 8)])
def test_heads_sharing_a_block_with_values_that_are_not_finite(lava, dtype, d, G, w, what):
    """A head whose attention is not a number takes no part in its group's maximum, and a group of such heads scores zero,
    whether its heads share a row block or not: the same heads twice in the group, too many for one block, give the same
    scores."""
    print(f"heads sharing a block, {what}, {dtype} d{d} G{G} w{w}", flush=True)
    s = shape_of(dtype, d, G, w, 900)
    i = synth.gen_layer(s, 12)
    q, k, v = (lava.to_device(x, dtype).clone() for x in (i.q_win, i.k, i.v))
    if what == "nan key":
        k[0, 50, 3] = float("nan")
    elif what == "inf key":
        k[0, 50, 3], k[1, 60, 4] = float("inf"), float("-inf")
    elif what == "inf query":
        q[0, 1, 5] = float("inf")
    else:
        k[0, s.n - 1, 3] = float("nan")                          # seen by the last window row alone
    twice = torch.cat([x.repeat(2, 1, 1) for x in q.view(2, G, w, d)])
    out = []
    for heads, x in ((G, q), (2 * G, twice)):
        desc = lava.LayerDesc.make(2 * heads, 2, d, w, dtype)
        out.append([t.cpu().numpy() for t in lava.lava_window_scores(desc, [s.n], x.contiguous(), k, v)])
    assert not np.isnan(out[0][0]).any()
    for got, want in zip(*out):
        np.testing.assert_allclose(got, want, rtol=1e-5)
