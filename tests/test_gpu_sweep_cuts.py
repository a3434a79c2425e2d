"""How a launch is cut into workgroups: short sequences (spans of a few tiles), and batches whose workgroups fill whole
rounds.  Scores against the oracle, and canaries behind the workspace the library asked for."""
import numpy as np
import pytest

from oracle import lava_oracle as O
from paper_2509_09754_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def lava():
    from paper_2509_09754_amd import lava as L
    return L


def run(lava, desc, shapes, inps):
    """The scores of a batch, with a guarded workspace."""
    q, k, v = (torch.cat([lava.to_device(getattr(i, n), s.dtype).reshape(-1) for s, i in zip(shapes, inps)])
               for n in ("q_win", "k", "v"))
    lens = [s.n for s in shapes]
    need = lava.lava_window_scores_workspace_bytes(desc, len(lens), sum(lens))
    buf = torch.full((need + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
    out = lava.lava_window_scores(desc, lens, q, k, v, workspace=buf[:need])
    torch.cuda.synchronize()
    assert bool((buf[need:] == 0x5A).all())
    return [x.cpu().numpy() for x in out]


def check(shapes, inps, out):
    """Scores: fp32 sums of exact products, 1e-5 of the value; the statistic: 1e-4 (its logarithms are fp32)."""
    scores, vbar, stat = out
    at = 0
    for b, (s, i) in enumerate(zip(shapes, inps)):
        want = O.lava_scores(*i.f64(), s.window, s.pool_kernel)[0]
        got = scores[at: at + s.n_kv_heads * s.n].reshape(s.n_kv_heads, s.n).astype(np.float64)
        at += s.n_kv_heads * s.n
        mask = want > 1e-30 * want.max()
        assert np.max(np.abs(got[:, : s.n_prefix][mask] - want[mask]) / want[mask]) < 1e-5
        assert np.all(np.isposinf(got[:, s.n_prefix:]))
        e = O.layer_entropy(want)
        assert abs(stat[b] - e) <= 1e-4 * abs(e) + 2e-5 / want.size


# one tile, one span, several spans with a ragged last one; one round of wavefronts per span and two
@pytest.mark.parametrize("cfg,n", [(1, 9), (1, 128), (1, 129), (1, 1000), (1, 2049), (1, 4097), (2, 33), (2, 191), (2, 193), (2, 1537),
                                   (2, 6143 + 32)])
def test_short_sequences(lava, cfg, n):
    print(f"short sequence cfg{cfg} n={n}", flush=True)
    s = synth.config(cfg, n=n, budget=0, heavy_count=8 if n > 64 else 1)
    i = synth.gen_layer(s, n)
    desc = lava.LayerDesc.make(s.n_q_heads, s.n_kv_heads, s.head_dim, s.window, s.dtype)
    check([s], [i], run(lava, desc, [s], [i]))


def test_batch_of_whole_rounds(lava):
    """Sequences of very different length in one launch of several rounds (2 KV heads: few workgroups per token)."""
    print("batch cut into whole rounds", flush=True)
    base = synth.LayerShape(8, 2, 64, 0, 8, "bf16", 0, heavy_frac=0.01)
    import dataclasses
    lens = [40000, 33, 3000, 131071, 9, 50001, 77777, 131072, 64, 100000] + [90000 + 17 * j for j in range(10)]
    shapes = [dataclasses.replace(base, n=n, heavy_count=4 if n > 64 else 1) for n in lens]
    inps = [synth.gen_layer(s, 3 + j) for j, s in enumerate(shapes)]
    desc = lava.LayerDesc.make(8, 2, 64, 8, "bf16")
    check(shapes, inps, run(lava, desc, shapes, inps))


# 5 heads a group: its parts meet in one workgroup or, with 8 tiles a compute unit, in memory; 9: always in memory
@pytest.mark.parametrize("heads", [5, 9])
@pytest.mark.parametrize("n", [40, 1024 + 8, 2049 + 8, 8000, 8500])
@pytest.mark.parametrize("kind", ["lava", "lse", "attention"])
def test_split_group(lava, n, kind, heads, launches):
    """A group swept in parts: the raw scores the parts join start from zero whichever kernel is the call's first
    (statistics, value norms, the fill of the attention score), also in a workspace full of large floats, and the
    pooling launch takes 4 or 8 entries per thread (8 where 64 heads leave the workspace few partials)."""
    print(f"split group {kind} n={n} {heads} heads", flush=True)
    hq = 64 * heads
    s = synth.LayerShape(hq, 64, 64, n, 8, "bf16", 0, heavy_count=64)
    i = synth.gen_layer(s, n)
    desc = lava.LayerDesc.make(hq, 64, 64, 8, "bf16", score_kind=lava.LAVA_SCORE_ATTENTION if kind == "attention" else lava.LAVA_SCORE_LAVA)
    q, k, v = (lava.to_device(a, "bf16") for a in (i.q_win, i.k, i.v))
    lse = torch.from_numpy(O.window_lse(*i.f64()[:2]).astype(np.float32)).cuda() if kind == "lse" else None
    need = lava.lava_window_scores_workspace_bytes(desc, 1, n)
    ws = torch.full((need,), 0x7E, dtype=torch.uint8, device="cuda")
    (scores, _, _), count = launches(lambda: lava.lava_window_scores(desc, [n], q, k, v, lse=lse, workspace=ws))
    assert count["poolstat"] == (1 if heads == 9 or (n == 1024 + 8 and kind != "lse") else 0)
    want = O.lava_scores(*i.f64(), 8, 7, use_value_norm=kind != "attention")[0]
    got = scores.cpu().numpy().reshape(64, n)[:, : n - 8].astype(np.float64)
    mask = want > 1e-30 * want.max()
    assert np.max(np.abs(got[mask] - want[mask]) / want[mask]) < 1e-5


# either side of the lines between which a sequence alone has its group's parts in workgroups of their own (tiles of 32 keys, of
# all heads, a compute unit, of which there are 256)
@pytest.mark.parametrize("dtype,d,G,n,apart", [("bf16", 128, 5, 128, 0), ("bf16", 64, 8, 129, 1), ("bf16", 128, 6, 1280, 1),
                                               ("bf16", 64, 5, 1281, 0), ("f32", 64, 3, 129, 1), ("f32", 64, 4, 1281, 0),
                                               ("f32", 64, 6, 500, 0), ("f32", 128, 4, 10, 1), ("f32", 128, 3, 640, 1),
                                               ("f32", 128, 4, 641, 0), ("f32", 128, 5, 40, 1), ("f32", 128, 6, 2561, 1),
                                               ("f32", 128, 8, 2560, 1), ("f32", 128, 7, 2561, 0)])
@pytest.mark.parametrize("kind", ["lava", "lse", "attention"])
def test_sequence_alone_and_its_groups_parts(lava, dtype, d, G, n, apart, kind, launches):
    """A sequence alone and as one of a batch of two: the same scores, to the order of their sums, wherever the parts meet.
    The workspace of the longer length does for the shorter one."""
    print(f"parts of a group, {dtype} d{d} G{G} n={n} {kind}", flush=True)
    hkv, w = 64, 9
    s = synth.LayerShape(G * hkv, hkv, d, n, w, dtype, 0, heavy_count=1)
    i = synth.gen_layer(s, n)
    desc = lava.LayerDesc.make(G * hkv, hkv, d, w, dtype, score_kind=lava.LAVA_SCORE_ATTENTION if kind == "attention" else lava.LAVA_SCORE_LAVA)
    q, k, v = (lava.to_device(a, dtype) for a in (i.q_win, i.k, i.v))
    lse = torch.from_numpy(O.window_lse(*i.f64()[:2]).astype(np.float32)).cuda() if kind == "lse" else None
    need = lava.lava_window_scores_workspace_bytes(desc, 1, n + 1)
    assert need >= lava.lava_window_scores_workspace_bytes(desc, 1, n)
    buf = torch.full((need + 4096,), 0x7E, dtype=torch.uint8, device="cuda")
    (one, vbar, stat), count = launches(lambda: lava.lava_window_scores(desc, [n], q, k, v, lse=lse, workspace=buf[:need]))
    if kind == "lse" and not (dtype == "f32" and d == 128):
        apart = 0                                                # one sweep
    assert count["poolstat"] == apart and bool((buf[need:] == 0x7E).all())
    twice = [torch.cat([x.reshape(-1)] * 2) for x in (q, k, v)]
    (two, vbar2, stat2), count = launches(lambda: lava.lava_window_scores(
        desc, [n, n], *twice, lse=None if lse is None else torch.cat([lse.reshape(-1)] * 2).view(2 * G * hkv, w)))
    assert count["poolstat"] == 0
    for b in range(2):
        np.testing.assert_allclose(two.view(2, -1)[b].cpu().numpy(), one.cpu().numpy().ravel(), rtol=1e-5)
        assert torch.equal(vbar2[b], vbar[0])
        np.testing.assert_allclose(stat2[b].cpu().numpy(), stat[0].cpu().numpy(), rtol=1e-4)
    want = O.lava_scores(*i.f64(), w, 7, use_value_norm=kind != "attention")[0]
    got = one.cpu().numpy().reshape(hkv, n)[:, : n - w].astype(np.float64)
    mask = want > 1e-30 * want.max()
    assert np.max(np.abs(got[mask] - want[mask]) / want[mask]) < 1e-5


# the lines that depend on the number of KV heads and on the score
@pytest.mark.parametrize("d,hkv,n,kind,apart", [(64, 1, 229376, "lava", 1), (64, 1, 229377, "lava", 0), (128, 2, 81920, "lava", 1),
                                                (128, 2, 81921, "lava", 0), (128, 1, 229377, "attention", 1), (64, 1, 458753, "attention", 0),
                                                (128, 8, 57344, "attention", 0), (128, 8, 57345, "attention", 1), (128, 8, 73728, "lse", 0),
                                                (128, 8, 73729, "lse", 1), (64, 8, 131072, "lse", 0), (64, 8, 131073, "lse", 1),
                                                (64, 8, 131072, "attention", 0), (64, 8, 131073, "attention", 1), (64, 2, 524288, "lava", 0),
                                                (64, 2, 524289, "lava", 1), (64, 8, 131073, "lava", 0)])
def test_long_sequence_alone_and_its_groups_parts(lava, d, hkv, n, kind, apart, launches):
    """A long sequence alone and beside a short one: the same scores, to the order of their sums, wherever the parts meet."""
    print(f"parts of a group, d{d} on {hkv} n={n} {kind}", flush=True)
    G, w, short = 5, 9, 10
    g = torch.Generator(device="cuda").manual_seed(3)
    rand = lambda *shape: torch.randn(*shape, device="cuda", generator=g).bfloat16().reshape(-1)
    q, k, v = rand(2, G * hkv, w, d), rand(hkv, n, d), rand(hkv, n, d)
    desc = lava.LayerDesc.make(G * hkv, hkv, d, w, "bf16", score_kind=lava.LAVA_SCORE_ATTENTION if kind == "attention" else lava.LAVA_SCORE_LAVA)
    lse = torch.full((2 * G * hkv, w), 13.0, device="cuda") if kind == "lse" else None
    need = lava.lava_window_scores_workspace_bytes(desc, 1, n)
    buf = torch.full((need + 4096,), 0x7E, dtype=torch.uint8, device="cuda")
    (one, vbar, stat), count = launches(lambda: lava.lava_window_scores(
        desc, [n], q[: q.numel() // 2], k, v, lse=None if lse is None else lse[: G * hkv], workspace=buf[:need]))
    assert count["poolstat"] == apart and bool((buf[need:] == 0x7E).all())
    k2, v2 = torch.cat([k, rand(hkv, short, d)]), torch.cat([v, rand(hkv, short, d)])
    (two, vbar2, stat2), count = launches(lambda: lava.lava_window_scores(desc, [n, short], q, k2, v2, lse=lse))
    assert count["poolstat"] == 0
    torch.testing.assert_close(two[: hkv * n], one, rtol=1e-5, atol=0)
    assert torch.equal(vbar2[0], vbar[0])
    torch.testing.assert_close(stat2[0], stat[0], rtol=1e-4, atol=0)


# a group split by the length of its sequence, and one that is always split: both clear raw scores
@pytest.mark.parametrize("hq", [28, 36])
def test_split_group_fill_is_no_sweep(lava, hq, launches):
    """The attention score's fill launch writes a float per token and head (2 MB here), the score kernel reads a row of 128:
    cleared by one or two workgroups the fill took longer than the scores (58 us of events against 48), by many 6."""
    import ctypes
    print("split group: time of the fill", flush=True)
    hkv, n = 4, 131072
    g = torch.Generator(device="cuda").manual_seed(1)
    q, k, v = (torch.randn(h, m, 128, device="cuda", generator=g).bfloat16() for h, m in ((hq, 32), (hkv, n), (hkv, n)))
    desc = lava.LayerDesc.make(hq, hkv, 128, 32, "bf16", score_kind=lava.LAVA_SCORE_ATTENTION)
    ws = torch.empty(lava.lava_window_scores_workspace_bytes(desc, 1, n), dtype=torch.uint8, device="cuda")
    names = [lava.lib.lava_prof_kernel_name(i) for i in range(lava.lib.lava_prof_kernel_count())]
    _, count = launches(lambda: lava.lava_window_scores(desc, [n], q, k, v, workspace=ws))
    assert count["poolstat"] == 1
    best = {b"vnorm": 1e9, b"scores": 1e9}
    try:
        for _ in range(8):
            lava.lib.lava_prof_enable(1), lava.lib.lava_prof_reset()
            lava.lava_window_scores(desc, [n], q, k, v, workspace=ws)
            torch.cuda.synchronize()
            for name in best:
                ms, launches = ctypes.c_double(), ctypes.c_int64()
                lava.lib.lava_prof_read(names.index(name), ctypes.byref(ms), ctypes.byref(launches))
                assert launches.value == 1
                best[name] = min(best[name], ms.value)
    finally:
        lava.lib.lava_prof_enable(0), lava.lib.lava_prof_reset()
    print(best, flush=True)
    assert best[b"vnorm"] < 0.5 * best[b"scores"]


# two to four rounds of few workgroups (spans of at most 128 tiles of 32 keys, narrow 96), one chunk and several
@pytest.mark.parametrize("dtype,d,hq,hkv,wgs,n", [("bf16", 64, 5, 1, 1, 128 * 32 + 1), ("bf16", 128, 4, 2, 2, 4500), ("f32", 64, 8, 1, 1, 7000),
                                                  ("bf16", 64, 3, 1, 3, 3 * 4096 + 40), ("f32", 128, 2, 1, 1, 3 * 4096 + 1),
                                                  ("bf16", 128, 6, 3, 2, 4096 + 50)])
@pytest.mark.parametrize("shape", ["wide", "narrow"])
@pytest.mark.parametrize("schedule", ["separate", "persistent", "prepass"])
def test_sequence_alone_of_several_rounds(lava, dtype, d, hq, hkv, wgs, n, shape, schedule, tuning):
    """A sequence alone whose spans are longer than a workgroup holds is cut into whole rounds of workgroups: the scores are the
    oracle's, and the workspace of that length holds the partials."""
    print(f"several rounds, {dtype} d{d} {hq} on {hkv}, {wgs} workgroups, n={n} {shape} {schedule}", flush=True)
    s = synth.LayerShape(hq, hkv, d, n, 17, dtype, 0, heavy_count=32)
    i = synth.gen_layer(s, n)
    tuning(sweep_workgroups=wgs, sweep_shape=shape, sweep_schedule=schedule)
    desc = lava.LayerDesc.make(hq, hkv, d, 17, dtype)
    need = lava.lava_window_scores_workspace_bytes(desc, 1, n)
    buf = torch.full((need + 4096,), 0x7E, dtype=torch.uint8, device="cuda")
    q, k, v = (lava.to_device(a, dtype) for a in (i.q_win, i.k, i.v))
    scores, _, _ = lava.lava_window_scores(desc, [n], q, k, v, workspace=buf[:need])
    torch.cuda.synchronize()
    assert bool((buf[need:] == 0x7E).all())
    want = O.lava_scores(*i.f64(), 17, 7)[0]
    got = scores.cpu().numpy().reshape(hkv, n)[:, : n - 17].astype(np.float64)
    mask = want > 1e-30 * want.max()
    assert np.max(np.abs(got[mask] - want[mask]) / want[mask]) < 1e-5


@pytest.mark.parametrize("dtype,d,hq,hkv,n", [("bf16", 128, 28, 4, 270000), ("bf16", 128, 32, 8, 140000), ("f32", 128, 32, 8, 140000)])
def test_sequence_alone_fills_its_rounds(lava, dtype, d, hq, hkv, n, tuning):
    """Just more spans than the device takes at a time: the library's own cut against one of two full rounds, events around
    the scores.  A last round that is nearly empty takes 1.3 to 1.5 times as long (368 us against 255, 228 against 177, 888 against
    582)."""
    print(f"rounds of a sequence alone, {dtype} {hq} on {hkv}, {n}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(1)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    q, k, v = (torch.randn(h, m, d, device="cuda", generator=g).to(dt) for h, m in ((hq, 32), (hkv, n), (hkv, n)))
    desc = lava.LayerDesc.make(hq, hkv, d, 32, dtype)
    best = {}
    for wgs in (0, 512):
        tuning(sweep_workgroups=wgs)
        ws = torch.empty(lava.lava_window_scores_workspace_bytes(desc, 1, n), dtype=torch.uint8, device="cuda")
        for _ in range(8):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            lava.lava_window_scores(desc, [n], q, k, v, workspace=ws)
            b.record()
            torch.cuda.synchronize()
            best[wgs] = min(best.get(wgs, 1e9), a.elapsed_time(b))
    print(best, flush=True)
    assert best[0] < 1.12 * best[512]


def test_ragged_batch_of_one_round(lava):
    """32-bit sequences of d_h 128 whose shares of the device, rounded up, are a few workgroups more than it has: the batch takes
    little longer than one of equal lengths and as many tokens (254 us and 234), and not a second round (437)."""
    print("ragged 32-bit batch of one round", flush=True)
    hq, hkv, d = 12, 2, 128
    lens = [35828, 21654, 34808, 42833]
    desc, best = lava.LayerDesc.make(hq, hkv, d, 32, "f32"), {}
    g = torch.Generator(device="cuda").manual_seed(1)
    q, k, v = (torch.randn(m * d, device="cuda", generator=g) for m in (4 * hq * 32, hkv * sum(lens), hkv * sum(lens)))
    for name, ls in (("ragged", lens), ("equal", [33781, 33781, 33781, 33780])):
        ws = torch.empty(lava.lava_window_scores_workspace_bytes(desc, 4, sum(ls)), dtype=torch.uint8, device="cuda")
        for _ in range(8):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            lava.lava_window_scores(desc, ls, q, k, v, workspace=ws)
            b.record()
            torch.cuda.synchronize()
            best[name] = min(best.get(name, 1e9), a.elapsed_time(b))
    print(best, flush=True)
    assert best["ragged"] < 1.35 * best["equal"]
