"""The selection's paths by size and by where the scores lie, against the oracle (integer-exact): one or several
workgroups per problem at every number of keys per lane, an interval of the first histogram with more keys than are
collected at once, one workgroup that holds more of them than its segment takes, the histogram's end bins, and the step
launches; plain and prepared problems alone and in one table."""
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


def flat(kind, n, seed):
    """n scores: 'plateau' as pooling leaves them; 'narrow' within 2 %, so that one interval holds thousands; 'burst'
    a run of nearly equal large scores; 'tiny' / 'huge' beyond the first histogram's range; 'signed'; 'equal'."""
    r = np.random.Generator(np.random.PCG64(seed))
    if kind == "plateau":
        return synth.random_scores(1, n, seed).ravel()
    if kind == "narrow":
        return (1.0 + 0.02 * r.random(n)).astype(np.float32)
    if kind == "burst":
        s = np.exp(r.standard_normal(n) * 2.0).astype(np.float32)
        k = min(n, 3000)
        at = int(r.integers(0, n - k + 1))
        s[at: at + k] = (40.0 + 1e-4 * r.random(k)).astype(np.float32)
        return s
    if kind == "tiny":
        return (np.exp(r.standard_normal(n)) * 2.0 ** -60).astype(np.float32)
    if kind == "huge":
        return (np.exp(r.standard_normal(n)) * 2.0 ** 40).astype(np.float32)
    if kind == "signed":
        s = r.standard_normal(n).astype(np.float32)
        s[r.random(n) < 0.1] = np.float32(-0.0)
        s[r.random(n) < 0.1] = np.float32(0.0)
        return s
    return np.full(n, 0.5, dtype=np.float32)


def want(s, nh, budget):
    offs = (np.arange(nh + 1) * (s.size // nh)).astype(np.int64)
    return O.select_topk(s.astype(np.float64), offs, budget)


def check(got, s, nh, budget):
    counts, offs, idx, kept = (x.cpu().numpy() for x in got)
    rc, ro, ri, _ = want(s, nh, budget)
    assert np.array_equal(counts, rc) and np.array_equal(offs, ro) and np.array_equal(idx[:budget], ri)
    flat_idx = np.concatenate([g * (s.size // nh) + ri[ro[g]: ro[g + 1]] for g in range(nh)]).astype(np.int64)
    assert np.array_equal(kept[:budget].view(np.uint32), s[flat_idx].view(np.uint32))   # bit for bit, -0 included


# 2, 4, 8 and 12 keys per lane; one workgroup and several; the last one full, with one entry, and empty rows
SIZES = [1, 63, 2047, 2048, 2049, 20 * 2048, 20 * 2048 + 1, 64 * 4096, 64 * 4096 + 4, 64 * 8192 - 4, 64 * 8192 + 4]


@pytest.mark.parametrize("n", SIZES)
def test_select_sizes(lava, n):
    print(f"select sizes n={n}", flush=True)
    s = flat("plateau", n, n)
    sc = torch.from_numpy(s).cuda()
    for budget in sorted({0, 1, n // 100, n // 3, n - 1, n}):
        check(lava.lava_select_topk(1, sc, budget), s, 1, budget)


@pytest.mark.parametrize("kind", ["narrow", "burst", "tiny", "huge", "signed", "equal"])
@pytest.mark.parametrize("n", [2000, 3 * 4096 + 12, 8 * 20000])
def test_select_values(lava, kind, n):
    print(f"select values {kind} n={n}", flush=True)
    nh = 4
    s = flat(kind, n, 7 + n)
    sc = torch.from_numpy(s).cuda()
    for budget in (1, n // 50, n // 2, n - 3):
        check(lava.lava_select_topk(nh, sc, budget), s, nh, budget)


def test_select_crowded_interval_beyond_the_list(lava):
    print("select: 2 M narrow scores (several histograms), and the step launches on 3.4 M", flush=True)
    for n in (2_000_000, 3_400_000):
        for kind in ("narrow", "burst"):
            s = flat(kind, n, n)
            check(lava.lava_select_topk(8, torch.from_numpy(s).cuda(), n // 100), s, 8, n // 100)


def test_select_table_mixes_sizes_and_needs_one_clearing(lava):
    """40 problems of one or several workgroups (two groups of a table): the second group's choice of keys per lane
    differs from the first's, and every problem's region is cleared when its selection needs that."""
    print("select table: 40 mixed problems", flush=True)
    nh, sizes = 2, [int(x) for x in np.linspace(10, 60000, 39).astype(int) // 2 * 2] + [300000]
    data, probs = [], []
    for i, n in enumerate(sizes):
        s = flat(("plateau", "narrow", "signed")[i % 3], n, i)
        budget = max(1, n // 7)
        out = (torch.full((nh,), -7, dtype=torch.int32, device="cuda"), torch.full((nh + 1,), -7, dtype=torch.int64, device="cuda"),
               torch.full((budget,), -7, dtype=torch.int32, device="cuda"), torch.empty(budget, device="cuda"))
        sc = torch.from_numpy(s).cuda()
        probs.append(lava.select_problem(sc, budget, out[0], out[1], out[2], out[3]))
        data.append((s, sc, budget, out))
    ws = torch.randint(0, 256, (lava.lava_select_batch_workspace_bytes(len(probs), max(sizes)),), dtype=torch.uint8, device="cuda")
    for _ in range(2):
        lava.lava_select_topk_batch(nh, probs, max(sizes), workspace=ws)
        torch.cuda.synchronize()
        for s, _, budget, out in data:
            check(out, s, nh, budget)
    assert lava.lava_select_batch_status(ws, len(probs), max(sizes)) == lava.LAVA_OK


@pytest.mark.parametrize("n", [257, 3000, 40000])
def test_prepared_equals_plain(lava, n):
    """The histogram the score kernels prepare leads to the same selection as the plain call's own."""
    print(f"prepared selection n={n}", flush=True)
    sh = synth.config(2, n=n, budget=8 * 40)
    inp = synth.gen_layer(sh, n)
    desc = lava.LayerDesc.make(sh.n_q_heads, sh.n_kv_heads, sh.head_dim, sh.window, sh.dtype)
    q, k, v = (lava.to_device(a, sh.dtype) for a in (inp.q_win, inp.k, inp.v))
    a = lava.evict_layer(desc, n, q, k, v, sh.budget, primed=True)
    b = lava.evict_layer(desc, n, q, k, v, sh.budget, primed=False)
    for key in ("scores", "head_counts", "head_offsets", "kept_idx", "kept_scores", "k_hat"):
        assert torch.equal(a[key], b[key]), key


@pytest.mark.parametrize("kind", ["narrow", "tiny", "huge", "signed", "equal"])
def test_select_step_launches(lava, kind):
    """Two digits behind a bin of the first histogram or of its end bins' one, none where all keys are equal."""
    n, nh = 3_400_000, 4
    print(f"select step launches {kind}", flush=True)
    s = flat(kind, n, 11)
    sc = torch.from_numpy(s).cuda()
    for budget in (n // 50, n // 2):
        check(lava.lava_select_topk(nh, sc, budget), s, nh, budget)


# one workgroup, several, the step launches; values scaled so that all scores lie in the first histogram's range, or in
# either of its end bins, of which a prepared region holds no further histogram
@pytest.mark.parametrize("scale", [1.0, 2.0 ** -70, 2.0 ** 50])
@pytest.mark.parametrize("n", [200, 20011, 400003])
def test_prepared_equals_plain_in_every_bin(lava, n, scale):
    print(f"prepared selection n={n} scale={scale}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(n)
    q = torch.randn(8, 16, 64, device="cuda", generator=g).bfloat16()
    k, v = (torch.randn(8, n, 64, device="cuda", generator=g).bfloat16() for _ in range(2))
    v = (v.float() * scale).bfloat16()
    desc = lava.LayerDesc.make(8, 8, 64, 16, "bf16")
    ws = torch.full((lava.lava_select_workspace_bytes(8 * n),), 0x5A, dtype=torch.uint8, device="cuda")
    scores, _, _ = lava.lava_window_scores(desc, [n], q, k, v, select_workspace=ws)
    for i, budget in enumerate((8 * 20, 8 * n // 3)):
        if i > 0:
            lava.lava_window_scores(desc, [n], q, k, v, scores=scores, select_workspace=ws)
        a = lava.lava_select_topk(8, scores, budget, workspace=ws, primed=True)
        b = lava.lava_select_topk(8, scores, budget)
        for x, y in zip(a, b):
            assert torch.equal(x, y)
        top = torch.sort(scores, descending=True, stable=True).indices[:budget].sort().values
        assert torch.equal(b[2].long(), top % n)
