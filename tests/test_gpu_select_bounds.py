"""Selections whose workgroups of 12 keys per lane do not divide their workspace region, with the threshold's interval
crowded into the last, partly filled workgroup: survivors against the oracle (integer-exact), canaries behind the
workspace, and the neighbours of a problem in a table."""
import numpy as np
import pytest

from oracle import lava_oracle as O

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

CHUNK = 12 * 1024
NH = 8
CANARY = 0x5A


@pytest.fixture(scope="module")
def lava():
    from paper_2509_09754_amd import lava as L
    return L


def crowded_end(n, inside, seed):
    """(scores, budget): `inside` distinct scores of one interval of the first histogram lie in the last workgroup, no
    others in that interval; some scores lie above it, the budget cuts in the middle of it."""
    r = np.random.Generator(np.random.PCG64(seed))
    s = (1e-3 * np.exp(0.3 * r.standard_normal(n))).astype(np.float32)
    first = (n - 1) // CHUNK * CHUNK
    assert first >= CHUNK and n - first >= inside
    above = r.choice(first, 500, replace=False)
    s[above] = (2.0 + r.random(500)).astype(np.float32)
    at = first + r.choice(n - first, inside, replace=False)
    s[at] = (1.0 + r.permutation(inside) * (0.04 / inside)).astype(np.float32)
    return s, 500 + inside // 2


def check(out, s, budget):
    counts, offs, idx, kept = (x.cpu().numpy() for x in out)
    starts = (np.arange(NH + 1) * (s.size // NH)).astype(np.int64)
    rc, ro, ri, _ = O.select_topk(s.astype(np.float64), starts, budget)
    assert np.array_equal(counts, rc) and np.array_equal(offs, ro) and np.array_equal(idx, ri)
    flat = np.concatenate([starts[g] + ri[ro[g]: ro[g + 1]] for g in range(NH)]).astype(np.int64)
    assert np.array_equal(kept.view(np.uint32), s[flat].view(np.uint32))


def outputs(budget):
    return (torch.empty(NH, dtype=torch.int32, device="cuda"), torch.empty(NH + 1, dtype=torch.int64, device="cuda"),
            torch.empty(budget, dtype=torch.int32, device="cuda"), torch.empty(budget, device="cuda"))


# the last workgroup's keys: fewer than its segment takes, its last word, one more (1048576 entries: 762 words), and more
@pytest.mark.parametrize("inside", [300, 577, 762, 763, 768, 769, 1500])
@pytest.mark.parametrize("n", [557056, 573440, 1048576])
def test_last_workgroup_of_a_problem(lava, n, inside):
    print(f"select bounds n={n} inside={inside}", flush=True)
    s, budget = crowded_end(n, inside, n + inside)
    need = lava.lava_select_workspace_bytes(n)
    buf = torch.full((need + 8192,), CANARY, dtype=torch.uint8, device="cuda")
    out = outputs(budget)
    lava.lava_select_topk(NH, torch.from_numpy(s).cuda(), budget, head_counts=out[0], head_offsets=out[1], kept_idx=out[2],
                          kept_scores=out[3], workspace=buf[:need])
    torch.cuda.synchronize()
    assert bool((buf[need:] == CANARY).all())
    check(out, s, budget)


@pytest.mark.parametrize("n", [81920, 262144])
def test_last_workgroup_of_every_problem_of_a_table(lava, n):
    """32 problems of one size: as many workgroups as make 12 keys per lane, regions back to back."""
    print(f"select bounds table n={n}", flush=True)
    data, probs = [], []
    for p in range(32):
        s, budget = crowded_end(n, 400 + 12 * p, n + p)
        sc, out = torch.from_numpy(s).cuda(), outputs(budget)
        data.append((s, sc, budget, out))
        probs.append(lava.select_problem(sc, budget, *out))
    need = lava.lava_select_batch_workspace_bytes(len(probs), n)
    buf = torch.full((need + 8192,), CANARY, dtype=torch.uint8, device="cuda")
    lava.lava_select_topk_batch(NH, probs, n, workspace=buf[:need])
    torch.cuda.synchronize()
    assert bool((buf[need:] == CANARY).all())
    assert lava.lava_select_batch_status(buf[:need], len(probs), n) == lava.LAVA_OK
    for s, _, budget, out in data:
        check(out, s, budget)


@pytest.mark.parametrize("short", [0, 1, 63, 2046, 2048])
def test_totals_up_to_31_bits(lava, short):
    """2^31 - 1 entries and a little fewer: the last wavefront's entries end at the last index there is, heads start in it,
    and its scores are ranked.  All scores are 0 but a few, so the survivors are known."""
    n = (1 << 31) - 1 - short
    if torch.cuda.mem_get_info()[0] < 4 * n + (1 << 30):
        pytest.skip("not enough free memory for 2^31 scores")
    print(f"select bounds n={n}", flush=True)
    buf = torch.zeros(n + 4096, device="cuda")
    buf[n:] = 9.0                                                    # nobody may rank these
    at = sorted({0, 5, n // 2, n - 2048, n - 1900, n - 1000, n - 700, n - 2, n - 1})
    buf[torch.tensor(at, device="cuda")] = torch.arange(1, len(at) + 1, device="cuda", dtype=torch.float32)
    starts = [0, n // 2 + 1, n - 1900, n - 1900, n - 1500, n - 700, n - 1, n, n]      # NH heads, two of them empty
    budget = len(at) + 3                                             # three zeros: the first ones in flat order
    flat = sorted(at + [1, 2, 3])
    head = [max(h for h in range(NH) if starts[h] <= p) for p in flat]
    out = outputs(budget)
    ws = torch.empty(lava.lava_select_workspace_bytes(n), dtype=torch.uint8, device="cuda")
    lava.lava_select_topk(NH, buf, budget, seg_offsets=torch.tensor(starts, device="cuda"), total_entries=n, head_counts=out[0],
                          head_offsets=out[1], kept_idx=out[2], kept_scores=out[3], workspace=ws)
    counts, offs, idx, kept = (x.cpu().numpy() for x in out)
    want = np.bincount(head, minlength=NH)
    assert counts.tolist() == want.tolist() and offs.tolist() == np.concatenate([[0], np.cumsum(want)]).tolist()
    assert idx.tolist() == [p - starts[h] for p, h in zip(flat, head)]
    assert kept.tolist() == [at.index(p) + 1.0 if p in at else 0.0 for p in flat]


def image(bits):
    """The order-preserving integer image of a float's bits."""
    return np.where(bits >> 31, ~bits, bits | 0x80000000).astype(np.uint32)


# one workgroup, several (2 and 12 keys per lane), the step launches
@pytest.mark.parametrize("n", [1001, 30001, 600001, 3_400_001])
def test_every_slot_is_written_whatever_the_bits(lava, n):
    """NaN is no valid score, but every slot that head_offsets counts holds an index all the same, also where the budget
    reaches the NaN with all bits set: survivors are ranked by the image of their bits, and kept_scores repeats them."""
    print(f"select bits n={n}", flush=True)
    r = np.random.Generator(np.random.PCG64(n))
    bits = r.standard_normal(n).astype(np.float32).view(np.uint32).copy()
    odd = r.choice(n, 40, replace=False)
    bits[odd] = np.array([0xffffffff, 0xffffffff, 0xffc00000, 0x7fc00000, 0x7fffffff, 0x7f800000, 0xff800000, 0x80000000], np.uint32)[np.arange(40) % 8]
    bits[n - 1] = 0xffffffff
    image_of = image(np.where(bits == 0x80000000, np.uint32(0), bits))
    order = np.argsort(-image_of.astype(np.int64), kind="stable")
    sc = torch.from_numpy(bits.view(np.int32)).cuda().view(torch.float32)
    for budget in (10, n - 11, n - 3, n):
        keep = np.sort(order[:budget])
        out = (torch.empty(1, dtype=torch.int32, device="cuda"), torch.empty(2, dtype=torch.int64, device="cuda"),
               torch.full((budget,), -7, dtype=torch.int32, device="cuda"), torch.empty(budget, device="cuda"))
        lava.lava_select_topk(1, sc, budget, head_counts=out[0], head_offsets=out[1], kept_idx=out[2], kept_scores=out[3])
        assert out[0].tolist() == [budget] and out[1].tolist() == [0, budget]
        assert np.array_equal(out[2].cpu().numpy(), keep)
        assert np.array_equal(out[3].view(torch.int32).cpu().numpy().view(np.uint32), bits[keep])
