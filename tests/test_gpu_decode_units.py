"""Units of the decode step: heads of one unit and of many, packed and appended rows in one unit, partials exchanged through a
workspace of any contents, and the launch replayed from a graph on changing head sizes."""
import numpy as np
import pytest

from paper_2509_09754_amd import synth
from test_gpu_decode import compare, run_oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def lava():
    from paper_2509_09754_amd import lava as L
    yield L
    L.set_tuning()


class Call:
    """A decode call with its buffers; canaries behind a workspace filled with `fill`."""

    def __init__(self, lava, di, H, Hkv, d, fill=0xFF):
        self.lava, self.di, self.batch = lava, di, di.q.shape[0]
        self.desc = lava.LayerDesc.make(H, Hkv, d, 1, di.dtype)
        dev = "cuda"
        self.q, self.k, self.v, self.kt, self.vt = (lava.to_device(x, di.dtype, dev) for x in (di.q, di.k_hat, di.v_hat, di.k_tail, di.v_tail))
        self.offs = torch.from_numpy(di.head_offsets).to(dev)
        self.out = torch.full((self.batch, H, d), 777.0, device=dev)
        self.lse = torch.full((self.batch, H), 777.0, device=dev)
        self.need = lava.lava_decode_workspace_bytes(self.desc, self.batch, di.rows_capacity, di.tail_len)
        self.ws = torch.full((self.need + 4096,), fill, dtype=torch.uint8, device=dev)
        self.ws[self.need:] = 0x5A

    def run(self):
        tail = self.di.tail_len
        self.lava.lava_decode_attention(self.desc, self.batch, self.q, self.k, self.v, self.offs, self.di.rows_capacity,
                                        k_tail=self.kt if tail else None, v_tail=self.vt if tail else None, tail_len=tail,
                                        tail_capacity=self.di.k_tail.shape[2], out=self.out, lse=self.lse, workspace=self.ws[: self.need])

    def check(self, di):
        torch.cuda.synchronize()
        compare(self.out.cpu().numpy(), self.lse.cpu().numpy(), *run_oracle(di))
        assert bool((self.ws[self.need:] == 0x5A).all())


# one unit per head, a few, more than a wavefront reads flags at once (64) and than one merge takes (32); appended rows
# in the last packed unit, in units of their own, alone
@pytest.mark.parametrize("H,Hkv,d,dtype,rows,tail,unit", [
    (8, 2, 128, "bf16", [200, 3], 0, 2048), (8, 2, 128, "bf16", [5000], 7, 128), (4, 1, 128, "bf16", [9000], 0, 128),
    (4, 1, 64, "f32", [4300], 300, 128), (8, 1, 128, "bf16", [127, 128, 129], 1, 128), (16, 2, 64, "bf16", [0, 40], 129, 128),
    (2, 2, 128, "f32", [33, 0], 31, 128), (6, 2, 128, "bf16", [2048], 200, 256)])
def test_units(lava, H, Hkv, d, dtype, rows, tail, unit):
    print(f"decode units H{H}/{Hkv} d{d} {dtype} rows {rows} tail {tail} unit {unit}", flush=True)
    lava.set_tuning(decode_rows_per_unit=unit)
    di = synth.gen_decode(H, Hkv, d, dtype, rows, 2, tail_len=tail, tail_capacity=tail + 2 if tail else 0)
    for fill in (0xFF, 0x00):
        c = Call(lava, di, H, Hkv, d, fill)
        c.run()
        c.check(di)
        first = c.out.clone()
        for _ in range(3):                                     # the workspace as the call before left it
            c.run()
        torch.cuda.synchronize()
        assert torch.equal(first.view(torch.int32), c.out.view(torch.int32))
    lava.set_tuning()


def test_replays_on_changing_heads(lava):
    """A captured step leaves no flag behind that a replay could take for its own, whatever units it has."""
    print("decode units: graph replays on changing heads", flush=True)
    H, Hkv, d, cap = 8, 2, 128, 4000
    dis = [synth.gen_decode(H, Hkv, d, "bf16", [r, 4000 - r], 20 + i, rows_capacity=cap, tail_len=5) for i, r in enumerate((3900, 17, 1300, 2600))]
    lava.set_tuning(decode_rows_per_unit=128)
    c = Call(lava, dis[0], H, Hkv, d)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        c.run()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        c.run()
    lava.set_tuning()
    for di in dis + dis:
        for dst, src in ((c.q, di.q), (c.k, di.k_hat), (c.v, di.v_hat), (c.kt, di.k_tail), (c.vt, di.v_tail)):
            dst.copy_(lava.to_device(src, "bf16"))
        c.offs.copy_(torch.from_numpy(di.head_offsets))
        c.out.fill_(777.0)
        graph.replay()
        c.check(di)
        c.run()                                                # an ordinary call in between, on the same workspace
        c.check(di)


# numbers of sequences that are turned by one a unit, after two or four units, and not at all; one round of 512 workgroups (in
# turn) and two that are not full (one after the other)
@pytest.mark.parametrize("units", [510, 760])
@pytest.mark.parametrize("batch", [2, 3, 4, 6, 8, 9, 16, 33])
def test_sequences_take_turns(lava, batch, units):
    """Sequences of very different length, some with nothing, one of them alone with many units: every unit of every sequence is
    done by one workgroup, whatever the batch."""
    print(f"decode units: {batch} sequences in turn, {units} units", flush=True)
    H, Hkv, d = 8, 2, 64
    # capacity / 128 + 1 (two appended tiles a head) + 1 (half a unit a head) units a sequence are expected
    cap = (units // batch - 2) * 128
    rows = [min((0, 1, 130, 700, 40)[i % 5], cap) for i in range(batch)]
    rows[batch // 2] = cap - 40
    lava.set_tuning(decode_rows_per_unit=128)
    di = synth.gen_decode(H, Hkv, d, "bf16", rows, 4, rows_capacity=cap, tail_len=33, tail_capacity=40)
    c = Call(lava, di, H, Hkv, d)
    for _ in range(2):
        c.run()
        c.check(di)
    lava.set_tuning()


@pytest.mark.parametrize("dtype,d,Hkv,batch,rows", [("bf16", 128, 8, 12, 32768), ("f32", 64, 2, 48, 8192), ("f32", 128, 8, 8, 8192),
                                                    ("bf16", 128, 1, 1, 32768)])
def test_cut_is_no_slower_than_others(lava, dtype, d, Hkv, batch, rows):
    """The library's own cut into units against forced ones, kernel time.  A cut that just misses a round of workgroups, a
    round spread unevenly, or a merge of too many units costs 20 to 70 % (52 us against 41, 59 against 46, 35 against 27,
    39 against 23)."""
    print(f"decode cut {dtype} d{d} {batch} x {rows} on {Hkv}", flush=True)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    gen = torch.Generator(device="cuda").manual_seed(1)
    q, k, v = (torch.randn(*n, d, device="cuda", generator=gen).to(dt) for n in ((batch, 4 * Hkv), (batch * rows,), (batch * rows,)))
    share = 0.5 + torch.rand(batch, Hkv, device="cuda", generator=gen, dtype=torch.float64)
    offs = torch.zeros(batch, Hkv + 1, dtype=torch.int64, device="cuda")
    offs[:, 1:] = (share.cumsum(1) / share.sum(1, keepdim=True) * rows).round().long()
    desc = lava.LayerDesc.make(4 * Hkv, Hkv, d, 1, dtype)
    best = {}
    try:
        for unit in (0, 384, 512, 1024):
            lava.set_tuning(**({"decode_rows_per_unit": unit} if unit else {}))
            ws = torch.empty(lava.lava_decode_workspace_bytes(desc, batch, rows, 0), dtype=torch.uint8, device="cuda")
            out = torch.empty(batch, 4 * Hkv, d, device="cuda")
            lava.prof_enable(True)
            for _ in range(12):
                lava.prof_reset()
                lava.lava_decode_attention(desc, batch, q, k, v, offs, rows, out=out, workspace=ws)
                torch.cuda.synchronize()
                best[unit] = min(best.get(unit, 1e9), lava.prof_read()["decode"][0])
            lava.prof_enable(False)
    finally:
        lava.prof_enable(False), lava.prof_reset(), lava.set_tuning()
    print(best, flush=True)
    assert best[0] < 1.15 * min(best.values())
