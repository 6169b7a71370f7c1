"""Calls that must not cost more than others of the same data.  Each pair is
timed in turn on the same pools, and the least times are compared: the bounds
lie between what the call takes and what it took when it was at fault."""
import numpy as np
import pytest

from paper_2606_31093_amd import workloads as W
from paper_2606_31093_amd.workloads import BufSpec, PoolSpec

pytestmark = pytest.mark.gpu
TOKEN, HEAD = "LPCTHD", "PLCHTD"


@pytest.fixture
def kvx():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_31093_amd import kvx
    kvx.lib()
    return kvx


def least(*calls, rounds=9, reps=20):
    """Least time of each call, in us: the calls take turns."""
    import torch
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    best = [float("inf")] * len(calls)
    for k in range(rounds):
        for i, call in enumerate(calls):
            a.record()
            for _ in range(reps if k else 3):
                call()
            b.record()
            b.synchronize()
            if k:
                best[i] = min(best[i], a.elapsed_time(b) * 1e3 / reps)
    return best


class Pools:
    """Two pools and tables of `per` pages for each of n records."""

    def __init__(self, kvx, src, dst, n, per):
        self.kvx, self.src, self.dst = kvx, src, dst
        self.mem = [W.alloc_side(s, "cuda").zero_() for s in (src, dst)]
        rng = np.random.default_rng(n)
        self.tables = [rng.permutation(s.N)[:n * per].astype(np.int32) for s in (src, dst)]
        self.n, self.per = n, per

    def rows(self, tokens, src_start=0, dst_start=0):
        r = np.arange(self.n) * self.per
        one = np.ones(self.n, np.int64)
        return np.stack([r, r, 0 * r, one * src_start, one * dst_start, one * tokens], axis=1)

    def transfer(self, rows, pad=0):
        k = self.kvx
        pt = [k.device_table(np.concatenate([t, np.zeros(pad, np.int32)]), "cuda") for t in self.tables]
        reqs = k.device_reqs(rows, "cuda")
        return lambda: k.kvx_transfer(self.mem[0], self.src, self.mem[1], self.dst, pt[0], pt[1], reqs)


def check(got, bound, what):
    assert got <= bound, f"{what}: {got:.2f} of the other's time, bound {bound}"


@pytest.mark.parametrize("n,tokens", [(64, 3), (1, 200)])
@pytest.mark.parametrize("ls,ld", [(TOKEN, TOKEN), (HEAD, HEAD), (TOKEN, HEAD), (HEAD, TOKEN)])
def test_table_longer_than_the_records_need(kvx, ls, ld, n, tokens):
    """A padded table must not take a short call to a way made for long ones
    (at fault 1.25 to 1.9; 1.0 to 1.1)."""
    S, D = (PoolSpec(36, 2, 8, 128, T=64, N=256, e=2, layout=x) for x in (ls, ld))
    p = Pools(kvx, S, D, n, 4 if n == 1 else 1)
    rows = p.rows(tokens)
    padded, exact = least(p.transfer(rows, pad=64 * 64), p.transfer(rows))
    check(padded / exact, 1.22, f"{n} x {tokens} tokens {ls} -> {ld}, padded table")


def test_many_short_records(kvx):
    """16384 records of 2 tokens against 256 of 128 tokens, of a small model
    (at fault 30; 6)."""
    S = PoolSpec(2, 2, 2, 64, T=64, N=1024, e=2, layout=TOKEN)
    p = Pools(kvx, S, S, 256, 2)
    few = p.transfer(p.rows(128))
    r = np.arange(16384)
    many = np.stack([r // 32, r // 32, 0 * r, r % 32 * 2, r % 32 * 2, 0 * r + 2], axis=1)
    many, few = least(p.transfer(many), few)
    check(many / few, 14, "16384 short records")


@pytest.mark.parametrize("layout", [TOKEN, HEAD])
def test_few_pages_over_the_link(kvx, layout):
    """One page of 2 layers out to host memory and back, against 18 times the
    data (at fault 0.5; 0.08)."""
    def trip(L):
        S = PoolSpec(L, 2, 8, 128, T=64, N=8, e=2, layout=layout)
        B = BufSpec(L, 2, 8, 128, 2, cap=L * 2 * 64 * 8 * 128)
        p = Pools(kvx, S, S, 1, 1)
        buf = W.alloc_side(B, "cuda", pinned=True)
        reqs, pt = kvx.device_reqs(p.rows(64), "cuda"), kvx.device_table(p.tables[0], "cuda")

        def call():
            kvx.kvx_gather(p.mem[0], S, buf, B, pt, reqs)
            kvx.kvx_scatter(buf, B, p.mem[1], S, pt, reqs)
        return call
    few, many = least(trip(2), trip(36))
    check(few / many, 0.25, f"{layout}, one page of 2 layers")


@pytest.mark.parametrize("H,D,T", [(1, 576, 64), (5, 80, 48)])
def test_source_pages_that_begin_inside_pieces(kvx, H, D, T):
    """Long records from and to the middle of pages, whose source pages begin
    inside the destination's kilobytes, against the same between starts of
    pages (at fault 1.35 to 1.45; 1.0 to 1.1)."""
    S = PoolSpec(36, 2, H, D, T=T, N=512, e=2, layout=TOKEN)
    p = Pools(kvx, S, S, 8, 32)
    s, d = np.random.default_rng(4).integers(0, T, size=(2, 8))
    shift, zero = least(p.transfer(p.rows(31 * T, s, d)), p.transfer(p.rows(31 * T)))
    check(shift / zero, 1.25, f"{H} x {D}, shifted")


def test_units_in_turns_of_several_source_pages(kvx):
    """MLA pages of 128 tokens (144 KiB, which an XCD's wavefronts take in
    turns) from pages of 64 tokens, against the same from 128 (at fault 1.4;
    1.1)."""
    D = PoolSpec(36, 1, 1, 576, T=128, N=128, e=2, layout=TOKEN)
    S = PoolSpec(36, 1, 1, 576, T=64, N=256, e=2, layout=TOKEN)
    halves, whole = Pools(kvx, S, D, 8, 16), Pools(kvx, D, D, 8, 16)
    rows = halves.rows(15 * 128)
    rows[:, 0] = np.arange(8) * 32
    halves.tables[0] = np.random.default_rng(1).permutation(256).astype(np.int32)
    halves, whole = least(halves.transfer(rows), whole.transfer(whole.rows(15 * 128)))
    check(halves / whole, 1.2, "64 to 128 token pages of 1 x 576")


@pytest.mark.parametrize("ls,ld", [(TOKEN, TOKEN), (HEAD, TOKEN), (TOKEN, HEAD)])
def test_layered_sparse_pages(kvx, ls, ld):
    """Planned layered calls always sweep: of 256 KiB pages with 16 of 64
    tokens they must cost no more than unplanned ones (at fault 1.5 to 1.8;
    0.75 to 0.85)."""
    import torch
    S, D = (PoolSpec(36, 2, 8, 128, T=64, N=256, e=2, layout=x) for x in (ls, ld))
    p = Pools(kvx, S, D, 256, 1)
    rows = p.rows(16)
    spt, dpt = (kvx.device_table(t, "cuda") for t in p.tables)
    reqs, plan = kvx.device_reqs(rows, "cuda"), kvx.device_plan(rows, 64, 64, "cuda")
    events = [torch.cuda.Event() for _ in range(9)]

    def planned():
        kvx.kvx_transfer_layered_planned(p.mem[0], S, p.mem[1], D, spt, dpt, reqs, 4, events, *plan)

    def unplanned():
        kvx.kvx_transfer_layered(p.mem[0], S, p.mem[1], D, spt, dpt, reqs, 4, events)
    a, b = least(planned, unplanned)
    check(a / b, 1.1, f"{ls} -> {ld}, 16 of 64 tokens a page")


@pytest.mark.parametrize("ls,ld", [(HEAD, TOKEN), (TOKEN, HEAD), (HEAD, HEAD)])
def test_short_records_of_rows(kvx, ls, ld):
    """2048 records of 6 tokens whose rows are resolved, against the same
    records between token-major pools (at fault
    1.04 to 1.11; 0.89 to 0.95)."""
    def call(ls, ld):
        S, D = (PoolSpec(36, 2, 4, 128, T=64, N=256, e=2, layout=x) for x in (ls, ld))
        p = Pools(kvx, S, D, 256, 1)
        r = np.arange(2048)
        return p.transfer(np.stack([r // 8, r // 8, 0 * r, r % 8 * 8, r % 8 * 8, 0 * r + 6], axis=1))
    rows, runs = least(call(ls, ld), call(TOKEN, TOKEN))
    check(rows / runs, 1.0, f"{ls} -> {ld}, short records")


@pytest.mark.parametrize("H,D", [(8, 80), (5, 112), (8, 48)])
def test_rows_narrower_than_a_line(kvx, H, D):
    """Head-major rows that are no whole 128-byte lines, against 64-byte rows of
    the same data (at fault 1.5 to 1.8; 1.0)."""
    def call(H, D, L):
        S = PoolSpec(L, 2, H, D, T=64, N=288, e=1, layout=HEAD)
        p = Pools(kvx, S, S, 17, 16)
        return p.transfer(p.rows(1000)), L * H * D
    (narrow, n), (even, m) = call(H, D, 5120 // (H * D)), call(8, 64, 10)
    a, b = least(narrow, even)
    check(a / n / (b / m), 1.2, f"{H} x {D} bytes")
