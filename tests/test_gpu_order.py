"""Unplanned calls, bit for bit against the oracle: runs on both sides in order
(the test build copies every such call in order, the product library those of
long records), rows by teams of wavefronts (the test build all of them, the
product library those of much data), and the rest in parts.  The product library
decides on the device, from the records, which of them a call takes; tests named
for one choose sizes for which it does, and compare bytes and error bits."""
import numpy as np
import pytest

import cases
from paper_2606_31093_amd.workloads import BufSpec, PoolSpec, Step, Workload
from runner import assert_same, initial_bytes, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(params=["test", "product"])
def library(request, monkeypatch):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_31093_amd import build_lib, kvx
    kvx.lib()    # the product library first: raises if it is missing
    if request.param == "test":
        monkeypatch.setattr(kvx, "_LIB", kvx.load(build_lib.TEST_LIBRARY))
    return request.param


def check(wl):
    init = initial_bytes(wl)
    want, werr = run_oracle(wl, init)
    got, gerr = run_gpu(wl, init)
    assert gerr == werr, f"{wl.title}: device error bits {gerr}, oracle {werr}"
    assert_same(got, want, wl.title)


@pytest.mark.parametrize("Ts,Td", [(4, 4), (16, 64), (64, 16), (1, 16), (16, 1), (3, 5)])
@pytest.mark.parametrize("ls,ld", [("LPCTHD", "LPCTHD"), ("PLCTHD", "LPCTHD"), ("LPCTHD", "PLCTHD")])
def test_page_sizes(library, ls, ld, Ts, Td):
    check(cases.transfer_case(ls, ld, Ts, Td, seed=Ts * 100 + Td, D=64))


@pytest.mark.parametrize("seed", range(60))
def test_random(library, seed):
    """Random transfers (damaged tables, slices, shared pages), copies inside
    a pool, layered transfers, and gathers and scatters with bad blocks."""
    check((cases.random_case, cases.random_cow_case, cases.random_layered_case,
           cases.random_gs_case)[seed % 4](seed))


@pytest.mark.parametrize("T,H,D,L,n", [(160, 8, 128, 2, 333),    # 640 pieces: more than an XCD's wavefronts
                                       (150, 4, 128, 3, 700),    # 300: no divisor of them
                                       (64, 8, 128, 5, 260),     # 256
                                       (64, 1, 576, 7, 500)])    # one kv component, 72
@pytest.mark.parametrize("shift", [0, 7])
def test_large_pages(library, T, H, D, L, n, shift):
    """Pages of as many pieces as a team has wavefronts, and more; with a
    shift, pieces that lie in two source pages."""
    C = 1 if D == 576 else 2
    spec = [(shift, 0, n, None), (3, 3, 2 * T, None), (T - 1, 0, 1, None)]
    check(cases.transfer_case("LPCTHD", "PLCTHD", T, T, seed=T + shift, D=D, L=L, C=C, H=H, spec=spec))


@pytest.mark.parametrize("Ts,Td", [(48, 48), (64, 64), (32, 64)])
@pytest.mark.parametrize("H,D", [(5, 80), (8, 128), (3, 56)])
def test_source_pages_that_begin_inside_pieces(library, Ts, Td, H, D):
    """1 KiB pieces hold 1.28 tokens, a quarter or 3.05 of them: long records whose
    source pages begin between and inside pieces (the product library's judge
    tells them apart), and a page id that is bad."""
    spec = [(0, 0, 700, None), (37, 5, 500, None), (8, 24, 611, None), (Ts - 1, Td - 1, 300, None)]
    wl = cases.transfer_case("LPCTHD", "LPCTHD", Ts, Td, seed=Ts + H, D=D, L=16, H=H, spec=spec)
    check(wl)
    wl.steps[0].src_pt[9] = -1
    check(wl)


@pytest.mark.parametrize("Ts,Td", [(64, 128), (128, 128), (256, 128), (128, 96)])
def test_units_in_turns(library, Ts, Td):
    """Pages of 144 and 108 pieces, the first taken in turns: the product
    library keeps their order where each lies in one source page."""
    spec = [(0, 0, 900, None), (0, 0, 1000, None), (128 % Ts, 0, 800, None)]
    wl = cases.transfer_case("LPCTHD", "LPCTHD", Ts, Td, seed=Ts + Td, D=576, L=32, C=1, H=1, spec=spec)
    check(wl)
    wl.steps[0].src_pt[1] = -1
    check(wl)


@pytest.mark.parametrize("n_reqs", [63, 64, 65, 1023, 1024, 1025, 2100])
def test_many_records(library, n_reqs):
    """Around the 64 records of a wavefront and the 1024 of a workgroup, every
    fifth of them empty."""
    spec = [(i % 3, (i * 5) % 4, 0 if i % 5 == 4 else 1 + i % 7, None) for i in range(n_reqs)]
    check(cases.transfer_case("LPCTHD", "LPCTHD", 4, 4, seed=n_reqs, D=8, L=3, H=1, spec=spec))


@pytest.mark.parametrize("n_reqs", [64, 65, 511, 512, 513, 1100])
@pytest.mark.parametrize("ls,ld", [("LPCTHD", "PLCHTD"), ("PLCHTD", "LPCTHD"), ("LPCHTD", "PLCHTD")])
def test_many_records_of_rows(library, ls, ld, n_reqs):
    """The same around the records that a workgroup shares its look at: every
    seventh record is empty, some begin in the middle of a page or span two."""
    spec = [(i % 3, (i * 5) % 4, 0 if i % 7 == 4 else 1 + i % 6, None) for i in range(n_reqs)]
    check(cases.transfer_case(ls, ld, 4, 4, seed=n_reqs, D=8, L=3, H=3, spec=spec))


@pytest.mark.parametrize("layout", ["LPCTHD", "PLCHTD"])
@pytest.mark.parametrize("n_reqs,pinned", [(65, False), (600, False), (600, True)])
def test_many_records_through_a_buffer(library, layout, n_reqs, pinned):
    """Gathered and scattered; the last record's block does not fit the buffer."""
    rng = np.random.default_rng(n_reqs)
    n = rng.integers(0, 9, size=n_reqs)
    S = PoolSpec(2, 2, 2, 8, T=4, N=2 * n_reqs + 8, e=2, layout=layout)
    block = 2 * 2 * n * 2 * 8
    off = np.concatenate([[0], np.cumsum(block)[:-1]])
    n[-1] = 9
    buf = BufSpec(2, 2, 2, 8, 2, cap=int(block.sum()))
    r = np.arange(n_reqs)
    start = rng.integers(0, 4, size=n_reqs) * (n < 5)
    src, dst = (rng.permutation(S.N)[:3 * n_reqs].astype(np.int32) for _ in range(2))
    src[5], dst[9] = S.N, -1
    gather = np.stack([2 * r, 0 * r, off, start, 0 * r, np.minimum(n, 8 - start)], axis=1)
    scatter = np.stack([0 * r, 2 * r, off, 0 * r, start, np.minimum(n, 8 - start)], axis=1)
    gather[-1, 5] = scatter[-1, 5] = 9
    check(Workload("case", "many records through a buffer", {"A": S, "buf": buf, "B": S},
                   [Step("gather", "A", "buf", src, None, gather), Step("scatter", "buf", "B", None, dst, scatter)],
                   host_sides=("buf",) if pinned else (), value_seed=9, prefill_tag=4))


@pytest.mark.parametrize("Ts,Td", [(16, 64), (64, 16), (3, 7), (1, 130)])   # 130: more source pages than lanes
@pytest.mark.parametrize("H,D,L", [(3, 8, 2), (8, 128, 3), (5, 80, 2)])
@pytest.mark.parametrize("ls,ld", [("LPCTHD", "LPCHTD"), ("PLCHTD", "LPCTHD"), ("LPCHTD", "PLCHTD")])
def test_rows(library, ls, ld, H, D, L, Ts, Td):
    """Head-major sides: odd first slots (half a slot block masked), one token,
    an empty record, pages left and entered in the middle."""
    spec = [(1, 3, 1, None), (0, 0, 0, None), (Ts - 1, Td - 1, 2 * Td + 3, None), (0, 1, Ts, None), (2, 0, 3 * Ts + 1, None)]
    check(cases.transfer_case(ls, ld, Ts, Td, seed=Ts + 3 * Td + H, D=D, L=L, H=H, spec=spec))


@pytest.mark.parametrize("Ts,Td", [(16, 64), (64, 13), (7, 7)])
@pytest.mark.parametrize("H,D", [(3, 16), (2, 32), (8, 48), (1, 64), (5, 80), (4, 96), (3, 112)])
@pytest.mark.parametrize("ls,ld", [("LPCTHD", "LPCHTD"), ("PLCHTD", "LPCHTD")])
def test_narrow_rows(library, ls, ld, H, D, Ts, Td):
    """Rows narrower than a 128-byte line, which a head-major destination takes in
    blocks of 2 to 8 slots: blocks masked at both ends, pages that end inside one."""
    spec = [(1, 3, 1, None), (0, 0, 0, None), (Ts - 1, Td - 1, 2 * Td + 3, None), (0, 1, Ts, None), (2, 5, 3 * Ts + 9, None)]
    check(cases.transfer_case(ls, ld, Ts, Td, seed=Ts + 3 * Td + H, e=1, D=D, L=3, H=H, spec=spec))


@pytest.mark.parametrize("pinned", [False, True])
@pytest.mark.parametrize("layout", ["LPCHTD", "PLCHTD"])
def test_rows_through_a_buffer(library, layout, pinned):
    check(cases.gather_scatter_case(layout, 24, 2, 80, seed=31, H=5, pinned=pinned))


@pytest.mark.parametrize("ls,ld,Ts,Td", [("PLCHTD", "LPCTHD", 64, 16), ("PLCHTD", "LPCHTD", 64, 64), ("LPCTHD", "PLCHTD", 16, 64)])
@pytest.mark.parametrize("n_reqs", [1, 12, 80])
def test_product_library_copies_much_data_of_rows_by_teams(ls, ld, Ts, Td, n_reqs):
    """4000 tokens over 16 layers, 262 MB, in 1, 12 or 80 records (many or few
    table entries for each), above the size from which the product library's
    wavefronts share parts; odd starts, and a bad id on each side."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n = 4000 // n_reqs
    per_s, per_d = -(-(n + 5) // Ts), -(-(n + 3) // Td)
    S = PoolSpec(16, 2, 8, 128, T=Ts, N=per_s * n_reqs + 6, e=2, layout=ls)
    D = PoolSpec(16, 2, 8, 128, T=Td, N=per_d * n_reqs + 6, e=2, layout=ld)
    rng = np.random.default_rng(6)
    src = rng.permutation(S.N)[:per_s * n_reqs].astype(np.int32)
    dst = rng.permutation(D.N)[:per_d * n_reqs].astype(np.int32)
    dst[7] = D.N
    src[11] = -1
    r = np.arange(n_reqs)
    rows = np.stack([r * per_s, r * per_d, 0 * r, 0 * r + 5, 0 * r + 3, 0 * r + n], axis=1)
    check(Workload("case", "much data of rows", {"A": S, "B": D}, [Step("transfer", "A", "B", src, dst, rows)],
                   value_seed=8, prefill_tag=3))


@pytest.mark.parametrize("T,pinned", [(16, False), (64, False), (64, True)])
def test_gather_and_scatter(library, T, pinned):
    """Through a flat buffer, in device memory (long records, in order) and in
    pinned host memory (in parts)."""
    check(cases.gather_scatter_case("LPCTHD", T, 2, 128, seed=T, H=8, pinned=pinned))


def test_product_library_keeps_the_order_of_long_records():
    """One record of 20 pages of 256 KiB over 16 layers: 84 MB, above the size
    from which the product library copies in order; its table's first entry
    is out of range and one page id is bad."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    S = PoolSpec(16, 2, 8, 128, T=64, N=24, e=2, layout="LPCTHD")
    rng = np.random.default_rng(5)
    src, dst = rng.permutation(24)[:21].astype(np.int32), rng.permutation(24)[:21].astype(np.int32)
    dst[7] = 24
    src[11] = -1
    rows = np.asarray([[0, -1, 0, 5, 5, 20 * 64]], np.int64)
    wl = Workload("case", "long record", {"A": S, "B": S}, [Step("transfer", "A", "B", src, dst, rows)],
                  value_seed=8, prefill_tag=3)
    check(wl)
    block = 16 * 2 * 1280 * 8 * 128
    buf = BufSpec(16, 2, 8, 128, 2, cap=block)
    rows = np.asarray([[0, 0, 0, 0, 0, 1280]], np.int64)
    good = rng.permutation(24)[:20].astype(np.int32)
    wl = Workload("case", "long block", {"A": S, "buf": buf, "B": S},
                  [Step("gather", "A", "buf", good, None, rows), Step("scatter", "buf", "B", None, good[::-1].copy(), rows)],
                  value_seed=9, prefill_tag=4)
    check(wl)
