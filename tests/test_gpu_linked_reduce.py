"""Irregular reductions in one launch: the part of a tile's first result that lies in front of the tile, added up by the tile's
own wavefronts (up to 512 elements each) or out of the sums that the tiles in front publish (64 or 512 of them per step), or
again from the elements where those are not waited for.  Whole numbers: exact."""
import numpy as np
import pytest
import torch

from paper_1811_09736_amd import workloads

pytestmark = pytest.mark.gpu

TILE = 8192


@pytest.fixture(scope="module")
def tcr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1811_09736_amd import binding
    binding.set_variant("reset")
    binding.tuning_import("")
    yield binding
    binding.set_variant("reset")
    binding.check_device_flags()


def check(tcr, oracle, x, xd, off):
    off = np.asarray(off, dtype=np.int64)
    od = torch.from_numpy(off).cuda()
    a, q = tcr.irregular_moments(xd, od)
    wa, wq = oracle.irregular_moments(x, off)
    assert np.max(wq) < 2 ** 24
    assert np.array_equal(tcr.irregular_reduce(xd, od).cpu().numpy().astype(np.float64), wa)
    assert np.array_equal(a.cpu().numpy().astype(np.float64), wa) and np.array_equal(q.cpu().numpy().astype(np.float64), wq)


# elements in front of a tile: the share of one wavefront, of four and of eight (wide tiles up to 1024), whole tiles
@pytest.mark.parametrize("tiles", [3, 1025])
@pytest.mark.parametrize("back", [1, 7, 8, 511, 512, 513, 2047, 2048, 2049, 4095, 4096, 4097, TILE - 1, TILE, TILE + 1])
def test_parts_of_every_length(tcr, oracle, tiles, back):
    n = tiles * TILE
    base = workloads.make_input(n + 8, "int1", back)
    bd = torch.from_numpy(base).cuda()
    edges = [TILE, 2 * TILE] if tiles == 3 else [TILE, 700 * TILE, 1024 * TILE]
    for shift in (0, 3):
        x, xd = base[shift:shift + n].copy(), bd[shift:shift + n]
        off = [0]
        for e in edges:                                           # a segment that begins `back` elements in front of the edge
            off += sorted({max(e - shift - back, off[-1]), e - shift + 5})
        check(tcr, oracle, x, xd, off + [n])


# tiles between a segment's start and its end: one step of 64, of 512, and more
@pytest.mark.parametrize("wait", ["bounded", "none"])
@pytest.mark.parametrize("span", [1, 2, 63, 64, 65, 511, 512, 513, 1100, 2050])
def test_published_sums(tcr, oracle, wait, span):
    n = (span + 3) * TILE - 1
    x = workloads.make_input(n, "int1", span)
    xd = torch.from_numpy(x).cuda()
    tcr.set_variant("scan_wait", wait)
    try:
        for first in (TILE - 1, TILE, TILE + 1):
            check(tcr, oracle, x, xd, [0, first, first + span * TILE, n])
        check(tcr, oracle, x, xd, [0, n])
        check(tcr, oracle, x, xd, workloads.make_offsets(n, "few4", 3).view(np.int64))
    finally:
        tcr.set_variant("reset")


@pytest.mark.parametrize("wait", ["bounded", "none"])
@pytest.mark.parametrize("seg_len,nseg", [(16, 5000), (513, 400), (4096, 33), (8192, 9), (65536, 40), (1 << 20, 5), (3 * TILE + 8, 11)])
def test_regular_segments_of_unaligned_arrays(tcr, oracle, wait, seg_len, nseg):
    n = seg_len * nseg
    base = workloads.make_input(n + 8, "int1", seg_len)
    bd = torch.from_numpy(base).cuda()
    tcr.set_variant("scan_wait", wait)
    try:
        for shift in (1, 7):
            x, xd = base[shift:shift + n].copy(), bd[shift:shift + n]
            off = np.arange(nseg + 1, dtype=np.int64) * seg_len
            wa, wq = oracle.irregular_moments(x, off)
            a, q = tcr.segmented_moments(xd, seg_len)
            assert np.array_equal(tcr.segmented_reduce(xd, seg_len).cpu().numpy().astype(np.float64), wa)
            assert np.array_equal(a.cpu().numpy().astype(np.float64), wa) and np.array_equal(q.cpu().numpy().astype(np.float64), wq)
            assert float(tcr.reduce(xd).cpu()[0]) == float(np.sum(wa))
    finally:
        tcr.set_variant("reset")


def test_recorded_on_a_stream_whose_epochs_the_device_keeps(tcr, oracle):
    # a recorded chained scan leaves the stream's epochs to the device; linked reductions then run recorded and eagerly
    n = 70 * TILE + 11
    inputs = [workloads.make_input(n, "int1", (9, k)) for k in range(2)]
    off = workloads.make_offsets(n, "few4", 2).view(np.int64)
    od = torch.from_numpy(off).cuda()
    x = torch.from_numpy(inputs[0]).cuda()
    out = torch.empty(off.size - 1, dtype=torch.float32, device="cuda")
    scanned = torch.empty(n, dtype=torch.float32, device="cuda")
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        tcr.irregular_reduce(x, od, out=out)
        tcr.scan(x, out=scanned)
    side.synchronize()
    for _ in range(2):                                            # the second recording finds them on the device
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            tcr.irregular_reduce(x, od, out=out)
            tcr.scan(x, out=scanned)
            tcr.irregular_reduce(x, od, out=out)
        for k in (1, 0, 1):
            x.copy_(torch.from_numpy(inputs[k]).cuda())
            out.fill_(float("nan"))
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            want = oracle.irregular_reduce(inputs[k], off)
            assert np.array_equal(out.cpu().numpy().astype(np.float64), want)
            assert np.array_equal(scanned.cpu().numpy().astype(np.float64), oracle.scan(inputs[k]))
            with torch.cuda.stream(side):
                again = tcr.irregular_reduce(x, od)
            side.synchronize()
            assert torch.equal(again, out)
