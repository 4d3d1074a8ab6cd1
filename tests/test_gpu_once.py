"""The chained scan of arrays that the chip holds at once: one tile per workgroup, the tile size by the size of the array, a
last tile cut anywhere, and every sum of an earlier tile either waited for or added up again.  Whole numbers: exact."""
import numpy as np
import pytest
import torch

from paper_1811_09736_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tcr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1811_09736_amd import binding
    binding.set_variant("reset")
    binding.tuning_import("")
    yield binding
    binding.set_variant("reset")
    binding.set_workspace(None)
    binding.check_device_flags()


@pytest.fixture(params=["bounded", "none"])
def wait(request, tcr):
    tcr.set_variant("scan_wait", request.param)
    yield request.param
    tcr.set_variant("reset")


U1, U2, U4, U8 = (256 * 8192 * u for u in (1, 2, 4, 8))       # the most that tiles of 1, 2, 4 and 8 x 8192 elements cover


# one tile and less, two, a last tile of one element or one group or all but one, the first and last size of every tile
# size, and the first that is pipelined; sizes that are no multiple of 8 from 65536 elements on (below: another kernel)
@pytest.mark.parametrize("n", [8200, 16384, 32776, 65536, 65537, 65543, 8192 * 9 + 1, 8192 * 9 + 511, 8192 * 9 + 515, 8192 * 10 - 1, U1 - 1,
                               U1, U1 + 8, U1 + 9, U2 - 3, U2 + 5, U4, U4 + 1, U8 - 7, U8, U8 + 8, U8 + 13])
def test_full_scans(tcr, oracle, wait, n):
    if wait == "none" and n > U2 + 5:
        pytest.skip("every tile would add up a large array")
    x = workloads.make_input(n, "int4", n % 991)
    xd = torch.from_numpy(x).cuda()
    ref = oracle.scan(x)
    assert np.max(np.abs(ref)) < 2 ** 24
    assert np.array_equal(tcr.scan(xd).cpu().numpy().astype(np.float64), ref)
    out = torch.full((n + 8,), -3.0, dtype=torch.float32, device="cuda")
    tcr.scan_ex(xd, tcr.SCAN_EXCLUSIVE, out=out[:n])
    assert np.array_equal(out[:n].cpu().numpy().astype(np.float64), ref - x)
    assert torch.all(out[n:] == -3.0)                    # nothing behind the last element
    half = torch.full((n + 8,), -3.0, dtype=torch.float16, device="cuda")
    tcr.scan_ex(xd, tcr.OUT_F16, out=half[:n])
    assert np.array_equal(half[:n].cpu().numpy(), ref.astype(np.float16))
    assert torch.all(half[n:] == -3.0)


@pytest.mark.parametrize("nseg,seg", [(3, 32768), (70, 32768), (5, 65536), (2, 1 << 19), (255, 65544), (3, 65544), (41, 100000), (83, 100000),
                                      (167, 100000), (16, 1 << 20), (31, 524288 + 8)])
def test_segments(tcr, oracle, wait, nseg, seg):
    n = nseg * seg
    if wait == "none" and n > 1 << 23:
        pytest.skip("every tile would add up a large array")
    assert tcr.kernel_name(tcr.OP_SEGMENTED_SCAN, n, seg) == "scan_chain_kernel<mfma>"
    x = workloads.make_input(n, "int8", seg % 983)
    xd = torch.from_numpy(x).cuda()
    ref = oracle.segmented_scan(x, seg)
    assert np.array_equal(tcr.segmented_scan(xd, seg).cpu().numpy().astype(np.float64), ref)
    assert np.array_equal(tcr.segmented_scan_ex(xd, seg, tcr.SCAN_EXCLUSIVE).cpu().numpy().astype(np.float64), ref - x)


@pytest.mark.parametrize("seg,nseg", [(8192, 1), (8192, 3), (8192, 700), (16384, 3), (16384, 700)])
def test_segments_of_one_workgroup(tcr, oracle, seg, nseg):
    x = workloads.make_input(nseg * seg, "int8", nseg)
    got = tcr.segmented_scan(torch.from_numpy(x).cuda(), seg).cpu().numpy().astype(np.float64)
    assert np.array_equal(got, oracle.segmented_scan(x, seg))


@pytest.mark.parametrize("n,descriptors", [(1 << 20, 32), ((1 << 20) + 2, 33), (1 << 18, 32)])
def test_a_small_caller_workspace(tcr, oracle, n, descriptors):
    # a descriptor per 32768 elements (and one for what is left) has always been enough: the smaller tiles of an ordinary
    # call need more
    x = workloads.make_input(n, "int4", 7)
    xd = torch.from_numpy(x).cuda()
    buf = torch.full((256 + 2 * 256 * -(-descriptors * 8 // 256),), 0x5A, dtype=torch.uint8, device="cuda")
    try:
        tcr.set_workspace(buf)
        for _ in range(2):
            assert np.array_equal(tcr.scan(xd).cpu().numpy().astype(np.float64), oracle.scan(x))
    finally:
        torch.cuda.synchronize()
        tcr.set_workspace(None)


def test_recorded_and_between_other_chained_scans(tcr, oracle):
    # replays, eager calls of the same kernel, the pipelined chain and the look-back kernel take turns on one workspace
    sizes = [(1 << 17) + 3, 1 << 20, (1 << 24) + 4096]
    xs = [workloads.make_input(n, "int4", n % 89) for n in sizes]
    xd = [torch.from_numpy(x).cuda() for x in xs]
    want = [torch.from_numpy(oracle.scan(x).astype(np.float32)).cuda() for x in xs]
    outs = [torch.empty(n, dtype=torch.float32, device="cuda") for n in sizes]
    side = torch.cuda.Stream()

    def calls():
        for x, o in zip(xd, outs):
            tcr.scan(x, out=o)

    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        calls()
    side.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        calls()
    for _ in range(4):
        for o in outs:
            o.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for o, w in zip(outs, want):
            assert torch.equal(o, w)
        with torch.cuda.stream(side):
            again = [tcr.scan(x) for x in xd[:2]]
        side.synchronize()
        assert torch.equal(again[0], want[0]) and torch.equal(again[1], want[1])
    tcr.check_device_flags(side)
