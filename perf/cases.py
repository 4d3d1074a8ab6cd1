"""What a user of this library has it do, as cases that can be timed and compared: one pass of each public entry
point over the sizes, segment lengths, data types and options that it is called with.

A case is a dict of plain values:

  op      the entry point: "reduce", "scan" (one segment), "segmented_reduce", "segmented_scan", "segmented_moments",
          "irregular_reduce", "irregular_scan", "irregular_moments"
  n       elements of the input (a multiple of seg_len for the segmented calls)
  seg_len elements per segment (the segmented calls)
  segs    the mix of segment lengths (the irregular calls): "uniform16" lengths spread evenly from nothing to twice 16,
          "lognormal256" a heavy tail (median 256, sigma 2: most segments short, most elements in long ones), "few7"
          seven long segments
  flags   scans: 0, or a combination of the library's SCAN_EXCLUSIVE and OUT_F16
  dist    values: "uniform_01", "uniform_pm1", "normal" or "int4" (whole numbers from -4 to 4)
"""
import torch

from paper_1811_09736_amd import binding


def listed():
    return [
        # a running sum over one short, odd-sized array: the smallest call, all launches and latency
        {"name": "scan_64k_ragged", "op": "scan", "n": 65541, "flags": 0, "dist": "uniform_01"},
        # sums of the rows of one small batch (configuration 1)
        {"name": "segreduce_1m_256", "op": "segmented_reduce", "n": 1 << 20, "seg_len": 256, "dist": "uniform_pm1"},
        # running sums along the rows of an ordinary matrix (configuration 2)
        {"name": "segscan_16m_1024", "op": "segmented_scan", "n": 1 << 24, "seg_len": 1024, "flags": 0, "dist": "uniform_pm1"},
        # the sum of one large array (configuration 3)
        {"name": "reduce_256m", "op": "reduce", "n": 1 << 28, "dist": "uniform_01"},
        # the running sum of one large array (configuration 4): the largest call
        {"name": "scan_256m", "op": "scan", "n": 1 << 28, "flags": 0, "dist": "int4"},
        # the shortest segments of the segment-size sweep (configuration 5)
        {"name": "segreduce_256m_16", "op": "segmented_reduce", "n": 1 << 28, "seg_len": 16, "dist": "uniform_01"},
        # a few hundred long rows, as many as there are compute units: the sweep's long segments at an ordinary size
        {"name": "segreduce_16m_64k", "op": "segmented_reduce", "n": 1 << 24, "seg_len": 1 << 16, "dist": "uniform_01"},
        # exclusive running sums kept in binary16, the output precision of the paper
        {"name": "segscan_f16_64m_4096", "op": "segmented_scan", "n": 1 << 26, "seg_len": 4096,
         "flags": binding.SCAN_EXCLUSIVE | binding.OUT_F16, "dist": "uniform_01"},
        # the statistics of a normalisation layer: 32 images of 256 channels of 28 x 28 values
        {"name": "moments_784", "op": "segmented_moments", "n": 784 * 32 * 256, "seg_len": 784, "dist": "normal"},
        # running sums along rows of an odd length
        {"name": "segscan_odd_1001", "op": "segmented_scan", "n": 1001 * 16384, "seg_len": 1001, "flags": 0, "dist": "uniform_01"},
        # sums over many short lists of different lengths (the neighbours of a graph's nodes, the words of a document)
        {"name": "irregular_reduce_64m", "op": "irregular_reduce", "n": 1 << 26, "segs": "uniform16", "dist": "uniform_01"},
        # running sums over a batch of sequences with a heavy tail of lengths
        {"name": "irregular_scan_16m", "op": "irregular_scan", "n": 1 << 24, "segs": "lognormal256", "flags": 0, "dist": "uniform_01"},
    ]


# The ranges that the listed cases stand for.
_OPS = ("reduce", "scan", "segmented_reduce", "segmented_reduce", "segmented_scan", "segmented_scan", "segmented_moments",
        "irregular_reduce", "irregular_scan", "irregular_moments")
_LOG2_N = (16.0, 27.0)          # elements
_LOG2_SEG = (2.0, 20.0)         # elements per segment


def draw(rng):
    case = {"op": rng.choice(_OPS), "n": int(2.0 ** rng.uniform(*_LOG2_N))}
    if rng.random() < 0.4:
        case["n"] -= case["n"] % 8          # an array whose size somebody chose
    if case["op"].startswith("segmented"):
        length = 2.0 ** rng.uniform(*_LOG2_SEG)
        while length > case["n"]:
            length /= 2.0
        case["seg_len"] = 1 << (int(length).bit_length() - 1) if rng.random() < 0.4 else int(length)
        case["n"] -= case["n"] % case["seg_len"]
    if case["op"].startswith("irregular"):
        case["segs"] = rng.choice(("uniform16", "lognormal256", "few7"))
    if "scan" in case["op"]:
        # (binary16 holds sums up to 65504: not for long segments of positive values)
        case["flags"] = rng.choice((0, 0, binding.SCAN_EXCLUSIVE))
        if case.get("seg_len", 1 << 30) <= 8192 and rng.random() < 0.25:
            case["flags"] |= binding.OUT_F16
    # (a single sum of values around zero may come out near zero, where it has no relative error to speak of)
    case["dist"] = rng.choice(("uniform_01", "uniform_pm1", "int4") if "scan" in case["op"] else ("uniform_01", "uniform_01", "int4"))
    return case


def _values(n, dist, gen):
    dev = gen.device
    if dist == "normal":
        return torch.randn(n, generator=gen, device=dev, dtype=torch.float16)
    if dist == "int4":
        return torch.randint(-4, 5, (n,), generator=gen, device=dev, dtype=torch.int8).to(torch.float16)
    x = torch.rand(n, generator=gen, device=dev, dtype=torch.float32)
    return (x if dist == "uniform_01" else 2.0 * x - 1.0).to(torch.float16)


def _segments(case):
    n = case["n"]
    return {"uniform16": max(1, n // 16), "lognormal256": max(1, n // 1892), "few7": 7}[case["segs"]]


def _offsets(case, gen):
    """nseg + 1 offsets from 0 to n: lengths drawn from the mix and scaled together so that they cover the array."""
    n, nseg = case["n"], _segments(case)
    u = torch.rand(nseg, generator=gen, device=gen.device, dtype=torch.float64)
    if case["segs"] == "lognormal256":
        u = torch.exp(2.0 * torch.randn(nseg, generator=gen, device=gen.device, dtype=torch.float64))
    ends = torch.cumsum(u, 0)
    ends = torch.floor(ends * (n / ends[-1])).to(torch.int64).clamp_(0, n)
    ends[-1] = n
    return torch.cat([ends.new_zeros(1), ends])


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    state = dict(case, x=_values(case["n"], case["dist"], gen))
    if "segs" in case:
        state["offsets"] = _offsets(case, gen)
    return state


def run(state):
    op, x, flags = state["op"], state["x"], state.get("flags", 0)
    if op == "reduce":
        return binding.reduce(x)
    if op == "scan":
        return binding.scan_ex(x, flags) if flags else binding.scan(x)
    if op == "segmented_reduce":
        return binding.segmented_reduce(x, state["seg_len"])
    if op == "segmented_scan":
        return binding.segmented_scan_ex(x, state["seg_len"], flags) if flags else binding.segmented_scan(x, state["seg_len"])
    if op == "segmented_moments":
        return binding.segmented_moments(x, state["seg_len"])
    if op == "irregular_reduce":
        return binding.irregular_reduce(x, state["offsets"])
    if op == "irregular_scan":
        return binding.irregular_scan_ex(x, state["offsets"], flags) if flags else binding.irregular_scan(x, state["offsets"])
    return binding.irregular_moments(x, state["offsets"])


def work(case):
    """The input read once and every result written once; an addition per element (and a product, for the squares)."""
    n, op = case["n"], case["op"]
    nseg = _segments(case) if "segs" in case else n // case.get("seg_len", n)
    read = 2 * n + (8 * (nseg + 1) if "segs" in case else 0)
    if "scan" in op:
        written = n * (2 if case["flags"] & binding.OUT_F16 else 4)
    else:
        written = 4 * nseg * (2 if "moments" in op else 1)
    return {"bytes": read + written, "flops": n * (3 if "moments" in op else 1)}


def tolerance(case):
    if case.get("flags", 0) & binding.OUT_F16:
        return {"rel": 1e-3, "max": 2e-3}         # results rounded to 11 bits
    return {"rel": 1e-6, "max": 1e-5}             # binary32 sums in some order: up to 2e-7 off the 64-bit ones, measured


def exact(case, seed):
    state = prepare(case, seed)
    x = state["x"].double()
    op, excl = case["op"], bool(case.get("flags", 0) & binding.SCAN_EXCLUSIVE)
    if "segs" not in case:
        rows = x.view(-1, case.get("seg_len", case["n"]))
        if "scan" in op:
            sums = torch.cumsum(rows, 1)
            return ((sums - rows) if excl else sums).view(-1)
        return (rows.sum(1), (rows * rows).sum(1)) if "moments" in op else rows.sum(1)
    offsets = state["offsets"]

    def in_front(v):
        return torch.cat([v.new_zeros(1), torch.cumsum(v, 0)])

    c = in_front(x)
    if "scan" in op:
        starts = torch.repeat_interleave(c[offsets[:-1]], offsets[1:] - offsets[:-1])
        return (c[:-1] if excl else c[1:]) - starts
    sums = c[offsets[1:]] - c[offsets[:-1]]
    if op == "irregular_reduce":
        return sums
    q = in_front(x * x)
    return sums, q[offsets[1:]] - q[offsets[:-1]]
