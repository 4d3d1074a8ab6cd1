"""The ordinary calls of binding.py through the extension module: what it leaves to binding.py's own checks, and that both ways give the
same results, errors and effects."""
import pytest
import torch

from paper_1811_09736_amd import binding, workloads

N = 3 * 8192 + 24


def calls(x, off, out=None):
    """Every operation as (name, call(**more), native call)."""
    n = x.numel()
    nat = binding._native
    return [
        ("segmented_reduce", lambda **k: binding.segmented_reduce(x, 8, **k), lambda: nat.segmented_reduce(x, 8, None)),
        ("segmented_scan", lambda **k: binding.segmented_scan(x, 24, **k), lambda: nat.segmented_scan(x, 24, 0, None, "")),
        ("segmented_scan_ex", lambda **k: binding.segmented_scan_ex(x, 8, 3, **k), lambda: nat.segmented_scan(x, 8, 3, None, "")),
        ("scan", lambda **k: binding.scan(x, **k), lambda: nat.scan(x, 0, None, "")),
        ("scan_ex", lambda **k: binding.scan_ex(x, 1, **k), lambda: nat.scan(x, 1, None, "")),
        ("reduce", lambda **k: binding.reduce(x, **k), lambda: nat.reduce(x, None)),
        ("segmented_moments", lambda **k: binding.segmented_moments(x, n // 8, **k), lambda: nat.segmented_moments(x, n // 8)),
        ("irregular_reduce", lambda **k: binding.irregular_reduce(x, off, **k), lambda: nat.irregular_reduce(x, off, None)),
        ("irregular_moments", lambda **k: binding.irregular_moments(x, off, **k), lambda: nat.irregular_moments(x, off)),
        ("irregular_scan", lambda **k: binding.irregular_scan(x, off, **k), lambda: nat.irregular_scan(x, off, 0, None, "")),
        ("irregular_scan_ex", lambda **k: binding.irregular_scan_ex(x, off, 1, **k), lambda: nat.irregular_scan(x, off, 1, None, "")),
    ]


@pytest.mark.parametrize("x", [torch.zeros(N, dtype=torch.float16), torch.zeros(N), torch.zeros(8, N // 8, dtype=torch.float16), [0.0] * 8, None], ids=str)
def test_what_is_no_gpu_tensor_is_left_to_binding(x):
    off = torch.tensor([0, 5])
    nat = binding._native
    for got in (nat.segmented_reduce(x, 8, None), nat.segmented_scan(x, 8, 0, None, ""), nat.scan(x, 0, None, ""), nat.reduce(x, None),
                nat.segmented_moments(x, 8), nat.irregular_reduce(x, off, None), nat.irregular_moments(x, off), nat.irregular_scan(x, off, 0, None, "")):
        assert got is None
    if isinstance(x, torch.Tensor):
        with pytest.raises(TypeError, match="input must be a contiguous 1-D float16 CUDA tensor"):
            binding.segmented_reduce(x, 8)


@pytest.fixture(scope="module")
def data():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    x = torch.from_numpy(workloads.make_input(N, "int4", 3)).cuda()
    return x, torch.tensor([3, 3, 100, 9000, N - 7], device="cuda")


def flat(r):
    return list(r) if isinstance(r, tuple) else [r]


@pytest.mark.gpu
def test_both_ways_agree(data):
    for name, call, native in calls(*data):
        here, there, direct = flat(call()), flat(call(stream=torch.cuda.current_stream())), flat(native())
        for a, b, c in zip(here, there, direct):
            assert torch.equal(a, b) and torch.equal(a, c), name
            assert a.dtype == b.dtype and a.shape == b.shape and a.device == b.device and not a.requires_grad, name


@pytest.mark.gpu
def test_given_results(data):
    x, off = data
    for name, call, _ in calls(x, off):
        if "moments" in name:
            continue
        want = call()
        out = torch.full_like(want, -3)
        assert call(out=out) is out
        if name.startswith("irregular_scan"):            # (given results stay as they are where no segment lies)
            assert torch.equal(out[3:N - 7], want[3:N - 7]) and (out[:3] == -3).all() and (out[N - 7:] == -3).all()
        else:
            assert torch.equal(out, want), name
        for wrong in (torch.empty(want.numel() + 1, device="cuda"), torch.empty(want.numel(), dtype=torch.float64, device="cuda"), torch.empty(want.numel()),
                      torch.empty(2 * want.numel(), device="cuda")[::2] if want.numel() > 1 else torch.empty(2, device="cuda")):
            with pytest.raises(TypeError, match="out must be a contiguous"):
                call(out=wrong)


@pytest.mark.gpu
def test_wrong_arguments_fail_as_before(data):
    x, off = data
    invalid = [lambda: binding.segmented_reduce(x, 7 * 11), lambda: binding.segmented_reduce(x, 0), lambda: binding.segmented_reduce(x, -8),
               lambda: binding.segmented_scan(x, 0), lambda: binding.segmented_scan_ex(x, 0, 1), lambda: binding.segmented_scan_ex(x, 77, 0),
               lambda: binding.segmented_scan_ex(x, 8, 4), lambda: binding.scan_ex(x, 8), lambda: binding.irregular_scan_ex(x, off, 4),
               lambda: binding.segmented_moments(x, 7 * 11), lambda: binding.segmented_moments(x, 0)]
    for call in invalid:
        with pytest.raises(binding.TcrError) as e:
            call()
        assert e.value.status == binding.ERR_INVALID_ARG
    for wrong in (off.int(), off.cpu(), off.view(1, -1), off[:0], torch.stack([off, off], 1)[:, 0]):
        with pytest.raises(TypeError, match="offsets must be"):
            binding.irregular_reduce(x, wrong)
    for wrong in (x.float(), x.view(2, -1), x[::2]):
        with pytest.raises(TypeError, match="input must be"):
            binding.scan(wrong)
    # an error that only the library sees, in the middle of a native call
    with pytest.raises(binding.TcrError, match="tcr_scan_ex"):
        binding._native.scan(x, 4, None, "tcr_scan_ex")


class Marked(torch.Tensor):
    pass


@pytest.mark.gpu
def test_special_tensors_and_modes_take_binding(data):
    x, off = data
    from torch.overrides import TorchFunctionMode
    from torch.utils._python_dispatch import TorchDispatchMode

    class Functions(TorchFunctionMode):
        seen = 0

        def __torch_function__(self, func, types, args=(), kwargs=None):
            Functions.seen += func is torch.empty
            return func(*args, **(kwargs or {}))

    class Dispatches(TorchDispatchMode):
        seen = 0

        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            Dispatches.seen += "empty" in str(func)
            return func(*args, **(kwargs or {}))

    want = binding.scan(x)
    assert binding._native.scan(x.as_subclass(Marked), 0, None, "") is None
    assert torch.equal(binding.scan(x.as_subclass(Marked)), want)
    with Functions():
        assert torch.equal(binding.scan(x), want) and Functions.seen == 1
    with Dispatches():
        assert torch.equal(binding.scan(x), want) and Dispatches.seen == 1
    with torch.inference_mode():
        got = binding.scan(x)
        assert got.is_inference()
    assert torch.equal(got, want)
    assert torch.equal(binding.scan(torch.nn.Parameter(x.clone())), want)


@pytest.mark.gpu
def test_the_current_stream(data):
    x, _ = data
    want = binding.scan(x)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        y = torch.zeros(1 << 26, device="cuda").half()          # (some time on the stream in front of the copy)
        y[:N].copy_(x)
        got = binding.scan(y[:N])
    side.synchronize()
    assert torch.equal(got, want)


# An allocation that has to free what is cached waits for the device; other threads of Python run meanwhile.  (The device is kept busy for a while, and the
# process is allowed no more memory than it has.)
@pytest.mark.gpu
def test_allocations_give_the_interpreter_up(data):
    import threading
    import time

    x = torch.ones(1 << 28, dtype=torch.float16, device="cuda")
    binding.scan(x)                                                      # (so that the library has what it needs)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    parked = torch.empty(1 << 29, dtype=torch.uint8, device="cuda")      # (half of what the call asks for: no use to it, but cached)
    total = torch.cuda.get_device_properties(x.device).total_memory
    calls, ticks, stop = [], [], threading.Event()

    def tick():
        while not stop.is_set():
            ticks.append(time.perf_counter())
            time.sleep(0.0005)

    thread = threading.Thread(target=tick)
    try:
        del parked
        torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + (768 << 20)) / total)
        thread.start()
        busy = x[:1 << 26]
        for _ in range(4000):
            busy.mul_(1.0)
        begin = time.perf_counter()
        got = binding._native.scan(x, 0, None, "tcr_scan")
        calls = [begin, time.perf_counter()]
    finally:
        stop.set()
        thread.join()
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert torch.equal(got[:1 << 24], torch.arange(1, (1 << 24) + 1, device="cuda").float())
    during = [t for t in ticks if calls[0] < t < calls[1]]
    assert calls[1] - calls[0] > 0.02, "the call did not wait"
    assert len(during) > (calls[1] - calls[0]) / 0.02


@pytest.mark.parametrize("missing", [True, False])
def test_binding_without_the_module(missing):
    """Where _native cannot be imported the calls take ctypes; where it can, it is used."""
    import subprocess
    import sys

    code = ("import sys, torch\n"
            + ("sys.modules['paper_1811_09736_amd._native'] = None\n" if missing else "")
            + "from paper_1811_09736_amd import binding\n"
            "assert (type(binding._native).__name__ == '_NoNative') is %s\n"
            "assert binding.kernel_name(binding.OP_SCAN, 1 << 20, 1 << 20)\n"
            "for call in (lambda x: binding.scan(x), lambda x: binding.segmented_moments(x, 8)):\n"
            "    try: call(torch.zeros(8, dtype=torch.float16))\n"
            "    except TypeError as e: assert 'input must be' in str(e)\n"
            "    else: raise AssertionError('accepted')\n"
            "print('ok')\n") % missing
    run = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=300)
    assert run.returncode == 0 and run.stdout.strip().endswith("ok"), run.stderr
