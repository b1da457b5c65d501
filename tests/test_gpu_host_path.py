"""The host side of the per-token calls: how it behaves out of memory, under capture and beside threads."""
import ctypes
import threading
import time

import pytest
import torch

import paper_2602_03681_amd as nats
from paper_2602_03681_amd import binding as nb

pytestmark = pytest.mark.gpu
NAMES = ("state", "k_cache", "v_cache", "cache_len", "q", "k", "v", "alpha", "beta", "mask")


def _step(B, H, d, cap, dtype=torch.bfloat16, seed=0, length=None):
    gen = torch.Generator().manual_seed(seed)
    rnd = lambda *s: torch.randn(*s, generator=gen)
    unit = lambda *s: torch.nn.functional.normalize(rnd(*s), dim=-1).to(dtype)
    x = dict(state=0.02 * rnd(B, H, d, d), k_cache=unit(B, H, cap, d), v_cache=rnd(B, H, cap, d).to(dtype),
             cache_len=torch.full((B, H), cap - 1 if length is None else length, dtype=torch.int32), q=unit(B, H, d), k=unit(B, H, d),
             v=rnd(B, H, d).to(dtype), alpha=torch.sigmoid(2 + rnd(B, H)), beta=torch.sigmoid(rnd(B, H)),
             mask=torch.zeros(B, H, dtype=torch.uint8))
    return {k: v.cuda() for k, v in x.items()}


@pytest.fixture
def no_memory():
    """From the call on, no block of 1 MB or more can be had: torch may take nothing from the device and what it holds is taken."""
    total, held = torch.cuda.get_device_properties(0).total_memory, []

    def close():
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        torch.cuda.set_per_process_memory_fraction(torch.cuda.memory_reserved() / total)
        for size in (1 << 26, 1 << 22, 1 << 20):
            with pytest.raises(torch.cuda.OutOfMemoryError):
                while True:
                    held.append(torch.empty(size, dtype=torch.uint8, device="cuda"))
    yield close
    held.clear()
    torch.cuda.set_per_process_memory_fraction(1.0)


def test_out_of_memory_for_the_output_is_torchs_error(no_memory):
    B, H, d = 512, 100, 128                      # an output of 13 MB
    x = _step(B, H, d, 1)
    no_memory()
    with pytest.raises(torch.cuda.OutOfMemoryError):
        nats.hybrid_attn_decode(*(x[k] for k in NAMES))


def test_a_step_without_memory_for_a_workspace_runs_without(no_memory):
    B, H, d, cap = 1, 128, 128, 2048             # partial results of 2.2 MB where there is room
    x = _step(B, H, d, cap)
    y = {k: v.clone() for k, v in x.items()}
    want = nats.hybrid_attn_decode(*(y[k] for k in NAMES))
    out = torch.empty_like(want)
    no_memory()
    nats.hybrid_attn_decode(*(x[k] for k in NAMES), out=out)
    torch.cuda.synchronize()
    assert float((out.float() - want.float()).abs().max()) <= 2.0 ** -7 * float(want.float().abs().max())


def test_other_threads_run_while_a_launch_waits():
    """Behind a kernel of a second the stream's queue fills up and a launch waits for room."""
    x = _step(1, 2, 64, 96)
    out = torch.empty_like(x["q"])
    run = lambda: nats.hybrid_attn_decode(*(x[k] for k in NAMES), out=out)
    run()
    torch.cuda._sleep(1000)
    torch.cuda.synchronize()
    gaps, stop = [0.0], threading.Event()

    def ticks():
        last = time.perf_counter()
        while not stop.is_set():
            time.sleep(0.001)
            now = time.perf_counter()
            gaps[0] = max(gaps[0], now - last)
            last = now
    other = threading.Thread(target=ticks)
    other.start()
    longest = 0.0
    t0 = time.perf_counter()
    torch.cuda._sleep(2_000_000_000)             # about a second
    while time.perf_counter() - t0 < 0.5 and longest < 0.2:
        t1 = time.perf_counter()
        run()
        longest = max(longest, time.perf_counter() - t1)
    stop.set()
    other.join()
    torch.cuda.synchronize()
    # (where the queue had room for all of it, nothing was seen)
    assert longest < 0.2 or gaps[0] < longest / 2, (gaps[0], longest)


def _hip():
    path = next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line)
    return ctypes.CDLL(path)


@pytest.mark.parametrize("chunked", [False, True])
def test_a_captured_step_allocates_nothing(chunked):
    """A capture outside torch's own graphs has no pool for what torch allocates meanwhile: with an output given, a step makes
    no allocation there, and the graph computes what the eager call does."""
    B, H, d, cap = 1, 16, 128, 512
    x, hip = _step(B, H, d, cap, length=300), _hip()
    st = dict(state_start=torch.empty_like(x["state"]), chunk_decay=torch.ones(B, H, device="cuda"),
              chunk_pos=torch.zeros(B, H, dtype=torch.int32, device="cuda"), **{k: x[k] for k in NAMES[:4]})
    out, first = torch.empty_like(x["q"]), {k: v.clone() for k, v in dict(x, **st).items()}
    if chunked:
        run = lambda: nats.hybrid_attn_decode_chunk(st, *(x[k] for k in NAMES[4:9]), out=out)
    else:
        run = lambda: nats.hybrid_attn_decode(*(x[k] for k in NAMES), out=out)
    run()
    want = out.clone()
    s, graph, exe = torch.cuda.Stream(), ctypes.c_void_p(), ctypes.c_void_p()
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        handle = ctypes.c_void_p(s.cuda_stream)
        assert hip.hipStreamBeginCapture(handle, 2) == 0        # relaxed
        before = torch.cuda.memory_stats()["allocation.all.allocated"]
        run()
        made = torch.cuda.memory_stats()["allocation.all.allocated"] - before
        assert hip.hipStreamEndCapture(handle, ctypes.byref(graph)) == 0
    assert made == 0
    assert hip.hipGraphInstantiate(ctypes.byref(exe), graph, None, None, ctypes.c_size_t(0)) == 0
    for _ in range(3):
        for k, v in dict(x, **st).items():
            v.copy_(first[k])
        out.zero_()
        torch.cuda.synchronize()
        assert hip.hipGraphLaunch(exe, handle) == 0
        torch.cuda.synchronize()
        assert float((out.float() - want.float()).abs().max()) <= 2.0 ** -7 * float(want.float().abs().max())
    hip.hipGraphExecDestroy(exe)
    hip.hipGraphDestroy(graph)
