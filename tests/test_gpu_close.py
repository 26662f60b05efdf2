"""sllm_close waits for the handle's device work, also for work that ran on
the caller's stream alone: a load from cached chunks by the kernel engine
(one launch on that stream) and a repack.  Without that wait the pool chunks
a load still reads could be evicted and refilled under it.  Each case
enqueues about 0.5 GB of work, closes the handle at once and checks that the
stream is then idle; the cached case then evicts the checkpoint, caches
another one into the same chunks and compares the first load's image with
the oracle's."""

import sys

import numpy as np
import pytest

import oracle
from paper_2401_14351_amd import binding, synth

pytestmark = pytest.mark.gpu

MiB = 1 << 20
C = 16 * MiB


def say(*a):
    print("[gpu-close]", *a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def torch_cuda():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    binding.lib()
    return torch


def write(tmp_path, name, seed, A=4096):
    spec = synth.CheckpointSpec(name, seed, alignment=A, chunk_size=C,
                                tensors=[synth.TensorSpec(f"w{i}", "i8", (128 * MiB + 4096 * i + 7,), "bytes")
                                         for i in range(4)])
    tensors = [(t.name, t.dtype, t.shape, d) for t, d in zip(spec.tensors, synth.materialize(spec))]
    d = str(tmp_path / name)
    binding.convert(iter(tensors), d, A, C)
    return d, tensors


@pytest.mark.parametrize("A2", [0, 256])
def test_close_waits_for_a_cached_kernel_load(torch_cuda, tmp_path, A2):
    torch = torch_cuda
    d, tensors = write(tmp_path, "first", 41)
    d2, _ = write(tmp_path, "second", 42)
    index = oracle.make_index(tensors, 4096, C)
    image = bytes(oracle.partition_bytes(tensors, 4096)[:index.total_bytes])
    want = bytes(oracle.repack(image, index, A2)) if A2 else image
    n = -(-index.total_bytes // C)
    s = torch.cuda.Stream()
    with binding.Pool(C, n) as pool:
        pool.cache(d)
        buf = torch.empty(len(want), dtype=torch.uint8, device="cuda:0")
        ck = binding.Checkpoint(d, pool=pool, dev_alignment=A2)
        ck.load_into(buf, s)
        ck.close()
        idle = s.query()
        say("A2", A2, "stream idle after close:", idle)
        assert idle, "close returned while the load still ran on the caller's stream"
        pool.evict(d)
        pool.cache(d2)  # refills the chunks the load read
        torch.cuda.synchronize()
        got = buf.cpu().numpy().tobytes()
        if got != want:
            bad = np.nonzero(np.frombuffer(got, np.uint8) != np.frombuffer(want, np.uint8))[0]
            raise AssertionError(f"{bad.size} bytes differ, first at {bad[:4].tolist()}")
        pool.evict(d2)


def test_close_waits_for_a_repack(torch_cuda, tmp_path):
    torch = torch_cuda
    d, tensors = write(tmp_path, "third", 43, A=1)
    index = oracle.make_index(tensors, 1, C)
    image = bytes(oracle.partition_bytes(tensors, 1)[:index.total_bytes])
    want = bytes(oracle.repack(image, index, 4096))
    src = torch.frombuffer(bytearray(image), dtype=torch.uint8).to("cuda:0")
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    out = torch.empty(len(want), dtype=torch.uint8, device="cuda:0")
    ck = binding.Checkpoint(d, dev_alignment=4096)
    for _ in range(8):  # about 8 GB of HBM traffic queued
        ck.repack(src, out, s)
    ck.close()
    idle = s.query()
    say("repack: stream idle after close:", idle)
    assert idle, "close returned while a repack still ran on the caller's stream"
    assert out.cpu().numpy().tobytes() == want


@pytest.mark.parametrize("grid", [None, "997"])
def test_close_waits_for_repacks_on_two_streams(torch_cuda, tmp_path, monkeypatch, grid):
    """More repacks in flight than end events looked at per call, on two
    streams, whole and split into several launches (the end rides on the last).
    Long copies ahead of them keep all of them waiting until close."""
    torch = torch_cuda
    if grid:
        monkeypatch.setenv("SLLM_K2_MAX_GRID", grid)
    spec = synth.stress(n=400, max_bytes=1 << 20, seed=44)
    tensors = [(t.name, t.dtype, t.shape, d) for t, d in zip(spec.tensors, synth.materialize(spec))]
    d = str(tmp_path / "two")
    binding.convert(iter(tensors), d, 4096, 1 << 20)
    index = oracle.make_index(tensors, 4096, 1 << 20)
    image = bytes(oracle.partition_bytes(tensors, 4096)[:index.total_bytes])
    want = bytes(oracle.repack(image, index, 256))
    src = torch.frombuffer(bytearray(image), dtype=torch.uint8).to("cuda:0")
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    outs = [torch.full((len(want),), 0xA5, dtype=torch.uint8, device="cuda:0") for _ in streams]
    ahead = [torch.zeros(4 << 30, dtype=torch.uint8, device="cuda:0") for _ in range(2)]
    torch.cuda.synchronize()
    ck = binding.Checkpoint(d, dev_alignment=256)
    ck.repack(src, outs[0], streams[0])  # the first call's own costs
    torch.cuda.synchronize()
    for s in streams:
        with torch.cuda.stream(s):
            for _ in range(30):  # 1.5 ms or more each
                ahead[0].copy_(ahead[1])
    for i in range(60):
        ck.repack(src, outs[i % 2], streams[i % 2])
    assert not any(s.query() for s in streams), "the copies ended too soon to show anything"
    ck.close()
    assert all(s.query() for s in streams), "close returned while a repack still ran"
    for o in outs:
        assert o.cpu().numpy().tobytes() == want


def test_repack_captured_in_a_graph(torch_cuda, tmp_path):
    """sllm_repack under capture: recorded once, replayed with the handle open,
    eager repacks and synchronizations between the replays."""
    torch = torch_cuda
    spec = synth.stress(n=60, max_bytes=256 << 10, seed=45)
    tensors = [(t.name, t.dtype, t.shape, d) for t, d in zip(spec.tensors, synth.materialize(spec))]
    d = str(tmp_path / "cap")
    binding.convert(iter(tensors), d, 4096, 1 << 20)
    index = oracle.make_index(tensors, 4096, 1 << 20)
    image = bytes(oracle.partition_bytes(tensors, 4096)[:index.total_bytes])
    want = bytes(oracle.repack(image, index, 256))
    src = torch.frombuffer(bytearray(image), dtype=torch.uint8).to("cuda:0")
    out = torch.empty(len(want), dtype=torch.uint8, device="cuda:0")
    other = torch.empty_like(out)
    with binding.Checkpoint(d, dev_alignment=256) as ck:
        side = torch.cuda.Stream()
        with torch.cuda.stream(side):
            ck.repack(src, out, side)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            ck.repack(src, out, torch.cuda.current_stream())
        for k in range(3):
            out.fill_(0xA5)
            ck.repack(src, other, torch.cuda.current_stream())
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            assert out.cpu().numpy().tobytes() == want, f"replay {k}"
            assert other.cpu().numpy().tobytes() == want, f"eager {k}"
        del g


@pytest.mark.parametrize("what,A2", [("kernel", 0), ("kernel", 256), ("sdma", 0), ("sdma", 256), ("repack", 256)])
def test_two_calls_in_one_capture(torch_cuda, tmp_path, what, A2):
    """A second call of a handle in one capture leaves the capture whole: cached
    loads by either engine and repacks, replayed with eager ones between the
    replays."""
    torch = torch_cuda
    spec = synth.stress(n=60, max_bytes=256 << 10, seed=48)
    tensors = [(t.name, t.dtype, t.shape, d) for t, d in zip(spec.tensors, synth.materialize(spec))]
    d = str(tmp_path / "loads")
    binding.convert(iter(tensors), d, 4096, 1 << 20)
    index = oracle.make_index(tensors, 4096, 1 << 20)
    image = bytes(oracle.partition_bytes(tensors, 4096)[:index.total_bytes])
    want = bytes(oracle.repack(image, index, A2)) if A2 else image
    outs = [torch.zeros(len(want), dtype=torch.uint8, device="cuda:0") for _ in range(3)]
    with binding.Pool(1 << 20, -(-index.total_bytes // (1 << 20))) as pool:
        pool.cache(d)
        with binding.Checkpoint(d, pool=pool, engine="sdma" if what == "sdma" else "kernel", dev_alignment=A2) as ck:
            src = torch.frombuffer(bytearray(image), dtype=torch.uint8).to("cuda:0")

            def work(o):
                s = torch.cuda.current_stream()
                ck.repack(src, o, s) if what == "repack" else ck.load_into(o, s)

            work(outs[2])  # its copy streams exist before the capture
            torch.cuda.synchronize()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g):
                for o in outs[:2]:
                    work(o)
            for k in range(3):
                for o in outs:
                    o.fill_(0xA5)
                work(outs[2])
                torch.cuda.synchronize()
                g.replay()
                torch.cuda.synchronize()
                for i, o in enumerate(outs):
                    assert o.cpu().numpy().tobytes() == want, (k, i)
            del g
        pool.evict(d)


def test_open_while_another_stream_captures(torch_cuda, tmp_path):
    """A handle that opens on idle blocks, while a stream captures, leaves the
    capture whole, and loads as ever."""
    torch = torch_cuda
    spec = synth.stress(n=60, max_bytes=256 << 10, seed=47)
    tensors = [(t.name, t.dtype, t.shape, d) for t, d in zip(spec.tensors, synth.materialize(spec))]
    d = str(tmp_path / "open")
    binding.convert(iter(tensors), d, 4096, 1 << 20)
    index = oracle.make_index(tensors, 4096, 1 << 20)
    want = bytes(oracle.repack(bytes(oracle.partition_bytes(tensors, 4096)[:index.total_bytes]), index, 256))
    out = torch.zeros(len(want), dtype=torch.uint8, device="cuda:0")
    x = torch.zeros(1 << 16, device="cuda:0")
    y = torch.zeros_like(x)
    side = torch.cuda.Stream()
    with binding.Pool(1 << 20, -(-index.total_bytes // (1 << 20))) as pool:
        pool.cache(d)
        binding.Checkpoint(d, pool=pool, dev_alignment=256).close()  # its blocks stay idle
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            y.copy_(x)
            ck = binding.Checkpoint(d, pool=pool, dev_alignment=256)
            y.add_(1)
        ck.load_into(out, side)
        torch.cuda.synchronize()
        assert out.cpu().numpy().tobytes() == want
        for k in range(3):
            x.fill_(k)
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            assert (y == k + 1).all(), k
        ck.close()
        del g
        pool.evict(d)


@pytest.mark.parametrize("what", ["repack", "load"])
def test_close_waits_for_replays(torch_cuda, tmp_path, what):
    """A captured repack, or cached load into a device layout, replayed on a
    non-blocking stream: close waits for the replays, which no event of the
    handle ends, so the next handle's tables cannot take the place of those
    they read."""
    torch = torch_cuda
    d, tensors = write(tmp_path, "graph", 46, A=1)
    index = oracle.make_index(tensors, 1, C)
    image = bytes(oracle.partition_bytes(tensors, 1)[:index.total_bytes])
    want = bytes(oracle.repack(image, index, 256))
    src = torch.frombuffer(bytearray(image), dtype=torch.uint8).to("cuda:0")
    out = torch.empty(len(want), dtype=torch.uint8, device="cuda:0")
    n = -(-index.total_bytes // C)
    with binding.Pool(C, n) as pool:
        pool.cache(d)
        ck = binding.Checkpoint(d, pool=pool, dev_alignment=256)

        def work(stream):
            ck.repack(src, out, stream) if what == "repack" else ck.load_into(out, stream)

        side = torch.cuda.Stream()
        work(side)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            work(torch.cuda.current_stream())
        out.fill_(0xA5)
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            for _ in range(8 if what == "repack" else 2):
                g.replay()
        assert not side.query(), "the replays ended too soon to show anything"
        ck.close()
        idle = side.query()
        with binding.Checkpoint(d, pool=pool, dev_alignment=4096):  # other tables of the same size
            torch.cuda.synchronize()
        assert idle, "close returned while a replay still ran"
        assert out.cpu().numpy().tobytes() == want
        del g
        pool.evict(d)
