"""The HBM repack at the edges of its tiles: slots that end a byte before,
at and after a wave's kilobyte, a tile (8 KiB) and a plan block (16 KiB), runs
of zero-size tensors longer than the 64 entries a wave loads at a time, and
launches split so that they start and end inside plan blocks; the tables of the
allocation-free repack around the ends of their batches, with the plan written
in both ways; and the tables of an open at many widths of the packed sizes.
Byte for byte against the oracle."""

import numpy as np
import pytest

import oracle
from paper_2401_14351_amd import binding

pytestmark = pytest.mark.gpu

SENTINEL = 0xA5


def edge_sizes():
    sizes = []
    for base in (1 << 10, 8 << 10, 16 << 10):
        for k in (1, 2, 3):
            sizes += [k * base + d for d in (-17, -16, -1, 0, 1, 15, 16)]
    sizes += [0] * 70 + [5000] + [0] * 130  # more empty slots in one place than a wave loads
    sizes += [1 + i % 16 for i in range(300)] + [40_000] + [16] * 65 + [0] + [2000]
    return sizes


def checkpoint(d, A, large):
    rng = np.random.default_rng(A)
    sizes = edge_sizes() + ([large] if large else [])
    tensors = [(f"t{i}", "i8", (n,), rng.integers(0, 256, n, dtype=np.uint8)) for i, n in enumerate(sizes)]
    binding.convert(iter(tensors), d, A, 1 << 16)
    index = oracle.make_index(tensors, A, 1)
    return index, bytes(oracle.partition_bytes(tensors, A)[:index.total_bytes])


# with the large tensor the mean slot passes the line between 2 and 1 KiB a wave
@pytest.mark.parametrize("A", [1, 16, 256])
@pytest.mark.parametrize("grid,large", [(0, 0), (1, 0), (3, 0), (0, 36 << 20), (997, (36 << 20) + 3)])
def test_repack_edges(tmp_path, monkeypatch, A, grid, large):
    import torch

    index, image = checkpoint(str(tmp_path), A, large)
    src = torch.frombuffer(bytearray(image), dtype=torch.uint8).to("cuda:0")
    if grid:
        monkeypatch.setenv("SLLM_K2_MAX_GRID", str(grid))
        monkeypatch.setenv("SLLM_NOALLOC_PLAN_BLOCKS", "5")
    for A2 in (16, 64, 4096):
        print("[gpu-test] repack edges", A, grid, A2, flush=True)
        want = bytes(oracle.repack(image, index, A2))
        for noalloc in (False, True):
            dst = torch.full((len(want) + 64,), SENTINEL, dtype=torch.uint8, device="cuda:0")
            with binding.Checkpoint(str(tmp_path), dev_alignment=A2) as ck:
                (ck.repack_noalloc if noalloc else ck.repack)(src, dst)
                torch.cuda.synchronize()
            got = dst.cpu().numpy()
            bad = np.nonzero(got[:len(want)] != np.frombuffer(want, np.uint8))[0]
            assert bad.size == 0, (A2, noalloc, bad[:8].tolist())
            assert (got[len(want):] == SENTINEL).all(), "bytes past the image were written"


def bits16(n):
    """n sizes that pack into 16 bits each, 1,984 to a batch."""
    sizes = [1 + (i * 40503) % 4999 + (60_000 if i % 900 == 0 else 0) for i in range(n)]
    assert (max(sizes) - min(sizes)).bit_length() == 16
    return sizes


# sizes of n tensors: all equal (no bits), multiples of a power of two, one
# large among small (wide values), batch ends at 1,984 (16 bits) and 2,048
# tensors, and batches, the last of them partial, whose plan is spread over the
# grid (more than 4 blocks of 16 KiB a tensor)
TABLES = {
    "equal": [513] * 2049,
    "shifted": [4096 * (1 + i % 5) for i in range(700)],
    "wide": [(i * 7919) % 301 for i in range(2500)] + [(9 << 20) + 5] + [i % 3 for i in range(40)],
    "16 bits, a batch less one": bits16(1983),
    "16 bits, a batch": bits16(1984),
    "16 bits, two batches": bits16(1990),
    "one": [77],
    "zeros": [0] * 2047 + [3, 0, 0],
    "spread": bits16(1984) + [i % 700 for i in range(90)] + [(40 << 20) + 3] + [0, 5000, 16384],
    "spread first": [(36 << 20) + 1] + [(i * 7919) % 301 for i in range(400)],
    "spread, then not": [(1 << 18) - (i * 4099) % 30_000 for i in range(200)] + [(36 << 20) + 1] + [0] * 2000 + [77] * 60,
}


@pytest.mark.parametrize("name", sorted(TABLES))
def test_noalloc_tables(tmp_path, monkeypatch, name):
    import torch

    rng = np.random.default_rng(7)
    tensors = [(f"t{i}", "i8", (n,), rng.integers(0, 256, n, dtype=np.uint8)) for i, n in enumerate(TABLES[name])]
    binding.convert(iter(tensors), str(tmp_path), 64, 1 << 16)
    index = oracle.make_index(tensors, 64, 1)
    image = bytes(oracle.partition_bytes(tensors, 64)[:index.total_bytes])
    src = torch.frombuffer(bytearray(image), dtype=torch.uint8).to("cuda:0")
    for A2, blocks in ((16, None), (256, "7"), (4096, None)):
        print("[gpu-test] noalloc tables", name, A2, flush=True)
        if blocks:
            monkeypatch.setenv("SLLM_NOALLOC_PLAN_BLOCKS", blocks)
        want = np.frombuffer(bytes(oracle.repack(image, index, A2)), np.uint8)
        dst = torch.full((len(want) + 64,), SENTINEL, dtype=torch.uint8, device="cuda:0")
        with binding.Checkpoint(str(tmp_path), index_only=True) as ck:
            ck.repack_noalloc(src, dst, A2)
            torch.cuda.synchronize()
        got = dst.cpu().numpy()
        assert np.array_equal(got[:len(want)], want)
        assert (got[len(want):] == SENTINEL).all(), "bytes past the image were written"
        monkeypatch.delenv("SLLM_NOALLOC_PLAN_BLOCKS", raising=False)


@pytest.mark.parametrize("streams", [2, 12])
@pytest.mark.parametrize("C", [24 << 20, (17 << 20) + 24])
@pytest.mark.parametrize("source", ["cached", "streamed", "keep"])
def test_staging_pieces(tmp_path, C, source, streams):
    """Copy-engine loads into a device layout, with chunks no larger than a
    stream's HBM staging (two streams) and larger than it (twelve: 16 MiB each),
    which go through it in pieces; two handles in a row, the second on the
    device blocks the first gave back."""
    import torch

    rng = np.random.default_rng(3)
    sizes = [(15 << 20) + 5, 1000, 0, (19 << 20) + 1, 77, 300_000]
    tensors = [(f"t{i}", "i8", (n,), rng.integers(0, 256, n, dtype=np.uint8)) for i, n in enumerate(sizes)]
    binding.convert(iter(tensors), str(tmp_path), 16, C)
    index = oracle.make_index(tensors, 16, C)
    image = bytes(oracle.partition_bytes(tensors, 16)[:index.total_bytes])
    for A2 in (256, 4096):
        print("[gpu-test] staging pieces", C, source, streams, A2, flush=True)
        want = np.frombuffer(bytes(oracle.repack(image, index, A2)), np.uint8)
        with binding.Pool(C, 2 if source == "streamed" else 4) as pool:
            if source == "cached":
                pool.cache(str(tmp_path))
            with binding.Checkpoint(str(tmp_path), pool=pool, engine="sdma", dev_alignment=A2, ring_slots=2,
                                    n_streams=streams, cache=source == "keep") as ck:
                for rep in range(2):
                    dst = torch.full((len(want) + 64,), SENTINEL, dtype=torch.uint8, device="cuda:0")
                    ck.load_into(dst, torch.cuda.current_stream())
                    torch.cuda.synchronize()
                    got = dst.cpu().numpy()
                    assert np.array_equal(got[:len(want)], want), rep
                    assert (got[len(want):] == SENTINEL).all(), "bytes past the image were written"
            if source != "streamed":
                pool.evict(str(tmp_path))


def test_open_after_a_failed_allocation(tmp_path):
    """An open whose staging no device could hold fails and leaves no HIP error
    behind: the next open and load of the thread, which need none, succeed."""
    import torch

    rng = np.random.default_rng(5)
    tensors = [(f"t{i}", "i8", (n,), rng.integers(0, 256, n, dtype=np.uint8)) for i, n in enumerate([(20 << 20) + 5, 77, 3000])]
    binding.convert(iter(tensors), str(tmp_path), 16, 4 << 20)
    index = oracle.make_index(tensors, 16, 4 << 20)
    want = np.frombuffer(bytes(oracle.repack(bytes(oracle.partition_bytes(tensors, 16)[:index.total_bytes]), index, 256)), np.uint8)
    with binding.Pool(4 << 20, 6) as pool:
        pool.cache(str(tmp_path))
        with pytest.raises(binding.SllmError) as ei:  # 4 MiB a stream at least: 64 TiB
            binding.Checkpoint(str(tmp_path), pool=pool, engine="sdma", dev_alignment=256, n_streams=1 << 24)
        assert ei.value.code == -5 and "hipMalloc" in ei.value.message
        dst = torch.full((len(want) + 64,), SENTINEL, dtype=torch.uint8, device="cuda:0")
        with binding.Checkpoint(str(tmp_path), pool=pool, dev_alignment=256) as ck:
            ck.load_into(dst, torch.cuda.current_stream())
            torch.cuda.synchronize()
        assert np.array_equal(dst.cpu().numpy()[:len(want)], want)
        pool.evict(str(tmp_path))


@pytest.mark.parametrize("width", [1, 2, 15, 16, 17, 24, 31, 32, 33])
def test_tables_of_every_width(tmp_path, width):
    """The tables an open computes, from sizes packed into `width` bits with
    counts just below, at and above a batch's capacity, are those of the host:
    open compares them, entry by entry.  The files are sparse, and no data is
    read."""
    most = min(2048, 31744 // width)
    rng = np.random.default_rng(width)
    for n in (most - 1, most, most + 1):
        print("[gpu-test] tables of width", width, n, flush=True)
        sizes = [int(x) for x in rng.integers(0, 1 << min(width, 12), n)]
        sizes[0], sizes[-1] = 0, (1 << width) - 1
        offsets, total = oracle.plan_layout(sizes, 64)
        entries = tuple(oracle.Entry(f"t{i}", "i8", (x,), 0, o, x) for i, (x, o) in enumerate(zip(sizes, offsets)))
        index = oracle.Index(64, 1 << 20, total, oracle.file_length(total), entries)
        d = tmp_path / str(n)
        d.mkdir()
        (d / "sllm.index").write_bytes(oracle.encode_index(index))
        with open(d / "sllm.part0", "wb") as f:
            f.truncate(index.file_bytes)
        for A2 in (16, 4096):
            with binding.Checkpoint(str(d), dev_alignment=A2, ring_slots=1) as ck:
                offsets2, total2 = oracle.device_layout(index, A2)
                assert ck.total_bytes == total2 and [t.offset for t in ck.tensors()] == offsets2
