"""Cases of test_host_hip.py, each run in a process of its own (usage:
fake_hip_cases.py FAKE_LIBRARY CASE DIRECTORY): the library's host code over
the HIP runtime of tests/native/fake_hip.cpp, which stands in for the real one
and must be loaded first.  Nothing here may import torch, which brings the real
runtime with it."""

import ctypes as C
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
sys.modules["torch"] = None  # "import torch" raises ImportError

fake = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
for _name in ("fake_mallocs", "fake_frees", "fake_launches", "fake_used", "fake_records_captured", "fake_bad_calls",
              "fake_waits", "fake_spread"):
    getattr(fake, _name).restype = C.c_uint64
fake.fake_bad_list.restype = C.c_char_p
fake.fake_last_kernel.restype = C.c_char_p
fake.fake_limit.argtypes = [C.c_uint64]
fake.fake_corrupt.argtypes = [C.c_uint64]
fake.fake_fail_launch.argtypes = [C.c_int64]
fake.fake_stream.restype = C.c_void_p
fake.fake_capture.argtypes = [C.c_void_p, C.c_int]
fake.fake_device_alloc.restype = C.c_void_p
fake.fake_device_alloc.argtypes = [C.c_uint64]

import numpy as np  # noqa: E402

from paper_2401_14351_amd import binding  # noqa: E402

KiB, MiB = 1 << 10, 1 << 20
NO_LIMIT = (1 << 64) - 1


def convert(d, sizes, A=16, chunk=64 * KiB):
    d = os.path.join(sys.argv[3], d)
    binding.convert(((f"t{i}", "i8", (n,), np.full(n, i % 251, np.uint8)) for i, n in enumerate(sizes)), d, A, chunk)
    return d


def total(sizes, A):
    return sum(-(-n // A) * A for n in sizes)


class Buffers:
    """Device buffers for a repack of `sizes` from A into A2."""

    def __init__(self, sizes, A, A2):
        self.n, self.n2 = total(sizes, A), total(sizes, A2)
        self.src, self.dst = fake.fake_device_alloc(self.n), fake.fake_device_alloc(self.n2)

    def repack(self, ck, stream):
        return binding.lib().sllm_repack(ck._h, self.src, self.n, self.dst, self.n2, stream)


SIZES = [1000, 0, 70_000, 5, 333_333]


def case_events_under_capture():
    """Captured loads and repacks record no event, and no event of a capture is
    queried or waited for: neither by calls of the same capture, nor by eager
    ones on another stream meanwhile, nor at close."""
    d = convert("c", SIZES)
    b = Buffers(SIZES, 16, 256)
    s, other = fake.fake_stream(), fake.fake_stream()
    pool = binding.Pool(64 * KiB, 32)
    pool.cache(d)
    ck = binding.Checkpoint(d, pool=pool, dev_alignment=256)
    assert b.repack(ck, s) == 0
    fake.fake_capture(s, 1)
    for _ in range(3):
        assert b.repack(ck, s) == 0
        ck.load(b.dst, b.n2, s)
        assert b.repack(ck, other) == 0  # eager
    fake.fake_capture(s, 0)
    for _ in range(6):  # more than the events a call looks at
        assert b.repack(ck, s) == 0
        ck.load(b.dst, b.n2, other)
    ck.close()
    assert fake.fake_records_captured() == 0
    assert fake.fake_bad_calls() == 0, fake.fake_bad_list()
    assert fake.fake_pending() == 0


def case_close_after_capture():
    """The device tables and staging of a handle whose loads or repacks were
    captured are freed at close (hipFree waits for the device, so for replays
    too); those of other handles stay for the next one."""
    d = convert("c", SIZES)
    b = Buffers(SIZES, 16, 256)
    s = fake.fake_stream()
    pool = binding.Pool(64 * KiB, 32)
    pool.cache(d)

    def frees(engine, work):
        """Blocks the close of a handle frees."""
        ck = binding.Checkpoint(d, pool=pool, dev_alignment=256, engine=engine)
        work(ck)
        before = fake.fake_frees()
        ck.close()
        return fake.fake_frees() - before

    def captured(f):
        def run(ck):
            f(ck)  # also eagerly
            fake.fake_capture(s, 1)
            f(ck)
            fake.fake_capture(s, 0)
            f(ck)
        return run

    def repack(ck):
        assert b.repack(ck, s) == 0

    def load(ck):
        ck.load(b.dst, b.n2, s)

    for engine, blocks in (("kernel", 1), ("sdma", 2)):
        for work in (repack, load):
            if engine == "sdma" and work is load:
                continue  # its copy streams would have to leave the capture again
            assert frees(engine, work) == 0, (engine, work)
            assert frees(engine, captured(work)) == blocks, (engine, work)
            assert frees(engine, work) == 0, (engine, work)


def case_open_under_capture():
    """While another stream captures, a handle opens on idle blocks by no call
    that would end the capture, and closes the same way."""
    d = convert("c", SIZES)
    s = fake.fake_stream()
    pool = binding.Pool(64 * KiB, 32)
    pool.cache(d)
    for engine in ("kernel", "sdma"):
        opts = {"pool": pool, "dev_alignment": 256, "engine": engine}
        binding.Checkpoint(d, **opts).close()
        fake.fake_capture(s, 1)
        binding.Checkpoint(d, **opts).close()
        fake.fake_capture(s, 0)
        assert fake.fake_bad_calls() == 0, fake.fake_bad_list()
        assert fake.fake_pending() == 0


def case_refused_free():
    """A close whose hipFree is refused, while another stream captures, leaves no
    HIP error behind: the next launch of the thread is no failure."""
    d = convert("c", SIZES)
    b = Buffers(SIZES, 16, 256)
    s, other = fake.fake_stream(), fake.fake_stream()
    ck = binding.Checkpoint(d, dev_alignment=256, ring_slots=1)
    next_one = binding.Checkpoint(d, dev_alignment=256, ring_slots=1)
    fake.fake_capture(s, 1)
    assert b.repack(ck, s) == 0
    fake.fake_capture(s, 0)
    fake.fake_capture(other, 1)
    ck.close()
    assert b"hipFree" in fake.fake_bad_list()
    assert fake.fake_pending() == 0
    assert b.repack(next_one, s) == 0
    fake.fake_capture(other, 0)
    next_one.close()


def case_failure_under_capture():
    """A repack or load that fails under capture returns its error and makes no
    call that HIP refuses on a capturing stream; eagerly it waits for the stream."""
    d = convert("c", SIZES)
    b = Buffers(SIZES, 16, 256)
    s = fake.fake_stream()
    pool = binding.Pool(64 * KiB, 32)
    pool.cache(d)
    with binding.Checkpoint(d, pool=pool, dev_alignment=256) as ck:
        for capture in (1, 0):
            for work in (lambda: b.repack(ck, s), lambda: binding.lib().sllm_load(ck._h, b.dst, b.n2, s)):
                fake.fake_capture(s, capture)
                fake.fake_fail_launch(0)
                waits = fake.fake_waits()
                assert work() == -5
                fake.fake_capture(s, 0)
                assert (fake.fake_waits() > waits) == (not capture)
    assert fake.fake_bad_calls() == 0, fake.fake_bad_list()
    assert fake.fake_pending() == 0


def case_error_not_left_pending():
    """An open whose device memory cannot be had, and a load, repack or pool
    whose HIP call fails, leave no error for the next call's launch check."""
    d = convert("c", SIZES)
    b = Buffers(SIZES, 16, 256)
    s = fake.fake_stream()
    pool = binding.Pool(64 * KiB, 32)
    pool.cache(d)
    for room in (0, 300 * KiB):  # not for the tables; for the tables, not for the staging
        fake.fake_limit(fake.fake_used() + room)
        for _ in range(2):
            try:
                binding.Checkpoint(d, pool=pool, dev_alignment=256, engine="sdma", n_streams=4)
            except binding.SllmError as e:
                assert e.code == -5, e
            else:
                raise AssertionError("the open succeeded")
            assert fake.fake_pending() == 0
        if room:
            with binding.Checkpoint(d, pool=pool, dev_alignment=256) as ck:  # the kernel engine stages nothing
                ck.load(b.dst, b.n2, s)
        fake.fake_limit(NO_LIMIT)
    with binding.Checkpoint(d, pool=pool, dev_alignment=256) as ck:
        for work in (lambda: b.repack(ck, s), lambda: binding.lib().sllm_load(ck._h, b.dst, b.n2, s)):
            fake.fake_fail_launch(0)
            assert work() == -5
            assert work() == 0
    pool.evict(d)
    fake.fake_limit(fake.fake_used())
    try:
        pool.cache(d)  # its chunk table
    except binding.SllmError as e:
        assert e.code == -5, e
    else:
        raise AssertionError("the fill succeeded")
    assert fake.fake_pending() == 0


def case_idle_blocks():
    """Blocks of closed handles wait for the next one, at most 256 MiB in 32
    blocks, the oldest given up first: sizes no handle takes any more do not
    keep later ones out."""
    small, large = convert("s", [100]), convert("l", [1] * 20_000)
    pool = binding.Pool(64 * KiB, 64)
    pool.cache(small)
    pool.cache(large)

    def reopened(**opts):
        """Allocations of the second of two handles opened and closed in a row."""
        for _ in range(2):
            before = fake.fake_mallocs()
            binding.Checkpoint(pool=pool, **opts).close()
        return fake.fake_mallocs() - before

    base = fake.fake_used()
    handles = [binding.Checkpoint(small, pool=pool, dev_alignment=256) for _ in range(40)]
    for ck in handles:
        ck.close()
    assert fake.fake_used() - base == 32 * 64 * KiB
    # 20,000 tensors' tables do not fit a 64 KiB block, whose place they take
    assert reopened(ckpt_dir=large, dev_alignment=16) == 0
    assert reopened(ckpt_dir=small, dev_alignment=16) == 0
    # staging of sizes that are not asked for again
    big = convert("b", [20 * MiB], chunk=64 * KiB)
    with binding.Pool(64 * KiB, 320) as p2:
        p2.cache(big)
        for n in (10, 9, 8):
            binding.Checkpoint(big, pool=p2, dev_alignment=16, engine="sdma", n_streams=n, io_threads=1).close()
            assert fake.fake_used() - base <= 256 * MiB
    assert reopened(ckpt_dir=large, dev_alignment=16) == 0
    # more than all idle blocks may hold: freed at once, without the others
    with binding.Pool(64 * KiB, 320) as p2:
        p2.cache(big)
        held = fake.fake_used()
        binding.Checkpoint(big, pool=p2, dev_alignment=16, engine="sdma", n_streams=100).close()
        assert abs(fake.fake_used() - held) <= MiB  # the tables only
    # no memory: the idle blocks are given up for an allocation that needs it
    fake.fake_limit(fake.fake_used())
    with binding.Checkpoint(convert("x", [1] * 60_000), pool=None, dev_alignment=16, ring_slots=1):
        pass


def case_tables_are_checked():
    """A wrong entry in any of the device's tables fails the open: file offset,
    device offset or size, of the first, a middle and the last tensor of each
    batch, and the totals."""
    sizes = [(i * 7919) % 60_000 for i in range(2500)]
    d = convert("c", sizes)
    n = len(sizes)
    for what in [3 * i + k for i in (0, 1, 1023, 1983, 1984, 1985, n - 1) for k in (0, 1, 2)] + [3 * n, 3 * n + 1]:
        fake.fake_corrupt(what)
        try:
            binding.Checkpoint(d, dev_alignment=256, ring_slots=1).close()
        except binding.SllmError as e:
            assert e.code == -5 and "disagree" in e.message, e
        else:
            raise AssertionError(f"entry {what} was not checked")
    fake.fake_corrupt(NO_LIMIT)
    with binding.Checkpoint(d, dev_alignment=256, ring_slots=1):
        pass


def sparse(name, sizes, A, chunk):
    """A converted checkpoint whose data file has no blocks."""
    import oracle

    offsets, t = oracle.plan_layout(sizes, A)
    entries = tuple(oracle.Entry(f"t{i}", "i8", (n,), 0, o, n) for i, (n, o) in enumerate(zip(sizes, offsets)))
    index = oracle.Index(A, chunk, t, oracle.file_length(t), entries)
    d = os.path.join(sys.argv[3], name)
    os.mkdir(d)
    with open(os.path.join(d, "sllm.index"), "wb") as f:
        f.write(oracle.encode_index(index))
    with open(os.path.join(d, "sllm.part0"), "wb") as f:
        f.truncate(index.file_bytes)
    return d


def case_staging_sizes():
    """Copy-engine staging: a chunk for streams, merged runs of 64 MiB for
    resident images, never more than the image; all streams' together 192 MiB,
    or the image in up to 64 MiB each, and kept with the tables up to 256."""
    d = sparse("c", [100 * MiB + 5], 16, MiB)
    large = sparse("l", [1200 * MiB], 16, 16 * MiB)
    pool = binding.Pool(MiB, 101)
    wide = binding.Pool(96 * MiB, 2)

    def staging(pool, n, d=d, **opts):
        before = fake.fake_used()
        with binding.Checkpoint(d, pool=pool, engine="sdma", dev_alignment=16, n_streams=n, **opts):
            held = fake.fake_used() - before
        kept = fake.fake_used()
        with binding.Checkpoint(d, pool=pool, engine="sdma", dev_alignment=16, n_streams=n, **opts):
            again = fake.fake_used() - kept
        fake.fake_limit(0)  # drop the idle blocks
        try:
            binding.Checkpoint(d, pool=pool, engine="sdma", dev_alignment=16, n_streams=1 << 20, **opts)
        except binding.SllmError:
            pass
        fake.fake_limit(NO_LIMIT)
        return held // MiB, again < 64 * KiB  # SLLM_OPEN_CACHE has a small table of its own

    assert staging(pool, 2, ring_slots=4) == (2, True)  # streamed
    assert staging(wide, 1, ring_slots=2) == (96, True)
    pool.cache(d)
    wide.cache(d)
    for n, held in ((1, 64), (2, 128), (3, 192), (4, 192), (8, 192), (12, 192), (24, 192), (48, 192)):
        assert staging(pool, n) == (held, True), n
    assert staging(pool, 100) == (400, False)
    assert staging(wide, 1) == (96, True)
    assert staging(wide, 3) == (192, True)
    with binding.Pool(16 * MiB, 75) as p3:
        for n, held in ((1, 64), (2, 128), (3, 192), (4, 256), (16, 1024), (24, 1200)):
            assert staging(p3, n, large, cache=True) == (held, held < 256), n


def case_scatter_unroll():
    """Vectors per lane of cached loads into a device layout: 2 for images below
    4 MiB, else 8; SLLM_K2_UNROLL gives 8, or 4 for any other value."""
    for sizes, default in (([3 * MiB], 2), ([5 * MiB], 8)):
        d = convert(f"c{default}", sizes, chunk=MiB)
        n2 = total(sizes, 256)
        dst = fake.fake_device_alloc(n2)
        with binding.Pool(MiB, 8) as pool:
            pool.cache(d)
            with binding.Checkpoint(d, pool=pool, dev_alignment=256) as ck:
                for knob, want in ((None, default), ("2", 4), ("4", 4), ("8", 8), ("16", 8), ("x", default)):
                    os.environ.pop("SLLM_K2_UNROLL", None)
                    if knob:
                        os.environ["SLLM_K2_UNROLL"] = knob
                    ck.load(dst, n2, fake.fake_stream())
                    assert f"k_scatterILj{want}E".encode() in fake.fake_last_kernel(), (knob, fake.fake_last_kernel())


def case_pack_sizes():
    """Sizes packed into kernel arguments and unpacked again, at every width and
    every shift it leaves room for, with counts just below, at and above a
    batch's capacity."""
    rng = np.random.default_rng(1)
    u64 = C.POINTER(C.c_uint64)
    fake.fake_pack.restype = C.c_uint64
    fake.fake_pack.argtypes = [u64, C.c_uint64, u64, u64, u64]

    def pack(s):
        s = np.ascontiguousarray(s, dtype=np.uint64)
        out, counts, widths = np.zeros_like(s), np.zeros_like(s), np.zeros_like(s)
        k = fake.fake_pack(*(a.ctypes.data_as(u64) if isinstance(a, np.ndarray) else a for a in (s, len(s), out, counts, widths)))
        assert np.array_equal(out, s)
        return counts[:k].tolist(), widths[:k].tolist()

    for width in range(65):
        most = min(2048, 31744 // width) if width else 2048
        for shift in range(65 - width if width else 1):
            top = (1 << width) - 1  # odd, so the shift is exact
            base = int(rng.integers(0, (1 << 64) - (top << shift), dtype=np.uint64, endpoint=False)) if width + shift < 64 else 0
            for n in (most - 1, most, most + 1):
                v = rng.integers(0, top, n, dtype=np.uint64, endpoint=True) if top else np.zeros(n, np.uint64)
                v[0], v[-2 if n > most else -1] = 0, top
                counts, widths = pack((v << np.uint64(shift)) + np.uint64(base))
                assert counts[0] == min(n, most) and sum(counts) == n, (width, shift, n, counts)
                assert widths[0] == width, (width, shift, n, widths)
    for n in (1, 2, 3, 5000):
        pack(rng.integers(0, 1 << 40, n, dtype=np.uint64))


def case_plan_writers():
    """Which writer a batch's plan gets: spread over a grid beyond four blocks of
    16 KiB a tensor, and from one on where more than 4 % of the tensors hold
    more than eight; and no empty grid where a window ends in or before a batch."""
    small, wide = 14 * KiB, 144 * KiB
    for sizes, spread in (([64 * KiB] * 1000, 0), ([64 * KiB] * 1000 + [3 * MiB], 1),
                          ([wide] * 40 + [small] * 960, 0), ([wide] * 41 + [small] * 959, 1),
                          ([wide] * 41 + [256] * 959, 0), ([128 * KiB] * 100 + [small] * 900, 0),
                          ([wide] * 2048 + [77] * 30 + [small] * 2018, 1), ([0] * 50, 0)):
        d = sparse(f"c{len(sizes)}-{sizes.count(wide)}-{sum(sizes)}", sizes, 16, MiB)
        before = fake.fake_spread()
        with binding.Checkpoint(d, dev_alignment=16, ring_slots=1):
            assert fake.fake_spread() - before == spread, (len(sizes), spread)
        buf = Buffers(sizes, 16, 16)
        with binding.Checkpoint(d, index_only=True) as ck:
            for window in ("1", "1001", "5000"):
                os.environ["SLLM_NOALLOC_PLAN_BLOCKS"] = window
                st = binding.lib().sllm_repack_noalloc(ck._h, 16, buf.src, buf.n, buf.dst, buf.n2, fake.fake_stream())
                assert st == 0 or buf.n2 == 0, (window, binding.lib().sllm_last_error())


if __name__ == "__main__":
    globals()["case_" + sys.argv[2]]()
    print("ok")
