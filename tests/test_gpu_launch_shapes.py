"""Cached kernel-engine loads on both sides of the sizes where the launch shape
changes (K1 at 5,000,000 bytes, K1-scatter at 4 MiB of device image), with
ragged ends, every byte against the oracle."""

import numpy as np
import pytest

import oracle
from paper_2401_14351_amd import binding

pytestmark = pytest.mark.gpu

SENTINEL = 0xA5


@pytest.mark.parametrize("total", [15, 4097, (4 << 20) - 1, 4 << 20, (4 << 20) + 16, 4_999_999, 5_000_000, 5_000_017])
@pytest.mark.parametrize("chunk", [1 << 20, (3 << 20) + 48])
def test_cached_load_at_shape_changes(tmp_path, total, chunk):
    import torch

    rng = np.random.default_rng(total)
    sizes = [min(777, total // 3), total // 2]
    sizes.append(total - sum(sizes))  # packed densely, the image has exactly `total` bytes
    tensors = [(f"t{i}", "i8", (n,), rng.integers(0, 256, n, dtype=np.uint8)) for i, n in enumerate(sizes)]
    binding.convert(iter(tensors), str(tmp_path), 1, chunk)
    index = oracle.make_index(tensors, 1, chunk)
    image = bytes(oracle.partition_bytes(tensors, 1)[:index.total_bytes])
    assert len(image) == total
    with binding.Pool(chunk, -(-total // chunk)) as pool:
        pool.cache(str(tmp_path))
        for A2 in (0, 16, 4096):
            print("[gpu-test] shapes", total, chunk, A2, flush=True)
            want = np.frombuffer(bytes(oracle.repack(image, index, A2)) if A2 else image, np.uint8)
            dst = torch.full((len(want) + 64,), SENTINEL, dtype=torch.uint8, device="cuda:0")
            with binding.Checkpoint(str(tmp_path), pool=pool, dev_alignment=A2) as ck:
                ck.load_into(dst, torch.cuda.current_stream())
                torch.cuda.synchronize()
            got = dst.cpu().numpy()
            assert np.array_equal(got[:len(want)], want)
            assert (got[len(want):] == SENTINEL).all(), "bytes past the image were written"
        pool.evict(str(tmp_path))
