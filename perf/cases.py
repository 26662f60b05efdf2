"""The work a program has this library do, as measurable cases.

A case is one call path over one converted checkpoint:

* ``load``     open, load the checkpoint cached in the pinned DRAM tier into a
               device buffer, build the tensor views, close: what a model
               manager does for each request that needs a checkpoint.
* ``stream``   the same from the checkpoint's file, through a ring of pinned
               chunks that reader threads fill.
* ``repack``   move a loaded file-layout image into another device alignment,
               by a handle that a program keeps open (sllm_repack).
* ``noalloc``  the same with no device allocation, by a handle that holds only
               the index (sllm_repack_noalloc): code under graph capture or in
               a serving loop.

Conversion is left out: it is done once per checkpoint, has no device work and
runs at the rate its disk writes.

The checkpoints are those of ``synth``: LoRA adapters, OPT-125M, Llama-2
shaped models (their first layers, so that inputs are made quickly) and sets
of many small tensors under the stress law (sizes log-uniform), which stand
for checkpoints made mostly of biases, norms, scales and small experts.  Every
output is the whole device image, compared byte for byte.
"""

import math
import os
import shutil
import tempfile
import weakref

import numpy as np
import torch

from paper_2401_14351_amd import binding, synth

KiB, MiB = 1 << 10, 1 << 20
_TORCH = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16, "i8": torch.int8}


def listed():
    return [
        # a small adapter swapped in from DRAM: fixed costs of a load count
        {"name": "load adapter 7b r8", "do": "load", "set": "lora", "size": "7b", "rank": 8,
         "align": 256, "chunk": 16 * MiB, "dev_align": 0, "engine": "kernel"},
        # a small model from DRAM
        {"name": "load opt-125m", "do": "load", "set": "opt", "align": 256, "chunk": 16 * MiB,
         "dev_align": 0, "engine": "kernel"},
        # the large case: a Llama-2-7B shaped partition from DRAM
        {"name": "load llama 7b 4 layers", "do": "load", "set": "llama", "size": "7b", "layers": 4,
         "align": 256, "chunk": 16 * MiB, "dev_align": 0, "engine": "kernel"},
        # an adapter into page-aligned device slots: the device tables are built at open
        {"name": "load adapter 13b r16 a2", "do": "load", "set": "lora", "size": "13b", "rank": 16,
         "align": 256, "chunk": 16 * MiB, "dev_align": 4096, "engine": "kernel"},
        # densely packed small tensors, relocated while they cross the link
        {"name": "load small dense a2", "do": "load", "set": "small", "n": 4001, "min": 256, "max": 256 * KiB,
         "sizes": 11, "align": 1, "chunk": 1 * MiB, "dev_align": 256, "engine": "kernel"},
        # the copy engines, staging in HBM and repacking from there
        {"name": "load opt-125m sdma a2", "do": "load", "set": "opt", "align": 256, "chunk": 16 * MiB,
         "dev_align": 4096, "engine": "sdma"},
        # a small model from its page-cached file
        {"name": "stream opt-125m", "do": "stream", "set": "opt", "align": 256, "chunk": 16 * MiB,
         "dev_align": 0, "engine": "kernel"},
        # the smallest call: an adapter already in HBM, into page-aligned slots
        {"name": "repack adapter 7b r4", "do": "repack", "set": "lora", "size": "7b", "rank": 4, "align": 256,
         "chunk": 16 * MiB, "dev_align": 4096},
        # the stress law's prefix: every tensor moves
        {"name": "repack stress 2g", "do": "repack", "set": "small", "n": 20000, "min": 256, "max": 64 * MiB,
         "sizes": 1005, "cap": 2 << 30, "align": 4096, "chunk": 1 * MiB, "dev_align": 256},
        # many small tensors, densely packed: most 16 KiB of the image meet several
        {"name": "repack small dense", "do": "repack", "set": "small", "n": 20000, "min": 256, "max": 64 * KiB,
         "sizes": 12, "align": 1, "chunk": 1 * MiB, "dev_align": 256},
        # a large adapter in a serving loop that may not allocate
        {"name": "noalloc adapter 70b r32", "do": "noalloc", "set": "lora", "size": "70b", "rank": 32,
         "align": 256, "chunk": 16 * MiB, "dev_align": 4096},
        # many small tensors without allocation: the tables are a large part of the work
        {"name": "noalloc small", "do": "noalloc", "set": "small", "n": 20000, "min": 256, "max": 64 * KiB,
         "sizes": 13, "align": 4096, "chunk": 1 * MiB, "dev_align": 16},
    ]


def draw(rng):
    def log_uniform(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    do = rng.choice(["load", "load", "load", "stream", "repack", "repack", "noalloc", "noalloc"])
    kind = rng.choice(["lora", "small"] if do == "noalloc" else ["lora", "opt", "llama", "small", "small"])
    case = {"do": do, "set": kind, "align": rng.choice([64, 256, 4096]), "chunk": rng.randint(2, 64) * MiB}
    if kind == "lora":
        case["size"] = rng.choice(["7b", "13b", "70b"])
        case["rank"] = log_uniform(2, 64)
    elif kind == "llama":
        case["size"] = rng.choice(["7b", "13b"])
        case["layers"] = rng.randint(1, 3 if case["size"] == "7b" else 2)
    elif kind == "small":
        case["max"] = log_uniform(4 * KiB, 64 * MiB)
        case["n"] = log_uniform(500, 30000)
        case["min"] = rng.choice([1, 64, 256, 1000])
        case["sizes"] = rng.randrange(1 << 20)
        case["cap"] = log_uniform(64 * MiB, 1900 * MiB)
        case["align"] = rng.choice([1, 16, 256, 4096])
        case["chunk"] = rng.choice([1, 16]) * MiB
    if do in ("load", "stream"):
        case["dev_align"] = rng.choice([0, 256, 4096])
        case["engine"] = rng.choice(["kernel", "kernel", "sdma"])
    else:
        case["dev_align"] = rng.choice([16, 64, 256, 4096])
    return case


def _spec(case):
    """The checkpoint's tensor list."""
    if case["set"] == "lora":
        spec = synth.lora(case["size"], case["rank"])
    elif case["set"] == "opt":
        spec = synth.opt_125m()
    elif case["set"] == "llama":
        spec = synth.llama2(case["size"])
        keep = 1 + 9 * case["layers"]  # the embedding, then nine tensors a layer; the norm and the head end the list
        spec.tensors = spec.tensors[:keep] + spec.tensors[-2:]
    else:
        spec = synth.stress(case["n"], case["sizes"], case["min"], case["max"], case.get("cap"))
    return spec


def _align_up(x, a):
    return -(-x // a) * a


def _payload(case, seed):
    """The tensors' bytes, one after another: N(0, 0.02) weights, random bytes for the stress law."""
    spec = _spec(case)
    n = spec.payload_bytes
    gen = torch.Generator(device="cuda").manual_seed(seed)
    if case["set"] == "small":
        words = torch.randint(-(1 << 63), (1 << 63) - 1, (n // 8 + 1,), dtype=torch.int64, device="cuda", generator=gen)
        data = words.view(torch.uint8)[:n]
    else:
        dtype = _TORCH[spec.tensors[0].dtype]
        data = torch.empty(n // 2, dtype=dtype, device="cuda").normal_(0.0, 0.02, generator=gen).view(torch.uint8)
    return spec, data.cpu().numpy()


class _State:
    """What a program holds: the converted checkpoint, its pool or handle, and its device buffers."""

    def __init__(self, case, seed):
        self.do = case["do"]
        spec, data = _payload(case, seed)
        self.dir = tempfile.mkdtemp(prefix="sllm-case-", dir="/dev/shm" if os.path.isdir("/dev/shm") else None)
        self.pool = self.handle = None
        self._end = weakref.finalize(self, shutil.rmtree, self.dir, True)

        def tensors():
            at = 0
            for t in spec.tensors:
                yield t.name, t.dtype, t.shape, data[at:at + t.nbytes]
                at += t.nbytes

        binding.convert(tensors(), self.dir, case["align"], case["chunk"])
        total = sum(_align_up(t.nbytes, case["align"]) for t in spec.tensors)
        total2 = sum(_align_up(t.nbytes, case["dev_align"] or case["align"]) for t in spec.tensors)
        chunks = -(-total // case["chunk"])
        self.dst = torch.empty(total2, dtype=torch.uint8, device="cuda")
        self.opts = {}
        if self.do in ("load", "stream"):
            # a stream's ring holds 256 MiB, at least 16 chunks; a load's pool all of the checkpoint
            ring = max(16, (256 * MiB) // case["chunk"])
            self.pool = binding.Pool(case["chunk"], chunks if self.do == "load" else ring)
            self.opts = {"pool": self.pool, "engine": case["engine"], "dev_alignment": case["dev_align"]}
            if self.do == "load":
                self.pool.cache(self.dir, io_threads=8)
            else:
                self.opts.update(io_threads=8, ring_slots=ring)
        else:
            self.src = torch.empty(total, dtype=torch.uint8, device="cuda")
            with binding.Checkpoint(self.dir, io_threads=8, ring_slots=16) as ck:
                ck.load_into(self.src, torch.cuda.current_stream())
            self.dev_align = case["dev_align"]
            self.handle = binding.Checkpoint(self.dir, index_only=True) if self.do == "noalloc" else \
                binding.Checkpoint(self.dir, dev_alignment=self.dev_align, ring_slots=1, chunk_size=MiB)

    def __del__(self):
        if self.handle is not None:
            self.handle.close()
        if self.pool is not None:
            self.pool.close()


def prepare(case, seed):
    return _State(case, seed)


def run(state):
    stream = torch.cuda.current_stream()
    if state.do in ("load", "stream"):
        with binding.Checkpoint(state.dir, **state.opts) as ck:
            ck.load_with_views(state.dst, stream)
    elif state.do == "repack":
        state.handle.repack(state.src, state.dst, stream)
    else:
        state.handle.repack_noalloc(state.src, state.dst, state.dev_align, stream)
    return {"image": state.dst}


def work(case):
    spec = _spec(case)
    src = sum(_align_up(t.nbytes, case["align"]) for t in spec.tensors)
    dst = sum(_align_up(t.nbytes, case["dev_align"] or case["align"]) for t in spec.tensors)
    return {"bytes": src + dst, "flops": 0}


def tolerance(case):
    return "exact"  # bytes are moved, never converted


def exact(case, seed):
    """The device image by its definition: tensors in order at the next multiple of the alignment, zeros between."""
    spec, data = _payload(case, seed)
    align = case["dev_align"] or case["align"]
    image = np.zeros(sum(_align_up(t.nbytes, align) for t in spec.tensors), dtype=np.uint8)
    at = to = 0
    for t in spec.tensors:
        image[to:to + t.nbytes] = data[at:at + t.nbytes]
        at += t.nbytes
        to += _align_up(t.nbytes, align)
    return {"image": image}
