"""Timed cases of the library's hot path: run_layers on packed batches, as a serving program calls it.

A case is one serving situation on one of the decoder shapes of this repository (a few layers of it: the layers
of a model are alike, and every layer's weights are larger than the caches keep).  One pass is what the program
does for one step of it: rebuild the batch in place (membership changes every step), bring in the step's hidden
states, run the layers; where the situation has them, the decode steps that follow, the hand-off to a second
instance at a layer boundary, or the layers' trip from page-locked host memory.  Outputs are the hidden states of
every step and the KV cache with the positions the pass has appended.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2412_17246_amd import Instance

# hidden, query heads, kv heads, head dim, feed-forward width, rotary base
SHAPES = {
    "tiny": (256, 4, 4, 64, 688, 10000.0),
    "7b": (4096, 32, 32, 128, 11008, 10000.0),
    "8b_gqa": (4096, 32, 8, 128, 14336, 500000.0),
    "13b": (5120, 40, 40, 128, 13824, 10000.0),
    "70b": (8192, 64, 8, 128, 28672, 500000.0),
}

# A case's keys: `prompts` sequences bring several new tokens each, their numbers lognormal around `median`
# (sigma 0.6) within [lo, hi], on top of `cached` positions of earlier chunks; `decodes` sequences bring one, on
# caches uniform in [cache_lo, cache_hi]; `follow` further decode steps of all sequences come after the first run.
# `split`: the first half of the layers runs on one instance, the second on another.  `streamed`: the layers come
# from page-locked host memory while they run.
NONE = {"prompts": 0, "median": 0, "lo": 0, "hi": 0, "cached": 0, "decodes": 0, "cache_lo": 0, "cache_hi": 0,
        "follow": 0, "split": False, "streamed": False, "lengths": 1}


def _case(shape, layers, **more):
    return dict(NONE, shape=shape, layers=layers, **more)


def listed():
    def named(name, shape, layers, **more):
        return dict(_case(shape, layers, **more), name=name)

    return [
        # the smallest session there is: a 64-token prompt and eight tokens after it; launches and latency only
        named("tiny_session", "tiny", 2, prompts=1, median=64, lo=64, hi=64, follow=8),
        # one user's answer being written, four tokens of it: every weight is read for one row
        named("8b_decode_1", "8b_gqa", 4, decodes=1, cache_lo=1171, cache_hi=1171, follow=3),
        # a lightly loaded pair of instances during scaling: half of the layers on each, hand-off in between
        named("8b_split_decode_24", "8b_gqa", 4, decodes=24, cache_lo=200, cache_hi=2500, split=True),
        # the benchmark's continuous decode
        named("8b_decode_64", "8b_gqa", 4, decodes=64, cache_lo=256, cache_hi=4096),
        # the same on the largest shape
        named("70b_decode_32", "70b", 2, decodes=32, cache_lo=512, cache_hi=4096),
        # a full house of short chats, no grouped heads
        named("7b_decode_161", "7b", 2, decodes=161, cache_lo=128, cache_hi=1024),
        # a single prompt of ordinary length
        named("7b_prompt_301", "7b", 4, prompts=1, median=301, lo=301, hi=301),
        # a chunk of a long prompt beside running answers (prefill and decode colocated)
        named("8b_chunk_512_decode_40", "8b_gqa", 4, prompts=1, median=512, lo=512, hi=512, cached=3000, decodes=40,
              cache_lo=256, cache_hi=4096),
        # the benchmark's batch of eight requests
        named("7b_prefill_8", "7b", 2, prompts=8, median=512, lo=16, hi=2048),
        # the benchmark's mixed batch: sixteen prompts and forty-eight running answers
        named("13b_mixed_16_48", "13b", 2, prompts=16, median=768, lo=32, hi=4096, decodes=48, cache_lo=128, cache_hi=2048),
        # the benchmark's headline batch on the largest shape
        named("70b_prefill_4x2048", "70b", 2, prompts=4, median=2048, lo=2048, hi=2048),
        # scale start to first token: layers arrive over the host link behind a waiting prompt
        named("7b_streamed_2000", "7b", 4, prompts=1, median=2000, lo=2000, hi=2000, streamed=True),
    ]


def _spread(rng, lo, hi):
    """A whole number, spread over the logarithm of the range."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "decode", "prefill", "prefill", "mixed", "mixed", "split", "session", "streamed"])
    shape = rng.choice(["7b", "8b_gqa", "8b_gqa", "13b", "70b"])
    lengths = rng.randrange(1, 1 << 20)
    lo = _spread(rng, 16, 1024)
    cache = dict(cache_lo=lo, cache_hi=_spread(rng, lo, 4096))
    if kind == "decode":
        return _case(shape, 2, decodes=_spread(rng, 1, 256 if shape == "8b_gqa" else 160), follow=rng.choice([0, 0, 1, 2]),
                     lengths=lengths, **cache)
    if kind == "split":
        return _case(shape, 2, decodes=_spread(rng, 1, 128), split=True, lengths=lengths, **cache)
    if kind == "session":
        return _case("tiny", 2, prompts=_spread(rng, 1, 8), median=_spread(rng, 16, 400), lo=2, hi=1000,
                     follow=rng.randrange(4, 12), lengths=lengths)
    prompts = _spread(rng, 1, 8)
    few = dict(prompts=prompts, median=_spread(rng, 16, 8000 // prompts if shape != "70b" else 4000 // prompts), lo=8,
               hi=min(4096, (8192 if shape != "70b" else 4096) // prompts), cached=rng.choice([0, 0, 0, rng.randrange(1, 2000)]),
               lengths=lengths)
    if kind == "prefill":
        return _case(shape, 2, **few)
    if kind == "streamed":
        return _case(rng.choice(["7b", "8b_gqa"]), 2, streamed=True, **dict(few, cached=0))
    return _case(shape, 2, decodes=_spread(rng, 1, 96), **few, **cache)


def _shape(case):
    H, Hq, Hkv, d, F, base = SHAPES[case["shape"]]
    return SimpleNamespace(L=case["layers"], H=H, Hq=Hq, Hkv=Hkv, d=d, F=F, eps=1e-5, rope_base=base)


def _sequences(case):
    """New tokens and cached positions of every sequence of the first run."""
    rng = np.random.default_rng(case["lengths"])
    new = np.exp(rng.normal(math.log(max(1, case["median"])), 0.6, case["prompts"]))
    new = np.clip(np.rint(new), max(1, case["lo"]), max(1, case["hi"])).astype(int).tolist()
    old = [case["cached"]] * case["prompts"]
    new += [1] * case["decodes"]
    old += rng.integers(case["cache_lo"], case["cache_hi"] + 1, case["decodes"]).tolist()
    return new, old


_STREAMS = []


def _streams():
    """The process's compute and copy stream: created once, shared by every instance (a process has few hardware queues)."""
    if not _STREAMS:
        _STREAMS.extend((torch.cuda.Stream(), torch.cuda.Stream()))
    return _STREAMS


def _normal(gen, n, scale=1.0, shift=0.0):
    return torch.randn(n, generator=gen, device="cuda", dtype=torch.float32).mul_(scale).add_(shift).to(torch.bfloat16)


def _blob(inst, shape, gen):
    """One layer's weights, N(0, 0.02^2), gains 1 + N(0, 0.02^2), as the library takes them."""
    blob = torch.empty(inst.layer_bytes // 2, dtype=torch.bfloat16, device="cuda")
    blob.copy_(_normal(gen, blob.numel(), 0.02))
    for at in (inst.layout.g1 // 2, inst.layout.g2 // 2):
        blob[at:at + shape.H].add_(1.0)
    return blob.view(torch.uint8)


def prepare(case, seed):
    shape = _shape(case)
    new, old = _sequences(case)
    n, T, follow = len(new), sum(new), case["follow"]
    room = [a + b + follow for a, b in zip(new, old)]
    compute, copy = _streams()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    s = SimpleNamespace(case=case, compute=compute, shape=shape, T=T, instances=[], sources=None)
    with torch.cuda.stream(compute):
        for _ in range(2 if case["split"] else 1):
            s.instances.append(Instance(shape, max_seqs=n, max_seq_len=max(room), max_tokens=T,
                                        kv_tokens=sum(room) + 32 * n, compute_stream=compute, copy_stream=copy))
        half = shape.L // 2
        owner = [s.instances[-1 if case["split"] and l >= half else 0] for l in range(shape.L)]
        if case["streamed"]:
            s.sources = []
            for l in range(shape.L):
                host = torch.empty(owner[l].layer_bytes, dtype=torch.uint8, pin_memory=True)
                host.copy_(_blob(owner[l], shape, gen))
                s.sources.append(host)
        else:
            for l in range(shape.L):
                blob = _blob(owner[l], shape, gen)
                compute.synchronize()
                owner[l].load_layer_from_device(l, blob)
                owner[l].wait_layer(l)
                owner[l].drop_sources()
        for inst in s.instances:
            for slot in range(n):
                inst.kv_reserve(slot, room[slot])
        for l in range(shape.L):
            for slot in range(n):
                if old[slot]:
                    k, v = (_normal(gen, old[slot] * shape.Hkv * shape.d) for _ in range(2))
                    owner[l].kv_write(l, slot, 0, old[slot], k, v)
        s.first = ([0] + np.cumsum(new).tolist(), list(range(n)), old)
        s.after = (list(range(n + 1)), list(range(n)), [a + b for a, b in zip(new, old)])
        s.batch = s.instances[0].batch(*s.first, storage=s.instances[0].batch_storage(n, T, max(room)))
        s.inputs = [_normal(gen, T * shape.H).view(T, shape.H)] + [_normal(gen, n * shape.H).view(n, shape.H) for _ in range(follow)]
        s.hidden = [torch.empty_like(x) for x in s.inputs]
        s.handed = torch.empty_like(s.hidden[0]) if case["split"] else None
    torch.cuda.synchronize()
    return s


def run(s):
    L, inst = s.shape.L, s.instances[0]
    outputs = []
    with torch.cuda.stream(s.compute):
        if s.sources is not None:                 # a new scale-out: nothing is resident
            for l in range(L):
                inst.unload_layer(l)
            for l in range(L):
                inst.load_layer(l, s.sources[l])
        s.batch.rebuild(*s.first)
        for step, (given, x) in enumerate(zip(s.inputs, s.hidden)):
            if step == 1 and s.case["prompts"]:   # the prompts are in: from here on every sequence brings one token
                s.batch.rebuild(*s.after)
            elif step:
                inst.batch_advance(s.batch)
            x.copy_(given)
            if s.handed is None:
                inst.run_layers(0, L, s.batch, x)
                outputs.append(x)
            else:
                inst.run_layers(0, L // 2, s.batch, x)
                second = s.instances[1]
                second.import_boundary(s.handed, s.T, x)
                second.run_layers(L // 2, L, s.batch, s.handed)
                outputs.append(s.handed)
    return {"hidden": outputs, "cache": [i.kv_arena.view(torch.bfloat16) for i in s.instances]}


def work(case):
    """The weights once per run (a later step's input waits for the earlier step's output), every cached position
    once, the new positions and the hidden states in and out; products, and attention over the visible pairs."""
    s = _shape(case)
    new, old = _sequences(case)
    params = s.H * s.d * (2 * s.Hq + 2 * s.Hkv) + 3 * s.H * s.F
    position = 2 * s.Hkv * s.d * 2
    nbytes = flops = 0
    for step in range(1 + case["follow"]):
        if step:
            new, old = [1] * len(new), [a + b for a, b in zip(new, old)]
        pairs = sum(a * b + a * (a + 1) / 2 for a, b in zip(new, old))
        nbytes += s.L * (2 * params + 4 * s.H + position * (sum(old) + sum(new))) + 4 * sum(new) * s.H
        flops += s.L * (2 * params * sum(new) + 4 * s.Hq * s.d * pairs)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # bf16 storage between the kernels, sums in fp32: with every sequence in a batch of its own (other kernels, other
    # orders of the sums) the hidden states after two to four layers move by 3.4e-3 to 6.6e-3, single ones by 0.04
    return {"rel": 1.5e-2, "max": 0.16}

