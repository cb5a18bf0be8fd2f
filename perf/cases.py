"""What the framework's speed is measured on: steps of a decoding program as it makes them through the binding.

A pass is one engine step over a batch: the metadata call, then for every layer the rotary append of the new tokens
and the attention call (the model's own projections are not part of it: queries, keys and values of the new tokens
are inputs).  Layers have a KV pool each, as in a model, so consecutive calls do not find each other's pages in a
cache; the number of layers is what is kept small here, the step is otherwise whole.  So that a pass can be repeated,
it starts with the decode state put back to where the step found it (one small copy) and with the queries fresh, as
the projection would leave them (one copy; aspd_rope_append turns them in place).

Kinds of step:
  decode     one token per branch of sequences in a parallel stage
  serial     the stage ends (merge) and one main-branch token per sequence attends everything
  mixed      some sequences in a parallel stage, some serial, one token per branch / per serial sequence
  chunk      forced tokens per branch (the branch prefix that opens a stage, or teacher-forced pieces)
  prefill    prompts: all tokens of a batch of empty sequences as one serial append
  sequences  whole multi-stage sequences rebuilt from slot 0 (re-prefill, teacher forcing), with the log-sum-exp
"""
import math
import random

import numpy as np
import torch

from paper_2508_08895_amd import binding as A

BLOCK = 16
THETA = 1e6

# Head layouts: the 7B shape of the benchmark configurations, and the others the tests run.
_7B = dict(dtype="bf16", hq=32, hkv=8, hd=128)


def _case(kind, name=None, *, layers, batch, prefix, branches=(1, 1), held=(0, 0), new=(1, 1), shape=1, **heads):
    c = dict(kind=kind, layers=layers, batch=batch, prefix_lo=prefix[0], prefix_hi=prefix[1], branches_lo=branches[0],
             branches_hi=branches[1], held_lo=held[0], held_hi=held[1], new_lo=new[0], new_hi=new[1], shape=shape, **heads)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # benchmark configuration 1, the smallest call there is: one short sequence in fp32, one layer; launches and
        # host work are all of it
        _case("decode", "tiny_f32", layers=1, batch=1, prefix=(64, 64), branches=(3, 3), held=(4, 15), dtype="f32", hq=4,
              hkv=4, hd=64),
        # configuration 2: one user, a conversation of 2k tokens, four branches; the latency of interactive decoding
        _case("decode", "single_decode", layers=4, batch=1, prefix=(2048, 2048), branches=(4, 4), held=(63, 63), **_7B),
        # configuration 3: an ordinary serving batch, ragged contexts and branch counts
        _case("decode", "batch16_decode", layers=4, batch=16, prefix=(512, 4096), branches=(2, 8), held=(15, 255), **_7B),
        # configuration 4: long documents, few sequences, parallel stage and then the serial step after the merge
        _case("decode", "long_decode", layers=4, batch=4, prefix=(16384, 16384), branches=(6, 6), held=(31, 191), **_7B),
        _case("serial", "long_serial", layers=4, batch=4, prefix=(16384, 16384), branches=(6, 6), held=(32, 192), **_7B),
        # configuration 5: a large serving batch, bound by the bandwidth of the cache reads
        _case("decode", "batch64_decode", layers=4, batch=64, prefix=(1024, 8192), branches=(2, 10), held=(24, 144), **_7B),
        # continuous batching: sequences of a batch switch modes on their own; an odd batch and the smaller head size
        _case("mixed", "mixed_hd64", layers=4, batch=27, prefix=(37, 3001), branches=(1, 5), held=(1, 90), dtype="bf16",
              hq=16, hkv=4, hd=64),
        # a stage opens: branch prefixes of ragged length (title tokens) behind mid-sized contexts
        _case("chunk", "stage_open_chunk", layers=4, batch=12, prefix=(200, 5000), branches=(2, 5), held=(0, 0), new=(5, 21),
              **_7B),
        # configuration 5's 16-token chunk over the whole large batch
        _case("chunk", "batch64_chunk", layers=2, batch=64, prefix=(1024, 8192), branches=(2, 10), held=(8, 128), new=(16, 16),
              **_7B),
        # the engine's prefill: prompts of a small batch as one serial append
        _case("prefill", "prompts_prefill", layers=2, batch=8, prefix=(90, 2000), **_7B),
        # re-prefill of a few short sequences after a stage
        _case("sequences", "short_sequences", layers=2, batch=3, prefix=(301, 1500), branches=(2, 5), **_7B),
        # teacher forcing over a large batch of whole sequences (the repository's largest call)
        _case("sequences", "batch64_sequences", layers=1, batch=64, prefix=(1100, 9400), branches=(1, 10), **_7B),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["decode", "decode", "decode", "serial", "mixed", "chunk", "chunk", "prefill", "sequences"])
    heads = rng.choice([_7B, _7B, _7B, dict(dtype="bf16", hq=16, hkv=4, hd=64), dict(dtype="bf16", hq=8, hkv=8, hd=128)])
    shape = rng.randrange(1 << 20)
    if kind in ("decode", "serial") and rng.random() < 0.15:  # fp32 is for small calls
        heads = rng.choice([dict(dtype="f32", hq=4, hkv=4, hd=64), dict(dtype="f32", hq=8, hkv=2, hd=128)])
        hi = log_int(40, 600)
        return _case(kind, layers=1, batch=log_int(1, 6), prefix=(max(1, hi // 3), hi), branches=(1, rng.randint(2, 6)),
                     held=(1, rng.randint(4, 60)), shape=shape, **heads)
    if kind in ("prefill", "sequences"):
        hi = log_int(150, 8000)
        batch = log_int(1, max(1.5, min(48, 160_000 / hi)))
        return _case(kind, layers=rng.randint(1, 2), batch=batch, prefix=(max(1, hi // rng.randint(2, 9)), hi),
                     branches=(1, rng.randint(2, 9)), shape=shape, **heads)
    hi = log_int(100, 16000)
    batch = log_int(1, max(1.5, min(64, 300_000 / hi)))
    held = (rng.randint(0, 20), rng.randint(21, 200))
    return _case(kind, layers=rng.randint(2, 4), batch=batch, prefix=(max(1, hi // rng.randint(1, 8)), hi),
                 branches=(rng.randint(1, 3), rng.randint(3, 10)), held=held,
                 new=(rng.randint(2, 8), rng.randint(9, 24)) if kind == "chunk" else (1, 1), shape=shape, **heads)


# ------------------------------------------------------------------------------------------------ lengths
def _lengths(case):
    """The batch's lengths, from the case alone: per sequence its prefix (or whole length), its branches' tokens held
    and new; for `sequences` the runs [(branch, tokens)]."""
    r = random.Random(case["shape"])
    kind, B = case["kind"], case["batch"]
    prefix = [r.randint(case["prefix_lo"], case["prefix_hi"]) for _ in range(B)]
    d = dict(prefix=prefix, serial=[False] * B)
    if kind == "sequences":
        d["runs"] = [_runs(r, n, case["branches_lo"], case["branches_hi"]) for n in prefix]
        return d
    if kind == "prefill":
        return d
    count = [r.randint(case["branches_lo"], case["branches_hi"]) for _ in range(B)]
    d["held"] = [[r.randint(case["held_lo"], case["held_hi"]) for _ in range(k)] for k in count]
    d["new"] = [[r.randint(case["new_lo"], case["new_hi"]) for _ in range(k)] for k in count]
    if kind == "mixed":
        d["serial"] = [r.random() < 0.5 for _ in range(B)]
    return d


def _runs(r, tokens, lo, hi):
    """Runs of one sequence of `tokens` tokens: serial and parallel stages in turn, up to three of the latter."""
    stages = r.randint(0, 3)
    w = [r.random() + 0.05 for _ in range(2 * stages + 1)]
    part = [int(tokens * x / sum(w)) for x in w]
    part[0] += tokens - sum(part)
    runs = []
    for i, n in enumerate(part):
        if i % 2 == 0:
            runs.append((0, n))
            continue
        k = r.randint(lo, hi)
        cut = [0] + sorted(r.randint(0, n) for _ in range(k - 1)) + [n]
        runs += [(b + 1, cut[b + 1] - cut[b]) for b in range(k)]
    return runs


def _totals(case):
    """(tokens per sequence after the step, new tokens, keys that the new tokens attend, over the batch)."""
    d, kind = _lengths(case), case["kind"]
    if kind == "prefill":
        return d["prefix"], sum(d["prefix"]), sum(n * (n + 1) // 2 for n in d["prefix"])
    if kind == "sequences":
        keys = 0
        for runs in d["runs"]:
            slot = base = 0
            for b, n in runs:
                base = slot if b <= 1 else base
                keys += n * base + n * (n + 1) // 2
                slot += n
        return d["prefix"], sum(d["prefix"]), keys
    total, rows, keys = [], 0, 0
    for p, held, new, serial in zip(d["prefix"], d["held"], d["new"], d["serial"]):
        t = p + sum(held)
        if kind == "serial" or serial:
            total.append(t + 1)
            rows += 1
            keys += t + 1
        else:
            total.append(t + sum(new))
            rows += sum(new)
            keys += sum((p + h) * n + n * (n + 1) // 2 for h, n in zip(held, new))
    return total, rows, keys


# ------------------------------------------------------------------------------------------------ state
class _State:
    pass


def _i32(x, dev):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.int32)).to(dev)


def prepare(case, seed):
    st = _State()
    dev = torch.device("cuda")
    dtype = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    kind, B, nl = case["kind"], case["batch"], case["layers"]
    d = _lengths(case)
    total, rows, _ = _totals(case)
    hq, hkv, hd = case["hq"], case["hkv"], case["hd"]
    gen = torch.Generator(device=dev).manual_seed(seed)

    def normal(*shape):
        return torch.randn(*shape, generator=gen, device=dev, dtype=dtype)

    # a pool with some room to spare, its blocks dealt to the sequences at random
    blocks = [(t + BLOCK - 1) // BLOCK for t in total]
    pool = sum(blocks) + sum(blocks) // 8 + 1
    order = np.random.default_rng(seed).permutation(pool)
    tables = np.full((B, max(blocks)), -1, dtype=np.int32)
    at = 0
    for s, n in enumerate(blocks):
        tables[s, :n] = order[at:at + n]
        at += n
    tables = torch.from_numpy(tables).to(dev)
    st.kv = [A.KVCache(normal(pool, hkv, BLOCK, hd), normal(pool, hkv, BLOCK, hd), tables, hq) for _ in range(nl)]
    st.state = A.BatchState(B, max(blocks) * BLOCK, dev)
    st.fresh_q = normal(nl, rows, hq, hd)
    st.q = torch.empty_like(st.fresh_q)
    st.k_new, st.v_new = normal(nl, rows, hkv, hd), normal(nl, rows, hkv, hd)
    st.out = torch.empty_like(st.q)
    st.lse = torch.empty(nl, rows, hq, device=dev, dtype=torch.float32) if kind == "sequences" else None
    st.workspace = A.new_workspace(st.kv[0], B, rows)
    st.merge_first = kind == "serial"

    if kind == "sequences":
        runs = d["runs"]
        st.attention = A.aspd_attn_full_sequence
        st.layout = (_i32(np.cumsum([0] + [len(r) for r in runs]), dev), _i32([b for r in runs for b, _ in r], dev),
                     _i32([n for r in runs for _, n in r], dev))
        st.rows = rows
        st.step = A.Step(rows, 0, B, dev)
        st.step.plan = torch.empty(A.aspd_sequence_plan_bytes(st.kv[0], B, rows), dtype=torch.uint8, device=dev)
        return st
    st.layout = None
    if kind == "prefill":
        st.stage, st.attention = A.STAGE_SERIAL, A.aspd_attn_serial_decode
        st.new_len = _i32(d["prefix"], dev)
        hint, parts = max(d["prefix"]), B
    else:
        _history(st, d, dev)
        if kind == "serial":
            st.stage, st.attention = A.STAGE_SERIAL, A.aspd_attn_serial_decode
            st.new_len = _i32([1] * B, dev)
            hint, parts = 1, B
        elif kind == "mixed":
            # the serial sequences' stages have ended before the step
            A.aspd_build_branch_meta(st.kv[0], st.state, A.STAGE_MERGE, _i32(d["serial"], dev))
            open_new = [n for n, ser in zip(d["new"], d["serial"]) if not ser]
            count = [0 if ser else len(n) for n, ser in zip(d["new"], d["serial"])]
            A.aspd_renumber_branches(st.state, torch.from_numpy(np.cumsum([0] + count).astype(np.int32)))
            st.stage, st.attention = A.STAGE_MIXED, A.aspd_attn_parallel_decode
            st.new_len = _i32([x for n in open_new for x in n] + [int(ser) for ser in d["serial"]], dev)
            hint, parts = max([1] + [sum(n) for n in open_new]), st.state.NB
        else:
            st.stage = A.STAGE_PARALLEL
            st.attention = A.aspd_attn_branch_chunk if kind == "chunk" else A.aspd_attn_parallel_decode
            st.new_len = _i32([x for n in d["new"] for x in n], dev)
            hint, parts = max(sum(n) for n in d["new"]), st.state.NB
    # the decode state's small arrays live side by side, so that one copy puts all of them back
    s = st.state
    names = [n for n in ("stage_base", "seq_len", "stage_open", "main_pos", "branch_len") if getattr(s, n) is not None]
    st.found = torch.cat([getattr(s, n) for n in names])
    st.live = st.found.clone()
    at = 0
    for n in names:
        size = getattr(s, n).numel()
        setattr(s, n, st.live[at:at + size])
        at += size
    st.step = A.Step(rows, parts, B, dev, max_new_per_seq=hint)
    st.step.plan = torch.empty(A.aspd_plan_bytes(st.kv[0], B, rows), dtype=torch.uint8, device=dev)
    return st


def _history(st, d, dev):
    """The appends before the step: the prefixes, then the branches one token per step, as decoding lays them."""
    kv, s = st.kv[0], st.state
    A.aspd_build_branch_meta(kv, s, A.STAGE_SERIAL, _i32(d["prefix"], dev), NQ=sum(d["prefix"]), plan=False)
    s.open_parallel(torch.from_numpy(np.cumsum([0] + [len(h) for h in d["held"]]).astype(np.int32)))
    held = np.array([x for h in d["held"] for x in h], dtype=np.int32)
    for t in range(int(held.max())):
        new_len = (held > t).astype(np.int32)
        A.aspd_build_branch_meta(kv, s, A.STAGE_PARALLEL, _i32(new_len, dev), NQ=int(new_len.sum()), plan=False)


def run(st):
    st.q.copy_(st.fresh_q)
    kv, state, step = st.kv, st.state, st.step
    if st.layout is not None:
        A.aspd_build_sequence_meta(kv[0], state, *st.layout, st.rows, step=step)
    else:
        st.live.copy_(st.found)
        if st.merge_first:
            A.aspd_build_branch_meta(kv[0], state, A.STAGE_MERGE, None)
        A.aspd_build_branch_meta(kv[0], state, st.stage, st.new_len, step=step)
    for i in range(len(kv)):
        q, lse = st.q[i], None if st.lse is None else st.lse[i]
        A.aspd_rope_append(kv[i], step, q, st.k_new[i], st.v_new[i], THETA)
        st.attention(kv[i], state, step, q, st.workspace, out=st.out[i], lse=lse)
    return {"out": st.out, "q": st.q, "lse": st.lse, "position_ids": step.position_ids, "slot_mapping": step.slot_mapping,
            "logical_slot": step.logical_slot, "kv_len": step.kv_len, "seq_len": state.seq_len}


# ------------------------------------------------------------------------------------------------ what it takes
def work(case):
    """Per layer: the visible cache once (for `prefill` and `sequences` what the step itself wrote), the new tokens' K
    and V read and written, Q read, turned and written, O written; 4 D flops per query head and visible key."""
    total, rows, keys = _totals(case)
    elt = 4 if case["dtype"] == "f32" else 2
    kv_row = 2 * case["hkv"] * case["hd"] * elt
    q_row = case["hq"] * case["hd"] * elt
    per_layer = sum(total) * kv_row + rows * (2 * kv_row + 3 * q_row)
    if case["kind"] == "sequences":
        per_layer += 4 * rows * case["hq"]
    flops = 4 * case["hd"] * case["hq"] * keys
    return {"bytes": case["layers"] * per_layer, "flops": case["layers"] * flops}


def tolerance(case):
    """bf16: P and O are rounded to bf16 (2^-9 each, 2.4e-3 measured against float64 and between two runs whose sums
    differ in order); fp32: sums in another order (2.4e-7 measured against float64)."""
    return {"rel": 2e-6, "max": 2e-5} if case["dtype"] == "f32" else {"rel": 1e-2, "max": 0.08}
