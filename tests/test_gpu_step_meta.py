"""The metadata calls and the plan where they can go wrong: steps that are refused in part (the plan stays inside its buffer
and names rows of the step only), batches over several waves of the plan, sequences over several workgroups."""
import numpy as np
import pytest
import torch

from paper_2508_08895_amd import binding as A

pytestmark = pytest.mark.gpu

_GUARD = 0x5a5a5a5a


def _batch(B, count, max_blocks=24):
    pool = torch.zeros(B * max_blocks, 2, 16, 64, dtype=torch.bfloat16, device="cuda")
    tables = torch.arange(B * max_blocks, dtype=torch.int32).reshape(B, max_blocks).cuda()
    kv = A.KVCache(pool, pool, tables, 8)
    st = A.BatchState(B, max_blocks * 16, "cuda")
    st.cu_branches = torch.from_numpy(np.append(0, np.cumsum(count)).astype(np.int32)).cuda()
    st.NB = int(sum(count))
    st.branch_len = torch.zeros(st.NB, dtype=torch.int32, device="cuda")
    st.stage_base.fill_(100)
    st.seq_len.fill_(100)
    return kv, st


@pytest.mark.parametrize("B", [1, 3, 64, 500])
@pytest.mark.parametrize("hint", [0, 7, 60])   # streaming kernel without and with a hint, row-splitting kernel
@pytest.mark.parametrize("kind", ["main tokens under open branches", "more tokens than rows"])
def test_plan_of_a_refused_step_stays_in_its_buffer(B, hint, kind):
    count = np.where(np.arange(B) % 2 == 0, 2, 0)
    kv, st = _batch(B, count)
    main = np.full(B, 3)
    if kind == "more tokens than rows":
        main[count > 0] = 0
    new = np.full(st.NB, 2)
    rows = int(new.sum() + main.sum()) if kind != "more tokens than rows" else 5
    step = A.Step(rows, st.NB, B, "cuda", max_new_per_seq=hint)
    step.cu_seq_new.copy_((torch.arange(B + 1) % 2 * 4000).int())   # as earlier steps may have left them
    words = A.aspd_plan_bytes(kv, B, rows) // 4
    whole = torch.full((words + 4096,), _GUARD, dtype=torch.int32, device="cuda")
    step.plan = whole[:words]
    lens = torch.from_numpy(np.concatenate([new, main]).astype(np.int32)).cuda()
    A.aspd_build_branch_meta(kv, st, A.STAGE_MIXED, lens, step=step)
    assert bool((whole[words:] == _GUARD).all())
    fault = int(st.fault[0])
    assert fault & (A.FAULT_ROW_COUNT if kind == "more tokens than rows" else A.FAULT_STAGE) or (B == 1 and rows == 5)
    # every sequence's rows begin where those before it end, refused or not
    per_seq = np.add.reduceat(np.append(new, 0), np.append(0, np.cumsum(count))[:-1]) * (count > 0) + main
    assert np.array_equal(step.cu_seq_new.cpu().numpy(), np.append(0, np.cumsum(per_seq)))
    # no segment of the plan names a row that the step does not have
    plan = step.plan.cpu().numpy()
    nwg = step.plan_key >> 27 & 2047
    for w in range(nwg):
        n, at = plan[32 * w + 8], plan[32 * w + 9]
        segs = [plan[32 * w:32 * w + 8]] if n > 0 else []
        segs += [plan[32 * nwg + 8 * (at + i):32 * nwg + 8 * (at + i + 1)] for i in range(n - 1)]
        for d in segs:
            assert 0 <= d[1] and 1 <= d[2] and d[1] + d[2] <= rows, (w, d)


@pytest.mark.parametrize("B,blocks", [(65, 3), (100, 9), (128, 40), (512, 6)])   # sequences in two to eight waves
@pytest.mark.parametrize("new", [1, 90])                                         # streaming, row-splitting kernel
def test_plan_of_large_batches_covers_every_page(B, blocks, new):
    """Even pieces, shares and queue, as the batch and its lengths select them."""
    rng = np.random.default_rng(B + new)
    kv, st = _batch(B, np.ones(B, dtype=int), blocks + 8)
    have = rng.integers(0, 16 * blocks, B).astype(np.int32)
    have[rng.integers(B)] = 16 * blocks
    st.stage_base.copy_(torch.from_numpy(have))
    st.seq_len.copy_(torch.from_numpy(have))
    lens = rng.integers(0, new + 1, B).astype(np.int32)
    lens[0] = new
    step = A.aspd_build_branch_meta(kv, st, A.STAGE_SERIAL, torch.from_numpy(lens).cuda(), NQ=int(lens.sum()),
                                    max_new_per_seq=new)
    assert int(st.fault[0]) == 0
    plan, nwg, qpg = step.plan.cpu().numpy().view(np.int32), step.plan_key >> 27 & 2047, step.plan_key >> 18 & 511
    first = np.append(0, np.cumsum(lens))
    total = have + lens
    read = {}   # (sequence, head, first row): how often each page is read
    for w in range(nwg):
        n, at = plan[32 * w + 8], plan[32 * w + 9]
        segs = [plan[32 * w:32 * w + 8]] if n > 0 else []
        segs += [plan[32 * nwg + 8 * (at + i):32 * nwg + 8 * (at + i + 1)] for i in range(n - 1)]
        for d in segs:
            s, h = int(d[0]) & 0xffff, int(d[0]) >> 16
            assert first[s] <= d[1] and d[1] + d[2] <= first[s + 1] and (d[1] - first[s]) % qpg == 0
            assert 0 <= d[3] < d[4] <= d[5] and d[7] == total[s]
            # no row of the group sees past its last slot; a plan may say more pages, up to the sequence's
            last = have[s] + d[1] - first[s] + d[2] - 1
            assert last // 16 + 1 <= d[5] <= (total[s] + 15) // 16
            pages = read.setdefault((s, h, int(d[1])), np.zeros(d[5], dtype=int))
            assert len(pages) == d[5]
            pages[d[3]:d[4]] += 1
    assert all((p == 1).all() for p in read.values())
    assert set(read) == {(s, h, q) for s in range(B) for h in range(2) for q in range(first[s], first[s + 1], qpg)}


@pytest.mark.parametrize("hkv,held,new,cap,queue", [
    (8, [8000] * 33, 64, 0, False),    # 264 like items on 256 workgroups: two rounds, the second nearly empty
    (8, [8000] * 64, 64, 0, True),     # two full rounds
    (8, [8000] * 65, 64, 0, False),    # and eight items more
    (8, [8000] * 48, 64, 0, False),
    (8, [4000] * 33 + [8000] * 33, 64, 0, False),    # like items of two kinds
    (8, [3900 + 9 * i for i in range(128)], 64, 0, True),
    (8, [1000] * 36, 64, 0, False),
    (8, [1000] * 48, 64, 0, True),     # short items: what a cut costs is more than the round that is half empty
    (8, [0] * 33, 64, 0, True),
    (8, [4000] * 33, 27, 0, False),
    (2, [2000] * 3, 60, 5, False),     # six items, five workgroups
    (2, [2000] * 5, 60, 5, True),
    (1, [2000] * 500, 60, 1, True),    # (one workgroup takes them all, whole or not)
    (8, [6000] + [100] * 300, 64, 0, False),         # one item long against a share
])
def test_whole_items_where_their_rounds_fill_the_workgroups(hkv, held, new, cap, queue):
    """Chunks of like lengths, the number of items just above the workgroups and at whole rounds of them: whole items from a
    queue (plan word 10) only where the last round costs no more than cutting does.  Either way every page of every item is
    read once."""
    B, have = len(held), np.asarray(held, dtype=np.int32)
    blocks = (int(have.max()) + new + 15) // 16
    pool = torch.zeros(1, hkv, 16, 64, dtype=torch.bfloat16, device="cuda")
    kv = A.KVCache(pool, pool, torch.zeros(B, blocks, dtype=torch.int32, device="cuda"), 4 * hkv)
    st = A.BatchState(B, blocks * 16, "cuda")
    st.stage_base.copy_(torch.from_numpy(have))
    st.seq_len.copy_(torch.from_numpy(have))
    step = A.aspd_build_branch_meta(kv, st, A.STAGE_SERIAL, torch.full((B,), new, dtype=torch.int32, device="cuda"), NQ=B * new,
                                    max_new_per_seq=new, max_workgroups=cap)
    assert int(st.fault[0]) == 0
    plan, nwg = step.plan.cpu().numpy().view(np.int32), step.plan_key >> 27 & 2047
    assert nwg == (cap or 256) and B * hkv > nwg and (plan[10] > 0) == queue
    read = {}
    for w in range(nwg):
        n, at = plan[32 * w + 8], plan[32 * w + 9]
        segs = [plan[32 * w:32 * w + 8]] if n > 0 else []
        segs += [plan[32 * nwg + 8 * (at + i):32 * nwg + 8 * (at + i + 1)] for i in range(n - 1)]
        for d in segs:
            s, h = int(d[0]) & 0xffff, int(d[0]) >> 16
            assert d[1] == s * new and d[2] == new and d[5] == (have[s] + new + 15) // 16
            assert 0 <= d[3] < d[4] <= d[5] and (not queue or (d[3] == 0 and d[4] == d[5]))
            read.setdefault((s, h), np.zeros(d[5], dtype=int))[d[3]:d[4]] += 1
    assert all((p == 1).all() for p in read.values())
    assert set(read) == {(s, h) for s in range(B) for h in range(hkv)}


@pytest.mark.parametrize("pages,new", [(433, 64), (432, 64), (2063, 1), (2062, 1), (40, 64)])
def test_as_many_items_as_workgroups_stay_whole(pages, new):
    """256 items of two nearly like lengths on 256 workgroups, an item each, also where only the last of the candidates for the
    even pieces' cost reaches that of the longest (433 and 2063 pages)."""
    B, hkv = 32, 8
    have = 16 * (pages - 10 * (np.arange(B) >= 16)) - new
    pool = torch.zeros(1, hkv, 16, 64, dtype=torch.bfloat16, device="cuda")
    kv = A.KVCache(pool, pool, torch.zeros(B, pages, dtype=torch.int32, device="cuda"), 4 * hkv)
    st = A.BatchState(B, pages * 16, "cuda")
    st.stage_base.copy_(torch.from_numpy(have))
    st.seq_len.copy_(torch.from_numpy(have))
    step = A.aspd_build_branch_meta(kv, st, A.STAGE_SERIAL, torch.full((B,), new, dtype=torch.int32, device="cuda"), NQ=B * new,
                                    max_new_per_seq=new, max_workgroups=256)
    plan, nwg = step.plan.cpu().numpy().view(np.int32), step.plan_key >> 27 & 2047
    hdr = plan[:32 * nwg].reshape(nwg, 32)
    assert int(st.fault[0]) == 0 and nwg == B * hkv and (hdr[:, 8] == 1).all()
    assert (hdr[:, 3] == 0).all() and np.array_equal(hdr[:, 4], ((have + new) // 16)[hdr[:, 0] & 0xffff])


@pytest.mark.parametrize("lengths", [[9001], [1, 513, 0, 2300], [300] * 70, [40, 0, 7] * 60])
def test_metadata_of_whole_sequences_that_workgroups_share(lengths):
    """One to sixteen workgroups per sequence, sequences in one to three waves of the row groups' list."""
    from oracle.sequence_layout import replay_layout
    rng = np.random.default_rng(len(lengths))
    blocks = max(lengths) // 16 + 1
    layouts = []
    for n in lengths:
        cut = np.sort(rng.integers(0, n + 1, 4))
        part = np.diff(np.concatenate([[0], cut, [n]])).tolist()
        layouts.append([(0, part[0]), (1, part[1]), (2, part[2]), (0, part[3]), (1, part[4])])
    B = len(lengths)
    kv, st = _batch(B, np.ones(B, dtype=int), blocks)
    tt, meta = replay_layout(kv.block_tables.cpu().numpy(), 16, layouts)
    dev = [torch.from_numpy(np.asarray(x, dtype=np.int32)).cuda() for x in
           (np.cumsum([0] + [5] * B), [b for r in layouts for b, _ in r], [n for r in layouts for _, n in r])]
    step = A.aspd_build_sequence_meta(kv, st, *dev, NQ=sum(lengths))
    assert int(st.fault[0]) == 0 and st.seq_len.cpu().tolist() == lengths
    assert np.array_equal(step.cu_seq_new.cpu().numpy(), np.append(0, np.cumsum(lengths)))
    for f in ("q_seq", "q_branch", "position_ids", "logical_slot", "slot_mapping", "kv_len"):
        assert np.array_equal(getattr(step, f).cpu().numpy(), getattr(meta, f)), f
    # the row groups: all rows once
    plan, rows = step.plan.cpu().numpy().view(np.int32), sum(lengths)
    items = plan[16 + (rows + 3 & ~3):][:4 * plan[0]].reshape(-1, 4)
    seen = np.zeros(rows, dtype=int)
    for s, q0, nq, pages in items.tolist():
        seen[q0:q0 + nq] += 1
        assert pages == (q0 + nq - int(step.cu_seq_new[s]) + 15) // 16
    assert (seen == 1).all()
